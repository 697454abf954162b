// Rules by which the host decides how a call is cut into chunks (pure host code).
#pragma once
#include <cstdint>

namespace vegas {

constexpr int kXcds = 8;

// Draft calls of up to kDraftRows rows per KV head (attn_draft16_kernel): the longest selection that one workgroup per
// column (sequence x KV head) streams by itself, writing the output rows; a longer one is cut into chunks that a second
// launch merges.  A single workgroup takes 0.3 us per 32 tokens at head dimension 128 (0.18 at 64) behind 3.4 us and no
// other helps it, the merge costs 2.5-4 us; with many columns the chip is full either way, with few it idles beside a
// long selection.  The rule sees the batch's bound only, so it has to hold for selections of unequal length as well.
// Microseconds of a draft call within a GPU-bound iteration (captured; 6 draft calls), one workgroup minus chunks; equal
// selections / between a tenth and all of the bound / one at the bound beside others of 256 tokens:
//   columns   head dimension 128                                  head dimension 64
//     8..48   416 tokens -0.1, 448 +0.2..-0.3, 544 +1.0             608 0.0, 672 +0.2, 800 +0.9, 1056 +2.1     (all equal)
//       64    544 -0.1/+0.1/+0.7, 800 +1.6                          800 0.0, 928 +0.6/+0.6/+0.7
//       80    544 -1.0/-0.4/+0.5                                    928 -0.1/-0.2/-0.4
//       96    800 -1.0/-0.8/-0.7, 1056 0.0/+1.5/+1.6                928 -0.7/-0.7/-0.7, 2080 -0.4/+2.5/+4.6
//      128    1312 -2.3/+0.7/+2.7, 2080 -1.5/+2.7/+7.7              2080 -3.4/+0.8/+3.8, 3104 -3.4/+4.1/+7.8
//      136    1312 -5.4/-2.4/+0.7, 2080 -6.6/+2.5/+6.5              3104 -6.7/-0.9/+6.5
//      144    2080 -5.9/-1.2/+6.7                                   3104 -6.7/-3.6/+6.5
//      176    2080 -5.1/-5.2/+2.6                                   3104 -5.9/-4.5/+3.8
//      192    3200 -8.0/-4.9/+8.5, 6176 -7.9/-6.1/+23               3200 -5.6/-4.1/+4.2, 6176 -7.4/-5.7/+12
//      256    3200 -6.2/-3.3/+8.6, 6176 -18/-24/+30                 3200 -6.3/-3.7/+3.4, 6176 -17/-14/+14
//      320    3200 +0.4/-10/+5.4, 4128 +7.2/+21/+14                 3200 -2.6/-3.2/+0.9, 4128 +11/-1.6/+5.4
// The lines lie where a call gains with equal and with spread lengths (0.8 us lost at most) and a lone long selection takes no
// more than half as long again (192 columns, 3200 tokens, head dimension 128: 24 -> 32 us, in an iteration of 319).
// (With V in parts, draft_value_parts, 64 columns go on to win up to 928 tokens and 96 up to 1312: 64 x 608 7.7 -> 5.8 us a call, 96 x 928 11.7 -> 9.5.  But a live
// step of one workgroup per column has a launch of its own for its append: live iterations, with these lines at 640 from a
// quarter and 1056 from 3/8 / as they are: 64 x 600 109.4 / 104.7, 96 x 900 153.5 / 148.0, 120 x 800 176.4 / 169.1.)
inline int lone_workgroup_tokens(int64_t columns, int num_cu, int head_dim) {
  struct Line { int per32, tokens128, tokens64; };        // from that many 32nds of the compute units on
  constexpr Line lines[] = {{24, 3200, 3200}, {18, 2176, 3200}, {17, 1312, 3200}, {16, 1312, 2176},
                            {12, 800, 928}, {9, 544, 928}, {0, 448, 672}};
  for (const Line& l : lines)
    if (32 * columns >= static_cast<int64_t>(l.per32) * num_cu) return head_dim == 64 ? l.tokens64 : l.tokens128;
  return 0;
}

// Chunk length of a draft call of `columns` that workgroups of a whole unit (128 tokens, a tile per wave) would leave much of the chip idle: 64 or
// 96 tokens, with a wave or two of every workgroup idle, while there are at most three workgroups for four compute units and 24
// partials to merge.  Fewer waves then share a compute unit's way to memory.  us a call (captured), 128 / 96 / 64 tokens, head
// dimension 128: 8 columns, 500 tokens 6.29 / 5.94 / 5.82, 1056 6.25 / 6.01 / 5.85, 1600 6.32 / 6.12 / 6.16, 2080 6.44 / 6.21 / 6.75,
// 2560 6.47 / 6.62 / 7.10; 16, 800 6.29 / 6.06 / 5.87, 1056 6.36 / 6.09 / 6.23, 1600 6.61 / 6.96 / 7.01; 32, 500 6.30 / 6.05 / 5.81,
// 800 6.55 / 6.62 / 6.68; 1, 2080 6.26 / 6.02 / 6.12; head dimension 64: 8, 1056 5.46 / 5.31 / 5.24, 2080 5.56 / 5.53 / 5.97.  An iteration of
// 32768 tokens with 2048 selected 68.5 / 67.6 / 68.0, of a live one 72.0 / 71.2 / 74.2.
// row_dims: a column's rows x head dimension.  Partials of more than 1.25 MB in all cost the merge what shorter chunks gain, and up to 3 %
// more on some cards: 16 rows of head dimension 128, 128 / 96 / 64 tokens, 8 columns, 1250 6.81 / 6.71 / 6.85 (1.25 MB of the last), 1400 6.85 / 6.72 /
// 6.92, 1900 7.06 / 7.03 / 7.35 (1.25 MB of 96), 2300 7.25 / 7.27 / 8.54; 12 columns, 1250 7.00 / 6.99 / 7.08, 1536 7.00 / 7.09 / 8.34; elsewhere, 128
// and what was chosen without the bound, 8 columns, 1536 6.83 / 7.07, 2300 7.26 / 7.47; 12, 1536 7.17 / 7.30.  (Groups of up to 12, and head dimension
// 64, stay below it.)
inline int draft_chunk_tokens(int64_t columns, int num_cu, int tokens, int unit, int row_dims) {
  for (int chunk = unit / 2; chunk < unit; chunk += unit / 4) {
    const int chunks = (tokens + chunk - 1) / chunk;
    if (chunks <= 24 && 4 * columns * chunks <= 3 * static_cast<int64_t>(num_cu) && columns * chunks * row_dims <= 320 * 1024) return chunk;
  }
  return unit;
}

// A draft call in which one workgroup streams each column's selection (head dimension 128, 16-token pages): through rings in LDS, which
// leave a compute unit room for no other workgroup, or through registers, a tile ahead?  us a call (captured), registers / rings, by
// columns and tokens: 8 128 4.1 / 4.1, 160 4.5 / 4.2, 272 6.0 / 5.3, 448 7.2 / 5.9; 96 800 13.1 / 9.6; 128 300 6.7 / 6.0, 1056 16.4 /
// 14.3; 160 2000 30.1 / 28.8; 192 300 7.4 / 6.7, 1040 19.4 / 19.0, 3000 54.5 / 51.6; 256 300 8.3 / 8.4, 1040 23.3 / 23.0, 3000 67.1 /
// 67.3.  (Head dimension 64: 8 400 5.0 / 5.2; 128 2000 14.4 / 15.2; 192 1040 11.2 / 12.7.  Calls cut into chunks: within 1 %.)
inline bool ring_draft(int64_t columns, int num_cu, int tokens) { return columns < num_cu && tokens > 128; }

// Parts of V, of 32 or 64 head dims, that a draft call of one workgroup per column is split into while there are compute units for them: a
// workgroup reads all of the column's K, its part of V, and writes its part of the output rows.  Such a call is bound by how fast one
// compute unit can read (about 50 GB/s), and no part has anything to merge.  us a call, captured, one / two / four workgroups, head dimension
// 128, 16-token pages: 8 columns, 128 tokens 3.96 / 3.70 / 3.46, 256 4.31 / 3.80 / 3.59, 448 5.71 / 5.03 / 4.71; 64 columns, 256 4.47 / 3.97 / 3.89,
// 448 5.91 / 5.24 / 5.08; 128 columns, 256 4.75 / 4.29 (four do not fit the chip: 6.51), 1300 15.8 / 15.3; one-token pages, 8 columns, 256 4.99 / - /
// 4.34, 448 6.74 / - / 5.85; head dimension 64, two parts, 8 columns, 256 3.93 / 3.46, 640 5.83 / 4.87, 128 columns, 1300 10.5 / 9.5.
inline int draft_value_parts(int64_t columns, int num_cu, int head_dim) {
  if (head_dim == 128 && 4 * columns <= num_cu) return 4;
  return 2 * columns <= num_cu ? 2 : 1;
}
// Their grid is (width, part, columns / width), workgroup x, y, z for column x + width z: workgroups go round the 8 XCDs in the order of the
// grid, and with a width of whole rounds a column's parts meet on one XCD, whose L2 fetches its K once.  A sequence's KV heads are such a width
// where they are a multiple of eight, other numbers of heads go by rounds of columns.  us a call, captured, one workgroup per column /
// parts with the heads for a width, on several XCDs / by rounds, head dimension 128, 16-token pages: 1 head, 128 sequences, 448 tokens 6.5 / 7.6 /
// 5.8, 1300 15.1 / 19.9 / 15.0; 2 heads, 64, 640 7.7 / 10.0 / 7.3; 4 heads, 32, 640 7.6 / 8.1 / 6.7; 7 heads, 18, 448 6.5 / 7.9 / 5.9; 5 heads, 3, 128 4.2 /
// 3.7 / 3.7; head dimension 64, 2 heads, 64, 1300 10.6 / 13.1 / 9.0.
inline int part_grid_width(int kv_heads) { return kv_heads % kXcds == 0 ? kv_heads : kXcds; }
// What a workgroup needs to find its sequence without a division: the number of columns (below 2048) and, above it, 2^16 / kv_heads rounded up; a
// column's sequence then is exact (the product is too large by at most column * kv_heads < 2^16).
inline int32_t column_rounds(int columns, int kv_heads) { return (65535 / kv_heads + 1) << 11 | columns; }
constexpr uint32_t round_columns(int32_t rounds) { return static_cast<uint32_t>(rounds) & 2047u; }
constexpr uint32_t round_sequence(int32_t rounds, uint32_t column) { return column * (static_cast<uint32_t>(rounds) >> 11) >> 16; }

// Verification with a local mask: does one workgroup per column (sequence x KV head x row block) stream the whole band
// (no row sees more than window + queries tokens, nor than the longest sequence has) and write the output rows, or is the context cut into chunks
// (`chunk` tokens, of which the band touches a few) and merged?  Cutting only helps where the chunks are shorter than the
// band: us, chunks + merge / one workgroup, head dimension 128, 20 rows, by chunk length and band:
//   128: 261 10.8 / 10.2, 389 10.8 / 10.0, 517 10.9 / 12.3, 1029 11.0 / 16.3;   256 (40 rows): 389 10.6 / 10.3, 517 10.6 / 12.6
//   1024: 517 15.3 / 12.4, 1029 16.9 / 16.7;   1792: 1029 19.8 / 17.6, 2053 26.4 / 29.1, 4101 28.8 / 52.9
//   3840: 1029 28.3 / 19.4, 2053 51.9 / 31.6;   7936: 1029 25.4 / 21.1, 4101 67.1 / 62.3
// head dimension 64:  128: 389 9.1 / 7.5, 517 9.1 / 9.5;  1024: 1029 13.2 / 12.6;  1792: 1029 15.1 / 12.7, 2053 17.7 / 18.6.
// (Where in its chunk a band of less than a chunk falls decides whether it is one part or two, which is worth up to half
// of the streaming time: the figures are for one place at batch 1, for a batch of many beyond.)
// These are workgroups of four waves that always took a second tile; with kBandWaves of them where eight_wave_band says so, and
// chunks of 128 (8 to 16 workgroups): head dimension 64, 20 rows: 424 7.2 / 6.0, 564 7.6 / 6.5 and 8.4 / 6.9, 704 7.3 / 7.1, 1004 7.6 / 8.0;
// 4 rows: 564 7.1 / 6.3, 1001 7.2 / 7.8; 128, 20 rows: 424 9.0 / 8.4, 564 9.3 / 9.2, 704 9.0 / 10.4; 4 rows: 420 8.1 / 7.9, 480 7.8 / 8.1.
// alone: the longest band that is not cut for being longer than a chunk (lone_band_tokens).
inline bool lone_workgroup_band(int window, int queries, int max_len, int chunk, int alone) {
  int64_t seen = static_cast<int64_t>(window) + queries;
  if (seen > max_len) seen = max_len;
  return seen <= alone || seen <= chunk;
}
constexpr int lone_band_tokens(int head_dim) { return head_dim == 64 ? 640 : 448; }

// Waves of such a workgroup: a wave's second tile is a round trip behind its first, and a band of 128 tokens has five or six.  Eight
// instead of four where the band can have more than four tiles (98 tokens; fewer lose the 0.2 to 0.3 us by which eight waves' rows are
// merged later), every workgroup has a compute unit to itself (384 and more are a second round, 8.2 -> 9.8), and what a row block's
// workgroups read in all is not itself the time (seen: tokens of the band).  us a call, captured, four waves / eight, window 128, 256,
// 384, 512, 1000 (both end at a wave's last tile): head dimension 64, 16 sequences x 8 heads, 40 rows (256 workgroups) 6.1 / 5.5, 6.9 / 6.7, 7.7 / 6.7,
// 8.5 / 7.9, 11.0 / 10.0; one sequence, 20 rows 5.8 / 5.4, 6.6 / 6.4, 7.3 / 6.4, 8.1 / 7.6, 10.2 / 9.2; 128, 8 sequences, 40 rows 7.6 / 7.1, 9.0 / 8.8,
// 10.1 / 8.9, 11.1 / 10.7, 14.4 / 14.1.
// A lone row block has K and V to itself, and one compute unit's way to memory is soon what counts.  Up to eleven tiles eight waves then gain
// with five or six (160 tokens), or where there are many rows to merge at head dimension 64: 8 heads, window 150, 200, 320, 20 rows, 64 5.6 / 5.3,
// 5.6 / 5.5, 6.4 / 6.3, but 16 rows 200 5.2 / 5.5; 128, 20 rows 7.0 / 6.7, 7.0 / 7.1, 8.2 / 8.3, and 16 sequences of 4 rows 256 7.0 / 7.4.  From
// twelve on a wave of four has a third or fourth round trip (head dimension 128, 20 rows, 384, four sequences 9.9 / 9.0, eight 10.4 / 10.2;
// 64, 4 rows, 440, eight 7.0 / 6.4), until the call reads enough for bandwidth to be what is left: 128, 20 rows, two of 630 (5.2 MB) 11.9 /
// 11.1, four of 440 10.2 / 10.4, of 512 11.4 / 11.8, 12 rows, one of 1000 13.7 / 14.5; 8 rows, two of 630 11.1 / 12.0; 64, 40 rows of 8 heads, one of
// 1000 10.2 / 8.7, 20 rows, two 10.0 / 10.0, three 10.8 / 11.2.
constexpr int kBandWaves = 8;
inline bool eight_wave_band(int64_t columns, int row_blocks, int num_cu, int64_t seen, int head_dim, int rows) {
  const int64_t bytes = columns * seen * head_dim * 4;
  if (columns * row_blocks > num_cu || seen <= 97 || bytes > (int64_t{18} << 20) * row_blocks) return false;
  if (row_blocks > 1) return true;
  const bool half_lines = head_dim == 64, few = !half_lines && rows < 12;
  if (seen <= 352) return seen <= 160 || (half_lines && rows > 16);
  if (seen > 640) return half_lines && bytes <= (int64_t{5} << 19);
  return half_lines || (!few && seen <= 420) || bytes <= (int64_t{5} << (few ? 19 : 20));
}

// Verification of more than 64 rows per KV head (with the two sum rows of the logit metric, and there of just above 32 as
// well): sibling workgroups of 32 rows (attn_split_kernel, two per compute unit, each reading K and V through the L2)
// instead of 64 rows each (attn_pair_kernel)?  The latter read half as often but take longer to begin and to end, so small
// calls keep the siblings; bound: sequences x KV heads x longest length, in tokens.  us, 32-row siblings / 64 rows, captured:
//   no collection: 1 sequence x 8 heads x 4096, 128 rows 15.3 / 17.7; 8 x 8 x 500..2000, 80 rows 27.2 / 30.1; 16 x 8 x
//     300..1200, 80 rows 30.9 / 36.1; head dimension 64, 80 rows: 1 x 4 x 32768 19.8 / 20.8; 1 x 8 x 32768 30.3 / 29.4;
//     4 x 8 x 16384 67.0 / 51.1
//   all rows: 1 x 4 x 4096, 80 rows 19.4 / 22.0; 1 x 8 x 12345, 80 rows 37.4 / 38.1, 128 rows 49.5 / 45.9; 2 x 8 x 8192,
//     80 rows 39.2 / 38.2; 8 x 8 x 500..2000, 80 rows 47.5 / 40.7
//   first and last token's rows: 2 x 8 x 8192, 80 rows 29.6 / 32.5; head dimension 64, 1 x 4 x 32768, 80 rows 23.6 / 28.1;
//     1 x 8 x 32768, 128 rows 51.3 / 50.1
//   more than 64 sequences (no plan, every chunk length one for all; 64-row workgroups take a whole sequence each, for an
//     empty one of them waits for a compute unit's LDS), 65 x 8 heads, 80 rows, all rows: 2048..16384 872 / 894, at head
//     dimension 64 540 / 659; 64 of 512 and one of 65536 496 / 1145
//   token sums, 1 sequence x 8 heads: head dimension 64, all rows: 12345, 32 rows 17.9 / 19.7; 32749, 32 rows 34.5 / 26.1,
//     80 rows 41.3 / 42.7; 128: 4096, 96 rows, first and last 17.2 / 18.7; 32749, 64 rows, first and last 39.7 / 41.8, all
//     51.9 / 52.6; 4 x 8 x 16384, head dimension 64, 80 rows 76.5 / 67.2; 16 x 8 x 300..1200, 64 rows 47.5 / 43.9
inline bool rows_as_siblings(int batch, int kv_heads, int max_len, int rows, int collect_rows, bool token_sums, int head_dim) {
  const int tile_rows = rows + (token_sums && collect_rows != 0 ? 2 : 0), blocks = (tile_rows + 31) / 32;
  if (tile_rows <= 64 && (rows > 32 || tile_rows <= 32)) return false;   // (33..62 rows: 64-row workgroups at any size)
  const int64_t bound = static_cast<int64_t>(batch) * kv_heads * max_len;
  if (collect_rows == 0) return bound <= 160000;
  if (batch >= 8) return batch > 64 && max_len < (1 << 24);        // (beyond, too many of a sibling's chunks for a launch grid)
  if (token_sums) return bound <= (blocks != 3 ? 100000 : collect_rows == 2 ? 1 << 18 : (1 << 24) / head_dim);
  if (collect_rows == 1) return bound <= (blocks <= 3 ? 100000 : 50000);
  return blocks <= 3 && bound * head_dim <= (1 << 24);
}

// Chunk length of 64-row workgroups where the columns alone are as many as the compute units and no plan evens out the
// lengths (more than 64 sequences): whole sequences up to 8192 tokens and halves beyond, with more than 64 rows at most 4096
// tokens.  A chunk past its sequence's end still waits for a compute unit, so shorter ones cost a batch of similar lengths
// more than they save; a single long sequence runs on by itself.  us, whole / as chosen, 65 x 8 heads, 40 rows: 16384 each
// 1015 / 949; 2048..16384 620 / 624 (100 sequences 887 / 945); 64 of 512 and one of 65536 1000 / 554; 80 rows without
// collection: 2048..16384 692 / 743, 64 of 512 and one of 65536 807 / 275
inline int unplanned_pair_chunk(int rows, int max_len) {
  if (rows > 64) {
    const int chunk = max_len < (1 << 24) ? 4096 : max_len / 4096;   // (chunks are a dimension of the launch grid)
    return max_len < chunk ? max_len : chunk;
  }
  return max_len > 8192 ? (max_len + 1) / 2 : max_len;
}

// Units of streaming that beginning one more piece costs a compute unit: 0, 1, 2, 3 of them, verification with collection, us:
// 16 sequences of 4000..16000 tokens, 20 rows 132 / 124 / 131 / 123; 8 of 1001..20011 75.4 / 81.5 / 70.6 / 70.3.
constexpr uint32_t kShareCost = 3;
// Units that cutting a batch into shares has to win at least (least_shared_chunk), with 32-row and with 64-row workgroups.  Not where two
// 64-row workgroups fit a compute unit: two waves of equal chunks all start at once there, and what one leaves idle the others
// stream with.  Shares instead, head dimension 64, us: token sums, 48 rows, 24 sequences of 4000..40000 tokens 286 (equal chunks
// 273), 16 190 (183), 31 of 2000..20000 191 (185); 32 rows 28 of 4000..40000 308 (299); 12 of 1000..4000 33.0 (33.0); no collection, 64
// rows, 28 of 4000..40000 275 (270), 12 of 2000..20000 69.3 (70.1).
constexpr int kShareMargin = 2, kPairShareMargin = 4;

// May the lengths of a batch be such that it is cut into shares (least_shared_chunk), if none is longer than `most` units?  With C the
// longest equal chunk of a plan for J workgroups, chunks of C - 1 take more than J, so that the sequences have at least
// (J + 1) (C - 1) - batch (C - 2) units, and C is at most ceil(most / (ceil((J + 1) / batch) - 1)); C >= S + margin then asks for
// C (batch - 1) >= J (margin - 1) - 4 + 5 batch (kShareCost is 3).  Fewer sequences than `batch` ask for a longer C.  (Slots for
// shares that cannot be: 3 sequences of 900..1500 tokens, 20 rows 15.1 us instead of 13.3, 6 of them 16.5 / 14.9; with a bound of
// 32768 they can be for all the host knows, and 14.5 and 16.2 remain.)
inline bool shares_possible(int J, int batch, int64_t most, int margin) {
  const int64_t per = (static_cast<int64_t>(J) + batch) / batch;                     // ceil((J + 1) / batch)
  const int64_t C = per > 1 ? (most + per - 2) / (per - 1) : most;
  return batch >= 2 && C * (batch - 1) >= static_cast<int64_t>(J) * (margin - 1) - 4 + 5 * static_cast<int64_t>(batch);
}

// Does a planned batch's 32-row workgroup that parks nothing have a compute unit to itself?  Sharing one, the pieces of a plan by
// shares all start at once, on some units two, so a batch that may be cut into shares is run as that plan assumes, from a bound of
// 12 units per workgroup on (16 at head dimension 64); below, workgroups run side by side and there are no shares.  us, side by side /
// alone, verification without collection, 20 rows, by bound per workgroup: 4.7 16 sequences of 300..1200 tokens 18.1 / 18.8; 11 18 of
// 1000..2500 32.2 / 33.3; 12.7 20 of 2000..2600 44.8 / 43.8 (head dimension 64 29.4 / 31.7); 14.6 30 of 300..2000 40.9 / 39.5 (27.4 /
// 30.5); 117 24 of 1001..20011 210 / 189; 192 12 of 8192..65536 365 / 302.  With more sequences than workgroups there are no shares,
// and the host cannot tell a long batch from a short one under a loose bound: 48 of 300..3000 83 / 72, but 64 of 400..800 under a
// bound of 131072 46.2 / 52.6.
inline bool alone_on_compute_unit(int J, int batch, int max_len, int unit, int head_dim) {
  return batch <= J && static_cast<int64_t>(batch) * max_len >= static_cast<int64_t>(head_dim == 64 ? 16 : 12) * J * unit;
}

// A batch whose chunk lengths are computed on the GPU (balanced_slot, vegas_common.hpp): the numbers that the plan works with,
// per KV head (and row block), and what of them a launch holds.  units: of kTile tokens per wave.
struct BatchPlan {
  int J = 0;                   // workgroups of one launch wave: one per compute unit
  int J2 = 0;                  // of two waves of equal chunks (= J where only one is planned for)
  int JS = 0;                  // workgroups launched and partial slots held
  int cap_units = 0;           // longest chunk
  int share_margin = -1;       // what shares have to win (least_shared_chunk); -1: the batch is not cut into shares
  bool alone = false;          // a workgroup has a compute unit to itself, whatever LDS it needs
};
inline BatchPlan batch_plan(int num_cu, int64_t per_head, int batch, int max_len, int unit, int cap_units, bool pair,
                            bool two_per_cu, bool collects, int head_dim) {
  BatchPlan p;
  p.cap_units = cap_units;
  p.J = static_cast<int>(num_cu / per_head);
  // Slots no plan uses still cost a workgroup that works that out, so only those that can be used are launched: two waves
  // of equal chunks are planned for where there are more sequences than workgroups, where workgroups that park nothing
  // run side by side, or where the mean share may be longer than a workgroup can park: shares are out of the question then, and
  // one wave of the longest chunks would be followed by a few more of them (verification with collection, us, without / with
  // the second plan: 16 sequences of 8192..65536 tokens, 24 rows 492 / 437; 8 of 10000..100000, 32 rows 418 / 364; 9 of 51202,
  // 4 rows, token sums 435 / 334; head dimension 64: 20 of 40945, 24 rows 444 / 354).
  p.alone = !pair && !collects && alone_on_compute_unit(p.J, batch, max_len, unit, head_dim);
  if (pair ? !two_per_cu : collects || p.alone) p.share_margin = pair ? kPairShareMargin : kShareMargin;
  const int64_t most_units = (static_cast<int64_t>(max_len) + unit - 1) / unit;
  const bool beyond_cap = batch >= 8 && batch * most_units + kShareCost * (batch - 1) > static_cast<int64_t>(cap_units) * p.J;
  const bool two_waves = batch > p.J || (two_per_cu && batch >= 8) || (!pair && !collects && 2 * batch > p.J) || beyond_cap;
  p.J2 = two_waves ? 2 * p.J : p.J;
  const int64_t capped = (most_units + cap_units - 1) / cap_units;
  // slots: a plan for J2 workgroups never takes more than max(J2, B) of them; a capped one B times the most of a sequence; J
  // shares one each and one more where a sequence ends inside a share (there are at most as many sequences as shares)
  int64_t js = p.J2 > batch ? p.J2 : batch;
  const int64_t shared = p.J + (batch < p.J ? batch : p.J) - 1;
  if (shared > js && p.share_margin >= 0 && shares_possible(p.J, batch, most_units, p.share_margin)) js = shared;
  if (batch * capped > js) js = batch * capped;
  p.JS = static_cast<int>(js);
  return p;
}

// Merge and page scores of a planned batch (attn_finalize.hpp): does one head dim per thread leave fewer than four workgroups per
// compute unit?  Then nothing waits for a workgroup to end, and that form, which requests all of a row's chunks at once, is
// the faster one.  us per verification, one head dim and page by page / four and by quads, by workgroups of the former, 20 rows:
// 160 12.8 / 13.3 (token sums 13.5 / 14.4), 320 13.8 / 14.1, 480 16.3 / 16.5, 960 19.2 / 19.4, 1280 21.1 / 20.9, 1920 25.4 / 24.4;
// 40 rows: 320 17.3 / 17.6, 960 21.9 / 21.9, 1920 25.1 / 24.3, 2560 27.8 / 25.9; head dimension 64: 160 11.7 / 12.1, 960 20.4 / 20.6,
// 1920 35.7 / 34.7; one KV head, 80 12.1 / 13.3.
inline bool planned_merge_is_small(int batch, int rows, int head_dim) {
  return static_cast<int64_t>(batch) * rows * head_dim < 1024 * 256;
}

// Merge and page scores of chunks that the host cuts (one sequence, more than 64, or a caller's chunk length): does a wave of a score
// workgroup have the (max, sum) pairs of five rounds of 64 rows in flight instead of three?  Three hold 192 rows; more are a second
// round trip, unless five hold them.  They are registers, which the merge workgroups of the same launch have as well: where a batch fills
// the chip that costs more.  us for merge and scores, captured, three / five, head dimension 128, 32 chunks or fewer: one sequence, 192 rows 4.3 / 4.7
// (4096 tokens), 196 7.2 / 7.1, 208 5.0 / 4.9, 256 5.4 / 5.2, 320 5.5 / 5.3, 384 5.6 / 6.5, 512 7.1 / 7.5; two, 256 5.0 / 4.8; four, 208 4.6 / 4.5, 320
// 5.5 / 5.4, in chunks of 512 5.4 / 5.1; eight, 224 5.4 / 5.1, 256 5.8 / 6.0, 320 6.3 / 6.6; 16, 256 7.5 / 7.7; 32 10.8 / 11.3; 65, 196 19.5 / 20.4, 320
// 22.1 / 23.4; 128, 256 31.3 / 33.5; but in 17 to 32 chunks, a round trip of twice as many requests, 65, 256 49.5 / 47.7, 320 62.5 / 61.0, 280 at head
// dimension 64 34.3 / 33.2.  96 chunks, one, 256 10.1 / 10.1, 320 10.5 / 10.6; 33 to 64 have three in any case (five are more registers than
// there are): 224 rows, 48 7.3, 64 7.2.
inline bool finalize_is_wide(int rows, int batch, int chunks) { return rows > 192 && rows <= 320 && chunks <= 32 && (batch <= 4 || chunks > 16); }

// Workgroups go round the 8 XCDs, on each round its 4 shader engines, so every 32nd starts on the same engine: of the
// consecutive ones of a head, whose grid has `per_slot` workgroups (KV heads x row blocks) between them, so many start on as
// many engines.
inline int share_group(int per_slot) {
  int group = 32;
  for (int step = per_slot; step % 2 == 0 && group > 1; step /= 2) group /= 2;
  return group;
}

}  // namespace vegas
