// Draft-attention streaming kernel for up to 16 query rows per KV head (one draft token, GQA groups of up to 16
// heads), gfx950; 16-token pages, or the 1, 2, 4, 8-token pages of Sec. 4 / App. D through a template argument.
//
// Same arithmetic, chunking, partial-result layout and merge kernels as attn_split_kernel (Eq. 1 over the selected
// pages of Sec. 3.2, split over the selection), but shaped for a call that is a few microseconds long and whose
// waves are bound by what they have to issue: a draft call stacks g (typically 4 or 8) rows on a KV head, so a
// 32-row MFMA tile is seven eighths padding, and the time goes into instructions around the contractions.
//   * 16x16x32 bf16 MFMAs: S^T = K Q^T per page (M = the page's 16 tokens, N = 16 query rows, K = 32 head dims per
//     instruction) and O^T += V^T P^T per 16 head dims (M = head dims, N = rows, K = the tile's 32 tokens): half the
//     matrix-core time of the 32-row tile, 8 logits and 32 (D = 128) accumulators per lane instead of 16 and 64.
//   * K needs no LDS: lane (token i, dim group kg) loads the 16 bytes K[i][32 kk + 8 kg ..] straight into the A
//     operand's register layout (four lanes read 64 consecutive bytes of a token row).
//   * Q needs no LDS and no barrier: lane (row n, kg) loads Q[n][32 kk + 8 kg ..] into the B operand's layout once (lanes of rows
//     past the group's heads the last row again).
//   * The softmax weights leave the first MFMA as P[token 4 kg + r of page pg][row n] in lane (n, kg): taking the
//     second contraction's index as k = 8 kg + e <-> (page e / 4, token 4 kg + e % 4) makes {P of page 0, P of page 1}
//     the B operand as it stands, and V is loaded to match: lane (m, kg) reads 16 bytes (D / 16 head dims from
//     (D / 16) m on) of those eight tokens; one byte-permute per register pair builds each A operand, and output
//     block blk then holds head dims (D / 16) m' + blk.
//   * A row's running maximum is shared by the four lanes (n, 0..3): two lane-swap instructions per reduction.
// Loads run one tile ahead as in attn_split_kernel (K back into its registers once the first contraction has
// consumed them, V into a second register set); the four waves merge through LDS and write one partial, or the
// finished bf16 rows when the workgroup's chunk is the whole selection.
#pragma once
#include <type_traits>

#include "attn_split.hpp"
#include "vegas_common.hpp"

namespace vegas {

// Reductions over the four lanes l % 16 + {0, 16, 32, 48}; every lane gets the result.
__device__ __forceinline__ float quad_rows_max(float x) {
  const auto r = __builtin_amdgcn_permlane16_swap(__float_as_uint(x), __float_as_uint(x), false, false);
  return half_max(fmaxf(__uint_as_float(r[0]), __uint_as_float(r[1])));
}
__device__ __forceinline__ float quad_rows_sum(float x) {
  const auto r = __builtin_amdgcn_permlane16_swap(__float_as_uint(x), __float_as_uint(x), false, false);
  return half_sum(__uint_as_float(r[0]) + __uint_as_float(r[1]));
}

// Tokens of a call's selections, in sixteens, rounded up for each: lane `lane`'s share of them; own: the length of sequence
// `lane`, if there is one.  (At most 2^25 a lane, far beyond what past_cache asks about.)
__host__ __device__ __forceinline__ uint32_t lane_sixteens(int own, const int32_t* lens, int batch, int max_tokens, int lane) {
  auto sixteens = [=](int n) { return static_cast<uint32_t>((n < 0 ? 0 : (n > max_tokens ? max_tokens : n)) + 15) >> 4; };
  uint32_t sum = lane < batch ? sixteens(own) : 0u;
  for (int first = 64; first < batch; first += 64) {
    if (first + lane < batch) sum += sixteens(lens[first + lane]);
    sum = sum < (1u << 25) ? sum : 1u << 25;
  }
  return sum;
}

// Are the selected K and V (sixteens: of tokens, of all sequences) more than the 256-MiB
// last-level cache keeps until the next draft step reads the same pages?  Then they are read past it.  us, 8 draft calls of the
// same selection in turn, through the cache / past it: 104 MB 18.8 / 22.7; 136 MB 28.4 / 33.0; 268 MB 45.5 / 49.4 (head
// dimension 64 51.9 / 56.7); 302 MB 53.3 / 55.8; 336 MB 60.9 / 60.9, with 16-token pages 58.0 / 59.3; 369 MB 66.6 / 64.4;
// 393 MB 74.1 / 68.1; 403 MB 76.6 / 71.4; 537 MB 106.7 / 95.0 (head dimension 64 117.7 / 106.2).  The rule takes the next reader
// of the pages to be the same layer's next step.  Where the steps of other layers come between, nothing is found in the
// cache at smaller sizes too, and reading past it would pay there as well (a first call on a selection, 537 MB: 179 -> 142).
__host__ __device__ __forceinline__ bool past_cache(uint64_t sixteens, int kv_heads, int head_dim) {
  return sixteens * 16u * static_cast<uint64_t>(kv_heads) * static_cast<uint64_t>(head_dim) * 4u >= static_cast<uint64_t>(352) << 20;
}

constexpr int kDraftWaves = 4;
constexpr int kDraftRows = 16;     // query rows (of one KV head) a workgroup can take

constexpr int kDraftRing = 32 * 1024;          // bytes of a wave's ring
static_assert(kDraftRing >= kDraftRows * red_pitch(128) * 4, "a wave's rows fit its ring");
// Dynamic LDS of attn_draft16_kernel with rings; the merge's rows alias them.
constexpr size_t draft_ring_lds_bytes() { return kDraftWaves * kDraftRing + 2 * kDraftWaves * kDraftRows * sizeof(float); }
// Dynamic LDS of attn_draft16_kernel for R (<= 16) rows: the waves' rows for the merge, their row maxima and sums.
inline size_t draft16_lds_bytes(int R, int D) {
  return static_cast<size_t>(kDraftWaves) * R * red_pitch(D) * sizeof(float) +
         2 * static_cast<size_t>(kDraftWaves) * kDraftRows * sizeof(float);
}

// PS: log2 of the tokens per page of the selection table (4: 16-token pages; 0..3: the 1, 2, 4, 8-token pages of
// Sec. 4 / App. D).  With small pages a tile spans 32 >> PS pages: their ids are loaded one tile ahead into one
// register (lane e <-> page e of the tile), every lane fetches the id of each of its tokens with a lane permute and
// forms a 64-bit address of its own; everything after the loads is the 16-token code.
// CHOOSE: calls whose bound allows selections that the last-level cache cannot hold until the next draft step reads them
// again.  Whether they are that long the lengths say (past_cache); if so, K and V are read with the non-temporal hint, K in
// whole 128-byte lines (half lines would fetch each of them twice then): 16 x 8192 tokens, one-token pages 106.7 -> 95.0 us
// (5.7 TB/s), 16-token pages 102.9 -> 92.4; 32 x 3000, two-token pages 74.1 -> 68.1.  A plain read of the same addresses takes 96
// us without the hint and 86 with it: what bounds the kernel then is HBM.  Whole lines alone change nothing.
// (The choice costs up to 1 us: 8 x 2048 tokens under a bound of 16384 43.6 -> 44.5, 16 x 200..8192 59.9 -> 60.5; taking the bound for
// the length cost 55.5 and 66.5.)
// Step: DraftStep in a draft step of a live drafting phase (16-token pages).  The new token's rows come from k_new and v_new instead of the
// cache: the wave that has the selection's last tile puts them in place of what it read there, so no launch has to go before this
// one, and the first workgroup of every KV head writes them into the cache for later calls.  Every workgroup works out for itself,
// from the lengths before the step, whether the sequence has room and how long the selection is; the lengths are stored by the
// merge, which reads copies of them.  (Figures: vegas_draft_step.)
// RING: K and V land in LDS, in a ring of two tiles per wave, instead of in registers: both are on their way from the start, where the
// registers hold one and the next is asked for when the first contraction has used its K.  One workgroup to a compute unit, so what
// bounds it is how much that unit has under way; the rule and its figures: ring_draft.
// DV: head dims of V that the workgroup reads and of the output rows that it writes: D, or a part of it in calls that one workgroup per
// column could finish (draft_value_parts, part_grid_width).
template <int D, int PS, bool CHOOSE, bool RING, int DV, typename... Step>
__device__ __forceinline__ void draft16(SplitParams& p, const Step&... step) {
  VEGAS_TL_DECL;
  VEGAS_TL(kTlEntry);
  static_assert(D == 128 || D == 64, "head dimension");
  extern __shared__ __attribute__((aligned(16))) unsigned char smem[];
  constexpr bool APPEND = sizeof...(Step) == 1;
  static_assert(!APPEND || (PS == 4 && !CHOOSE && !RING), "draft steps: 16-token pages through the cache");
  static_assert(DV == D || (!APPEND && !CHOOSE && (DV == 32 || (DV == 64 && D == 128))), "parts of V: 32 or 64 head dims, calls without a merge");
  static_assert(!RING || (PS == 4 && !CHOOSE && D == 128), "rings: 16-token pages through the cache, head dimension 128");
  constexpr int NW = kDraftWaves;
  constexpr int KK = D / 32;                 // steps of the first contraction = K loads per page
  constexpr int NBLK = DV / 16;              // 16-wide blocks of the output = head dims one V load covers
  constexpr int kRedPitch = red_pitch(DV);
  typedef unsigned int u32x1 __attribute__((ext_vector_type(1)));
  using VReg = typename std::conditional<NBLK == 8, u32x4, typename std::conditional<NBLK == 4, u32x2, u32x1>::type>::type;   // NBLK head dims of one token
  constexpr int TP = 32 >> (PS < 4 ? PS : 0);   // pages per tile on the small-page path
  const int tid = threadIdx.x;
  const int lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int half = lane >> 5;
  const int l32 = lane & 31;
  const int l16 = lane & 15;                 // token of a page (K), query row (Q, S^T, O^T), head-dim group (V)
  const int kg = lane >> 4;                  // which 8 of a contraction step's 32 indices
  int h = blockIdx.x, b = blockIdx.z;        // grid (KV head, chunk, sequence), or part_grid_width's
  const int split = DV == D ? blockIdx.y : 0;
  const int part = DV == D ? 0 : blockIdx.y;  // which DV head dims of V
  if constexpr (DV != D) {
    if (p.Hkv % kXcds != 0) {
      const uint32_t column = static_cast<uint32_t>(h + kXcds * b);
      if (column >= round_columns(p.row_blocks)) return;
      b = static_cast<int>(round_sequence(p.row_blocks, column));
      h = static_cast<int>(column) - b * p.Hkv;
    }
  }
  const int Rl = p.R;                        // rows of this KV head: one draft token, g heads (G = 1)

  int last_page = 0;                         // (set below, from arguments that are not there yet)
  // Physical page ids of the wave's next 32 tiles in one register, lane (k, half) <-> page `half` of tile
  // tile_first + k NW, requested before the length is known (see attn_split_kernel).
  const int32_t* table = p.table + static_cast<int64_t>(b) * p.table_stride;
  const int c0 = split * p.chunk_tokens;
  const int tile_first = c0 / kTile + wave;
  int pagevec = 0;
  auto table_entry = [&](int kbase) -> int {
    int page = 2 * (tile_first + (kbase + l32) * NW) + half;
    page = page < p.table_stride ? page : p.table_stride - 1;
    return table[page];
  };
  auto into_pool = [&](int raw) -> int { return min(max(raw, 0), last_page); };
  auto load_pagevec = [&](int kbase) { pagevec = into_pool(table_entry(kbase)); };
  // Small pages: ids of the TP pages of this wave's tile k, lane e (mod TP) <-> page e of the tile.
  auto ids_entry = [&](int k) -> int {
    int page = (tile_first + k * NW) * TP + (lane & (TP - 1));
    page = page < p.table_stride ? page : p.table_stride - 1;
    return table[page];
  };

  // ---- one round trip for everything the preloaded arguments can address: table entry, length, query rows; the
  //      rest of the argument block is pulled in one go meanwhile (see attn_split_kernel).  No wave has another beside it here, so
  //      every instruction before a request or after its arrival is time: no integer division (the group size is an argument),
  //      no masked query loads, addresses ready but for the page id.  With the merge kernel's the same, one sequence of 32768
  //      tokens 70.4 -> 69.0 us an iteration, 131072 157.2 -> 154.2.
  int first_entry = PS == 4 ? table_entry(0) : ids_entry(0);
  int zero = 0;
  asm("" : "+v"(zero));                      // (a vector load: a scalar one would wait in line behind the argument block's)
  int n = p.lens[b + zero];
  int n_seq = 0;                             // the sequence's length (APPEND: its address takes the plan's place)
  if constexpr (APPEND) n_seq = reinterpret_cast<const int32_t*>(p.plan)[b + zero];
  u32x4 qreg[KK];
  {
    const unsigned char* qbase = uniform_ptr(reinterpret_cast<const unsigned char*>(
        p.q + (static_cast<int64_t>(b) * p.Hq + h * p.g) * D));
#pragma unroll
    for (int kk = 0; kk < KK; ++kk) {
      // (rows past the group's heads: copies of the last one, which nobody reads)
      qreg[kk] = gload<u32x4, false>(qbase, static_cast<uint32_t>(min(l16, Rl - 1) * D + 32 * kk + 8 * kg) * 2u);
    }
  }
  int lane_len = 0;                          // length of sequence `lane` (the last one's beyond), used once the chunk is known to be live
  if constexpr (CHOOSE) lane_len = p.lens[min(lane, p.batch - 1)];
  asm volatile("" : "+s"(p.k), "+s"(p.v), "+s"(p.page_stride), "+s"(p.token_stride), "+s"(p.head_stride), "+s"(p.num_pages),
               "+s"(p.out_direct), "+s"(p.max_tokens), "+s"(p.nsplit), "+s"(p.scale_log2e), "+s"(p.part_o), "+s"(p.part_ml));
  last_page = static_cast<int>(p.num_pages < INT32_MAX ? p.num_pages - 1 : INT32_MAX);     // (an id is an int32)
  // What the first loads' addresses take besides page ids is worked out while those are on their way.
  const int64_t head_off = static_cast<int64_t>(h) * p.head_stride;
  const unsigned char* k_head = reinterpret_cast<const unsigned char*>(p.k + head_off);
  const unsigned char* v_head = reinterpret_cast<const unsigned char*>(p.v + head_off + part * DV);
  uint64_t page_bytes = static_cast<uint64_t>(p.page_stride) * 2u;
  const uint32_t ts_bytes = static_cast<uint32_t>(p.token_stride) * 2u;
  uint32_t k_cached_off = static_cast<uint32_t>(l16) * ts_bytes + static_cast<uint32_t>(kg) * 16u;
  uint32_t v_lane_off = static_cast<uint32_t>(4 * kg) * ts_bytes + static_cast<uint32_t>(l16) * (2u * NBLK);
  asm volatile("" : "+v"(k_cached_off), "+v"(v_lane_off), "+s"(k_head), "+s"(v_head), "+s"(page_bytes), "+s"(last_page));
  asm volatile("" : "+v"(first_entry), "+v"(n));
  n = __builtin_amdgcn_readfirstlane(n);
  if constexpr (APPEND) n_seq = __builtin_amdgcn_readfirstlane(n_seq);
  float* red = reinterpret_cast<float*>(smem);                     // [wave][row][D] (padded rows)
  float* sm_m = RING ? reinterpret_cast<float*>(smem + NW * kDraftRing) : red + NW * Rl * kRedPitch;   // [wave][16] row maxima
  float* sm_l = sm_m + NW * kDraftRows;                            // [wave][16] row sums
  const int64_t pbase = (static_cast<int64_t>(b) * p.Hkv + h) * p.nsplit + split;   // this workgroup's partial slot
  // (when the workgroup finishes the rows itself: G = 1, so the group's rows are consecutive)
  auto out_rows = [&]() -> uint16_t* { return p.out_direct + (static_cast<int64_t>(b) * p.Hq + h * p.g) * D; };
  int ids_cur = 0, ids_pending = 0;          // small pages: ids of the tile whose loads go out next; of the one after
  if constexpr (PS == 4) pagevec = into_pool(first_entry);
  else ids_cur = into_pool(first_entry);

  // ---- APPEND: room and growth as append_kv_kernel and extend_selection_row decide them
  const int covered = n;
  bool grows = false;
  bool appends = false;                      // this thread moves 16 bytes of the new rows into the cache
  int new_page = 0;
  u32x4 new_piece = {0u, 0u, 0u, 0u};
  constexpr int kPieces = D / 8;             // 16-byte pieces of a row
  if constexpr (APPEND) {
    const bool room = n_seq >= 0 && n_seq < the_one(step...).cap;
    grows = room && covered > 0 && (covered - 1) / kPage + 1 + (n_seq % kPage == 0 ? 1 : 0) <= p.table_stride;
    appends = room && split == 0 && tid < 2 * kPieces;
    if (appends) {
      new_page = the_one(step...).block_table[static_cast<int64_t>(b) * the_one(step...).max_blocks + n_seq / kPage];
      const uint16_t* const rows = tid < kPieces ? the_one(step...).k_new : the_one(step...).v_new;
      new_piece = *reinterpret_cast<const u32x4*>(rows + (static_cast<int64_t>(b) * p.Hkv + h) * D + tid % kPieces * 8);
    }
  }
  auto append_row = [&]() {
    if constexpr (APPEND) {
      if (appends) {
        uint16_t* const cache = const_cast<uint16_t*>(tid < kPieces ? p.k : p.v);
        *reinterpret_cast<u32x4*>(cache + static_cast<int64_t>(into_pool(new_page)) * p.page_stride +
                                  static_cast<int64_t>(n_seq % kPage) * p.token_stride + static_cast<int64_t>(h) * p.head_stride +
                                  tid % kPieces * 8) = new_piece;
      }
      if ((h | split | tid) == 0) {
        const int after = covered + (grows ? 1 : 0);
        if (grows && n_seq % kPage == 0) the_one(step...).sel_table[static_cast<int64_t>(b) * p.table_stride + (covered - 1) / kPage + 1] = new_page;
        the_one(step...).grown[b] = make_int2(appends ? n_seq + 1 : n_seq, after);
        the_one(step...).sel_lens[b] = after;
      }
    }
  };
  if constexpr (APPEND) n += grows ? 1 : 0;
  n = n < 0 ? 0 : (n > p.max_tokens ? p.max_tokens : n);
  if (__builtin_expect(c0 >= n, 0)) {        // nothing to do, no partial is read
    append_row();
    if (p.out_direct != nullptr) {           // no merge kernel follows: the rows of an empty sequence are zeros
      uint16_t* rows = out_rows();
      if constexpr (DV == D) {
        for (int e = tid; e < Rl * D; e += NW * 64) rows[e] = 0;
      } else {
        for (int e = tid; e < Rl * DV; e += NW * 64) rows[e / DV * D + part * DV + e % DV] = 0;
      }
    }
    // (The stores are waited for here.  The compiler lets this way out run into the stream below and counts stores and loads in one
    //  counter without an order between the two kinds: as long as a store may be under way it waits for everything where it wants the
    //  oldest load, the next tile's page ids.)
    __builtin_amdgcn_s_waitcnt(0x0f70);      // vmcnt(0)
    return;
  }
  VEGAS_TL(kTlLength);
  const int c1 = min(c0 + p.chunk_tokens, n);
  const int tile_end = (c1 + kTile - 1) / kTile;

  auto stream_chunk = [&](auto streamed) __attribute__((always_inline)) {
    constexpr bool STREAM = decltype(streamed)::value;
    // K: token and byte of its row this lane fetches with load (pg, kk) before the lane exchange (see exchange_k)
    const int k_tok = STREAM ? l16 & 7 : l16;
    const uint32_t k_byte = static_cast<uint32_t>(kg) * 16u + (STREAM ? static_cast<uint32_t>(l16 >> 3) * 64u : 0u);
    const uint32_t k_lane_off = STREAM ? static_cast<uint32_t>(k_tok) * ts_bytes + k_byte : k_cached_off;
    auto page_base = [&](const unsigned char* head, int ph) -> const unsigned char* {
      return uniform_ptr(head + static_cast<uint64_t>(static_cast<uint32_t>(ph)) * page_bytes);
    };
    // Small pages: byte address of token t (0..31, a per-lane value) of the tile whose page ids are in ids_cur.
    typedef const __attribute__((address_space(1))) unsigned char* gbytes;
    auto token_addr = [&](const uint16_t* cache, int t) -> gbytes {
      const int id = __shfl(ids_cur, t >> (PS & 3), 64);
      const int tokin = t & ((1 << (PS & 3)) - 1);
      const int64_t el = static_cast<int64_t>(id) * p.page_stride + static_cast<int64_t>(tokin) * p.token_stride + head_off;
      return (gbytes)cache + el * 2;
    };
    // K load (pg, kk): token l16 of page pg, head dims 32 kk + 8 kg .. + 7
    auto issue_k = [&](int k, u32x4 (&kr)[2][KK]) {
      if constexpr (PS != 4) {
#pragma unroll
        for (int pg = 0; pg < 2; ++pg) {
          if constexpr (STREAM) {
#pragma unroll
            for (int e = 0; e < 2; ++e) {
              const gbytes row = token_addr(p.k, 16 * pg + 8 * e + k_tok) + k_byte;
#pragma unroll
              for (int kk = e; kk < KK; kk += 2) kr[pg][kk] = gload_at<u32x4, STREAM>(row + (kk >> 1) * 128);
            }
          } else {
            const gbytes row = token_addr(p.k, 16 * pg + l16) + kg * 16;
#pragma unroll
            for (int kk = 0; kk < KK; ++kk) kr[pg][kk] = gload_at<u32x4, STREAM>(row + kk * 64);
          }
        }
        return;
      }
      if ((k & 31) == 0 && k > 0) load_pagevec(k);
      const unsigned char* kb0 = page_base(k_head, __builtin_amdgcn_readlane(pagevec, k & 31));
      const unsigned char* kb1 = page_base(k_head, __builtin_amdgcn_readlane(pagevec, 32 + (k & 31)));
#pragma unroll
      for (int pg = 0; pg < 2; ++pg)
#pragma unroll
        for (int kk = 0; kk < KK; ++kk)
          kr[pg][kk] = gload<u32x4, STREAM>((pg ? kb1 : kb0) + (STREAM ? (kk >> 1) * 128u + (kk & 1) * 8u * ts_bytes : kk * 64u), k_lane_off);
    };
    // V load e: token 4 kg + e % 4 of page e / 4, head dims NBLK l16 .. + NBLK - 1
    auto issue_v = [&](int k, VReg (&vr)[8]) {
      if constexpr (PS != 4) {
#pragma unroll
        for (int e = 0; e < 8; ++e) vr[e] = gload_at<VReg, STREAM>(token_addr(p.v, 16 * (e >> 2) + 4 * kg + (e & 3)) + (part * 2 * DV + l16 * (2 * NBLK)));
        return;
      }
      const unsigned char* vb0 = page_base(v_head, __builtin_amdgcn_readlane(pagevec, k & 31));
      const unsigned char* vb1 = page_base(v_head, __builtin_amdgcn_readlane(pagevec, 32 + (k & 31)));
#pragma unroll
      for (int e = 0; e < 8; ++e)
        vr[e] = gload<VReg, STREAM>((e < 4 ? vb0 : vb1) + static_cast<uint32_t>(e & 3) * ts_bytes, v_lane_off);
    };

    // Loads of whole 128-byte lines bring two tokens' pieces to the wrong lanes: of loads 2 q and 2 q + 1 the first holds, in
    // lanes l16 < 8, the first half of line q of token l16 and, in the others, the second half of token l16 - 8's; the second
    // load the same of tokens l16 + 8 and l16.  Lanes 8 apart exchange them.
    auto exchange_k = [&](u32x4 (&kr)[2][KK]) {
#pragma unroll
      for (int pg = 0; pg < 2; ++pg)
#pragma unroll
        for (int q = 0; q < KK / 2; ++q)
#pragma unroll
          for (int w = 0; w < 4; ++w) {
            const int a = static_cast<int>(kr[pg][2 * q][w]), b = static_cast<int>(kr[pg][2 * q + 1][w]);
            kr[pg][2 * q][w] = static_cast<unsigned>(__builtin_amdgcn_update_dpp(a, b, 0x128, 0xf, 0xc, false));       // row_ror:8
            kr[pg][2 * q + 1][w] = static_cast<unsigned>(__builtin_amdgcn_update_dpp(b, a, 0x128, 0xf, 0x3, false));
          }
    };

    // APPEND: the new token's rows in the layout of the loads, where the chunk holds the selection's end
    u32x4 k_row[APPEND ? KK : 1];
    VReg v_row = {};
    const bool has_new = APPEND && grows && c1 == n && n == covered + 1;       // (not where max_tokens ends the selection before it)
    if constexpr (APPEND) {
      if (has_new) {
        const int64_t row = (static_cast<int64_t>(b) * p.Hkv + h) * D;
        const unsigned char* const k_at = uniform_ptr(reinterpret_cast<const unsigned char*>(the_one(step...).k_new + row));
        const unsigned char* const v_at = uniform_ptr(reinterpret_cast<const unsigned char*>(the_one(step...).v_new + row));
#pragma unroll
        for (int kk = 0; kk < KK; ++kk) k_row[kk] = gload<u32x4, false>(k_at, static_cast<uint32_t>(64 * kk + 16 * kg));
        v_row = gload<VReg, false>(v_at, static_cast<uint32_t>(l16) * (2u * NBLK));
      }
    }
    // RING: 16-byte piece c of K row t sits at c ^ (t mod 16), V rows stay whole: reads without bank conflicts (attn_pair.hpp).
    constexpr int TPI = 64 / (D / 8);          // token rows of one load instruction
    constexpr int NP = kPage / TPI;            // load instructions per page (of K, of V)
    constexpr int NL = 2 * NP;                 // ... per tile
    constexpr int VPI = 64 / (DV / 8), NPV = kPage / VPI, NLV = 2 * NPV;       // the same of V
    constexpr int kRow = 2 * D, kVRow = 2 * DV, kHalfSlot = kTile * kRow, kSlot = kTile * (kRow + kVRow);
    constexpr int NS = 2;                      // tiles the ring holds
    static_assert(!RING || NS * kSlot <= kDraftRing, "the ring's tiles");
    unsigned char* const ring = smem + wave * kDraftRing;
    uint32_t ring_lds = 0, koff[NP] = {}, voff[NPV] = {};
    if constexpr (RING) {
      typedef const __attribute__((address_space(3))) unsigned char* lptr;
      ring_lds = __builtin_amdgcn_readfirstlane(static_cast<uint32_t>(reinterpret_cast<uintptr_t>((lptr)ring)));
#pragma unroll
      for (int i = 0; i < NP; ++i) {
        const int row = TPI * i + lane / (D / 8), piece = lane % (D / 8);     // where the 16 bytes land
        koff[i] = static_cast<uint32_t>(row) * ts_bytes + static_cast<uint32_t>(piece ^ row) * 16u;
      }
#pragma unroll
      for (int i = 0; i < NPV; ++i)
        voff[i] = static_cast<uint32_t>(VPI * i + lane / (DV / 8)) * ts_bytes + static_cast<uint32_t>(lane % (DV / 8)) * 16u;
#pragma unroll
      for (int kk = 0; kk < KK; ++kk) asm volatile("" : "+v"(qreg[kk]));      // (waited for before loads that the compiler does not count)
    }
    auto ring_k = [&](int k) {
      if ((k & 31) == 0 && k > 0) load_pagevec(k);
      const uint32_t at = ring_lds + static_cast<uint32_t>((k & (NS - 1)) * kSlot);
      load_to_lds<NP, false>(at, page_base(k_head, __builtin_amdgcn_readlane(pagevec, k & 31)), koff);
      load_to_lds<NP, false>(at + kHalfSlot / 2, page_base(k_head, __builtin_amdgcn_readlane(pagevec, 32 + (k & 31))), koff);
    };
    auto ring_v = [&](int k) {
      const uint32_t at = ring_lds + static_cast<uint32_t>((k & (NS - 1)) * kSlot + kHalfSlot);
      load_to_lds<NPV, false>(at, page_base(v_head, __builtin_amdgcn_readlane(pagevec, k & 31)), voff);
      load_to_lds<NPV, false>(at + kPage * kVRow, page_base(v_head, __builtin_amdgcn_readlane(pagevec, 32 + (k & 31))), voff);
    };
    const uint32_t k_first = static_cast<uint32_t>(l16 * kRow + ((kg ^ l16) * 16));
    // For tile k's K or V: what has been requested after it.  With a tile to follow behind the ring's, the other tile's K and V and
    // either its own V or the K that has just been asked for; in the ring's last tiles what is left of that.
    auto wait_k = [&](bool last) {
      if (last) wait_vm<NLV>();
      else wait_vm<NLV + NL + NLV>();
    };
    auto wait_v = [&](bool last) {
      if (last) wait_vm<0>();
      else wait_vm<NL + NLV>();
    };
    const int ntiles = tile_first < tile_end ? (tile_end - tile_first + NW - 1) / NW : 0;      // this wave's tiles
    u32x4 kr[2][KK];
    VReg va[8], vb[8];
    // (Brought into the pool when they are used: a wave of one tile never waits for them.  With that and the wait above, us a call in
    //  one-token pages, captured, before / after: 8 columns x 64 tokens 3.71 / 3.39, x 2048 6.37 / 6.06; 24 x 600 6.28 / 5.96; 2-token ones, 64 x
    //  120 4.32 / 4.03; head dimension 64, 8 x 2048 5.58 / 5.38; calls of many tiles per wave the same, 128 x 2000 23.7 / 23.55.)
    if constexpr (PS != 4) ids_pending = ids_entry(1);                // (requested before tile 0's loads: it is back first)
    if constexpr (RING) {
#pragma unroll
      for (int k = 0; k < NS; ++k) {
        if (k < ntiles) {
          ring_k(k);
          ring_v(k);
        }
      }
    } else if (PS == 4 && D == 128 ? tile_first < tile_end : ntiles > 0) {
      // (The stream below is under ntiles > 0.  Under the same condition the compiler sees that a wave that streams has these loads under
      //  way; under another it waits for all of a wave's loads in every second tile.  us a call, other condition / same, captured: one-token
      //  pages, 96 columns x 692 tokens 10.99 / 9.95, 128 x 840 13.0 / 12.2; 8-token ones, 8 x 393 7.14 / 6.70; 16-token ones at head dimension 64,
      //  128 x 1474 11.59 / 11.34, 192 x 5828 74.2 / 73.5.  At head dimension 128 16-token pages have the same waits either way and a better
      //  order of instructions under the other: 64 x 1246 12.36 / 12.68, 32 x 2427 12.42 / 12.78.)
      issue_k(0, kr);
      // (A part of V is few loads, which the compiler moves between K's halves; the stream's waits for K's second half, which have to hold for
      //  this order too, then waited for the V of every tile: us without / with this, two parts, 128 columns, 120 tokens: one-token pages
      //  4.03 / 3.86, 8-token ones 4.09 / 3.88.)
      if constexpr (D == 128 && DV < D) __builtin_amdgcn_sched_barrier(0);
      issue_v(0, va);
    }
    VEGAS_TL(kTlLoadsIssued);
    VEGAS_TL(kTlQueries);

    // ---- running state of lane (row n, kg): the row maximum (the same in the row's four lanes), this lane's share
    //      of the row sum, and acc[blk][r] = O[n][NBLK (4 kg + r) + blk]
    float m_run = -INFINITY, l_run = 0.f;
    f32x4 acc[NBLK];
#pragma unroll
    for (int blk = 0; blk < NBLK; ++blk) acc[blk] = f32x4{0.f, 0.f, 0.f, 0.f};

    auto step = [&](int k, VReg (&vcur)[8], VReg (&vnxt)[8], auto has_next_tag) {
      constexpr bool has_next = decltype(has_next_tag)::value;
      const int tok0 = (tile_first + k * NW) * kTile;
      if constexpr (STREAM) exchange_k(kr);
      const unsigned char* const kt = ring + (k & (NS - 1)) * kSlot;
      const unsigned char* const vt = kt + kHalfSlot;
      if constexpr (RING) {
        wait_k(!has_next && k + 1 == ntiles);
#pragma unroll
        for (int pg = 0; pg < 2; ++pg)
#pragma unroll
          for (int kk = 0; kk < KK; ++kk)
            kr[pg][kk] = *reinterpret_cast<const u32x4*>(kt + pg * (kPage * kRow) + (k_first ^ static_cast<uint32_t>(64 * kk)));
      }
      if constexpr (APPEND) {
        if (has_new && tok0 + kTile >= n) {    // the tile of the selection's last token, the new one
#pragma unroll
          for (int pg = 0; pg < 2; ++pg) {
            if (tok0 + 16 * pg + l16 != n - 1) continue;
#pragma unroll
            for (int kk = 0; kk < KK; ++kk) kr[pg][kk] = k_row[kk];
          }
#pragma unroll
          for (int e = 0; e < 8; ++e)
            if (tok0 + 16 * (e >> 2) + 4 * kg + (e & 3) == n - 1) vcur[e] = v_row;
        }
      }
      f32x4 st[2] = {f32x4{0.f, 0.f, 0.f, 0.f}, f32x4{0.f, 0.f, 0.f, 0.f}};     // st[pg][r]: token 4 kg + r of page pg, row l16
#pragma unroll
      for (int kk = 0; kk < KK; ++kk)
#pragma unroll
        for (int pg = 0; pg < 2; ++pg)
          st[pg] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8, kr[pg][kk]),
                                                           __builtin_bit_cast(bf16x8, qreg[kk]), st[pg], 0, 0, 0);
      if (has_next) {
        if constexpr (PS != 4) {               // the next tile's ids are here (requested a tile ago); ask for the ones after
          ids_cur = into_pool(ids_pending);
          ids_pending = ids_entry(k + 2);
        }
        if constexpr (RING) {
          wait_lds();
          ring_k(k + NS);
        } else {
          issue_k(k + 1, kr);
          issue_v(k + 1, vnxt);
        }
      }
      const bool tail = tok0 + kTile > n;      // (chunks are whole tiles: only the sequence's end cuts into one)
      if (tail) {
#pragma unroll
        for (int pg = 0; pg < 2; ++pg)
#pragma unroll
          for (int r = 0; r < 4; ++r)
            if (tok0 + 16 * pg + 4 * kg + r >= n) st[pg][r] = -INFINITY;
      }
      float tmax = fmaxf(fmaxf(fmaxf(st[0][0], st[0][1]), fmaxf(st[0][2], st[0][3])),
                         fmaxf(fmaxf(st[1][0], st[1][1]), fmaxf(st[1][2], st[1][3])));
      tmax = quad_rows_max(tmax) * p.scale_log2e;           // scale > 0: max commutes with scaling
      const float m_new = fmaxf(m_run, tmax);
      const float m_use = (m_new == -INFINITY) ? 0.f : m_new;
      const float alpha = fast_exp2(m_run - m_use);
      float pw[8];
#pragma unroll
      for (int i = 0; i < 8; ++i) pw[i] = fast_exp2(__builtin_fmaf(st[i >> 2][i & 3], p.scale_log2e, -m_use));
      // The row sum adds the weights as the second contraction sees them, i.e. rounded to bf16: numerator and
      // denominator of Eq. 1 then carry the same rounding errors, which cancel where one key dominates (the output
      // is a convex combination of V rows again) and do no harm elsewhere.
      bf16x8 pb;
      float pr[8];
#pragma unroll
      for (int i = 0; i < 8; ++i) {
        pb[i] = static_cast<__bf16>(pw[i]);
        pr[i] = static_cast<float>(pb[i]);
      }
      l_run = l_run * alpha + ((pr[0] + pr[1]) + (pr[2] + pr[3])) + ((pr[4] + pr[5]) + (pr[6] + pr[7]));
      const float m_before = m_run;
      m_run = m_new;
      if (__builtin_amdgcn_ballot_w64(alpha != 1.0f && m_before != -INFINITY) != 0) {   // (no key seen yet: sums still zero)
#pragma unroll
        for (int blk = 0; blk < NBLK; ++blk) acc[blk] *= alpha;
      }
      if constexpr (RING) {
        if constexpr (has_next) wait_vm<NL + NLV + NL>();
        else wait_v(k + 1 == ntiles);
#pragma unroll
        for (int e = 0; e < 8; ++e) {
          vcur[e] = *reinterpret_cast<const VReg*>(vt + (16 * (e >> 2) + 4 * kg + (e & 3)) * kVRow + l16 * (2 * NBLK));
        }
      }
      if (tail) {                              // slots past the end may hold anything: feed zeros
#pragma unroll
        for (int e = 0; e < 8; ++e)
          if (tok0 + 16 * (e >> 2) + 4 * kg + (e & 3) >= n) vcur[e] = VReg{};
      }
#pragma unroll
      for (int blk = 0; blk < NBLK; ++blk) {
        u32x4 raw;
#pragma unroll
        for (int j = 0; j < 4; ++j)              // head dim blk of this lane's group, tokens 2 j and 2 j + 1 of its eight
          raw[j] = __builtin_amdgcn_perm(vcur[2 * j + 1][blk >> 1], vcur[2 * j][blk >> 1],
                                         (blk & 1) ? 0x07060302u : 0x05040100u);
        acc[blk] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8, raw), pb, acc[blk], 0, 0, 0);
      }
      if constexpr (RING && has_next) {
        wait_lds();
        ring_v(k + NS);
      }
#ifdef VEGAS_TIMELINE
      if (tl_stamps[kTlFirstTile] == 0) VEGAS_TL(kTlFirstTile);
#endif
    };

    // ---- stream the chunk's tiles (the last one peeled: prefetches are unconditional, load-counter waits exact)
    if (ntiles > 0) {
      using yes = std::integral_constant<bool, true>;
      using no = std::integral_constant<bool, false>;
      int k = 0;
      if constexpr (RING) {
        for (; k + NS < ntiles; ++k) step(k, va, va, yes{});
        for (; k < ntiles; ++k) step(k, va, va, no{});
      } else {
        while (k + 2 < ntiles) {
          step(k, va, vb, yes{});
          step(k + 1, vb, va, yes{});
          k += 2;
        }
        if (k + 1 < ntiles) {
          step(k, va, vb, yes{});
          step(k + 1, vb, va, no{});
        } else {
          step(k, va, vb, no{});
        }
      }
    }

    // ---- merge the waves: every wave parks its rows as [wave][row][d], with their maxima and sums, and after the one barrier all threads
    //      scale and add the waves' copies and write the workgroup's partial (or the finished rows).  (Scaled by the common maximum before
    //      they are parked they need a barrier more.  us for the launch, captured, before / so: 8 columns of 2048 tokens 4.01 / 3.89, of 4096
    //      4.41 / 4.24, 256 tokens through rings 4.35 / 4.27.)
    // RING: a wave's copy lies in its own ring, which it is done with; another wave may still be streaming through its own.
    VEGAS_TL(kTlStreamed);
    const int copy_floats = RING ? kDraftRing / 4 : Rl * kRedPitch;
    {
      const float lsum = quad_rows_sum(l_run);
      if (kg == 0) {
        sm_m[wave * kDraftRows + l16] = m_run;
        sm_l[wave * kDraftRows + l16] = lsum;
      }
      if (l16 < Rl) {
        float* dst = red + wave * copy_floats + l16 * kRedPitch;
#pragma unroll
        for (int r = 0; r < 4; ++r) {
          const int d0 = NBLK * (4 * kg + r);
          if constexpr (NBLK == 2) *reinterpret_cast<f32x2*>(dst + d0) = f32x2{acc[0][r], acc[1][r]};
          else *reinterpret_cast<f32x4*>(dst + d0) = f32x4{acc[0][r], acc[1][r], acc[2 % NBLK][r], acc[3 % NBLK][r]};
          if constexpr (NBLK == 8) *reinterpret_cast<f32x4*>(dst + d0 + 4) = f32x4{acc[4 % NBLK][r], acc[5 % NBLK][r], acc[6 % NBLK][r], acc[7 % NBLK][r]};
        }
      }
    }
    __syncthreads();
    VEGAS_TL(kTlMerged);
    constexpr int V4 = DV / 4;
    constexpr int kSumTrips = (kDraftRows * V4 + NW * 64 - 1) / (NW * 64);
    f32x4 sums[kSumTrips];
    const int sum_trips = (Rl * V4 + NW * 64 - 1) / (NW * 64);       // (few rows: the later trips have nothing to do)
    // Scales of the waves' copies of a row to their common maximum.
    auto wave_scales = [&](int row, float (&sc)[NW]) {
      float mw[NW];
#pragma unroll
      for (int w = 0; w < NW; ++w) mw[w] = sm_m[w * kDraftRows + row];
      float top = mw[0];
#pragma unroll
      for (int w = 1; w < NW; ++w) top = fmaxf(top, mw[w]);
      const float m_fin = (top == -INFINITY) ? 0.f : top;
#pragma unroll
      for (int w = 0; w < NW; ++w) sc[w] = fast_exp2(mw[w] - m_fin);
      return top;
    };
#pragma unroll
    for (int it = 0; it < kSumTrips; ++it) {
      if (it < sum_trips) {
        const int e = min(tid + it * NW * 64, Rl * V4 - 1);
        const float* src = red + (e / V4) * kRedPitch + 4 * (e % V4);
        f32x4 part[NW];
#pragma unroll
        for (int w = 0; w < NW; ++w) part[w] = *reinterpret_cast<const f32x4*>(src + w * copy_floats);
        float sc[NW];
        wave_scales(e / V4, sc);
        f32x4 acc4 = part[0] * sc[0];
#pragma unroll
        for (int w = 1; w < NW; ++w) acc4 += part[w] * sc[w];
        sums[it] = acc4;
      }
    }
    if (p.out_direct != nullptr) {
      // The only chunk of its (sequence, KV head): divide by the softmax denominator and write the bf16 rows (Eq. 1).
      uint16_t* const rows = out_rows();
#pragma unroll
      for (int it = 0; it < kSumTrips; ++it) {
        const int e = tid + it * NW * 64;
        if (e < Rl * V4) {
          const int row = e / V4;
          float lw = 0.f, sc[NW];
          wave_scales(row, sc);
#pragma unroll
          for (int w = 0; w < NW; ++w) lw += sm_l[w * kDraftRows + row] * sc[w];
          const float inv = lw > 0.f ? 1.0f / lw : 0.f;       // (a row with no visible key: zeros)
          u32x2 packed;
          packed[0] = static_cast<uint32_t>(float_to_bf16_bits(sums[it][0] * inv)) |
                      (static_cast<uint32_t>(float_to_bf16_bits(sums[it][1] * inv)) << 16);
          packed[1] = static_cast<uint32_t>(float_to_bf16_bits(sums[it][2] * inv)) |
                      (static_cast<uint32_t>(float_to_bf16_bits(sums[it][3] * inv)) << 16);
          *reinterpret_cast<u32x2*>(rows + (DV == D ? 4 * e : row * D + part * DV + 4 * (e % V4))) = packed;
        }
      }
      VEGAS_TL(kTlExit);
      VEGAS_TL_FLUSH(p.timeline, NW);
      return;
    }
    float* po = p.part_o + pbase * p.R * D;
#pragma unroll
    for (int it = 0; it < kSumTrips; ++it) {
      const int e = tid + it * NW * 64;
      if (e < Rl * V4) *reinterpret_cast<f32x4*>(po + 4 * e) = sums[it];
    }
    if (tid < Rl) {
      float lw = 0.f, sc[NW];
      const float mw = wave_scales(tid, sc);
#pragma unroll
      for (int w = 0; w < NW; ++w) lw += sm_l[w * kDraftRows + tid] * sc[w];
      p.part_ml[pbase * p.R + tid] = make_float2(mw, lw);
    }
    VEGAS_TL(kTlExit);
    VEGAS_TL_FLUSH(p.timeline, NW);
  };
  if constexpr (CHOOSE) {
    if (past_cache(wave_sum(lane_sixteens(lane_len, p.lens, p.batch, p.max_tokens, lane)), p.Hkv, D)) {
      stream_chunk(std::true_type{});
      return;
    }
  }
  stream_chunk(std::false_type{});
  append_row();
}

template <int D, int PS = 4, bool CHOOSE = false, bool RING = false, typename... Step>
__global__ __launch_bounds__(kDraftWaves * 64, 2) void attn_draft16_kernel(VEGAS_SPLIT_HOT_PARAMS, const SplitParams pfull, const Step... step) {
  SplitParams p = pfull;                     // (see attn_split_kernel: the preloaded arguments)
  VEGAS_SPLIT_HOT_ASSIGN(p);
  draft16<D, PS, CHOOSE, RING, D>(p, step...);
}

// A workgroup for every DV head dims of V (draft_value_parts).
template <int D, int DV, int PS, bool RING>
__global__ __launch_bounds__(kDraftWaves * 64, 2) void attn_draft16_parts_kernel(VEGAS_SPLIT_HOT_PARAMS, const SplitParams pfull) {
  SplitParams p = pfull;
  VEGAS_SPLIT_HOT_ASSIGN(p);
  draft16<D, PS, false, RING, DV>(p);
}

}  // namespace vegas
