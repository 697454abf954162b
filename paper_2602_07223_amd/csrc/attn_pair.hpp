// KV-streaming verification kernel for more than 32 query rows per KV head, gfx950: two 32-row blocks per wave.
//
// Same arithmetic and the same partial-result layout as attn_split_kernel (Eq. 1 split over the context, page
// log-sum-exps for Eq. 2 / Eq. 3, or the token sums of the logit metric), but a wave serves 64 query rows from ONE read
// of K and V.  Two row blocks leave no registers for tiles in flight (128 accumulators), so K and V never pass through
// registers on their way in: they are loaded straight into LDS.
//   * A workgroup = 4 waves (8: pair_waves) on one (sequence, KV head, chunk); every wave takes a contiguous part of the chunk's
//     32-token tiles and owns a ring of LDS (2 tiles, or 4 at head dimension 64; pair_ring) that only it
//     fills and reads, so the streaming loop has no barrier and no wave waits for another one.
//   * K goes into a ring slot as soon as the first contraction has read the slot's old K, V as soon as the second one
//     has read the old V: 64 to 128 KB per compute unit are in flight all the time.  The load counter returns in
//     order: "all but the n newest" is an exact wait for a tile's K or V (stores in between only make it stricter).
//   * A load instruction lands 64 x 16 bytes side by side in LDS, whatever their addresses; the lanes therefore choose
//     WHICH 16 bytes they fetch so that the reads below are free of bank conflicts: a K row's 16-byte pieces are
//     exchanged by the token's number (piece c of token t sits at c ^ (t mod 16); at head dimension 64, where two rows
//     share a bank line, at c ^ (t / 2 mod 8)); V rows stay whole, at head dimension 64 in the order in which the two
//     halves of a wave read them.
//   * S^T = K Q^T and O^T += V^T P^T as in attn_split_kernel; each operand read from LDS feeds the MFMAs of both row
//     blocks.  Page ids come through the scalar path one tile ahead (their wait must not count loads).
//   * A row's running maximum is its true maximum, as in attn_split_kernel: raising it only when a tile exceeds it by 2^8
//     saves most of the rescaling (48 rows, 32K tokens 35.2 us instead of 36.1; 16 sequences 602.4, 603.4 per iteration),
//     but then the heaviest key's weight is no longer exactly 1 and its bf16 rounding shows: error against 64 bits
//     2.2e-3 instead of 1.9e-3 (2-norm).
//   * What is collected (2 % of the bytes read) must not trickle into the read stream: 47 MB written in 320-byte pieces
//     beside 2.4 GB read took 421 us instead of 347 in a stand-alone kernel, the same with a writing wave of its own, in
//     bursts of 5 KB per wave (417), and in bursts at common times too (416: dirty L2 lines are evicted later, into the
//     reads); bursts at common times that are written THROUGH the L2 took 362.  So a wave parks its tiles' values in
//     LDS and writes them through when the wall clock enters a new interval, or its part of the LDS is full.  (When a
//     value leaves depends on the clock; the value does not.)
// Streaming kernel, 40 rows, captured launches: 16 x 36864 tokens 403 us, 376 without collection (6.4 TB/s; a store per
// tile cost 90 us); 16 of 8192..65536 tokens 443 and 399; one of 32768 20.6 at head dimension 64; 48 rows, two of twelve
// tokens' collected, 28.5 at 128.  By the profiler within whole iterations 437, 22.8 and 29.9; the kernel this one replaced,
// which passed K and V through the registers of two waves and their LDS tiles between two barriers per 64 tokens, 483,
// 25.8 and 40.2.  What bounds it: HBM from 64K tokens on, its head and merge below.
// Rows beyond 64 go to sibling workgroups of 64 rows each; small calls of that kind stay with attn_split_kernel
// (rows_as_siblings).
#pragma once
#include <type_traits>

#include "attn_split.hpp"
#include "vegas_common.hpp"

namespace vegas {

constexpr int kPairWaves = 4;
constexpr int kPairRows = 64;               // query rows (of one KV head) of a workgroup
// At head dimension 64, unless page values are parked (they are many), the LDS is laid out for two workgroups per compute
// unit, in rings of two tiles instead of four.  No collection: 48 sequences of 300..3000 tokens, 49 rows, 4 KV heads 52.1 ->
// 35.1 us, 32 of 300..1500, 80 rows, 8 KV heads 49.3 -> 36.6, one of 32768, 40 rows 21.9 -> 20.0.  Token sums: 24 of
// 1000..8000, 80 rows, 8 KV heads 132.2 -> 110.6, 16 of 4000..16000, 64 rows, 4 KV heads 101.1 -> 77.8.  (Of page values
// only two tiles could be parked beside 64 rows, and short bursts are what slows the reads.)
constexpr bool pair_two_per_cu(int D, int collect) { return D == 64 && collect != 1; }
// Bytes of K and V tiles per wave, where there are kPairWaves of them.
constexpr int pair_ring(int D, int collect) { return pair_two_per_cu(D, collect) ? 16 * 1024 : 32 * 1024; }
// Waves of a workgroup that parks page values at head dimension 64 and so has its compute unit to itself.  One wave per SIMD
// leaves a tile's chain (first contraction, maximum, exponentials, second contraction: 1.3 us) nothing to run beside; two halve the
// ring and what is parked per wave (two tiles instead of four).  `share`: tokens of the call's bound per compute unit.  One row
// block is bound by HBM in long streams, where the deeper rings win; siblings, of which one reads from the L2, are bound by the chain.
// A workgroup of 128 tokens or fewer has a tile for each of four waves, and merging eight costs 1.1 us; batches reach that with a
// higher bound, being ragged.  us a call, four waves / eight, 8 KV heads: 40 rows, one sequence of 4096 15.5 / 16.5; 6000 16.7 / 16.1;
// 16384 23.0 / 21.5; 32768 29.6 / 27.6 (the kernel 22.8 / 19.7); 65536 41.7 / 41.9; 131072 67 / 71; 16 of 8192..65536 251 / 286; 12 of
// 375..1500 21.6 / 20.3; 64 rows, 4 of 4000..8000 31.1 / 29.4, of 12000..24000 51.7 / 52.1; 96 rows, one of 12000 32.8 / 32.7, 32768
// 47.0 / 38.7, 131072 122 / 101; 12 of 12500..50000 324 / 274; 112 rows, one of 1959 (share 122) +9 %, of 2268 (141) -3 %; 24 x 124, 96 rows
// 24.1 / 26.7.  Of 4200 batches drawn, four / eight by share: up to 128 0.923, 128..160 0.975, 160..200 0.996, 200..256 1.006, 256..512 1.024,
// 512..2048 1.09.
constexpr int pair_waves(int D, int collect, int row_blocks, int batch, int max_len, int64_t share) {
  return D == 64 && collect == 1 && max_len > 128 && share > (batch > 1 ? 200 : 128) && (row_blocks > 1 || share <= 2048) ? 2 * kPairWaves
                                                                                                                        : kPairWaves;
}
// What a second launch wave costs, in units of 128 tokens (see wants_second_wave): nothing where two workgroups fit.
constexpr int pair_second_cost(int D, int collect) { return pair_two_per_cu(D, collect) ? 0 : 11; }
constexpr int kPairFold = 32768;           // chunks per round of a folded grid

// Floats of one wave's parked values: park_tiles tiles of two pages x the collected rows a workgroup can have, or of the
// high and low token sums.  (A multiple of four: a wave reads them in 16-byte pieces; see pair_lds.)
__host__ __device__ __forceinline__ int pair_park_floats(int park_tiles, int Rc, int collect) {
  return park_tiles * 2 * (collect == 2 ? kTile : (Rc < kPairRows ? Rc : kPairRows));
}

// ONE: all rows fit one workgroup, which is then the only reader of its K/V lines (non-temporal loads); otherwise sibling
// workgroups read them too and want to find them in the L2.  NW: waves, kPairWaves or twice as many (pair_waves).
template <int COLLECT, int D, bool ONE, int NW = kPairWaves>
__global__ __launch_bounds__(NW * 64, 2) void attn_pair_kernel(VEGAS_SPLIT_HOT_PARAMS, const SplitParams pfull) {
  VEGAS_TL_DECL;                             // (profiling builds: per-wave phase stamps, see vegas_common.hpp)
  VEGAS_TL(kTlEntry);
  SplitParams p = pfull;                     // (see attn_split_kernel: the preloaded arguments)
  VEGAS_SPLIT_HOT_ASSIGN(p);
  static_assert(D == 128 || D == 64, "head dimension");
  // Dynamic LDS (pair_lds): [ring of every wave][queries][collected values of every wave][row maxima][row sums]; the
  // merge buffer aliases everything before the row maxima.
  extern __shared__ __attribute__((aligned(16))) unsigned char smem[];
  constexpr int NB = 2;                      // 32-row blocks of a wave
  constexpr int CH = D / 8;                  // 16-byte pieces of a K/V row
  constexpr int TPI = 64 / CH;               // token rows of one load instruction
  constexpr int kRing = pair_ring(D, COLLECT) * kPairWaves / NW;
  constexpr int NP = kPage / TPI;            // load instructions per page (of K, of V)
  constexpr int NL = 2 * NP;                 // ... per tile
  constexpr int NBLK = D / 32;               // 32-wide blocks of the output's head dimension
  constexpr int kRow = 2 * D;                // bytes of a K/V row
  constexpr int kHalfSlot = 32 * kRow;       // bytes of a tile's K (then as many of V)
  constexpr int NS = kRing / (2 * kHalfSlot);   // tiles the ring holds
  constexpr int kRowPitch = row_pitch(D);
  constexpr int kRedPitch = red_pitch(D);
  using VReg = typename std::conditional<D == 128, u32x2, uint32_t>::type;   // NBLK head dims of one token
  const int tid = threadIdx.x;
  const int lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int half = lane >> 5;
  const int l32 = lane & 31;
  unsigned char* const ring = smem + wave * kRing;
  unsigned char* const qlds = smem + NW * kRing;
  float* const sm_m = reinterpret_cast<float*>(smem + p.lds_q_off);             // [wave][64]
  float* const sm_l = sm_m + NW * kPairRows;

  // Grid (KV head, row block + row_blocks * chunk, sequence): the 8 KV heads of a chunk, whose rows interleave in memory,
  // run side by side on the 8 XCDs, and sibling row blocks share one (chunks fastest: 396 us instead of 380 for 16 x 36864
  // tokens without collection).
  // More than 65535 row blocks and chunks: the grid's third dimension goes round the sequences once per kPairFold of them.
  const int h = blockIdx.x;
  int b = blockIdx.z, yy = blockIdx.y;
  const int seqs = p.plan ? 1 : p.batch;
  if (b >= seqs) {
    yy += b / seqs * kPairFold;
    b %= seqs;
  }
  const int rb = ONE ? 0 : yy % p.row_blocks;
  const int split = ONE ? yy : yy / p.row_blocks;
  int chunk_tokens = p.chunk_tokens;
  int c0 = split * chunk_tokens;
  int slot = split;                          // this workgroup's partial slot, of the head's or the column's
  int n = 0;                                 // the sequence's length: a plan brings it
  if (p.plan) {                              // balanced chunking: workgroup `split` of this head -> (sequence, tokens)
    const BalancedSlot bs = balanced_slot(p.lens, p.batch, p.max_tokens, p.slots_target, p.slots_target2, p.share_group, p.slots_total,
                                          p.share_margin, pair_second_cost(D, COLLECT),
                                          p.chunk_cap_units, kTile * kPairWaves, split, ((blockIdx.x | yy) == 0 && wave == 0) ? p.plan : nullptr);
    if (bs.b < 0) return;
    b = __builtin_amdgcn_readfirstlane(bs.b);
    c0 = __builtin_amdgcn_readfirstlane(bs.c0);
    chunk_tokens = __builtin_amdgcn_readfirstlane(bs.chunk);
    slot = __builtin_amdgcn_readfirstlane(bs.slot);
    n = bs.n;
  }
  const int row0 = kPairRows * rb;           // first query row (of this KV head) of this workgroup
  const int Rl = max(min(kPairRows, p.R - row0), 0);   // valid rows (none in a block that only carries the sum rows)

  // Page ids through the scalar path: entry clamped to the table row, id to the pool.
  typedef const __attribute__((address_space(4))) int32_t* sptr;
  const sptr table = (sptr)(p.table + static_cast<int64_t>(b) * p.table_stride);
  auto into_pool = [&](int raw) -> int {
    return static_cast<int>(raw < 0 ? 0 : (static_cast<int64_t>(raw) >= p.num_pages ? p.num_pages - 1 : raw));
  };

  constexpr int QI = kPairRows * CH / (NW * 64);
  u32x4 qraw[QI];
  const int qrows = ONE ? p.R + (COLLECT == 2 ? 2 : 0) : kPairRows;      // rows the query tile holds
  const bool all_rows_here = COLLECT != 2 || ONE;
  if (all_rows_here) issue_query_loads<D, QI>(qraw, p, b, h, row0, Rl, tid, NW * 64);
  int zero = 0;
  asm("" : "+v"(zero));                      // (see attn_split_kernel)
  if (!p.plan) n = p.lens[b + zero];
  // A wave's tiles are a contiguous part of the chunk's: what it collects is contiguous too.  Where they begin depends on the
  // chunk's end, which is the sequence's in its last chunk only: the page ids of the others are requested beside the length.
  int tile_first, ntiles;
  auto place = [&](int end) {
    const int chunk_tiles = (end - c0 + kTile - 1) / kTile;
    tile_first = c0 / kTile + chunk_tiles * wave / NW;
    ntiles = c0 / kTile + chunk_tiles * (wave + 1) / NW - tile_first;
  };
  int first_ids[2 * NS];                     // of the ring's first tiles
  auto page_id = [&](int k, int pg) -> int {           // page pg of this wave's tile k
    const int page = min(2 * (tile_first + k) + pg, p.table_stride - 1);
    return table[page];
  };
  auto request_ids = [&]() {
#pragma unroll
    for (int i = 0; i < 2 * NS; ++i) first_ids[i] = page_id(i >> 1, i & 1);
  };
  place(c0 + chunk_tokens);
  request_ids();
  // (the rest of the argument block in one go, and what follows from it, while these are on their way; see attn_split_kernel)
  asm volatile("" : "+s"(p.k), "+s"(p.v), "+s"(p.page_stride), "+s"(p.token_stride), "+s"(p.head_stride), "+s"(p.num_pages),
               "+s"(p.max_tokens), "+s"(p.nsplit));
  // ---- which 16 bytes of a page this lane fetches with each load instruction
  const int64_t head_off = static_cast<int64_t>(h) * p.head_stride;
  const uint32_t ts_bytes = static_cast<uint32_t>(p.token_stride) * 2u;
  uint32_t koff[NP], voff[NP];
#pragma unroll
  for (int i = 0; i < NP; ++i) {
    const int row = TPI * i + lane / CH, piece = lane % CH;       // where the 16 bytes land
    if constexpr (D == 128) {
      koff[i] = static_cast<uint32_t>(row) * ts_bytes + static_cast<uint32_t>(piece ^ row) * 16u;
      voff[i] = static_cast<uint32_t>(row) * ts_bytes + static_cast<uint32_t>(piece) * 16u;
    } else {
      koff[i] = static_cast<uint32_t>(row) * ts_bytes + static_cast<uint32_t>(piece ^ (row >> 1)) * 16u;
      const int tok = (row & 8) | ((row >> 1) & 3) | ((row & 1) << 2);   // V row r holds this token of the page
      voff[i] = static_cast<uint32_t>(tok) * ts_bytes + static_cast<uint32_t>(piece) * 16u;
    }
  }
#pragma unroll
  for (int i = 0; i < NP; ++i) asm volatile("" : "+v"(koff[i]), "+v"(voff[i]));
  if constexpr (NS == 2) asm volatile("" : "+v"(n), "+s"(first_ids[0]), "+s"(first_ids[1]), "+s"(first_ids[2]), "+s"(first_ids[3]));
  else asm volatile("" : "+v"(n), "+s"(first_ids[0]), "+s"(first_ids[1]), "+s"(first_ids[2]), "+s"(first_ids[3]), "+s"(first_ids[4]),
                    "+s"(first_ids[5]), "+s"(first_ids[6]), "+s"(first_ids[7]));
  n = __builtin_amdgcn_readfirstlane(n);
  n = n < 0 ? 0 : (n > p.max_tokens ? p.max_tokens : n);
  if (c0 >= n) return;                       // whole workgroup: nothing to do, no partial is read
  const int64_t pbase = p.plan ? static_cast<int64_t>(h) * p.slots_total + slot : (static_cast<int64_t>(b) * p.Hkv + h) * p.nsplit + slot;
  VEGAS_TL(kTlLength);
  const int c1 = min(c0 + chunk_tokens, n);
  const int nblk = (n + kPage - 1) / kPage;
  if (c1 != c0 + chunk_tokens) {
    place(c1);
    request_ids();
  }

  // ---- query rows -> LDS [rows][CH pieces of 16 B], padded rows (lanes of later rows work on a copy of the last one).
  // COLLECT == 2: the last row block's rows Rl (high part) and Rl + 1 (low part) carry the sum of the collected rows.
  // (Before the first tile is requested: the wait for the queries would count its loads.)
  const bool has_extra = COLLECT == 2 && (ONE || rb == p.row_blocks - 1);
  if (all_rows_here) store_queries_to_lds<D, QI>(qlds, qraw, qrows, tid, NW * 64);
  else load_queries_to_lds<D>(qlds, p, b, h, qrows, row0, Rl, has_extra, tid, NW * 64);

  typedef const __attribute__((address_space(3))) unsigned char* lptr;
  const uint32_t ring_lds = __builtin_amdgcn_readfirstlane(static_cast<uint32_t>(reinterpret_cast<uintptr_t>((lptr)ring)));
  auto page_base = [&](const uint16_t* cache, int ph) -> const unsigned char* {
    return uniform_ptr(reinterpret_cast<const unsigned char*>(cache + static_cast<int64_t>(ph) * p.page_stride + head_off));
  };
  auto load_k = [&](int slot, int id0, int id1) {
    load_to_lds<NP, ONE>(ring_lds + static_cast<uint32_t>(slot * 2 * kHalfSlot), page_base(p.k, id0), koff);
    load_to_lds<NP, ONE>(ring_lds + static_cast<uint32_t>(slot * 2 * kHalfSlot + kHalfSlot / 2), page_base(p.k, id1), koff);
  };
  auto load_v = [&](int slot, int id0, int id1) {
    load_to_lds<NP, ONE>(ring_lds + static_cast<uint32_t>(slot * 2 * kHalfSlot + kHalfSlot), page_base(p.v, id0), voff);
    load_to_lds<NP, ONE>(ring_lds + static_cast<uint32_t>(slot * 2 * kHalfSlot + kHalfSlot + kHalfSlot / 2), page_base(p.v, id1), voff);
  };

  // ---- the ring's first tiles
#pragma unroll
  for (int k = 0; k < NS; ++k) {
    if (k < ntiles) {
      const int id0 = into_pool(first_ids[2 * k]), id1 = into_pool(first_ids[2 * k + 1]);
      load_k(k, id0, id1);
      load_v(k, id0, id1);
    }
  }
  int next0 = page_id(NS, 0), next1 = page_id(NS, 1);             // ids of the tile that enters the ring next
  VEGAS_TL(kTlLoadsIssued);

  // last visible token of this lane's row of each block: the causal bound, and nothing past this workgroup's chunk
  int limit[NB];
#pragma unroll
  for (int nb = 0; nb < NB; ++nb) {
    const int r = 32 * nb + l32;
    limit[nb] = min(n - p.G + ((r < Rl) ? (row0 + r) / p.g : 0), c1 - 1);
  }
  // ---- collection: index of this lane's rows among the collected ones (COLLECT 1), columns of the sum rows (COLLECT 2)
  int ci[NB];
  if constexpr (COLLECT == 1) {
#pragma unroll
    for (int nb = 0; nb < NB; ++nb) {
      const int r = row0 + 32 * nb + l32;
      const bool all = p.collect_rows == 1 || p.G <= 2;
      const int c = (all || r < p.g) ? r : (r >= (p.G - 1) * p.g ? r - (p.G - 2) * p.g : -1);
      ci[nb] = (32 * nb + l32 < Rl) ? c : -1;
    }
  }
  // Collected rows of this row block: ci runs over [ci_lo, ci_hi) (one contiguous range of a page's Rc values).
  int ci_lo = 0, nci = 0;
  int tile_vals = 0;                         // values a tile parks
  float* park = nullptr;                     // this wave's parked values, park_tiles tiles of them
  unsigned char* col_dst = nullptr;          // where the first of them belongs (wave-uniform)
  if constexpr (COLLECT == 1) {
    auto before = [&](int r) {                                    // collected rows below row r
      return (p.collect_rows == 1 || p.G <= 2) ? r : min(r, p.g) + max(r - (p.G - 1) * p.g, 0);
    };
    ci_lo = before(row0);
    nci = before(row0 + Rl) - ci_lo;
    tile_vals = 2 * nci;
    col_dst = reinterpret_cast<unsigned char*>(
        p.page_lse + ((static_cast<int64_t>(b) * p.Hkv + h) * p.lse_pages + 2 * tile_first) * p.Rc);
  }
  if constexpr (COLLECT == 2) {
    tile_vals = 2 * kTile;                   // high and low parts
    col_dst = reinterpret_cast<unsigned char*>(
        p.page_lse + (static_cast<int64_t>(b) * p.Hkv + h) * p.lse_pages + kTile * tile_first);
  }
  if constexpr (COLLECT != 0)
    park = reinterpret_cast<float*>(qlds + qrows * kRowPitch) + wave * pair_park_floats(p.park_tiles, p.Rc, COLLECT);
  int parked = 0, flushed = 0;               // tiles parked now; tiles that left before them
  uint32_t epoch = 0;
  auto clock_epoch = [&]() -> uint32_t {     // number of the wall-clock interval (100 MHz ticks, the same on every unit)
    return __umulhi(static_cast<uint32_t>(__builtin_amdgcn_s_memrealtime()), p.epoch_mul);
  };
  if constexpr (COLLECT != 0) epoch = clock_epoch();
  // The parked values leave.
  auto flush = [&]() {
    wave_lds_fence();
    if constexpr (COLLECT == 1) {
      const int pages = min(2 * parked, min(nblk, (c1 + kPage - 1) / kPage) - 2 * (tile_first + flushed));
      unsigned char* dst = uniform_ptr_mut(col_dst + static_cast<int64_t>(flushed) * (8 * p.Rc));
      if (nci == p.Rc) {                     // one contiguous run
        const int vals = pages * nci;
        for (int e = 4 * lane; e < vals; e += 256) {
          const f32x4 v = *reinterpret_cast<const f32x4*>(park + e);
          if (e + 4 <= vals) {
            store_through(dst, 4u * e, v);
          } else {
            for (int i = 0; e + i < vals; ++i) store_through(dst, 4u * (e + i), v[i]);
          }
        }
      } else {                               // a row block among several: a run per page
        for (int pg = 0; pg < pages; ++pg)
          if (lane < nci) store_through(dst, 4u * (pg * p.Rc + ci_lo + lane), park[pg * nci + lane]);
      }
    }
    if constexpr (COLLECT == 2) {
      if (has_extra) {
        unsigned char* dst = uniform_ptr_mut(col_dst + static_cast<int64_t>(flushed) * (4 * kTile));
        const int vals = min(kTile * parked, c1 - kTile * (tile_first + flushed));
        for (int e = lane; e < vals; e += 64) {
          const float* src = park + (e / kTile) * (2 * kTile) + e % kTile;
          store_through(dst, 4u * e, src[0] + src[kTile]);
        }
      }
    }
    wave_lds_fence();
    flushed += parked;
    parked = 0;
  };
  __syncthreads();                           // queries in LDS
  if constexpr (COLLECT == 2 && ONE) {
    add_query_sums<D>(qlds, p, Rl, tid);
    __syncthreads();
  }
  VEGAS_TL(kTlQueries);

  // ---- running state: lane (row, half) keeps the running maximum m (same in both halves), its half's partial sum l,
  //      and O^T accumulators acc[nb][blk][i] = O[row][NBLK*(8(i/4) + 4half + i%4) + blk]
  float m_run[NB], l_run[NB];
  f32x16 acc[NB][NBLK];
#pragma unroll
  for (int nb = 0; nb < NB; ++nb) {
    m_run[nb] = -INFINITY;
    l_run[nb] = 0.f;
#pragma unroll
    for (int blk = 0; blk < NBLK; ++blk)
#pragma unroll
      for (int i = 0; i < 16; ++i) acc[nb][blk][i] = 0.f;
  }
  // K reads of a slot: piece 2 kk + half of token l32, exchanged as above
  const uint32_t k_first = static_cast<uint32_t>(l32 * kRow + ((half ^ (D == 128 ? (l32 & 15) : ((l32 >> 1) & 7))) * 16));
  uint32_t q_row[NB];
#pragma unroll
  for (int nb = 0; nb < NB; ++nb) q_row[nb] = static_cast<uint32_t>(min(32 * nb + l32, qrows - 1) * kRowPitch + half * 16);

  // One tile.  load_next: the tile NS further enters the ring as this one leaves it.
  auto step = [&](int k, int slot, auto load_tag) {
    constexpr bool load_next = decltype(load_tag)::value;
    const int tok0 = (tile_first + k) * kTile;
    const uint32_t now = COLLECT != 0 ? clock_epoch() : 0u;
    const unsigned char* kt = ring + slot * (2 * kHalfSlot);
    const unsigned char* vt = kt + kHalfSlot;
    const int after = ntiles - 1 - k;        // (tail) tiles requested after this one
    const int id0 = into_pool(next0), id1 = into_pool(next1);
    if constexpr (load_next) {
      wait_vm<(2 * NS - 1) * NL>();
      next0 = page_id(k + NS + 1, 0);
      next1 = page_id(k + NS + 1, 1);
    } else {
      if (after == 0) wait_vm<NL>();
      else if (after == 1) wait_vm<3 * NL>();
      else if (after == 2) wait_vm<(NS > 2 ? 5 : 0) * NL>();
      else wait_vm<(NS > 3 ? 7 : 0) * NL>();
    }
    f32x16 st[NB];
#pragma unroll
    for (int nb = 0; nb < NB; ++nb)
#pragma unroll
      for (int i = 0; i < 16; ++i) st[nb][i] = 0.f;
    uint32_t k_at = k_first;
    asm volatile("" : "+v"(k_at));           // (the eight addresses are not worth eight registers of the whole loop)
#pragma unroll
    for (int kk = 0; kk < D / 16; ++kk) {
      const bf16x8 a = __builtin_bit_cast(
          bf16x8, *reinterpret_cast<const u32x4*>(kt + (k_at ^ static_cast<uint32_t>(32 * kk))));
#pragma unroll
      for (int nb = 0; nb < NB; ++nb) {
        const bf16x8 qb = __builtin_bit_cast(
            bf16x8, *reinterpret_cast<const u32x4*>(qlds + q_row[nb] + kk * 32));
        st[nb] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(a, qb, st[nb], 0, 0, 0);
      }
    }
    if constexpr (load_next) {
      wait_lds();
      load_k(slot, id0, id1);
    }

    if constexpr (COLLECT == 2) {
      // Columns Rl and Rl + 1 of S^T hold k_i . (high part) and k_i . (low part) for the tile's tokens.
      if (has_extra) {
#pragma unroll
        for (int nb = 0; nb < NB; ++nb) {
          const int r = 32 * nb + l32;
          if (r == Rl || r == Rl + 1) {
            float* dst = park + parked * tile_vals + (r - Rl) * kTile + 4 * half;
#pragma unroll
            for (int i4 = 0; i4 < 4; ++i4)
              *reinterpret_cast<f32x4*>(dst + 8 * i4) = f32x4{st[nb][4 * i4], st[nb][4 * i4 + 1], st[nb][4 * i4 + 2], st[nb][4 * i4 + 3]};
          }
        }
      }
    }

    const bool tail = (tok0 + kTile > c1) || (tok0 + kTile - 1 > n - p.G);
    bf16x8 pb[NB][2];
#pragma unroll
    for (int nb = 0; nb < NB; ++nb) {
      if (tail) {
#pragma unroll
        for (int i = 0; i < 16; ++i) {
          const int tok = tok0 + 8 * (i >> 2) + 4 * half + (i & 3);
          if (tok > limit[nb]) st[nb][i] = -INFINITY;
        }
      }
      float tmax = st[nb][0];
#pragma unroll
      for (int i = 1; i < 16; ++i) tmax = fmaxf(tmax, st[nb][i]);
      tmax = half_max(tmax) * p.scale_log2e;               // scale > 0: max commutes with scaling
      const float m_before = m_run[nb];
      const float m_new = fmaxf(m_before, tmax);
      const float m_use = (m_new == -INFINITY) ? 0.f : m_new;
      m_run[nb] = m_new;
      float pw[16];
#pragma unroll
      for (int i = 0; i < 16; ++i) pw[i] = fast_exp2(__builtin_fmaf(st[nb][i], p.scale_log2e, -m_use));
      float ps0 = 0.f, ps1 = 0.f;
#pragma unroll
      for (int i = 0; i < 8; ++i) { ps0 += pw[i]; ps1 += pw[8 + i]; }
      // (nothing to rescale where the row had seen no key yet: its sums are still zero)
      if (__builtin_amdgcn_ballot_w64(m_new != m_before && m_before != -INFINITY) != 0) {
        const float alpha = fast_exp2(m_before - m_use);
        l_run[nb] *= alpha;
#pragma unroll
        for (int blk = 0; blk < NBLK; ++blk)
#pragma unroll
          for (int i = 0; i < 16; ++i) acc[nb][blk][i] *= alpha;
      }
      l_run[nb] += ps0 + ps1;
      if constexpr (COLLECT == 1) {
        const float f0 = half_sum(ps0);
        const float f1 = half_sum(ps1);                    // page `half` of the tile
        if (ci[nb] >= 0) park[parked * tile_vals + half * nci + ci[nb] - ci_lo] = m_use + fast_log2(half ? f1 : f0);
      }
#pragma unroll
      for (int s2 = 0; s2 < 2; ++s2)
#pragma unroll
        for (int jj = 0; jj < 8; ++jj) pb[nb][s2][jj] = static_cast<__bf16>(pw[s2 * 8 + jj]);
    }

    if constexpr (load_next) {
      wait_vm<(2 * NS - 1) * NL>();
    } else {
      if (after == 0) wait_vm<0>();
      else if (after == 1) wait_vm<2 * NL>();
      else if (after == 2) wait_vm<(NS > 2 ? 4 : 0) * NL>();
      else wait_vm<(NS > 3 ? 6 : 0) * NL>();
    }
    const bool past_end = tok0 + kTile > n;              // slots past the end may hold anything: feed zeros
#pragma unroll
    for (int s2 = 0; s2 < 2; ++s2) {
      VReg vcur[8];
#pragma unroll
      for (int jj = 0; jj < 8; ++jj) {
        const int tl = 16 * s2 + 8 * (jj >> 2) + 4 * half + (jj & 3);
        const int row = D == 128 ? tl : (16 * s2 + 8 * (jj >> 2) + 2 * (jj & 3) + half);   // where that token's V sits
        vcur[jj] = *reinterpret_cast<const VReg*>(vt + row * kRow + l32 * (2 * NBLK));
        if (past_end && tok0 + tl >= n) vcur[jj] = VReg{};
      }
#pragma unroll
      for (int blk = 0; blk < NBLK; ++blk) {
        u32x4 raw;
#pragma unroll
        for (int pp = 0; pp < 4; ++pp) {
          unsigned lo, hi;                     // the dword that holds head dim blk of two consecutive tokens
          if constexpr (D == 128) {
            lo = (blk < 2) ? vcur[2 * pp][0] : vcur[2 * pp][1];
            hi = (blk < 2) ? vcur[2 * pp + 1][0] : vcur[2 * pp + 1][1];
          } else {
            lo = vcur[2 * pp];
            hi = vcur[2 * pp + 1];
          }
          raw[pp] = __builtin_amdgcn_perm(hi, lo, (blk & 1) ? 0x07060302u : 0x05040100u);
        }
#pragma unroll
        for (int nb = 0; nb < NB; ++nb)
          acc[nb][blk] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(bf16x8, raw), pb[nb][s2], acc[nb][blk], 0, 0, 0);
      }
    }
    if constexpr (load_next) {
      wait_lds();
      load_v(slot, id0, id1);
    }
    if constexpr (COLLECT != 0) {
      ++parked;
      if (parked == p.park_tiles || now != epoch) {
        flush();
        epoch = now;
      }
    }
#ifdef VEGAS_TIMELINE
    if (tl_stamps[kTlFirstTile] == 0) VEGAS_TL(kTlFirstTile);
#endif
  };

  // ---- stream the chunk's tiles
  {
    using yes = std::integral_constant<bool, true>;
    using no = std::integral_constant<bool, false>;
    int k = 0, slot = 0;
    for (; k + NS < ntiles; ++k) {
      step(k, slot, yes{});
      slot = slot + 1 == NS ? 0 : slot + 1;
    }
    for (; k < ntiles; ++k) {
      step(k, slot, no{});
      slot = slot + 1 == NS ? 0 : slot + 1;
    }
  }

  if constexpr (COLLECT != 0) {
    if (parked > 0) flush();
  }

  // ---- merge the waves: row maxima meet in LDS, every wave rescales and parks its valid rows as [wave][row][d], all
  //      threads add the waves' copies and write the workgroup's partial with consecutive threads on consecutive addresses
  VEGAS_TL(kTlStreamed);
  if (half == 0) {
#pragma unroll
    for (int nb = 0; nb < NB; ++nb) sm_m[wave * kPairRows + 32 * nb + l32] = m_run[nb];
  }
  __syncthreads();                           // also: every wave is done with its ring and the queries
  VEGAS_TL(kTlMerged);
  float* red = reinterpret_cast<float*>(smem);
#pragma unroll
  for (int nb = 0; nb < NB; ++nb) {
    const int row = 32 * nb + l32;
    float mw = -INFINITY;
#pragma unroll
    for (int w = 0; w < NW; ++w) mw = fmaxf(mw, sm_m[w * kPairRows + row]);
    const float m_fin = (mw == -INFINITY) ? 0.f : mw;
    const float sc = fast_exp2(m_run[nb] - m_fin);
    const float lsum = half_sum(l_run[nb] * sc);
    if (half == 0) sm_l[wave * kPairRows + row] = lsum;
    if (row < Rl) {
      float* dst = red + (wave * Rl + row) * kRedPitch;
#pragma unroll
      for (int i = 0; i < 16; ++i) {
        const int d0 = NBLK * (8 * (i >> 2) + 4 * half + (i & 3));
        if constexpr (D == 128) {
          *reinterpret_cast<f32x4*>(dst + d0) =
              f32x4{acc[nb][0][i] * sc, acc[nb][1][i] * sc, acc[nb][2][i] * sc, acc[nb][3][i] * sc};
        } else {
          *reinterpret_cast<f32x2*>(dst + d0) = f32x2{acc[nb][0][i] * sc, acc[nb][1][i] * sc};
        }
      }
    }
  }
  __syncthreads();
  constexpr int V4 = D / 4;
  float* po = p.part_o + (pbase * p.R + row0) * D;
#pragma unroll 2
  for (int e = tid; e < Rl * V4; e += NW * 64) {
    const float* src = red + (e / V4) * kRedPitch + 4 * (e % V4);
    f32x4 acc4 = *reinterpret_cast<const f32x4*>(src);
#pragma unroll
    for (int w = 1; w < NW; ++w) acc4 += *reinterpret_cast<const f32x4*>(src + w * Rl * kRedPitch);
    *reinterpret_cast<f32x4*>(po + 4 * e) = acc4;
  }
  if (tid < Rl) {
    float mw = -INFINITY, lw = 0.f;
#pragma unroll
    for (int w = 0; w < NW; ++w) {
      mw = fmaxf(mw, sm_m[w * kPairRows + tid]);
      lw += sm_l[w * kPairRows + tid];
    }
    p.part_ml[pbase * p.R + row0 + tid] = make_float2(mw, lw);
  }
  VEGAS_TL(kTlExit);
  VEGAS_TL_FLUSH(p.timeline, NW);
}

// Dynamic LDS of attn_pair_kernel: bytes, where the row maxima start, and how many tiles of collected values a wave parks.
struct PairLds {
  size_t bytes, off_max;
  int park_tiles;
};
inline PairLds pair_lds(int R, int Rc, int row_blocks, int collect, int D, int waves = kPairWaves) {
  const size_t q = static_cast<size_t>(row_blocks == 1 ? R + (collect == 2 ? 2 : 0) : kPairRows) * row_pitch(D);
  const size_t rows_ml = 2 * static_cast<size_t>(waves) * kPairRows * sizeof(float);
  size_t before = kPairWaves * pair_ring(D, collect) + q;
  PairLds l = {0, 0, 0};
  if (collect != 0) {
    const size_t tile = sizeof(float) * pair_park_floats(1, Rc, collect);
    const size_t room = (pair_two_per_cu(D, collect) ? 80 : 160) * 1024;
    l.park_tiles = static_cast<int>((room - rows_ml - before) / (waves * tile));
    if (l.park_tiles > 64) l.park_tiles = 64;
    if (tile % 16) l.park_tiles &= ~1;       // (an odd number of collected rows: tiles of 8 bytes more than a multiple of 16)
    before += waves * tile * l.park_tiles;
  }
  const size_t red = static_cast<size_t>(waves) * (R < kPairRows ? R : kPairRows) * red_pitch(D) * sizeof(float);
  if (red > before) before = red;
  l.off_max = (before + 15) / 16 * 16;
  l.bytes = l.off_max + rows_ml;
  return l;
}

}  // namespace vegas
