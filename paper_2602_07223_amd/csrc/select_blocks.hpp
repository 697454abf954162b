// Top-k page selection: workgroup-wide radix select over fp32 score bit patterns, then an
// order-preserving compaction that gathers physical page ids.
//
// The argmax of Eq. 2 / Eq. 3 over unions of pages is the k pages with the largest scores.  The
// pages overlapping the last G token positions are always kept (last sentence of Sec. 3.2) and
// are a suffix of the logical page range, so the search runs over the prefix [0, f0) only.
// Everything is integer work on the score bits: the result is defined bit for bit, ties go to the
// lower logical page index.
#pragma once
#include <type_traits>

#include "vegas_common.hpp"

namespace vegas {

constexpr int kSelectThreads = 1024;
constexpr int kSelectKeyCap = 16384;   // keys kept in LDS (64 KB); longer prefixes re-read the scores
constexpr int kSelectRegRows = 8;      // prefixes of up to 8 pages a thread keep their keys in registers instead
constexpr int kSelectFewThreads = 512; // threads for prefixes that these can hold in registers (select_blocks_kernel)

// Order-preserving key of a score (larger float <=> larger unsigned); -0 is folded onto +0 and every NaN onto
// key 0, below -infinity: a NaN score ranks last, NaNs among themselves by index like any other tie.
__device__ __forceinline__ uint32_t score_key(float s) {
  const uint32_t u = __float_as_uint(s + 0.0f);
  const uint32_t key = (u & 0x80000000u) ? ~u : (u | 0x80000000u);
  return (s != s) ? 0u : key;
}

// ---- selection among keys that the threads of a workgroup hold in registers ----
struct RegisterSelectShared {
  uint32_t hist[3][2048];                       // digit counts of the up to three passes
  uint32_t low[kSelectThreads / 64], high[kSelectThreads / 64];
  uint32_t bin, need, count;
};
// Taken are the keys above base + span and the first `need`, by position, of those in [base, base + span]; whole: these are all.
struct LastKey {
  uint32_t base, span, need;
  bool whole;
};

constexpr uint32_t kNoDigit = 0xFFFFFFFFu;      // of a key that is not counted
constexpr int kOften = 4;                       // digits that a crowded wave counts by itself
constexpr int kRunLanes = 32;                   // so many lanes with the digit of the lane beside them: one add per run of lanes
// The digit of the lane `BELOW` below, of sixteen; none for the first ones.
template <int BELOW = 1>
__device__ __forceinline__ uint32_t digit_beside(uint32_t digit) {
  return static_cast<uint32_t>(__builtin_amdgcn_update_dpp(static_cast<int>(kNoDigit), static_cast<int>(digit), 0x110 + BELOW, 0xf, 0xf,
                                                           false));   // row_shr
}
// Lanes that have the digit of the lane beside them: the chance that two keys share a digit, at the price of one comparison.
__device__ __forceinline__ int sharing_lanes(uint32_t digit) {
  return __popcll(__builtin_amdgcn_ballot_w64(digit == digit_beside(digit) && digit != kNoDigit));
}

// One full wave: from the top, the bin of the 2048 in `h` that holds key number `need` (0 < need <= keys counted), how many of its
// keys are wanted and how many it has.
__device__ __forceinline__ void walk_to_last_bin(const uint32_t* h, uint32_t need, RegisterSelectShared& sh) {
  const int lane = threadIdx.x & 63;
  // lane l owns the 32 bins from 32 (63 - l) on, read in an order that spreads the lanes over the banks; then lanes
  // 0..31 the bins of the lane that holds the wanted key, both from the top bin down
  const u32x4* g4 = reinterpret_cast<const u32x4*>(h) + 8 * (63 - lane);
  u32x4 s4 = {0u, 0u, 0u, 0u};
#pragma unroll
  for (int i = 0; i < 8; ++i) s4 += g4[(i + lane) & 7];
  const uint32_t mine = (s4[0] + s4[1]) + (s4[2] + s4[3]);
  const uint32_t above = wave_prefix_sum(mine) - mine;
  const uint64_t who = __builtin_amdgcn_ballot_w64(above < need && need <= above + mine);   // one lane: 0 < need <= all
  const int src = who ? __builtin_ctzll(who) : 0;
  const int top = 32 * (63 - src) + 31;
  const uint32_t left = need - __builtin_amdgcn_readlane(above, src);
  const uint32_t c = lane < 32 ? h[top - lane] : 0u;
  const uint32_t over = wave_prefix_sum(c) - c;
  const uint64_t in = __builtin_amdgcn_ballot_w64(over < left && left <= over + c);
  const int at = in ? __builtin_ctzll(in) : 0;
  if (lane == at) {
    sh.bin = static_cast<uint32_t>(top - at);
    sh.need = left - over;
    sh.count = c;
  }
}

// Radix select: where the `take` largest of the workgroup's keys end.  Keys below `full` of every thread hold positions, of
// those from there to `live` valid(u) says which; a key without a position is 0 and its place lies behind all positions.  0 <
// take < positions.  Followed by no barrier; the first thing it does is not ordered behind reads of `sh` either.
// A digit is 11 bits of key - smallest key, from the highest bit in which the keys differ: what the scores have in common
// (sign, most of the exponent) costs no pass, the counts spread over the bins so that one shared histogram and plain adds
// do, and two passes as a rule, three at most, find the end.  (With four passes over 8 fixed bits, a histogram per wave and
// one add for the lanes that share a digit, an iteration took, us: 2048 pages 70.2 instead of 69.7, 4096 pages of each of 16
// sequences 590.6 instead of 587.6, 8192 pages 161.0 instead of 158.0.)  What bounds it is latency, a barrier and one wave's walk
// through the counts per pass, and with 16 and more keys a thread the instructions issued per key.
// Scores need not spread: adds of many lanes to one bin wait for each other.  A wave whose first keys meet in few bins counts
// the digits of up to four of them in registers and adds the rest, or, where half its lanes have the digit of the lane beside
// them (scores that rise or fall with the position, or nearly all equal), adds once for each run of lanes; and where a bin holds
// an eighth of the keys, its own smallest and largest set the next digits, instead of passes that tell nothing apart.
// us per call, four passes of 8 bits (five launches for tokens) / plain adds and fixed digits / now.  8192 pages: normally
// distributed 9.2 / 7.75 / 8.1, four values 15.7 / 13.1 / 8.9, fifteen in sixteen 0 8.6 / 12.5 / 7.8, a twentieth -infinity beside
// scores within a percent 12.9 / 14.5 / 10.6, one far outlier there 13.0 / 15.0 / 10.6, ascending 9.9 / 12.8 / 8.3.  32768 tokens:
// 20.8 / 17.1 / 17.0, 20.5 / 39.0 / 19.9, 20.6 / 90.3 / 19.3, 20.6 / 42.8 / 23.4, 20.6 / 44.2 / 25.3, 20.6 / 39.1 / 19.0.
// !CROWDS: none of this, up to 2048 pages: 2048 pages 5.6 / 5.8 / 5.9, 8.3 / 7.4 / 5.7, 7.9 / 10.7 / 10.7, 6.9 / 7.6 / 7.8, 7.9 /
// 7.85 / 8.0, 5.7 / 6.7 / 6.8 (with the exact ranges 6.05, 6.5, 7.4, 8.9, 9.1, 7.0).  The passes are a loop, whose code is cold
// in an iteration: token selection at 32768 there 0.7 less than unrolled.  (A first range that leaves masks' scores and a lone
// low one out, with up to four passes: masked and outlier 8.6 and 18.2 at the larger two, but every other call 0.3 to 1.6 more.)
// given: a range that holds all keys taken and the last of them, [base, base + span], instead of the workgroup's smallest and largest key.
// CLEARED: the counts are zero already, with a range (no other call has one) since before a barrier.
template <bool CROWDS = true, int THREADS = kSelectThreads, bool CLEARED = false, int N, typename Valid>
__device__ __forceinline__ LastKey find_last_key(const uint32_t (&key)[N], int full, int live, Valid valid, uint32_t take,
                                                 RegisterSelectShared& sh, const LastKey* given = nullptr) {
  constexpr int kWaves = THREADS / 64;
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  if constexpr (!CLEARED)
    for (int i = tid; i < 3 * 2048 / 4; i += THREADS) reinterpret_cast<u32x4*>(sh.hist)[i] = u32x4{0u, 0u, 0u, 0u};
  LastKey r;
  r.need = take;
  r.whole = false;
  auto set_range = [&](uint32_t hi, uint32_t inv_lo) {              // (the smallest as the largest complement)
    hi = wave_max(hi);
    inv_lo = wave_max(inv_lo);
    if (lane == 0) {
      sh.high[wave] = hi;
      sh.low[wave] = inv_lo;
    }
    __syncthreads();
    hi = __builtin_amdgcn_readfirstlane(wave_max(sh.high[lane & (kWaves - 1)]));
    r.base = ~__builtin_amdgcn_readfirstlane(wave_max(sh.low[lane & (kWaves - 1)]));
    r.span = hi - r.base;
  };
  if (CLEARED && given != nullptr) {
    r.base = given->base;
    r.span = given->span;
  } else {
    uint32_t hi = 0u, inv_lo = 0u;
#pragma unroll
    for (int u = 0; u < N; ++u) {
      if (u >= live) continue;
      hi = max(hi, key[u]);
      if (u < full || valid(u)) inv_lo = max(inv_lo, ~key[u]);
    }
    set_range(hi, inv_lo);
  }
  uint32_t keys = static_cast<uint32_t>(live) * THREADS;     // in the range
  // (Keys without a position lie outside every range unless it starts at 0, the key of NaNs, and are the last there: a bin is
  //  then never taken whole, and of equal keys the first positions are.)
  int shift = max(32 - __builtin_clz(r.span | 1u) - 11, 0);
#pragma unroll 1                              // (later passes find the first one's instructions in the cache)
  for (int pass = 0; pass < 3; ++pass) {
    if (r.span == 0u) break;                                        // all keys are equal: nothing to find
    uint32_t* const h = sh.hist[pass];
    auto digit = [&](int u) { return (key[u] - r.base) >> shift; };
    auto counted = [&](int u) { return key[u] - r.base <= r.span; };
    const uint32_t first = counted(0) ? digit(0) : kNoDigit;
    // (later passes count a fraction of the keys, so that neighbours seldom are both among them)
    const int sharing = !CROWDS || live < 4 ? 0 : sharing_lanes(first);
    if (__builtin_expect(sharing < (pass == 0 ? 8 : 1), 1)) {
#pragma unroll
      for (int u = 0; u < N; ++u) {
        if (u >= live) continue;
        if (counted(u)) atomicAdd(&h[digit(u)], 1u);
      }
    } else if (sharing >= kRunLanes) {
#pragma unroll
      for (int u = 0; u < N; ++u) {
        if (u >= live) continue;
        const uint32_t d = counted(u) ? digit(u) : kNoDigit;
        const uint64_t heads = __builtin_amdgcn_ballot_w64(d != digit_beside(d) || (lane & 15) == 0);
        const uint64_t beyond = (heads >> lane) >> 1;
        if (((heads >> lane) & 1u) && d != kNoDigit) atomicAdd(&h[d], static_cast<uint32_t>(beyond ? __builtin_ctzll(beyond) + 1 : 64 - lane));
      }
    } else {
      uint32_t often[kOften], n[kOften];
      uint64_t left = __builtin_amdgcn_ballot_w64(first != kNoDigit);
#pragma unroll
      for (int c = 0; c < kOften; ++c) {
        n[c] = 0u;
        often[c] = left ? __builtin_amdgcn_readlane(first, __builtin_ctzll(left)) : kNoDigit - 1u;
        left &= ~__builtin_amdgcn_ballot_w64(first == often[c]);
      }
#pragma unroll
      for (int u = 0; u < N; ++u) {
        if (u >= live) continue;
        const uint32_t d = counted(u) ? digit(u) : kNoDigit;
        bool seldom = d != kNoDigit;
#pragma unroll
        for (int c = 0; c < kOften; ++c) {
          n[c] += d == often[c] ? 1u : 0u;
          seldom = seldom && d != often[c];
        }
        if (seldom) atomicAdd(&h[d], 1u);
      }
#pragma unroll
      for (int c = 0; c < kOften; ++c) {
        const uint32_t of_wave = wave_sum(n[c]);
        if (lane == 0 && of_wave != 0u) atomicAdd(&h[often[c]], of_wave);
      }
    }
    __syncthreads();
    if (wave == 0) walk_to_last_bin(h, r.need, sh);
    __syncthreads();
    const uint32_t start = __builtin_amdgcn_readfirstlane(sh.bin) << shift;
    r.base += start;
    r.need = __builtin_amdgcn_readfirstlane(sh.need);
    r.span = min((1u << shift) - 1u, r.span - start);               // (the last bin ends with the range: above it are taken keys)
    const uint32_t count = __builtin_amdgcn_readfirstlane(sh.count);
    r.whole = count == r.need;
    if (shift == 0 || r.whole) break;                       // equal keys, or the whole bin is taken
    shift = max(shift - 11, 0);
    if (CROWDS && __builtin_expect(8u * count >= keys, 0)) {
      uint32_t hi = 0u, inv_lo = 0u;
#pragma unroll
      for (int u = 0; u < N; ++u) {
        if (u >= live || key[u] - r.base > r.span) continue;
        hi = max(hi, key[u]);
        inv_lo = max(inv_lo, ~key[u]);
      }
      set_range(hi, inv_lo);
      shift = max(32 - __builtin_clz(r.span | 1u) - 11, 0);
    }
    keys = count;
  }
  return r;
}

// ROWS x waves cells in LDS, row-major, one per (row, wave), each with two 16-bit counts: lane kCellLanes u + wave / kCellsPerLane of
// the result holds the sum of the cells before cell (u, this wave).  `rows` of them are in use.
template <int ROWS, int THREADS = kSelectThreads>
struct CellWalk {
  static constexpr int kWaves = THREADS / 64;
  static constexpr int kPerLane = ROWS * kWaves > 64 ? ROWS * kWaves / 64 : 1;
  static_assert(kWaves % kPerLane == 0, "a wave's cells sit at one place of their lanes");
  // total: the sum of all cells
  static __device__ __forceinline__ uint32_t before(const uint32_t* cells, int rows, int wave, int lane, uint32_t* total = nullptr) {
    uint32_t part = 0u, all = 0u;
#pragma unroll
    for (int c = 0; c < kPerLane; ++c) {
      const int cell = kPerLane * lane + c;
      const uint32_t v = cell < rows * kWaves ? cells[cell] : 0u;
      if (c < (wave & (kPerLane - 1))) part += v;
      all += v;
    }
    const uint32_t incl = wave_prefix_sum(all);
    if (total != nullptr) *total = __builtin_amdgcn_readlane(incl, 63);
    return incl - all + part;
  }
  static __device__ __forceinline__ int lane_of(int u, int wave) { return (kWaves * u + wave) / kPerLane; }
};

// One workgroup a sequence; prefixes of up to 8 THREADS pages keep their keys in registers.  What bounds it there is latency: two
// dependent requests, then per digit a barrier, one wave's walk through 2048 counts and another barrier, and ahead of them the
// instructions of every wave; with four waves on each SIMD of the one CU these run in turn.  kSelectFewThreads (max_seq_len of up to
// 4096 pages; no general path, no LDS for keys): half the waves to start, to meet at each barrier and to walk for, more keys a thread.
// us per captured call, 1024 threads / 512: 256 pages 5.4 / 4.6 (equal scores 4.0 / 3.4), 1024 pages 5.6 / 4.8, 2048 pages 5.8 / 5.3
// (a twentieth -infinity 7.7 / 7.4), 24 x 1250 pages 6.1 / 5.4, 16 x 4096 pages 6.9 / 6.6; an iteration at 4096 tokens 38.5 -> 36.9,
// at 32768 65.5 -> 65.1.  With 256: 4.5, 5.1, 5.9, 5.8.  Past 4096 pages the keys of 512 would leave the registers.
template <int THREADS>
__global__ __launch_bounds__(THREADS) void select_blocks_kernel(const SelectParams p) {
  extern __shared__ uint32_t skeys[];                 // [min(prefix pages, key_cap)]
  __shared__ __align__(16) RegisterSelectShared reg_shared;
  constexpr bool kGeneral = THREADS == kSelectThreads;  // prefixes of any length
  uint32_t (*hist)[256] = reinterpret_cast<uint32_t (*)[256]>(reg_shared.hist);   // general path: one digit histogram per wave
  static_assert(sizeof(reg_shared.hist) >= (THREADS / 64) * 256 * sizeof(uint32_t), "a histogram per wave");
  __shared__ uint32_t sh_prefix, sh_need, sh_count;
  __shared__ uint32_t wave_take[THREADS / 64], wave_eq[THREADS / 64];
  __shared__ uint32_t cells[kSelectRegRows * (THREADS / 64)];

  const int b = blockIdx.x;
  const int tid = threadIdx.x;
  const int lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  int32_t* sel = p.sel_table + static_cast<int64_t>(b) * p.max_sel_blocks;
  const int32_t* table = p.block_table + static_cast<int64_t>(b) * p.max_blocks;
  const float* scores = p.block_scores + static_cast<int64_t>(b) * p.max_blocks;

  // With at most 8 THREADS pages per row the scores are requested before the sequence length is known (one memory
  // round trip less, and all requests in flight together): every index below max_blocks is a valid address, what
  // lies past the prefix is dropped.
  constexpr int kPre = 8;
  const bool prefetched = !kGeneral || p.max_blocks <= kPre * THREADS;   // (!kGeneral: the prefix fits, whatever the table's width)
  float pre[kPre];
  if (prefetched) {
#pragma unroll
    for (int i = 0; i < kPre; ++i) pre[i] = scores[min(tid + i * THREADS, p.max_blocks - 1)];
  }

  int n = p.seq_lens[b];
  n = n < 0 ? 0 : (n > p.max_tokens ? p.max_tokens : n);
  const int nblk = (n + kPage - 1) / kPage;
  if (nblk == 0) {
    for (int i = tid; i < p.max_sel_blocks; i += THREADS) sel[i] = -1;
    if (tid == 0) p.sel_seq_lens[b] = 0;
    return;
  }
  const int budget = sequence_budget(p.budgets, p.budget_ratio, p.budget_tokens, b, n);
  const int f0 = max(n - p.G, 0) / kPage;            // first forced page
  int nF = nblk - f0;                                // forced pages (1 or 2 for G <= 17)
  int k = min((budget + kPage - 1) / kPage, nblk);
  k = max(k, nF);
  k = min(k, p.max_sel_blocks);                      // device-side clamp; the host rejects this case
  nF = min(nF, k);
  const int kc = k - nF;                             // pages to take from the prefix [0, f0)
  const bool need_search = kc > 0 && kc < f0;
  const bool take_all = kc >= f0;

  // ---- the whole prefix is taken: its pages in order, nothing to search
  if (kc > 0 && take_all) {
    for (int j = tid; j < f0; j += THREADS) sel[j] = table[j];
  }

  // ---- up to 8 THREADS prefix pages: a thread keeps the keys of pages tid, tid + THREADS, ... and their table entries in registers
  auto register_path = [&]() {
    constexpr int kRows = kSelectRegRows;
    const int rows = (f0 + THREADS - 1) / THREADS;          // 1 .. kRows, uniform
    uint32_t key[kRows];
    int32_t page[kRows];
    // (rows past the prefix are skipped by uniform branches: loops stay fully unrolled, arrays in registers)
    float v[kRows];
#pragma unroll
    for (int u = 0; u < kRows; ++u) {
      v[u] = 0.f;
      page[u] = 0;
      if (u < rows) {
        v[u] = (prefetched && u < kPre) ? pre[u < kPre ? u : 0] : scores[min(u * THREADS + tid, f0 - 1)];
        page[u] = table[min(u * THREADS + tid, f0 - 1)];           // coalesced, used if the page is taken
      }
    }
#pragma unroll
    for (int u = 0; u < kRows; ++u) key[u] = tid < f0 - u * THREADS ? score_key(v[u]) : 0u;
    // 2048 pages at most: neither counting by waves nor exact ranges, which cost there what they save (find_last_key).
    auto valid = [&](int u) { return tid < f0 - u * THREADS; };
    LastKey last;
    constexpr int kFewRows = 2048 / THREADS;
    if (rows <= kFewRows) {
      uint32_t few[kFewRows];
#pragma unroll
      for (int u = 0; u < kFewRows; ++u) few[u] = key[u];
      last = find_last_key<false, THREADS>(few, f0 / THREADS, rows, valid, static_cast<uint32_t>(kc), reg_shared);
    } else {
      last = find_last_key<true, THREADS>(key, f0 / THREADS, rows, valid, static_cast<uint32_t>(kc), reg_shared);
    }
    // Cell (row u, wave w) covers the 64 pages from THREADS u + 64 w on; it counts its keys above the last bin (low half) and in
    // it.  A taken page's place: keys above before it + keys in the bin before it, of these at most as many as are taken.
    const uint32_t top = last.base + last.span;
    uint32_t packed = 0u;
#pragma unroll
    for (int u = 0; u < kRows; ++u) {
      if (u >= rows) continue;
      const uint32_t gt = __popcll(__builtin_amdgcn_ballot_w64(key[u] > top));
      const uint32_t eq = __popcll(__builtin_amdgcn_ballot_w64(key[u] - last.base <= last.span));
      if (lane == u) packed = gt | (eq << 16);
    }
    if (lane < rows) cells[lane * (THREADS / 64) + wave] = packed;
    __syncthreads();
    const uint32_t before = CellWalk<kRows, THREADS>::before(cells, rows, wave, lane);
#pragma unroll
    for (int u = 0; u < kRows; ++u) {
      if (u >= rows) continue;
      const bool gt = key[u] > top, eq = key[u] - last.base <= last.span;
      const uint64_t bgt = __builtin_amdgcn_ballot_w64(gt), beq = __builtin_amdgcn_ballot_w64(eq);
      const uint32_t w = __builtin_amdgcn_readlane(before, CellWalk<kRows, THREADS>::lane_of(u, wave));
      const uint32_t e = lanes_below(beq, w >> 16);
      const uint32_t rank = lanes_below(bgt, w & 0xFFFFu) + min(e, last.need);
      if ((gt || (eq && e < last.need)) && rank < static_cast<uint32_t>(p.max_sel_blocks)) sel[rank] = page[u];
    }
  };

  // ---- longer prefixes: keys go to LDS once (up to key_cap of them; beyond that they are recomputed from the scores)
  const bool in_regs = !kGeneral || f0 <= kSelectRegRows * THREADS;
  const bool in_lds = f0 <= p.key_cap;
  if (kGeneral && need_search && !in_regs && in_lds) {
    // groups of kPre independent requests (clamped, so that none sits behind a branch)
    for (int base = tid; base < f0; base += kPre * THREADS) {
      float v[kPre];
#pragma unroll
      for (int i = 0; i < kPre; ++i) v[i] = scores[min(base + i * THREADS, f0 - 1)];
#pragma unroll
      for (int i = 0; i < kPre; ++i)
        if (base + i * THREADS < f0) skeys[base + i * THREADS] = score_key(v[i]);
    }
    __syncthreads();
  }

  // The search and the compaction for prefixes of more than 8192 pages (only reached when a search is needed),
  // compiled once for keys held in LDS and once for keys recomputed from the scores (prefixes longer than the LDS
  // area): the choice is uniform for the workgroup and taken once.
  auto search_and_compact = [&](auto lds_tag) {
    constexpr bool kKeysInLds = decltype(lds_tag)::value;
    auto key_at = [&](int j) -> uint32_t {
      if constexpr (kKeysInLds) return skeys[j];
      else return score_key(scores[j]);
    };

    // ---- radix select: key of the kc-th largest prefix score, and how many of its ties to take.  The search
    //      stops as soon as the digit bin that holds the kc-th key is needed whole (distinct scores: after three
    //      passes as a rule): T then is a key PREFIX, kmask its resolved bits, and every key with that prefix is
    //      a "tie".
    uint32_t T, need_eq, kmask;
    {
      uint32_t prefix = 0u, mask = 0u, need = static_cast<uint32_t>(kc);
#pragma unroll 1
      for (int pass = 0; pass < 4; ++pass) {
        const int shift = 24 - 8 * pass;
        uint32_t* h = hist[wave];
#pragma unroll
        for (int i = 0; i < 4; ++i) h[lane + 64 * i] = 0u;     // wave-private: ordered by the wave's own LDS stream
        // Up to four key rows per trip (independent chains overlap; a wave is bound by instruction issue and
        // latency here).  A row whose active lanes all carry one digit -- the rule for the top byte, where scores
        // cluster -- is counted by one atomic of its first active lane; any other row adds lane by lane.
        auto count_rows = [&](int base, auto rows_tag) {
          constexpr int kR = decltype(rows_tag)::value;
          uint32_t d[kR];
          bool act[kR];
#pragma unroll
          for (int u = 0; u < kR; ++u) {
            const int j = base + u * THREADS + tid;
            const uint32_t key = key_at(min(j, f0 - 1));
            act[u] = j < f0 && (key & mask) == prefix;
            d[u] = (key >> shift) & 255u;
          }
          uint64_t am[kR], same[kR];
          uint32_t dl[kR];
#pragma unroll
          for (int u = 0; u < kR; ++u) {
            am[u] = __builtin_amdgcn_ballot_w64(act[u]);
            const int leader = am[u] ? __builtin_ctzll(am[u]) : 0;
            dl[u] = __builtin_amdgcn_readlane(d[u], leader);
            same[u] = __builtin_amdgcn_ballot_w64(act[u] && d[u] == dl[u]);
          }
#pragma unroll
          for (int u = 0; u < kR; ++u) {
            if (am[u] == 0ull) continue;
            if (same[u] == am[u]) {
              if (lane == 0) atomicAdd(&h[dl[u]], static_cast<uint32_t>(__popcll(am[u])));
            } else if (act[u]) {
              atomicAdd(&h[d[u]], 1u);
            }
          }
        };
        for (int base = 0; base < f0;) {
          const int rows = (f0 - base + THREADS - 1) / THREADS;
          if (rows >= 4) {
            count_rows(base, std::integral_constant<int, 4>{});
            base += 4 * THREADS;
          } else if (rows >= 2) {
            count_rows(base, std::integral_constant<int, 2>{});
            base += 2 * THREADS;
          } else {
            count_rows(base, std::integral_constant<int, 1>{});
            base += THREADS;
          }
        }
        __syncthreads();
        if (wave == 0) {
          // lane l owns bins 4l .. 4l+3; count from the top bin downwards
          uint32_t c[4] = {0u, 0u, 0u, 0u};
          for (int w = 0; w < THREADS / 64; ++w) {
#pragma unroll
            for (int i = 0; i < 4; ++i) c[i] += hist[w][4 * lane + i];
          }
          const uint32_t mine = c[0] + c[1] + c[2] + c[3];
          uint32_t incl = mine;                        // sum over lanes >= lane
#pragma unroll
          for (int off = 1; off < 64; off <<= 1) {
            const uint32_t o = __shfl_down(incl, off, 64);
            if (lane + off < 64) incl += o;
          }
          uint32_t above = incl - mine;                // elements in bins above this lane's bins
#pragma unroll
          for (int i = 3; i >= 0; --i) {
            if (above < need && need <= above + c[i]) {
              sh_prefix = prefix | (static_cast<uint32_t>(4 * lane + i) << shift);
              sh_need = need - above;
              sh_count = c[i];
            }
            above += c[i];
          }
        }
        __syncthreads();
        prefix = sh_prefix;
        need = sh_need;
        mask |= 255u << shift;
        if (sh_count == need) break;         // the whole bin is taken: its lower digits do not matter
      }
      T = prefix;
      need_eq = need;
      kmask = mask;
    }

    // ---- ordered compaction of the prefix: wave w owns the contiguous pages [w*span, (w+1)*span) and walks
    //      them 64 at a time (lane = page), so page order is (wave, step, lane) and every memory access is
    //      coalesced.  Ballots count the keys above T and the ties; a 16-entry prefix over the wave totals turns
    //      the counts into global tie ranks and output positions.
    {
      constexpr int kWaves = THREADS / 64;
      const int span = ((f0 + kWaves - 1) / kWaves + 63) / 64 * 64;
      const int w0 = min(wave * span, f0), w1 = min(w0 + span, f0);
      const uint64_t lt = (1ull << lane) - 1ull;
      // pass A: keys above T and ties in this wave's pages (up to four steps per trip).  A wave's takes follow
      //         from the counts: its keys above T plus as many of its ties as are still wanted.
      uint32_t eq_wave = 0u, gt_wave = 0u;
      {
        auto count_steps = [&](int base, auto steps_tag) {
          constexpr int kS = decltype(steps_tag)::value;
#pragma unroll
          for (int i = 0; i < kS; ++i) {
            const int j = base + 64 * i + lane;
            const uint32_t key = key_at(min(j, f0 - 1)) & kmask;
            eq_wave += __popcll(__builtin_amdgcn_ballot_w64(j < w1 && key == T));
            gt_wave += __popcll(__builtin_amdgcn_ballot_w64(j < w1 && key > T));
          }
        };
        int base = w0;
        for (; base + 64 * 3 < w1; base += 64 * 4) count_steps(base, std::integral_constant<int, 4>{});
        for (; base < w1; base += 64) count_steps(base, std::integral_constant<int, 1>{});
      }
      if (lane == 0) {
        wave_eq[wave] = eq_wave;
        wave_take[wave] = gt_wave;
      }
      __syncthreads();
      uint32_t eq_before = 0u, pos_run = 0u;
      for (int w = 0; w < wave; ++w) {
        const uint32_t e = wave_eq[w];
        const uint32_t wanted = need_eq > eq_before ? need_eq - eq_before : 0u;   // ties still wanted where wave w starts
        pos_run += wave_take[w] + min(e, wanted);
        eq_before += e;
      }
      // pass B: the decisions, now with positions; gather the physical page ids.  The page ids of kGather steps
      //         are requested together and unconditionally (coalesced, clamped): a request per taken page
      //         behind its decision would cost one memory round trip per step.
      constexpr int kGather = 8;
      uint32_t eq_run = eq_before;
      for (int base = w0; base < w1; base += 64 * kGather) {
        int32_t page[kGather];
#pragma unroll
        for (int i = 0; i < kGather; ++i) page[i] = table[min(base + 64 * i + lane, f0 - 1)];
#pragma unroll
        for (int i = 0; i < kGather; ++i) {
          if (base + 64 * i >= w1) break;
          const int j = base + 64 * i + lane;
          const uint32_t key = key_at(min(j, f0 - 1)) & kmask;
          const bool eq = j < w1 && key == T;
          const bool gt = j < w1 && key > T;
          const uint64_t beq = __builtin_amdgcn_ballot_w64(eq);
          const bool take = gt || (eq && eq_run + __popcll(beq & lt) < need_eq);
          eq_run += __popcll(beq);
          const uint64_t btk = __builtin_amdgcn_ballot_w64(take);
          if (take) {
            const uint32_t pos = pos_run + __popcll(btk & lt);
            if (pos < static_cast<uint32_t>(p.max_sel_blocks)) sel[pos] = page[i];
          }
          pos_run += __popcll(btk);
        }
      }
    }
  };
  if (need_search) {
    if (in_regs) register_path();
    if constexpr (kGeneral) {
      if (!in_regs && in_lds) search_and_compact(std::true_type{});
      if (!in_regs && !in_lds) search_and_compact(std::false_type{});
    }
  }

  // ---- forced tail pages, padding, covered length
  for (int i = tid; i < nF; i += THREADS) sel[kc + i] = table[nblk - nF + i];
  for (int i = k + tid; i < p.max_sel_blocks; i += THREADS) sel[i] = -1;
  if (tid == 0) p.sel_seq_lens[b] = kPage * (k - 1) + (n - kPage * (nblk - 1));
}

// Adds the num_new newest token positions of sequence b, whose length now is n_new, to its selection: a new table
// entry whenever a position starts a page of the selection's page size (one thread's work).
__device__ __forceinline__ void extend_selection_row(const ExtendParams& p, int b, int n_new) {
  const int covered = p.sel_seq_lens[b];
  if (covered <= 0) return;
  const int P = p.page_size;
  int32_t* sel = p.sel_table + static_cast<int64_t>(b) * p.max_sel_blocks;
  const int32_t* table = p.block_table + static_cast<int64_t>(b) * p.max_blocks;
  int count = (covered - 1) / P + 1;
  int added = 0;
  for (int i = n_new - p.num_new; i < n_new; ++i) added += (i >= 0 && i % P == 0) ? 1 : 0;
  if (count + added > p.max_sel_blocks) return;            // row full: left as it is
  for (int i = n_new - p.num_new; i < n_new; ++i) {
    if (i >= 0 && i % P == 0) {
      const int page16 = min(i / kPage, p.max_blocks - 1);
      sel[count++] = table[page16] * (kPage / P) + (i % kPage) / P;
    }
  }
  p.sel_seq_lens[b] = covered + p.num_new;
}

// One thread per sequence.
__global__ void extend_selection_kernel(const ExtendParams p) {
  const int b = blockIdx.x * blockDim.x + threadIdx.x;
  if (b >= p.batch) return;
  extend_selection_row(p, b, p.seq_lens[b]);
}

}  // namespace vegas
