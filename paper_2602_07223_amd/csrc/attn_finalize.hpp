// Merge of the per-chunk partial results, and the page-criticality finalisation.
#pragma once
#include <type_traits>

#include "vegas_common.hpp"

namespace vegas {

// Merge of the chunk partials of one output row with the usual max/sum bookkeeping (all in log2 units), for at
// most MAXS (<= 64) chunks, in ONE memory round trip: the sequence length, the
// chunks' (max, sum) pairs (lane s of every wave fetches chunk s) and the thread's element of every
// chunk's partial row are all requested before any of them is used.  Chunks at or past the end of the
// sequence were never written; their slots are loaded all the same (the workspace holds nsplit of them)
// and then discarded.  Addresses are a scalar base plus a 32-bit offset: the kernel is so short that
// 64-bit address arithmetic per load would show in its run time.
template <int MAXS, int SURE = MAXS < 8 ? 0 : MAXS / 2>
struct RowMerge {
  f32x2 mine;        // (max, sum) of chunk `lane`
  float x[MAXS];     // this thread's head dim of every chunk's partial row
  // ml, po: the row's first chunk (wave-uniform); d: head dim of this thread
  // last: the largest chunk index whose slot may be read, not negative (slots past the row's chunks are loaded and discarded)
  __device__ __forceinline__ void issue(const float2* ml, const float* po, int d, int R, int last, int D) {
    const int lane = threadIdx.x & 63;
    const unsigned char* mlb = uniform_ptr(reinterpret_cast<const unsigned char*>(ml));
    const unsigned char* pob = uniform_ptr(reinterpret_cast<const unsigned char*>(po));
    mine = gload<f32x2, false>(mlb, requested_slot(lane, last) * static_cast<uint32_t>(R) * 8u);
    const uint32_t stride = static_cast<uint32_t>(R) * static_cast<uint32_t>(D) * 4u;
    const uint32_t off = static_cast<uint32_t>(d) * 4u;
#pragma unroll
    for (int s = 0; s < MAXS; ++s) x[s] = gload<float, false>(pob, off + requested_slot(s, last) * stride);
    __builtin_amdgcn_sched_barrier(0);     // every request leaves before the first use
  }
  // Output element: sum_s 2^(m_s - m) x_s / sum_s 2^(m_s - m) l_s over the first ns chunks; 0 if no key was visible.
  // Chunks before s_lo were skipped by a call with local masking and hold nothing either.
  __device__ __forceinline__ float finish(int ns, int s_lo = 0) const {
    const int lane = threadIdx.x & 63;
    return finish(lane >= s_lo && lane < ns);
  }
  // The same for the chunks s whose lane s says `live`.
  __device__ __forceinline__ float finish(bool live) const {
    const uint64_t lives = __builtin_amdgcn_ballot_w64(live);
    const float ms = live ? mine[0] : -INFINITY;
    const float m = wave_max(ms);
    const float m_use = (m == -INFINITY) ? 0.f : m;
    const float w = fast_exp2(ms - m_use);              // 0 for lanes at or past ns
    const float L = wave_sum(live ? w * mine[1] : 0.f);
    // Four sums, whose steps do not wait for each other.  Elements are looked at only where a slot may not be live, so that one that is not
    // (unwritten, or the row's last one once more) never meets a weight: 0 times an infinity is no 0.  SURE: slots that are live if
    // all requested ones are, by the rule that chose MAXS; behind them four at a time, those that hold nothing left out.  us per iteration,
    // no slot looked at where all requested ones are live / all by fours / so: 32768 tokens 65.4 / 65.4 / 65.2, live 69.4 / 70.1 / 69.5,
    // 131072 (33 chunks) 150.5 / 147.4 / 147.0.  (One sum with a test per element, the merge alone, captured: 22 chunks 2.31 against 2.18 us, 33
    // 2.71 against 2.62.)
    float acc[4] = {0.f, 0.f, 0.f, 0.f};
    auto add_up = [&](auto first, auto end, auto all) {
#pragma unroll
      for (int s = decltype(first)::value; s < decltype(end)::value; ++s) {
        const float ws = __uint_as_float(__builtin_amdgcn_readlane(__float_as_uint(w), s));
        acc[s & 3] = __builtin_fmaf(ws, decltype(all)::value || ((lives >> s) & 1u) ? x[s] : 0.f, acc[s & 3]);
      }
    };
    using none = std::integral_constant<int, 0>;
    using sure = std::integral_constant<int, SURE>;
    if ((~lives & ((1ull << SURE) - 1ull)) == 0u) add_up(none{}, sure{}, std::true_type{});
    else add_up(none{}, sure{}, std::false_type{});
    auto rest = [&](auto at) {
      constexpr int s0 = SURE + 4 * decltype(at)::value;
      if constexpr (s0 < MAXS)
        if ((static_cast<uint32_t>(lives >> s0) & 15u) != 0u) add_up(std::integral_constant<int, s0>{}, std::integral_constant<int, s0 + 4>{}, std::false_type{});
    };
    static_assert(MAXS - SURE <= 32 && (MAXS - SURE) % 4 == 0, "eight groups of four");
    rest(std::integral_constant<int, 0>{});
    rest(std::integral_constant<int, 1>{});
    rest(std::integral_constant<int, 2>{});
    rest(std::integral_constant<int, 3>{});
    rest(std::integral_constant<int, 4>{});
    rest(std::integral_constant<int, 5>{});
    rest(std::integral_constant<int, 6>{});
    rest(std::integral_constant<int, 7>{});
    return (L > 0.f) ? ((acc[0] + acc[1]) + (acc[2] + acc[3])) / L : 0.f;
  }
};

// One workgroup of D threads (= head dims; 128 or 64) per (query row, KV head, sequence): merges the
// chunk partials of that row and writes the bf16 output row (Eq. 1), for any number of chunks and for balanced
// chunking, where a sequence has few of its head's slots and how many is known once the plan has been read: they, and
// no others, are then requested together.  Many chunks take two passes: the (max, sum) pairs, fetched by one thread
// each, then the partial rows.
// Lengths: GrownLengths in a draft step, otherwise nothing.
template <typename... Lengths>
__global__ __launch_bounds__(128) void attn_combine_kernel(const CombineParams p, const Lengths... lengths) {
  __shared__ float sw[128];
  __shared__ float sred[4];
  const int r = blockIdx.x, h = blockIdx.y, b = blockIdx.z;
  const int tid = threadIdx.x;
  const int wave = tid >> 6;
  const int T = p.D;                                              // threads of this workgroup = head dims
  int n = p.lens[b];
  n = n < 0 ? 0 : (n > p.max_tokens ? p.max_tokens : n);
  const ColumnSlots cs = column_slots(p.plan, p.slots_total, b, p.Hkv, p.nsplit, p.chunk_tokens);
  const ColumnChunks cc = column_chunks(cs, n);
  const int ns = cc.ns;
  const int64_t pbase = cs.off + static_cast<int64_t>(h) * cs.stride_h;
  const float2* ml = p.part_ml + pbase * p.R + r;                 // stride R between chunks
  const float* po = p.part_o + (pbase * p.R + r) * T + tid;       // stride R*D between chunks
  const int64_t ostride = static_cast<int64_t>(p.R) * T;

  const int s_lo = first_live_chunk(n, p.G, p.window, cs.chunk);   // earlier chunks were skipped (local masking)
  const int t = r / p.g, j = r % p.g;
  uint16_t* const out = p.out + ((static_cast<int64_t>(b) * p.G + t) * p.Hq + h * p.g + j) * T + tid;
  if ((r | h | tid) == 0) (lengths.store(b), ...);
  if (cc.last < 0) {                         // an empty sequence: it may own no slot, so nothing is requested
    *out = 0;
    return;
  }
  if (ns <= 32) {
    auto merge = [&](auto maxs) {
      RowMerge<decltype(maxs)::value> rm;
      rm.issue(ml, po - tid, tid, p.R, cc.last, T);
      return rm.finish(ns, s_lo);
    };
    float o;
    if (ns <= 4) o = merge(std::integral_constant<int, 4>{});
    else if (ns <= 8) o = merge(std::integral_constant<int, 8>{});
    else if (ns <= 16) o = merge(std::integral_constant<int, 16>{});
    else o = merge(std::integral_constant<int, 32>{});
    *out = float_to_bf16_bits(o);
    return;
  }
  // pass 1: global max over chunks
  float m = -INFINITY;
  for (int s = s_lo + tid; s < ns; s += T) m = fmaxf(m, ml[static_cast<int64_t>(s) * p.R].x);
  m = wave_max(m);
  if ((tid & 63) == 0) sred[wave] = m;
  __syncthreads();
  m = T > 64 ? fmaxf(sred[0], sred[1]) : sred[0];
  const float m_use = (m == -INFINITY) ? 0.f : m;

  // pass 2: weights of up to D chunks at a time, then the weighted sum of the partial rows
  float accv = 0.f, L = 0.f;
  for (int s0 = s_lo; s0 < ns; s0 += T) {
    const int cnt = min(T, ns - s0);
    float wl = 0.f;
    if (tid < cnt) {
      const float2 v = ml[static_cast<int64_t>(s0 + tid) * p.R];
      const float w = fast_exp2(v.x - m_use);
      sw[tid] = w;
      wl = w * v.y;
    }
    wl = wave_sum(wl);
    if ((tid & 63) == 0) sred[2 + wave] = wl;
    __syncthreads();
    L += T > 64 ? sred[2] + sred[3] : sred[2];
    int s = 0;
    for (; s + 4 <= cnt; s += 4) {
      const float x0 = po[(s0 + s) * ostride], x1 = po[(s0 + s + 1) * ostride];
      const float x2 = po[(s0 + s + 2) * ostride], x3 = po[(s0 + s + 3) * ostride];
      accv += sw[s] * x0 + sw[s + 1] * x1 + sw[s + 2] * x2 + sw[s + 3] * x3;
    }
    for (; s < cnt; ++s) accv += sw[s] * po[(s0 + s) * ostride];
    __syncthreads();
  }
  const float o = (L > 0.f) ? accv / L : 0.f;
  *out = float_to_bf16_bits(o);
}

// Numbers of chunks that the kernel below is built for.  A call takes the first that is not below its own, so it has more slots than the step before.
constexpr int kSmallMerges[] = {8, 12, 16, 20, 24, 32, 40, 48, 64};
constexpr int small_merge_below(int maxs) {
  int below = 0;
  for (int step : kSmallMerges) below = step < maxs ? step : below;
  return below;
}

// (Uniform chunking.  A chunk is live if the sequence reaches it, no count is needed; a row's token comes from one reciprocal, r <
// 128: integer divisions are two dozen instructions each, in a kernel of one round trip.)
template <int MAXS, typename... Lengths>
__global__ __launch_bounds__(128) void attn_combine_small_kernel(VEGAS_COMBINE_SMALL_PARAMS, const Lengths... lengths) {   // launched with D threads
  const int r = blockIdx.x, h = blockIdx.y, b = blockIdx.z;
  const int tid = threadIdx.x, lane = tid & 63;
  const int R = shape & 255, D = (shape >> 8) & 255, nsplit = shape >> 16;
  const int64_t row = (static_cast<int64_t>(b) * Hkv + h) * nsplit * R + r;
  int zero = 0;
  asm("" : "+v"(zero));                      // (a vector load, the first to come back: the compiler puts a scalar one last)
  int n = lens[b + zero];
  RowMerge<MAXS, small_merge_below(MAXS)> rm;
  rm.issue(part_ml + row, part_o + row * D, tid, R, nsplit - 1, D);
  if ((r | h | tid) == 0) (lengths.store(b), ...);
  const int t = static_cast<int>((static_cast<float>(r) + 0.5f) * __builtin_amdgcn_rcpf(static_cast<float>(g)));
  const int64_t at = ((static_cast<int64_t>(b) * R + t * g) * Hkv + h * g + (r - t * g)) * D;
  uint16_t* const dst = out + at + tid;
  n = __builtin_amdgcn_readfirstlane(n);
  n = n < 0 ? 0 : (n > max_tokens ? max_tokens : n);
  int s_lo = 0;
  if (window > 0) s_lo = first_live_chunk(n, R / g, window, chunk_tokens);
  // (a chunk that starts past 2^31 tokens is behind every end)
  const bool live = lane >= s_lo && static_cast<uint64_t>(static_cast<uint32_t>(lane)) * static_cast<uint32_t>(chunk_tokens) < static_cast<uint32_t>(n);
  *dst = float_to_bf16_bits(rm.finish(live));
}

// Verification epilogue in ONE launch (a kernel boundary costs ~3 us on this GPU): workgroups
// [0, nA) merge the chunk partials of a few query rows each (as the combine kernels do) and write
// the bf16 output rows (Eq. 1); workgroups [nA, nA + nB) turn the per-(row, page) log-sum-exps of
// 32 pages into page criticalities (Eq. 2 / Eq. 3 with weights, averaged over rows and heads as in the
// last paragraph of Sec. 3.3): score[b][j] = inv_norm * sum_h sum_{rows in R} 2^(page_lse - row_lse).
// A score workgroup derives the global row log-sum-exps itself from the chunks' (max, sum) pairs,
// so it does not depend on the merge workgroups.  Pages at or beyond the sequence's page count get 0.
// MAXS > 0: at most MAXS chunks, the merge workgroups take the one-round-trip path; 0: any number; kFinPlanned:
// balanced chunking (any number, usually few; merge_planned_rows).
// Loads are ordered so that a workgroup's dependent memory round trips are as few as possible: the
// kernel runs for a handful of microseconds and every trip is a sizeable part of that.
constexpr int kFinPlanned = -1;
constexpr int kFinPlannedSmall = -2;   // the same in a call of few rows: merged a head dim per thread, pages scored row by row
constexpr int kFinPre = 8;       // page log-sum-exps a score thread keeps in registers: 4 * kFinPre rows
constexpr int kFinRounds = 3, kFinWideRounds = 5;   // rounds of 64 rows whose pairs a wave of a score workgroup has in flight (finalize_is_wide)

// Merge under balanced chunking: 1024 / D consecutive rows of the Hkv R rows per workgroup, a thread has four head dims of
// one, and asks for the slots of its sequence (few as a rule, and known by now: the plan had to be read first) four or eight at a
// time, (max, sum) pairs and partial rows together.  A batch has thousands of rows, so it is not one row's round trip that
// counts but how many workgroups have to follow one another.  (With the page values below, by the profiler: 16 sequences of 8K..64K
// tokens, 40 rows 20.4 -> 17.3 us, 24 of 1K..20K, 32 rows 13.7 -> 10.0; 4 of 64K, 20 rows 7.9 -> 7.9.)
__device__ __forceinline__ void merge_planned_rows(const FinalizeParams& p, const ColumnSlots& cs, int b, int n, int HR) {
  const int per_row = p.D >> 2;                                   // threads
  const int rr = static_cast<int>(blockIdx.x) * (256 / per_row) + static_cast<int>(threadIdx.x) / per_row;
  const int d = 4 * (static_cast<int>(threadIdx.x) & (per_row - 1));
  if (rr >= HR) return;
  const int h = static_cast<int>((static_cast<float>(rr) + 0.5f) * __builtin_amdgcn_rcpf(static_cast<float>(p.R)));   // rr / R < 2^15
  const int r = rr - h * p.R;
  const int64_t row = (cs.off + static_cast<int64_t>(h) * cs.stride_h) * p.R + r;   // of the first slot; R rows between slots
  const float2* const ml = p.part_ml + row;
  const float* const po = p.part_o + row * p.D + d;
  const ColumnChunks cc = column_chunks(cs, n);
  float m = -INFINITY, L = 0.f;
  f32x4 acc = {0.f, 0.f, 0.f, 0.f};
  auto slots = [&](int s0, auto tag) {
    constexpr int N = decltype(tag)::value;
    float2 v[N];
    f32x4 x[N];
#pragma unroll
    for (int s = 0; s < N; ++s) {
      const int64_t at = static_cast<int64_t>(requested_slot(s0 + s, cc.last)) * p.R;
      v[s] = ml[at];
      x[s] = *reinterpret_cast<const f32x4*>(po + at * p.D);
    }
    __builtin_amdgcn_sched_barrier(0);       // every request leaves before the first use
    float top = m;
#pragma unroll
    for (int s = 0; s < N; ++s)
      if (s0 + s < cc.ns) top = fmaxf(top, v[s].x);
    const float use = (top == -INFINITY) ? 0.f : top;
    const float old = fast_exp2(m - use);
    L *= old;
    acc *= old;
    m = top;
#pragma unroll
    for (int s = 0; s < N; ++s) {
      if (s0 + s < cc.ns) {
        const float w = fast_exp2(v[s].x - use);
        L += w * v[s].y;
        acc += w * x[s];
      }
    }
  };
  if (cc.last >= 0) {                        // (an empty sequence may own no slot, so nothing is requested)
    if (cc.ns <= 4) slots(0, std::integral_constant<int, 4>{});
    else for (int s0 = 0; s0 < cc.ns; s0 += 8) slots(s0, std::integral_constant<int, 8>{});
  }
  f32x4 o;
#pragma unroll
  for (int e = 0; e < 4; ++e) o[e] = (L > 0.f) ? acc[e] / L : 0.f;
  const int t = r / p.g, j = r % p.g;
  u32x2 packed;
  packed[0] = static_cast<uint32_t>(float_to_bf16_bits(o[0])) | (static_cast<uint32_t>(float_to_bf16_bits(o[1])) << 16);
  packed[1] = static_cast<uint32_t>(float_to_bf16_bits(o[2])) | (static_cast<uint32_t>(float_to_bf16_bits(o[3])) << 16);
  *reinterpret_cast<u32x2*>(p.out + ((static_cast<int64_t>(b) * p.G + t) * p.Hq + h * p.g + j) * p.D + d) = packed;
}

// Role B's page sums of rows that no thread has in registers: page j, heads slot, slot + 8, ...
__device__ __forceinline__ float page_by_rows(const FinalizeParams& p, const float* sm_row, int b, int slot, int j) {
  const int Rc = p.Rc;
  float sc = 0.f;
  auto add = [&](float x, float rl) { sc += rl != -INFINITY ? fast_exp2(x - rl) : 0.f; };
  for (int h = slot; h < p.Hkv; h += 8) {
    const float* pl = p.page_lse + ((static_cast<int64_t>(b) * p.Hkv + h) * p.lse_pages + j) * Rc;
    const float* rl = sm_row + h * Rc;
    if ((Rc & 3) == 0) {
      for (int r = 0; r < Rc; r += 4) {
        const f32x4 x = *reinterpret_cast<const f32x4*>(pl + r);
        const f32x4 of = *reinterpret_cast<const f32x4*>(rl + r);
#pragma unroll
        for (int e = 0; e < 4; ++e) add(x[e], of[e]);
      }
    } else {
      // (Eight requests at a time: one by one a page's rows are as many round trips, 77 rows 48 us for the kernel.)
      for (int r = 0; r < Rc; r += 8) {
        float x[8];
#pragma unroll
        for (int e = 0; e < 8; ++e) x[e] = pl[min(r + e, Rc - 1)];
#pragma unroll
        for (int e = 0; e < 8; ++e)
          if (r + e < Rc) add(x[e], rl[r + e]);
      }
    }
  }
  return sc;
}
// The score of page j (lanes of the first 32 threads): the sums of the eight head slots.
__device__ __forceinline__ void store_page_scores(const FinalizeParams& p, const float* sm_sum, float* out_row, int j, int nblk) {
  if (threadIdx.x >= 32 || j >= p.max_blocks) return;
  float tot = 0.f;
#pragma unroll
  for (int q = 0; q < 8; ++q) tot += sm_sum[q * 32 + threadIdx.x];
  out_row[j] = (j < nblk) ? tot * p.inv_norm : 0.f;
}

// Page criticality of 32 pages for at most MAXS (<= 64) chunks (MANY: any number, MAXS at a time) that the host cut, all of a head's slots its own: the global log-sum-exp of
// every collected row from its chunks' (max, sum) pairs, then the sums over rows and heads.
// Wave w takes the chunks MAXS / 4 w .., lane and round the row: a pair's address is a uniform base per chunk and a 32-bit offset per row, one
// division (by a reciprocal) per round, and whether a chunk counts is uniform.  Four waves with a compute unit to themselves have nothing
// that hides an instruction: of 10600 cycles at 160 rows and 32 chunks 2500 went into the addresses of 24 pairs a thread (a unit of four
// chunks of one row each, with two integer divisions), 2900 into merging them in two stages.  us for merge and scores, captured, units of
// four chunks / this: 20 rows of 8 heads 4096 tokens 5.4 / 4.3, 32768 5.5 / 4.3; 28 rows, 131072 7.7 / 5.6; 32 rows, 50000 9.9 / 5.8; 40 rows,
// head dimension 64, 32768 7.8 / 5.5; 48 rows, 8192 10.8 / 5.8, two of twelve tokens', 32768 6.0 / 3.8; 56 rows, 131072 11.9 / 7.8; 96 rows, head
// dimension 64, 20000 14.8 / 8.0; one head, 700 4.1 / 3.1.
template <int MAXS, int ROUNDS, bool MANY>
__device__ __forceinline__ void score_pages(const FinalizeParams& p, float* smf, int b) {
  static_assert(MAXS > 0, "a bound on the chunks");
  constexpr int NC = MAXS / 4;                // chunks of a wave
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int Rc = p.Rc, rows = p.Hkv * Rc;     // the collected rows
  const int jbase = (static_cast<int>(blockIdx.x) - p.nA) * 32, pg = tid & 31, slot = tid >> 5;
  float2* const sm_pair = reinterpret_cast<float2*>(smf);          // [wave][rows] (max, sum) of a row over a wave's chunks
  float* const sm_row = smf + ((8 * rows + 3) & ~3);               // [rows] global log-sum-exp; -inf for rows that do not count
  float* const sm_sum = smf + ((8 * rows + 3) & ~3) + ((rows + 3) & ~3);     // [8][32]
  int zero = 0;
  asm("" : "+v"(zero));                       // (a vector load, the first to come back: a scalar one is waited for at once)
  int n = p.lens[b + zero];
  const unsigned char* const ml = reinterpret_cast<const unsigned char*>(p.part_ml + static_cast<int64_t>(b) * p.Hkv * p.nsplit * p.R);
  const uint32_t chunk_bytes = static_cast<uint32_t>(p.R) * 8u;
  const float rcp_rc = __builtin_amdgcn_rcpf(static_cast<float>(Rc));
  const bool all = p.collect_rows == 1 || p.G <= 2;
  f32x2 v[ROUNDS][NC];
  auto load_pairs = [&](int base, int first) {
#pragma unroll
    for (int a = 0; a < ROUNDS; ++a) {
      const int i = min(first + 64 * a + lane, rows - 1);
      const int h = static_cast<int>((static_cast<float>(i) + 0.5f) * rcp_rc), c = i - h * Rc;
      const int r = all || c < p.g ? c : c + (p.G - 2) * p.g;      // (collected_row)
      const uint32_t off = static_cast<uint32_t>(h) * static_cast<uint32_t>(p.nsplit) * chunk_bytes + static_cast<uint32_t>(r) * 8u;
#pragma unroll
      for (int q = 0; q < NC; ++q)
        v[a][q] = gload<f32x2, false>(uniform_ptr(ml + static_cast<uint64_t>(min(base + wave * NC + q, p.nsplit - 1)) * chunk_bytes), off);
    }
  };
  load_pairs(0, 0);
  // The thread's page values, where they are few, are requested behind the pairs: they are needed last.
  const bool pre_ok = (Rc & 3) == 0 && Rc <= 4 * kFinPre && p.Hkv <= 8;
  f32x4 pre[kFinPre];
  if (pre_ok && slot < p.Hkv) {
    const float* pl = p.page_lse + ((static_cast<int64_t>(b) * p.Hkv + slot) * p.lse_pages + min(jbase + pg, p.lse_pages - 1)) * Rc;
#pragma unroll
    for (int q = 0; q < kFinPre; ++q)
      if (4 * q < Rc) pre[q] = *reinterpret_cast<const f32x4*>(pl + 4 * q);
  }
  float* const out_row = p.block_scores + static_cast<int64_t>(b) * p.max_blocks;
  n = __builtin_amdgcn_readfirstlane(n);
  n = n < 0 ? 0 : (n > p.max_tokens ? p.max_tokens : n);
  const int nblk = (n + kPage - 1) / kPage;
  if (jbase >= nblk) {                        // whole workgroup past the sequence
    if (tid < 32 && jbase + tid < p.max_blocks) out_row[jbase + tid] = 0.f;
    return;
  }
  for (int base = 0; base == 0 || (MANY && static_cast<int64_t>(base) * p.chunk_tokens < n); base += MAXS) {
    int mine = 0;                             // chunks of this wave that the sequence reaches
#pragma unroll
    for (int q = 0; q < NC; ++q) mine += static_cast<int64_t>(base + wave * NC + q) * p.chunk_tokens < n ? 1 : 0;
    auto merge = [&](const f32x2 (&x)[NC], float2 before, auto whole) {
      float m = before.x, L = 0.f;
#pragma unroll
      for (int q = 0; q < NC; ++q)
        if (decltype(whole)::value || q < mine) m = fmaxf(m, x[q][0]);
      const float mu = (m == -INFINITY) ? 0.f : m;
      if constexpr (MANY) L = before.y * fast_exp2(before.x - mu);
#pragma unroll
      for (int q = 0; q < NC; ++q)
        if (decltype(whole)::value || q < mine) L += x[q][1] * fast_exp2(x[q][0] - mu);
      return make_float2(m, L);
    };
    for (int first = 0; first < rows; first += 64 * ROUNDS) {
      if ((MANY && base > 0) || first > 0) load_pairs(base, first);
#pragma unroll
      for (int a = 0; a < ROUNDS; ++a) {
        const int i = first + 64 * a + lane;
        if (first + 64 * a >= rows) continue;
        float2 pair = make_float2(-INFINITY, 0.f);
        if (MANY && base > 0) pair = sm_pair[wave * rows + min(i, rows - 1)];
        pair = mine == NC ? merge(v[a], pair, std::true_type{}) : merge(v[a], pair, std::false_type{});
        if (i < rows) sm_pair[wave * rows + i] = pair;
      }
    }
  }
  __syncthreads();
  for (int i = tid; i < rows; i += 256) {
    float2 w[4];
#pragma unroll
    for (int q = 0; q < 4; ++q) w[q] = sm_pair[q * rows + i];
    const float m = fmaxf(fmaxf(w[0].x, w[1].x), fmaxf(w[2].x, w[3].x));
    const float mu = (m == -INFINITY) ? 0.f : m;
    float L = 0.f;
#pragma unroll
    for (int q = 0; q < 4; ++q) L += w[q].y * fast_exp2(w[q].x - mu);
    sm_row[i] = (L > 0.f) ? mu + fast_log2(L) : -INFINITY;
  }
  __syncthreads();
  const int j = jbase + pg;
  float sc = 0.f;
  auto add = [&](float x, float rl) { sc += rl != -INFINITY ? fast_exp2(x - rl) : 0.f; };
  if (j < nblk) {
    if (pre_ok) {
      if (slot < p.Hkv) {
#pragma unroll
        for (int q = 0; q < kFinPre; ++q) {
          if (4 * q < Rc) {
            const f32x4 rl = *reinterpret_cast<const f32x4*>(sm_row + slot * Rc + 4 * q);
#pragma unroll
            for (int e = 0; e < 4; ++e) add(pre[q][e], rl[e]);
          }
        }
      }
    } else {
      sc = page_by_rows(p, sm_row, b, slot, j);
    }
  }
  sm_sum[slot * 32 + pg] = sc;
  __syncthreads();
  store_page_scores(p, sm_sum, out_row, j, nblk);
}

// The same under balanced chunking, for sequence b of n tokens with the slots cs: the sequence has few chunks as a rule, so a thread has a
// row, and asks for four or eight of its pairs at a time, with one division by a reciprocal for their address.  us for merge and scores,
// captured, units of four chunks of a row behind integer divisions, length read after the plan / this: 24 sequences of 1001..20011, 32 rows
// 9.1 / 7.8; 16 of 8192..65536, 40 rows 15.0 / 14.5; 4 of 65536, 20 rows 6.0 / 5.2; 2 of 900..1500 5.5 / 4.5; 32 of 300..1500 5.9 / 5.3.
// SMALL: page values are read page by page, a thread those of its page and head, as in score_pages; otherwise as they lie: a wave has every
// fourth head, whose 32 pages are one run of quads of rows, and a quad's sum goes through LDS to the thread that adds up its page.
// (A thread that reads the rows of its page itself, 128 or 160 bytes apart from its neighbour's, touches every line of the run with every request;
// figures: merge_planned_rows.  One sequence, and calls of few rows, are better off with that all the same, their score workgroups wait
// for latency and not for requests: us per iteration, page by page / by quads, 4096 tokens 44.0 / 44.6, 32768 69.7 / 70.6, 131072 157.8 /
// 158.5.)
template <bool SMALL>
__device__ __forceinline__ void score_pages_planned(const FinalizeParams& p, const ColumnSlots& cs, float* smf, int b, int n) {
  constexpr int kRuns = 5;                    // requests per head in flight, of two heads
  constexpr int kFewHeads = 3;                // where a head's run is one or two requests: heads in flight
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int Rc = p.Rc, rows = p.Hkv * Rc;
  const int jbase = (static_cast<int>(blockIdx.x) - p.nA) * 32, pg = tid & 31, slot = tid >> 5, j = jbase + pg;
  float* const out_row = p.block_scores + static_cast<int64_t>(b) * p.max_blocks;
  const int nblk = (n + kPage - 1) / kPage;
  if (jbase >= nblk) {                        // whole workgroup past the sequence
    if (tid < 32 && j < p.max_blocks) out_row[j] = 0.f;
    return;
  }
  const ColumnChunks cc = column_chunks(cs, n);
  float* const sm_row = smf;                                       // [rows] global log-sum-exp; -inf for rows that do not count
  float* const sm_sum = smf + ((rows + 3) & ~3);                   // [8][32]
  float* const sm_quad = sm_sum + 256;                             // [Hkv * 32][pitch]
  const float rcp_rc = __builtin_amdgcn_rcpf(static_cast<float>(Rc));
  const bool all = p.collect_rows == 1 || p.G <= 2;
  const float2* const ml = p.part_ml + cs.off * p.R;
  auto row_pairs = [&](int i) {               // the first of row i's pairs
    const int h = static_cast<int>((static_cast<float>(i) + 0.5f) * rcp_rc), c = i - h * Rc;
    const int r = all || c < p.g ? c : c + (p.G - 2) * p.g;        // (collected_row)
    return ml + static_cast<int64_t>(h) * cs.stride_h * p.R + r;
  };
  float m = -INFINITY, L = 0.f;
  auto add_pairs = [&](const float2* at, int s0, auto tag) {
    constexpr int N = decltype(tag)::value;
    float2 v[N];
#pragma unroll
    for (int s = 0; s < N; ++s) v[s] = at[static_cast<int64_t>(requested_slot(s0 + s, cc.last)) * p.R];
    __builtin_amdgcn_sched_barrier(0);       // every request leaves before the first use
    const float old = m;
#pragma unroll
    for (int s = 0; s < N; ++s)
      if (s0 + s < cc.ns) m = fmaxf(m, v[s].x);
    const float mu = (m == -INFINITY) ? 0.f : m;
    L *= fast_exp2(old - mu);
#pragma unroll
    for (int s = 0; s < N; ++s)
      if (s0 + s < cc.ns) L += v[s].y * fast_exp2(v[s].x - mu);
  };
  auto row_lse = [&](int i) {
    const float2* const at = row_pairs(min(i, rows - 1));
    m = -INFINITY;
    L = 0.f;
    if (cc.ns <= 4) add_pairs(at, 0, std::integral_constant<int, 4>{});
    else for (int s0 = 0; s0 < cc.ns; s0 += 8) add_pairs(at, s0, std::integral_constant<int, 8>{});
    if (i < rows) sm_row[i] = (L > 0.f) ? (m == -INFINITY ? 0.f : m) + fast_log2(L) : -INFINITY;
  };
  // page values requested before the rows' pairs are back
  const int q4 = Rc >> 2, run = 32 * q4;                           // quads of a page, of a head's run
  const int run_live = min(32, p.lse_pages - jbase) * q4;          // quads of a run that exist
  const bool pre_ok = SMALL && (Rc & 3) == 0 && Rc <= 4 * kFinPre && p.Hkv <= 8;
  const bool by_quads = !SMALL && (Rc & 3) == 0;
  f32x4 pre[SMALL ? kFinPre : 2 * kRuns];
  const float* const lse_base = p.page_lse + (static_cast<int64_t>(b) * p.Hkv * p.lse_pages + jbase) * Rc;
  auto load_quads = [&](int h, int first) {
#pragma unroll
    for (int a = 0; a < 2 * kRuns; ++a) {
      const int hd = h + 4 * (a / kRuns), i = first + 64 * (a % kRuns) + lane;
      if (hd >= p.Hkv || first + 64 * (a % kRuns) >= run) continue;
      pre[SMALL ? 0 : a] = *reinterpret_cast<const f32x4*>(lse_base + static_cast<int64_t>(hd) * p.lse_pages * Rc + 4 * min(i, run_live - 1));
    }
  };
  if (pre_ok && slot < p.Hkv) {
    const float* pl = p.page_lse + ((static_cast<int64_t>(b) * p.Hkv + slot) * p.lse_pages + min(j, p.lse_pages - 1)) * Rc;
#pragma unroll
    for (int q = 0; q < kFinPre; ++q)
      if (4 * q < Rc) pre[SMALL ? q : 0] = *reinterpret_cast<const f32x4*>(pl + 4 * q);
  }
  // (At most two requests a head, up to 16 rows: three heads at a time, behind the rows.  Two, the first of them ahead, are as many round trips again where
  //  there are many heads: 64 heads x 12 rows, head dimension 128, 32 sequences of 1000 19.8 / 18.3, 3 of 30000 13.3 / 12.0; x 8 rows, 16 of 3000
  //  11.1 / 10.6.  More at a time are registers that cost two workgroups on a compute unit.)
  const bool few = run <= 128;
  if (by_quads && !few) load_quads(wave, 0);
  for (int first = 0; first < rows; first += 256) row_lse(first + tid);
  __syncthreads();
  auto add = [&](float& sum, float x, float rl) { sum += rl != -INFINITY ? fast_exp2(x - rl) : 0.f; };
  float sc = 0.f;
  if (by_quads) {
    const float rcp_q4 = __builtin_amdgcn_rcpf(static_cast<float>(q4));
    const int pitch = q4 | 1;
    if (few) {
      const int i0 = min(lane, run_live - 1), i1 = min(64 + lane, run_live - 1);
      const int page0 = static_cast<int>((static_cast<float>(lane) + 0.5f) * rcp_q4), page1 = static_cast<int>((static_cast<float>(64 + lane) + 0.5f) * rcp_q4);
      const int q0 = lane - page0 * q4, q1 = 64 + lane - page1 * q4;
      for (int h = wave; h < p.Hkv; h += 4 * kFewHeads) {
        f32x4 x[kFewHeads][2];
#pragma unroll
        for (int k = 0; k < kFewHeads; ++k) {
          const float* const head = lse_base + static_cast<int64_t>(min(h + 4 * k, p.Hkv - 1)) * p.lse_pages * Rc;
          x[k][0] = *reinterpret_cast<const f32x4*>(head + 4 * i0);
          x[k][1] = *reinterpret_cast<const f32x4*>(head + 4 * i1);
        }
#pragma unroll
        for (int k = 0; k < kFewHeads; ++k) {
          const int hd = h + 4 * k;
          if (hd >= p.Hkv) break;
          float s0 = 0.f, s1 = 0.f;
          const f32x4 r0 = *reinterpret_cast<const f32x4*>(sm_row + hd * Rc + 4 * q0), r1 = *reinterpret_cast<const f32x4*>(sm_row + hd * Rc + 4 * q1);
#pragma unroll
          for (int e = 0; e < 4; ++e) {
            add(s0, x[k][0][e], r0[e]);
            add(s1, x[k][1][e], r1[e]);
          }
          if (lane < run) sm_quad[(hd * 32 + page0) * pitch + q0] = s0;
          if (64 + lane < run) sm_quad[(hd * 32 + page1) * pitch + q1] = s1;
        }
      }
    }
    for (int h = wave; !few && h < p.Hkv; h += 8) {
      for (int first = 0; first < run; first += 64 * kRuns) {
        if (h != wave || first > 0) load_quads(h, first);
#pragma unroll
        for (int t = 0; t < kRuns; ++t) {
          const int i = first + 64 * t + lane;
          if (first + 64 * t >= run) continue;
          const int page = static_cast<int>((static_cast<float>(i) + 0.5f) * rcp_q4), q = i - page * q4;
#pragma unroll
          for (int two = 0; two < 2; ++two) {
            const int hd = h + 4 * two;
            if (hd >= p.Hkv || i >= run) continue;
            const f32x4 x = pre[SMALL ? 0 : two * kRuns + t], rl = *reinterpret_cast<const f32x4*>(sm_row + hd * Rc + 4 * q);
            float sum = 0.f;
#pragma unroll
            for (int e = 0; e < 4; ++e) add(sum, x[e], rl[e]);
            sm_quad[(hd * 32 + page) * pitch + q] = sum;
          }
        }
      }
    }
    __syncthreads();
    if (j < nblk) {
      for (int h = slot; h < p.Hkv; h += 8) {
        const float* const sums = sm_quad + (h * 32 + pg) * pitch;
        for (int q = 0; q < q4; ++q) sc += sums[q];
      }
    }
  } else if (j < nblk) {
    if (pre_ok) {
      if (slot < p.Hkv) {
#pragma unroll
        for (int q = 0; q < kFinPre; ++q) {
          if (4 * q < Rc) {
            const f32x4 rl = *reinterpret_cast<const f32x4*>(sm_row + slot * Rc + 4 * q);
#pragma unroll
            for (int e = 0; e < 4; ++e) add(sc, pre[SMALL ? q : 0][e], rl[e]);
          }
        }
      }
    } else {
      sc = page_by_rows(p, sm_row, b, slot, j);
    }
  }
  sm_sum[slot * 32 + pg] = sc;
  __syncthreads();
  store_page_scores(p, sm_sum, out_row, j, nblk);
}

// METRIC 1 (the paper's logit metric, token granularity) replaces the page-score role by workgroups
// [nA, nA + nC) that add the H_kv per-head token sums of 1024 tokens each: score[b][i] = tok_norm *
// sum_h partial[b][h][i] for prefix tokens i < n_b - G (Sec. 3.3, last paragraph), 0 elsewhere.
template <int MAXS, int METRIC = 0, int ROUNDS = kFinRounds>
__global__ __launch_bounds__(256) void verify_finalize_kernel(const FinalizeParams p) {
  // Merging, general path: [256 / D][D] weights + [256 / D][4].  Page scores, of rows = Hkv * Rc: score_pages 8 x rows + rows + [8][32] floats,
  // score_pages_planned rows + [8][32] + [Hkv * 32][pitch], pitch at most 3/8 Rc (Rc of 8): 12 x rows.
  extern __shared__ __attribute__((aligned(16))) float smf[];
  constexpr bool kPlanned = MAXS < 0;
  const int b = blockIdx.y;
  const int tid = threadIdx.x;
  const int HR = p.Hkv * p.R;
  ColumnSlots cs;
  int plan_n = 0;                             // kPlanned: the sequence's length
  if constexpr (kPlanned) {                   // (its entry of the plan and its length in one round trip: two after each other were 0.7 us)
    int zero = 0;
    asm("" : "+v"(zero));
    int2 e = p.plan[b + zero];
    plan_n = p.lens[b + zero];
    asm volatile("" : "+v"(e.x), "+v"(e.y), "+v"(plan_n));
    e = make_int2(__builtin_amdgcn_readfirstlane(e.x), __builtin_amdgcn_readfirstlane(e.y));
    plan_n = __builtin_amdgcn_readfirstlane(plan_n);
    plan_n = plan_n < 0 ? 0 : (plan_n > p.max_tokens ? p.max_tokens : plan_n);
    cs = planned_slots(e, p.slots_total);
  } else {
    cs = column_slots(nullptr, p.slots_total, b, p.Hkv, p.nsplit, p.chunk_tokens);
  }

  if (static_cast<int>(blockIdx.x) < p.nA) {
    if constexpr (MAXS == kFinPlanned) {
      merge_planned_rows(p, cs, b, plan_n, HR);
      return;
    }
    // ---- role A: 256 / D consecutive rows of the Hkv*R rows, D threads (= head dims) each
    const int T = p.D;
    const int sub = tid / T, t128 = tid % T, wv = (tid >> 6) % (T >> 6);
    const int rr_raw = (256 / T) * blockIdx.x + sub;
    const bool valid = rr_raw < HR;
    const int rr = valid ? rr_raw : HR - 1;
    const int h = rr / p.R, r = rr % p.R;
    const int64_t pbase = cs.off + static_cast<int64_t>(h) * cs.stride_h;
    const float2* ml = p.part_ml + pbase * p.R + r;
    float o;
    if constexpr (MAXS > 0) {
      int n = p.lens[b];
      RowMerge<MAXS> rm;
      rm.issue(ml, p.part_o + (pbase * p.R + r) * T, t128, p.R, cs.last, T);
      n = n < 0 ? 0 : (n > p.max_tokens ? p.max_tokens : n);
      o = rm.finish((n + cs.chunk - 1) / cs.chunk);
    } else {
      int n = plan_n;
      if constexpr (!kPlanned) {
        n = p.lens[b];
        n = n < 0 ? 0 : (n > p.max_tokens ? p.max_tokens : n);
      }
      const ColumnChunks cc = column_chunks(cs, n);
      const int ns = cc.ns;
      auto store = [&](uint16_t bits) {
        if (valid) {
          const int t = r / p.g, j = r % p.g;
          p.out[((static_cast<int64_t>(b) * p.G + t) * p.Hq + h * p.g + j) * T + t128] = bits;
        }
      };
      if (cc.last < 0) {                     // an empty sequence: nothing is requested
        store(0);
        return;
      }
      // A sequence may have few chunks although the host's bound on them is high (a loose max_seq_len or a caller's chunk
      // length): only its own slots are read, in one round trip.  (One sequence of 4000 tokens in chunks of 128 under a bound
      // of 131072, 20 rows, first and last collected: the whole call 22.0 -> 20.8 us.)
      if (ns <= 32) {
        const float* const po = p.part_o + (pbase * p.R + r) * T;
        auto merge = [&](auto maxs) {
          RowMerge<decltype(maxs)::value> rm;
          rm.issue(ml, po, t128, p.R, cc.last, T);
          return rm.finish(ns);
        };
        if (ns <= 4) o = merge(std::integral_constant<int, 4>{});
        else if (ns <= 8) o = merge(std::integral_constant<int, 8>{});
        else if (ns <= 16) o = merge(std::integral_constant<int, 16>{});
        else o = merge(std::integral_constant<int, 32>{});
        store(float_to_bf16_bits(o));
        return;
      }
      const float* po = p.part_o + (pbase * p.R + r) * T + t128;
      float* sw = smf + sub * T;
      float* sred = smf + 256 + sub * 4;
      const int64_t ostride = static_cast<int64_t>(p.R) * T;
      float m = -INFINITY;
      for (int s = t128; s < ns; s += T) m = fmaxf(m, ml[static_cast<int64_t>(s) * p.R].x);
      m = wave_max(m);
      if ((tid & 63) == 0) sred[wv] = m;
      __syncthreads();
      m = T > 64 ? fmaxf(sred[0], sred[1]) : sred[0];
      const float m_use = (m == -INFINITY) ? 0.f : m;
      float accv = 0.f, L = 0.f;
      for (int s0 = 0; s0 < ns; s0 += T) {
        const int cnt = min(T, ns - s0);
        float wl = 0.f;
        if (t128 < cnt) {
          const float2 v = ml[static_cast<int64_t>(s0 + t128) * p.R];
          const float w = fast_exp2(v.x - m_use);
          sw[t128] = w;
          wl = w * v.y;
        }
        wl = wave_sum(wl);
        if ((tid & 63) == 0) sred[2 + wv] = wl;
        __syncthreads();
        L += T > 64 ? sred[2] + sred[3] : sred[2];
        int s = 0;
        for (; s + 4 <= cnt; s += 4) {
          const float x0 = po[(s0 + s) * ostride], x1 = po[(s0 + s + 1) * ostride];
          const float x2 = po[(s0 + s + 2) * ostride], x3 = po[(s0 + s + 3) * ostride];
          accv += sw[s] * x0 + sw[s + 1] * x1 + sw[s + 2] * x2 + sw[s + 3] * x3;
        }
        for (; s < cnt; ++s) accv += sw[s] * po[(s0 + s) * ostride];
        __syncthreads();
      }
      o = (L > 0.f) ? accv / L : 0.f;
    }
    if (valid) {
      const int t = r / p.g, j = r % p.g;
      p.out[((static_cast<int64_t>(b) * p.G + t) * p.Hq + h * p.g + j) * T + t128] = float_to_bf16_bits(o);
    }
    return;
  }

  if constexpr (METRIC == 1) {
    // ---- role C: 1024 tokens; thread = 4 consecutive tokens
    const int i0 = (static_cast<int>(blockIdx.x) - p.nA) * 1024 + 4 * tid;
    const int cap = p.max_blocks * kPage;
    if (i0 >= cap) return;
    int n = p.lens[b];
    // The heads' partial sums are requested eight at a time, unconditionally (clamped), before the length is needed.
    const int iload = min(i0, p.lse_pages - 4);
    f32x4 sum = {0.f, 0.f, 0.f, 0.f};
    for (int h0 = 0; h0 < p.Hkv; h0 += 8) {
      f32x4 part[8];
#pragma unroll
      for (int u = 0; u < 8; ++u)
        part[u] = *reinterpret_cast<const f32x4*>(
            p.page_lse + (static_cast<int64_t>(b) * p.Hkv + min(h0 + u, p.Hkv - 1)) * p.lse_pages + iload);
#pragma unroll
      for (int u = 0; u < 8; ++u)
        if (h0 + u < p.Hkv) sum += part[u];
    }
    n = n < 0 ? 0 : (n > p.max_tokens ? p.max_tokens : n);
    const int p_len = max(n - p.G, 0);
    f32x4 o;
#pragma unroll
    for (int e = 0; e < 4; ++e) o[e] = (i0 + e < p_len) ? sum[e] * p.tok_norm : 0.f;
    *reinterpret_cast<f32x4*>(p.block_scores + static_cast<int64_t>(b) * cap + i0) = o;
    return;
  }

  // ---- role B: 32 pages; thread = (page, head slot)
  if constexpr (MAXS > 0) {
    score_pages<MAXS, ROUNDS, false>(p, smf, b);
  } else if constexpr (kPlanned) {
    score_pages_planned<MAXS == kFinPlannedSmall>(p, cs, smf, b, plan_n);
  } else {
    score_pages<32, ROUNDS, true>(p, smf, b);
  }
}

}  // namespace vegas
