// Top-k selection over single tokens (the paper's own granularity: Sec. 3.3 last paragraph, Sec. 4).
//
// A sequence has up to a few hundred thousand prefix tokens, too many for one workgroup, so the
// radix select of the page version is spread over workgroups that own 4096-token slices and meet in
// per-slice digit histograms between launches (plain stores, nothing to clear, no global atomics; up to 32768 tokens one
// workgroup does it all, token_select_one_kernel):
//   token_select_hist x 4  pass q: every workgroup sums the slices' histograms of passes < q, derives
//                          the key prefix they fix, counts digit q of its own slice's matching keys
//                          in LDS and stores its 256 counts
//   token_select_write     derives the k-th key T the same way; the keys > T and == T in the slices
//                          before its own follow from those slices' histograms, so it knows where its
//                          output starts; then an order-preserving compaction of the slice;
//                          physical slot = table[i / 16] * 16 + i % 16
// The last min(G, n) tokens are not part of the prefix and are always kept (Sec. 3.2, last sentence).
// Integer work on the score bits: defined bit for bit, ties go to the lower position.
#pragma once
#include "select_blocks.hpp"
#include "vegas_common.hpp"

namespace vegas {

constexpr int kTokSlice = 4096;       // prefix tokens per workgroup
constexpr int kTokThreads = 1024;

struct TokenSelectParams {
  const float* scores;        // [B, max_blocks * 16]
  const int32_t* block_table; // [B, max_blocks]
  const int32_t* seq_lens;
  const int32_t* budgets;     // or nullptr
  int32_t* sel_table;         // [B, max_sel] physical token slots
  int32_t* sel_seq_lens;
  uint32_t* hist;             // [B, 4, slices, 256] digit histogram of every (pass, slice)
  int32_t budget_tokens, G, max_blocks, max_sel, max_tokens, slices;
  float budget_ratio;         // > 0: budget = ceil(ratio * seq_len) unless per-sequence budgets are given
};

// What one sequence asks for.
struct TokenPlan {
  int n, p_len, tail, k, kc;
  bool need_search, take_all;
};

__device__ __forceinline__ TokenPlan token_plan(const TokenSelectParams& p, int b, int n) {       // n: seq_lens[b]
  TokenPlan t;
  t.n = n < 0 ? 0 : (n > p.max_tokens ? p.max_tokens : n);
  t.p_len = max(t.n - p.G, 0);
  t.tail = t.n - t.p_len;
  const int budget = sequence_budget(p.budgets, p.budget_ratio, p.budget_tokens, b, t.n);
  int k = min(budget, t.n);
  k = max(k, t.tail);
  t.k = min(k, p.max_sel);                           // device-side clamp; the host rejects this case
  t.kc = max(t.k - t.tail, 0);
  t.need_search = t.kc > 0 && t.kc < t.p_len;
  t.take_all = t.kc >= t.p_len;
  return t;
}

// All threads: sh_tot[q][bin] = sum over the sequence's slices of histogram (pass q, bin) for q < passes,
// and, if sh_bef is given, the same sum over the slices before `upto` only.  Followed by a barrier.
__device__ __forceinline__ void token_sum_hists(const TokenSelectParams& p, int b, int passes, int nslices, int upto,
                                                uint32_t (*sh_tot)[256], uint32_t (*sh_bef)[256]) {
  const int q = threadIdx.x >> 8, bin = threadIdx.x & 255;          // 1024 threads = 4 passes x 256 bins
  if (q < passes) {
    const uint32_t* h = p.hist + ((static_cast<int64_t>(b) * 4 + q) * p.slices) * 256 + bin;
    uint32_t tot = 0u, bef = 0u;
    for (int sl0 = 0; sl0 < nslices; sl0 += 8) {          // eight independent loads in flight per round trip
      uint32_t c[8];
#pragma unroll
      for (int u = 0; u < 8; ++u) c[u] = h[static_cast<int64_t>(min(sl0 + u, nslices - 1)) * 256];
#pragma unroll
      for (int u = 0; u < 8; ++u) {
        tot += sl0 + u < nslices ? c[u] : 0u;
        bef += sl0 + u < upto ? c[u] : 0u;
      }
    }
    sh_tot[q][bin] = tot;
    if (sh_bef) sh_bef[q][bin] = bef;
  }
  __syncthreads();
}

// Executed by ONE full wave: walks the summed histograms of passes 0 .. passes-1 and returns, in every
// lane, the key prefix they fix and how many keys are still wanted inside it.
__device__ __forceinline__ void token_prefix(const uint32_t (*sh_tot)[256], int passes, uint32_t kc,
                                             uint32_t* prefix_out, uint32_t* need_out) {
  const int lane = threadIdx.x & 63;
  uint32_t prefix = 0u, need = kc;
  for (int q = 0; q < passes; ++q) {
    const int shift = 24 - 8 * q;
    // lane l owns bins 255-4l .. 252-4l, so an inclusive prefix sum over lanes counts from the top bin down
    uint32_t c[4];
#pragma unroll
    for (int i = 0; i < 4; ++i) c[i] = sh_tot[q][255 - 4 * lane - i];
    const uint32_t mine = c[0] + c[1] + c[2] + c[3];
    uint32_t above = wave_prefix_sum(mine) - mine;
    uint32_t found = 0u, digit = 0u, rest = 0u;
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      if (above < need && need <= above + c[i]) {
        found = 1u;
        digit = static_cast<uint32_t>(255 - 4 * lane - i);
        rest = need - above;
      }
      above += c[i];
    }
    const uint64_t who = __builtin_amdgcn_ballot_w64(found != 0u);   // exactly one lane when need <= matching keys
    const int src = who ? __builtin_ctzll(who) : 0;
    digit = __builtin_amdgcn_readlane(digit, src);
    rest = __builtin_amdgcn_readlane(rest, src);
    prefix |= digit << shift;
    need = rest;
  }
  *prefix_out = prefix;
  *need_out = need;
}

__global__ __launch_bounds__(kTokThreads) void token_select_hist(const TokenSelectParams p, int pass) {
  __shared__ uint32_t hist[kTokThreads / 64][256];
  __shared__ uint32_t sh_tot[4][256];
  __shared__ uint32_t sh_prefix;
  const int b = blockIdx.y, s = blockIdx.x;
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const TokenPlan t = token_plan(p, b, p.seq_lens[b]);
  const int base = s * kTokSlice;
  if (!t.need_search || base >= t.p_len) return;
  const int nslices = (t.p_len + kTokSlice - 1) / kTokSlice;
  // The thread's scores do not depend on the earlier passes: they are requested first (together, clamped indices,
  // none behind a branch), so their round trip overlaps the one of the slices' histograms.
  const float* scores = p.scores + static_cast<int64_t>(b) * p.max_blocks * kPage;
  float sc[kTokSlice / kTokThreads];
#pragma unroll
  for (int it = 0; it < kTokSlice / kTokThreads; ++it) sc[it] = scores[min(base + it * kTokThreads + tid, t.p_len - 1)];
  uint32_t* h = hist[wave];
#pragma unroll
  for (int i = 0; i < 4; ++i) h[lane + 64 * i] = 0u;
  token_sum_hists(p, b, pass, nslices, 0, sh_tot, nullptr);
  if (wave == 0) {
    uint32_t prefix, need;
    token_prefix(sh_tot, pass, static_cast<uint32_t>(t.kc), &prefix, &need);
    if (lane == 0) sh_prefix = prefix;
  }
  __syncthreads();
  const uint32_t prefix = sh_prefix;
  const uint32_t mask = pass == 0 ? 0u : (0xFFFFFFFFu << (32 - 8 * pass));
  const int shift = 24 - 8 * pass;
#pragma unroll
  for (int it = 0; it < kTokSlice / kTokThreads; ++it) {
    const int j = base + it * kTokThreads + tid;
    const uint32_t key = score_key(sc[it]);
    bool act = j < t.p_len && (key & mask) == prefix;
    const uint32_t d = (key >> shift) & 255u;
    // lanes that share the leader's digit are counted by one atomic; what is left after two rounds adds itself
#pragma unroll
    for (int round = 0; round < 2; ++round) {
      const uint64_t am = __builtin_amdgcn_ballot_w64(act);
      const int leader = am ? __builtin_ctzll(am) : 0;
      const uint32_t dl = __builtin_amdgcn_readlane(d, leader);
      const bool hit = act && d == dl;
      const uint64_t same = __builtin_amdgcn_ballot_w64(hit);
      if (hit && lane == leader) atomicAdd(&h[dl], static_cast<uint32_t>(__popcll(same)));
      act = act && !hit;
    }
    if (act) atomicAdd(&h[d], 1u);
  }
  __syncthreads();
  if (tid < 256) {
    uint32_t c = 0u;
#pragma unroll
    for (int w = 0; w < kTokThreads / 64; ++w) c += hist[w][tid];
    p.hist[((static_cast<int64_t>(b) * 4 + pass) * p.slices + s) * 256 + tid] = c;
  }
}

__global__ __launch_bounds__(kTokThreads) void token_select_write(const TokenSelectParams p) {
  __shared__ uint32_t sh_tot[4][256], sh_bef[4][256];
  __shared__ uint32_t sh_T, sh_need_eq, sh_eq_before, sh_pos_before;
  __shared__ uint32_t wave_take[kTokThreads / 64], wave_eq[kTokThreads / 64];
  const int b = blockIdx.y, s = blockIdx.x;
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const TokenPlan t = token_plan(p, b, p.seq_lens[b]);
  int32_t* sel = p.sel_table + static_cast<int64_t>(b) * p.max_sel;
  const int32_t* table = p.block_table + static_cast<int64_t>(b) * p.max_blocks;
  const float* scores = p.scores + static_cast<int64_t>(b) * p.max_blocks * kPage;
  auto slot_of = [&](int i) -> int32_t { return table[i >> 4] * kPage + (i & 15); };

  // ---- the kept tail, the padding and the length: spread over the sequence's workgroups
  const int stride = gridDim.x * kTokThreads;
  for (int i = s * kTokThreads + tid; i < t.tail; i += stride)
    if (t.kc + i < p.max_sel) sel[t.kc + i] = slot_of(t.p_len + i);
  for (int i = t.k + s * kTokThreads + tid; i < p.max_sel; i += stride) sel[i] = -1;
  if (s == 0 && tid == 0) p.sel_seq_lens[b] = t.k;

  const int base = s * kTokSlice;
  if (t.kc == 0 || base >= t.p_len) return;
  // This thread's tokens (wave w owns tokens [base + 256 w, base + 256 (w + 1)), 64 per step, lane = token): their
  // scores and the table entries of their pages are requested now, unconditionally and together, so that the
  // round trip overlaps the one of the slices' histograms and no request waits behind a decision.
  constexpr int kSteps = kTokSlice / kTokThreads;
  const int w0 = base + wave * (64 * kSteps);
  uint32_t key[kSteps];
  int32_t page_of[kSteps];
  bool valid[kSteps];
#pragma unroll
  for (int st = 0; st < kSteps; ++st) {
    const int j = w0 + 64 * st + lane;
    valid[st] = j < t.p_len;
    key[st] = score_key(scores[min(j, t.p_len - 1)]);
    page_of[st] = table[min(j, t.p_len - 1) >> 4];
  }
  if (t.need_search) {
    const int nslices = (t.p_len + kTokSlice - 1) / kTokSlice;
    token_sum_hists(p, b, 4, nslices, s, sh_tot, sh_bef);
    if (wave == 0) {
      uint32_t T, need_eq;
      token_prefix(sh_tot, 4, static_cast<uint32_t>(t.kc), &T, &need_eq);
      // In the slices before this one: keys > T are, pass by pass, the keys that match T's prefix so far and
      // have a larger digit; keys == T are the last pass's count of T's low digit.
      uint32_t gt = 0u;
#pragma unroll
      for (int q = 0; q < 4; ++q) {
        const uint32_t digit = (T >> (24 - 8 * q)) & 255u;
#pragma unroll
        for (int i = 0; i < 4; ++i) {
          const uint32_t bin = static_cast<uint32_t>(4 * lane + i);
          gt += bin > digit ? sh_bef[q][bin] : 0u;
        }
      }
      gt = __builtin_amdgcn_readlane(wave_prefix_sum(gt), 63);
      const uint32_t eq_before = sh_bef[3][T & 255u];
      if (lane == 0) {
        sh_T = T;
        sh_need_eq = need_eq;
        sh_eq_before = eq_before;
        sh_pos_before = gt + min(eq_before, need_eq);        // ties are taken in order until need_eq are found
      }
    }
  }
  __syncthreads();
  const bool all = t.take_all;
  const uint32_t T = all ? 0u : sh_T, need_eq = all ? 0u : sh_need_eq;
  const uint32_t slice_eq_before = all ? 0u : sh_eq_before;
  const uint32_t slice_pos_before = all ? static_cast<uint32_t>(base) : sh_pos_before;

  // ---- ordered compaction
  const uint64_t lt = (1ull << lane) - 1ull;
  uint32_t eq_wave = 0u;
#pragma unroll
  for (int st = 0; st < kSteps; ++st) eq_wave += __popcll(__builtin_amdgcn_ballot_w64(valid[st] && !all && key[st] == T));
  if (lane == 0) wave_eq[wave] = eq_wave;
  __syncthreads();
  uint32_t eq_before = slice_eq_before;
  for (int w = 0; w < wave; ++w) eq_before += wave_eq[w];
  uint32_t take_wave = 0u, eq_run = eq_before;
  bool take[kSteps];
#pragma unroll
  for (int st = 0; st < kSteps; ++st) {
    const bool eq = valid[st] && !all && key[st] == T;
    const bool gt = valid[st] && !all && key[st] > T;
    const uint64_t beq = __builtin_amdgcn_ballot_w64(eq);
    take[st] = all ? valid[st] : (gt || (eq && eq_run + __popcll(beq & lt) < need_eq));
    eq_run += __popcll(beq);
    take_wave += __popcll(__builtin_amdgcn_ballot_w64(take[st]));
  }
  if (lane == 0) wave_take[wave] = take_wave;
  __syncthreads();
  uint32_t pos_run = slice_pos_before;
  for (int w = 0; w < wave; ++w) pos_run += wave_take[w];
#pragma unroll
  for (int st = 0; st < kSteps; ++st) {
    const uint64_t btk = __builtin_amdgcn_ballot_w64(take[st]);
    if (take[st]) {
      const uint32_t pos = pos_run + __popcll(btk & lt);
      if (pos < static_cast<uint32_t>(p.max_sel)) sel[pos] = page_of[st] * kPage + ((w0 + 64 * st + lane) & 15);
    }
    pos_run += __popcll(btk);
  }
}

// ---- up to 32768 tokens: one workgroup per sequence, thread tid has tokens 4096 g + 4 tid + e (row g, e = 0..3) in registers; token
// (g, e) is bit 4 g + e of a thread's set of tokens.
constexpr int kRowTokens = 4 * kTokThreads;
constexpr int kBinTies = 512;          // tokens of one bin that are ranked among each other at most
constexpr int kCrowd = 12;             // so many of 64 scores in one bin: bins do not tell them apart (take_by_bins)
constexpr int kFewValues = 2;          // so many of 64 scores equal to one of two sampled beside them: there are few values

struct TokenSelectShared : RegisterSelectShared {
  alignas(16) uint32_t bins[2048];     // counts of take_by_bins (hist: of find_last_key)
  uint32_t top[kTokThreads / 64], bound[kTokThreads / 64];      // of each wave: largest key, complement of the bound (key_bounds)
  uint32_t crowded, listed;
};

// Tokens of all threads before each of this thread's rows, and of all rows (the result); n[g] of row g (4 at most) are this thread's.
// One barrier inside.
template <int ROWS>
__device__ __forceinline__ uint32_t counts_before(const uint32_t (&n)[ROWS], uint32_t (&before)[ROWS], int rows, uint32_t* cells) {
  constexpr int kWaves = kTokThreads / 64, kPacks = (ROWS + 2) / 3;
  const int lane = threadIdx.x & 63;
  const int wave = __builtin_amdgcn_readfirstlane(static_cast<int>(threadIdx.x) >> 6);
  uint32_t lower[kPacks], own = 0u;                // (a wave's row has 256 tokens: three counts of ten bits in one sum)
#pragma unroll
  for (int q = 0; q < kPacks; ++q) {
    uint32_t pack = n[3 * q];
    if (3 * q + 1 < ROWS) pack |= n[3 * q + 1 < ROWS ? 3 * q + 1 : 0] << 10;
    if (3 * q + 2 < ROWS) pack |= n[3 * q + 2 < ROWS ? 3 * q + 2 : 0] << 20;
    const uint32_t incl = wave_prefix_sum(pack);
    lower[q] = incl - pack;
    const uint32_t of_wave = __builtin_amdgcn_readlane(incl, 63);
#pragma unroll
    for (int i = 0; i < 3; ++i)
      if (lane == 3 * q + i) own = (of_wave >> (10 * i)) & 1023u;
  }
  if (lane < rows) cells[lane * kWaves + wave] = own;
  __syncthreads();
  uint32_t total;
  const uint32_t cell = CellWalk<ROWS>::before(cells, rows, wave, lane, &total);
#pragma unroll
  for (int g = 0; g < ROWS; ++g)
    before[g] = ((lower[g / 3] >> (10 * (g % 3))) & 1023u) + __builtin_amdgcn_readlane(cell, CellWalk<ROWS>::lane_of(g, wave));
  return total;
}

// The same of a set of tokens.
template <int ROWS>
__device__ __forceinline__ uint32_t row_counts(uint32_t set, uint32_t (&before)[ROWS], int rows, uint32_t* cells) {
  uint32_t n[ROWS];
#pragma unroll
  for (int g = 0; g < ROWS; ++g) n[g] = __popc((set >> (4 * g)) & 15u);
  return counts_before<ROWS>(n, before, rows, cells);
}

// Places of the tokens above a last bin and of the first `need`, by position, of those in it, of two disjoint sets: `set` is made theirs
// and `before` counts them.  One barrier inside; the result is their number.
template <int ROWS>
__device__ __forceinline__ uint32_t keep_first(uint32_t& set, uint32_t in, uint32_t need, uint32_t (&before)[ROWS], int rows, uint32_t* cells) {
  constexpr int kWaves = kTokThreads / 64, kPacks = (2 * ROWS + 2) / 3;
  const int lane = threadIdx.x & 63;
  const int wave = __builtin_amdgcn_readfirstlane(static_cast<int>(threadIdx.x) >> 6);
  uint32_t n[3 * kPacks], lower[kPacks], of_wave[kPacks];
#pragma unroll
  for (int i = 0; i < 3 * kPacks; ++i) n[i] = i < ROWS ? __popc((set >> (4 * i)) & 15u) : i < 2 * ROWS ? __popc((in >> (4 * (i - ROWS))) & 15u) : 0u;
#pragma unroll
  for (int q = 0; q < kPacks; ++q) {
    const uint32_t pack = n[3 * q] | (n[3 * q + 1] << 10) | (n[3 * q + 2] << 20);
    const uint32_t incl = wave_prefix_sum(pack);
    lower[q] = incl - pack;
    of_wave[q] = __builtin_amdgcn_readlane(incl, 63);
  }
  auto field = [](const uint32_t (&packs)[kPacks], int i) { return (packs[i / 3] >> (10 * (i % 3))) & 1023u; };
  uint32_t own = 0u;                             // (a cell's two counts are 32768 at most in sum)
#pragma unroll
  for (int g = 0; g < ROWS; ++g)
    if (lane == g) own = field(of_wave, g) | (field(of_wave, ROWS + g) << 16);
  if (lane < rows) cells[lane * kWaves + wave] = own;
  __syncthreads();
  uint32_t total;
  const uint32_t cell = CellWalk<ROWS>::before(cells, rows, wave, lane, &total);
#pragma unroll
  for (int g = 0; g < ROWS; ++g) {
    const uint32_t c = __builtin_amdgcn_readlane(cell, CellWalk<ROWS>::lane_of(g, wave));
    const uint32_t in_before = field(lower, ROWS + g) + (c >> 16);
    before[g] = field(lower, g) + (c & 0xFFFFu) + min(in_before, need);
    // of the row's tokens in the last bin as many as are still wanted, the lower ones first
    const uint32_t left = need > in_before ? need - in_before : 0u;
    uint32_t row = (in >> (4 * g)) & 15u;
#pragma unroll
    for (int drop = 3; drop >= 0; --drop)
      if (__popc(row) > static_cast<int>(left)) row &= ~(1u << drop);
    set |= row << (4 * g);
  }
  return (total & 0xFFFFu) + min(total >> 16, need);
}

__device__ __forceinline__ float max3(float a, float b, float c) {      // (fmaxf quiets what it is given first: an instruction a key)
  float r;
  asm("v_max3_f32 %0, %1, %2, %3" : "=v"(r) : "v"(a), "v"(b), "v"(c));
  return r;
}
// set = 16 set + (bit e: y[e] >= bound), of floats or unsigned keys.  (Two instructions a bit; left to the compiler, a select, a shift
// and an or as well.)
#define VEGAS_SHIFT_IN_GE(TYPE, SUFFIX)                                                                                                \
  __device__ __forceinline__ void shift_in_ge(uint32_t& set, TYPE y0, TYPE y1, TYPE y2, TYPE y3, TYPE bound) {                        \
    uint64_t c0, c1, c2, c3;                                                                                                           \
    asm("v_cmp_le_" SUFFIX "_e64 %4, %9, %8\n\tv_cmp_le_" SUFFIX "_e64 %3, %9, %7\n\t"                                                 \
        "v_cmp_le_" SUFFIX "_e64 %2, %9, %6\n\tv_cmp_le_" SUFFIX "_e64 %1, %9, %5\n\t"                                                 \
        "v_addc_co_u32_e64 %0, vcc, %0, %0, %4\n\tv_addc_co_u32_e64 %0, vcc, %0, %0, %3\n\t"                                           \
        "v_addc_co_u32_e64 %0, vcc, %0, %0, %2\n\tv_addc_co_u32_e64 %0, vcc, %0, %0, %1"                                               \
        : "+v"(set), "=&s"(c0), "=&s"(c1), "=&s"(c2), "=&s"(c3)                                                                      \
        : "v"(y0), "v"(y1), "v"(y2), "v"(y3), "v"(bound)                                                                            \
        : "vcc");                                                                                                                      \
  }
VEGAS_SHIFT_IN_GE(float, "f32")
VEGAS_SHIFT_IN_GE(uint32_t, "u32")
#undef VEGAS_SHIFT_IN_GE

__device__ __forceinline__ float key_score(uint32_t key) { return __uint_as_float((key & 0x80000000u) ? key ^ 0x80000000u : ~key); }

// Scores by 2048 bins of equal width: a bin is a monotone function of the score, one multiply-add to a number whose low bits are the bin.
struct ScoreBins {
  static constexpr float kOne = 2097152.f;       // 2^21: numbers from there to its double have their quarters in bits 0 and 1
  static constexpr uint32_t kBytes = 2047u * 4u;
  float scale, shift;
  bool ok;                                       // false: the range is too near a point, or too far from 0 for its width
  __device__ __forceinline__ ScoreBins(float lo, float hi) {
    scale = 2040.f * __builtin_amdgcn_rcpf(hi - lo);
    shift = kOne + 3.f - lo * scale;
    ok = scale > 0.f && fabsf(lo) * scale < kOne && fabsf(hi) * scale < kOne;
  }
  __device__ __forceinline__ float place(float v) const { return __builtin_fmaf(v, scale, shift); }      // 2^21 + bin
  static __device__ __forceinline__ bool inside(float y) { return y >= kOne + 1.f; }
  static __device__ __forceinline__ uint32_t offset(float y) { return __float_as_uint(y) & kBytes; }
};

// Largest key of the workgroup, and a lower bound of the `take`-th largest: the smallest of the largest keys of groups of tokens that are
// disjoint and at least `take` (a quarter of all, or fewer) in number, so that masked and far low scores do not count.  False where it is no number.
// One barrier inside.
template <int ROWS>
__device__ __forceinline__ bool key_bounds(const float (&x)[4 * ROWS], int rows, int p_len, uint32_t take, TokenSelectShared& sh,
                                           LastKey& range) {
  constexpr int kWaves = kTokThreads / 64;
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  float m[ROWS], top = -INFINITY;
#pragma unroll
  for (int g = 0; g < ROWS; ++g) {
    m[g] = -INFINITY;
    if (g >= rows) continue;
    const float three = max3(x[4 * g], x[4 * g + 1], x[4 * g + 2]);
    m[g] = max3(three, x[4 * g + 3], x[4 * g + 3]);
    top = max3(top, m[g], m[g]);
  }
  uint32_t hi = score_key(top), inv_lo = 0u;
  // groups of N rows of a thread have 4 N tokens or fewer, so there are p_len / (4 N) of them or more
  auto group_bound = [&](auto rows_per) {
    constexpr int N = decltype(rows_per)::value;
#pragma unroll
    for (int g = 0; g < ROWS; g += N) {
      float of_group = m[g];
#pragma unroll
      for (int i = 1; i < N; ++i) of_group = max3(of_group, m[g + i], m[g + i]);
      if (kRowTokens * g + 4 * tid < p_len) inv_lo = max(inv_lo, ~score_key(of_group));
    }
  };
  if (ROWS >= 4 && 16u * take <= static_cast<uint32_t>(p_len)) group_bound(std::integral_constant<int, ROWS >= 4 ? 4 : 1>{});
  else if (ROWS >= 2 && 8u * take <= static_cast<uint32_t>(p_len)) group_bound(std::integral_constant<int, ROWS >= 2 ? 2 : 1>{});
  else group_bound(std::integral_constant<int, 1>{});
  hi = wave_max(hi);
  inv_lo = wave_max(inv_lo);
  if (lane == 0) {
    sh.top[wave] = hi;
    sh.bound[wave] = inv_lo;
  }
  __syncthreads();
  hi = __builtin_amdgcn_readfirstlane(wave_max(sh.top[lane & (kWaves - 1)]));
  range.base = ~__builtin_amdgcn_readfirstlane(wave_max(sh.bound[lane & (kWaves - 1)]));
  range.span = hi - range.base;
  return range.base > score_key(-INFINITY) && hi >= range.base && hi < score_key(INFINITY);
}

// The set of this thread's tokens among the `take` largest scores, found among the scores themselves: 2048 bins over the range, one pass
// that counts, one that takes what lies above the last bin, and the few tokens of that bin ranked among each other.  False where that bin
// has too many, or where a wave finds twelve of 64 scores in one bin before anything is counted: a far one leaves the others no bins.
// (Largest number found, 16 sequences of 2048 to 32768: normal 3, its exponential 5, rising or falling 7; exp of five times a normal one 59, one at
// 3e38 63.)  Whatever a bin rounds, the set is right if it has `take` tokens, and false is the result if it has not.
// before: tokens taken before this thread's of a row.  used: whether `hist` was written.
template <int ROWS>
__device__ __forceinline__ bool take_by_bins(const float (&x)[4 * ROWS], int rows, uint32_t take, const LastKey& range, TokenSelectShared& sh,
                                             uint32_t* cells, uint32_t& taken, uint32_t (&before)[ROWS], bool& used) {
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  uint32_t* const ranked = sh.hist[1];             // [thread] its tokens of the last bin that are kept
  uint64_t* const ties = reinterpret_cast<uint64_t*>(sh.hist[2]);
  static_assert(sizeof(sh.hist[1]) >= kTokThreads * 4 && sizeof(sh.hist[2]) >= kBinTies * 8, "sets and ties alias digit counts");
  const ScoreBins bins(key_score(range.base), key_score(range.base + range.span));
  if (!bins.ok) return false;
  const float first = bins.place(x[0]);
  const uint32_t digit = ScoreBins::inside(first) ? ScoreBins::offset(first) : kNoDigit;
  const uint64_t in_range = __builtin_amdgcn_ballot_w64(digit != kNoDigit);
  const uint32_t probe = in_range ? __builtin_amdgcn_readlane(digit, __builtin_ctzll(in_range)) : kNoDigit - 1u;
  if (__popcll(__builtin_amdgcn_ballot_w64(digit == probe)) < kCrowd) {
    uint32_t one = 1u;
    asm("" : "+v"(one));
#pragma unroll
    for (int u = 0; u < 4 * ROWS; ++u) {
      if ((u >> 2) >= rows) continue;
      const float y = bins.place(x[u]);
      if (ScoreBins::inside(y)) atomicAdd(reinterpret_cast<uint32_t*>(reinterpret_cast<unsigned char*>(sh.bins) + ScoreBins::offset(y)), one);
    }
  } else if (lane == 0) {
    sh.crowded = 1u;
  }
  __syncthreads();
  if (sh.crowded != 0u) return false;
  if (wave == 0) walk_to_last_bin(sh.bins, take, sh);
  __syncthreads();
  const uint32_t bin = __builtin_amdgcn_readfirstlane(sh.bin), need = __builtin_amdgcn_readfirstlane(sh.need);
  const uint32_t count = __builtin_amdgcn_readfirstlane(sh.count);
  const bool whole = need == count;                // the last bin is kept whole
  if (!whole && count > min(kBinTies, 128 * ROWS)) return false;       // (ranking 270 costs what digits take up to 4096 tokens)
  used = true;
  const float in = ScoreBins::kOne + static_cast<float>(bin), above = whole ? in : in + 1.f;
  uint32_t set = 0u;
#pragma unroll
  for (int g = ROWS - 1; g >= 0; --g) {
    if (g >= rows) continue;
    float y[4];
#pragma unroll
    for (int e = 0; e < 4; ++e) y[e] = bins.place(x[4 * g + e]);
    uint32_t at_least = 0u;
    shift_in_ge(set, y[0], y[1], y[2], y[3], above);
    shift_in_ge(at_least, y[0], y[1], y[2], y[3], in);
    const uint32_t tie = at_least ^ (set & 15u);
    if (__builtin_expect(__builtin_amdgcn_ballot_w64(tie != 0u) != 0, 0)) {
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        if ((tie >> e) & 1u) {                     // larger score, then lower position: larger entry
          const uint32_t at = atomicAdd(&sh.listed, 1u);
          if (at < kBinTies) ties[at] = (static_cast<uint64_t>(score_key(x[4 * g + e])) << 32) | ~static_cast<uint32_t>(kRowTokens * g + 4 * tid + e);
        }
      }
    }
  }
  if (!whole) {
    __syncthreads();
    if (tid < static_cast<int>(count)) {
      const uint64_t own = ties[tid];
      uint32_t before = 0u;
#pragma unroll 4
      for (uint32_t c = 0; c < count; ++c) before += ties[c] > own ? 1u : 0u;
      const uint32_t j = ~static_cast<uint32_t>(own);
      if (before < need) atomicOr(&ranked[(j >> 2) & (kTokThreads - 1)], 1u << ((4 * (j / kRowTokens) + (j & 3)) & 31u));
    }
    __syncthreads();
    set |= ranked[tid];
  }
  taken = set;
  return row_counts<ROWS>(set, before, rows, cells) == take;
}

// The same by find_last_key, for scores of any kind.
// RANGED: within the range, and if that does not yield `take` tokens (it is that of floating-point comparisons, which some NaNs upset) among
// all keys.  used: the counts are not zero.
template <int ROWS, bool RANGED>
__device__ __forceinline__ uint32_t take_by_digits(const float (&x)[4 * ROWS], int rows, int p_len, uint32_t take, bool used, const LastKey& range,
                                                   TokenSelectShared& sh, uint32_t* cells, uint32_t (&before)[ROWS]) {
  const int tid = threadIdx.x;
  uint32_t key[4 * ROWS];
#pragma unroll
  for (int u = 0; u < 4 * ROWS; ++u) {
    key[u] = score_key(x[u]);
    if (kRowTokens * ((u >> 2) + 1) > p_len && kRowTokens * (u >> 2) + 4 * tid + (u & 3) >= p_len) key[u] = 0u;
  }
  auto valid = [&](int u) { return kRowTokens * (u >> 2) + 4 * tid + (u & 3) < p_len; };
  uint32_t set;
  bool ranged = RANGED && !used;
#pragma unroll 1
  do {
    // (A barrier is behind the last use of the counts, and one ahead of the next: in find_last_key where it has no range.)
    if (RANGED && used)
      for (int i = tid; i < 3 * 2048 / 4; i += kTokThreads) reinterpret_cast<u32x4*>(sh.hist)[i] = u32x4{0u, 0u, 0u, 0u};
    const LastKey last = find_last_key<true, kTokThreads, true>(key, p_len / kRowTokens * 4, 4 * rows, valid, take, sh,
                                                                RANGED && ranged ? &range : nullptr);
    // (a last bin that ends with the largest key there is has nothing above it)
    const uint32_t above = last.base + last.span + 1u;
    uint32_t in = 0u;
    set = 0u;
#pragma unroll
    for (int g = ROWS - 1; g >= 0; --g) {
      if (g >= rows) continue;
      shift_in_ge(in, key[4 * g], key[4 * g + 1], key[4 * g + 2], key[4 * g + 3], last.base);
      if (above != 0u) shift_in_ge(set, key[4 * g], key[4 * g + 1], key[4 * g + 2], key[4 * g + 3], above);
    }
    in &= ~set;
    uint32_t found;
    if (last.whole) {
      set |= in;
      found = row_counts<ROWS>(set, before, rows, cells);
    } else {
      found = keep_first<ROWS>(set, in, last.need, before, rows, cells);
    }
    if (!RANGED || !ranged || found == take) break;
    ranged = false;
    used = true;
  } while (RANGED);
  return set;
}

// One workgroup per sequence, for prefixes of at most 4096 ROWS tokens, in one launch instead of five: a thread holds the scores
// of tokens 4096 g + 4 tid .. + 3 in registers; which are taken is a bit each, and their places come from prefix sums over a wave that
// count three rows at once.  The sequence's page ids wait in LDS.
// Bound by the instructions issued on one compute unit, 0.2 us for each one that every key of 32768 takes.  Digits of the keys
// (find_last_key) take some forty a key, most of them to make keys and to count and place one by one; bins over the scores take half.
// us, captured, five launches / by digits alone, as they were / now, normally distributed scores: 1 sequence of 4096 tokens 19.2 / 5.3 / 4.5,
// 8192 19.9 / 6.8 / 5.0, 16384 20.5 / 10.4 / 6.4, 32768 21.0 / 17.0 / 9.8; 16 of 32768 22.4 / 19.0 / 10.7; a twentieth -infinity 32768 20.6 / 18.9 /
// 10.1, a far low one 20.6 / 16.9 / 9.8, rising with the position 20.6 / 17.2 / 11.3, half 0 19.8 / 10.2.  Where bins do not tell the scores
// apart, digits as they were / now, 4096, 8192, 32768: four values 6.2 / 6.5, 7.9 / 8.0, 19.9 / 19.8; fifteen in sixteen 0 4.8 / 5.1, 6.5 / 6.4, 19.3 /
// 19.2; all equal 3.5 / 3.8, 4.5 / 4.6, 11.1 / 11.0 (seen in the sample: its request and test are the difference); one at 3e38 5.2 / 5.7,
// 6.8 / 7.0, 16.9 / 14.0; exp of a normal one 4.3 / 4.8, 6.4 / 5.5, 15.8 / 11.2, of five times one 5.2 / 5.9, 6.5 / 6.2, 15.7 / 14.3 (seen
// behind the bounds); over a quarter of the tokens taken, which has digits alone, 5.3 / 5.4, 6.8 / 6.7, 17.0 / 15.7.  What every wave does for
// one of its scores costs 7 ns: an instruction of 16 waves is 16 cycles of a SIMD.  In an iteration of 32768 tokens, whose instructions are
// cold, 80.3 -> 71.1.
template <int ROWS>
__global__ __launch_bounds__(kTokThreads) void token_select_one_kernel(const TokenSelectParams p) {
  static_assert(kTokThreads == kSelectThreads, "find_last_key");
  constexpr int kWaves = kTokThreads / 64;
  constexpr int kPageTrips = (ROWS * kRowTokens / kPage + kTokThreads - 1) / kTokThreads;
  __shared__ __align__(16) TokenSelectShared shared;
  __shared__ uint32_t cells[ROWS * kWaves];
  __shared__ int32_t pages[kPageTrips * kTokThreads];
  typedef float f32x4_any __attribute__((ext_vector_type(4), aligned(4)));     // (scores may start at any float)
  const int b = blockIdx.x;
  const int tid = threadIdx.x;
  const int32_t* table = p.block_table + static_cast<int64_t>(b) * p.max_blocks;
  const float* scores = p.scores + static_cast<int64_t>(b) * p.max_blocks * kPage;
  int32_t* sel = p.sel_table + static_cast<int64_t>(b) * p.max_sel;
  // Scores and page ids are requested before the sequence length is known: clamped to the row, what lies past the prefix is
  // dropped.
  const int cap = p.max_blocks * kPage;
  f32x4_any sc[ROWS];
#pragma unroll
  for (int g = 0; g < ROWS; ++g) sc[g] = *reinterpret_cast<const f32x4_any*>(scores + min(kRowTokens * g + 4 * tid, cap - 4));
  int32_t page[kPageTrips];
#pragma unroll
  for (int i = 0; i < kPageTrips; ++i) page[i] = table[min(i * kTokThreads + tid, p.max_blocks - 1)];
  // 64 scores, the same in every wave (eight in a row from eight places: 64 places are as many lines for each of 16 waves, 0.3 us)
  const int lane = tid & 63, sampled = (lane >> 3) * (p.max_tokens >> 3) + (lane & 7);
  const float sample = gload<float, false>(uniform_ptr(reinterpret_cast<const unsigned char*>(scores)), static_cast<uint32_t>(min(sampled, cap - 1)) * 4u);
  const int n = p.seq_lens[b];
  // (counts start at zero; these, and the pages, are ordered by the search's first barrier)
  static_assert(kTokThreads * 4 == 2 * 2048, "a thread clears four counts of two arrays each");
  reinterpret_cast<u32x4*>(shared.hist[0])[tid] = u32x4{0u, 0u, 0u, 0u};
  reinterpret_cast<u32x4*>(tid < kTokThreads / 2 ? shared.hist[2] : shared.bins)[tid & (kTokThreads / 2 - 1)] = u32x4{0u, 0u, 0u, 0u};
  if (tid == 0) shared.crowded = shared.listed = 0u;
  const TokenPlan t = token_plan(p, b, n);
#pragma unroll
  for (int i = 0; i < kPageTrips; ++i) pages[i * kTokThreads + tid] = page[i];
  auto slot_of = [&](int j) -> int32_t { return pages[j >> 4] * kPage + (j & 15); };
  if (t.need_search) {
    const int rows = (t.p_len + kRowTokens - 1) / kRowTokens;        // at most ROWS: the host's bound on the lengths says so
    const uint32_t take = static_cast<uint32_t>(t.kc);
    float x[4 * ROWS];
#pragma unroll
    for (int g = 0; g < ROWS; ++g) {
#pragma unroll
      for (int e = 0; e < 4; ++e) x[4 * g + e] = sc[g][e];
      if (kRowTokens * (g + 1) > t.p_len) {
        asm volatile("");                          // (a branch; as selects, three instructions for every key of every row)
#pragma unroll
        for (int e = 0; e < 4; ++e)
          if (kRowTokens * g + 4 * tid + e >= t.p_len) x[4 * g + e] = -INFINITY;
      }
    }
    // Few values, which bins do not tell apart (and to find that out with them costs half of what digits take): every wave sees it in the same
    // sample, so that nothing waits.  Not where a quarter of the sample is above all that occurs twice and groups of 16 tokens are asked for
    // a bound, which then is above it too (half of the scores 0: 18.5 us by digits, 10.0).
    auto few_values = [&]() {
      const uint32_t bits = __float_as_uint(sample);
      const uint64_t counts = __builtin_amdgcn_ballot_w64(sampled < t.p_len) & __builtin_amdgcn_ballot_w64(sample > -INFINITY);
      const uint64_t twice = counts & (__builtin_amdgcn_ballot_w64(sample == __uint_as_float(digit_beside<1>(bits))) |
                                       __builtin_amdgcn_ballot_w64(sample == __uint_as_float(digit_beside<2>(bits))));
      if (__popcll(twice) < kFewValues) return false;
      if (ROWS < 4 || 16u * take > static_cast<uint32_t>(t.p_len)) return true;
      const float most = key_score(wave_max((twice >> lane) & 1u ? score_key(sample) : 0u));
      return 4 * __popcll(__builtin_amdgcn_ballot_w64(sample > most) & counts) < __popcll(counts);
    };
    LastKey range;
    uint32_t taken, before[ROWS];
    bool used = false;
    if (4u * take > static_cast<uint32_t>(t.p_len) || few_values() || !key_bounds<ROWS>(x, rows, t.p_len, take, shared, range))
      taken = take_by_digits<ROWS, false>(x, rows, t.p_len, take, false, range, shared, cells, before);
    else if (!take_by_bins<ROWS>(x, rows, take, range, shared, cells, taken, before, used))
      taken = take_by_digits<ROWS, true>(x, rows, t.p_len, take, used, range, shared, cells, before);
    unsigned char* const out = uniform_ptr_mut(reinterpret_cast<unsigned char*>(sel));
#pragma unroll
    for (int g = 0; g < ROWS; ++g) {
      if (g >= rows) continue;
      const int32_t slot0 = slot_of(kRowTokens * g + 4 * tid);
      uint32_t at = before[g] * 4u;                // (take <= max_sel)
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        if ((taken >> (4 * g + e)) & 1u) {
          *reinterpret_cast<int32_t*>(out + at) = slot0 + e;
          at += 4u;
        }
      }
    }
  } else if (t.take_all) {
    __syncthreads();
    for (int j = tid; j < min(t.p_len, p.max_sel); j += kTokThreads) sel[j] = slot_of(j);
  }
  // ---- the kept tail, the padding and the length
  for (int i = tid; i < t.tail; i += kTokThreads)
    if (t.kc + i < p.max_sel) sel[t.kc + i] = table[(t.p_len + i) >> 4] * kPage + ((t.p_len + i) & 15);
  for (int i = t.k + tid; i < p.max_sel; i += kTokThreads) sel[i] = -1;
  if (tid == 0) p.sel_seq_lens[b] = t.k;
}

}  // namespace vegas
