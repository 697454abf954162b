// Shared device-side types and helpers for the gfx950 kernels (wave64, MFMA, LDS).
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

#include <type_traits>

#include "plan_rules.hpp"

namespace vegas {

constexpr int kPage = 16;       // tokens per KV page
constexpr int kHeadDim = 128;   // the larger of the two head dimensions (128, 64) the kernels are written for
constexpr int kTile = 32;       // tokens per MFMA tile (two pages)

typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef float f32x16 __attribute__((ext_vector_type(16)));
typedef float f32x4 __attribute__((ext_vector_type(4)));
typedef float f32x2 __attribute__((ext_vector_type(2)));
typedef unsigned int u32x4 __attribute__((ext_vector_type(4)));
typedef unsigned int u32x2 __attribute__((ext_vector_type(2)));

__device__ __forceinline__ float fast_exp2(float x) { return __builtin_amdgcn_exp2f(x); }
__device__ __forceinline__ float fast_log2(float x) { return __builtin_amdgcn_logf(x); }

// Reductions over the 64 lanes of a wave; every lane gets the result.  Four rotations within a row of 16 lanes (DPP operands
// of the instruction that combines), then the two row exchanges: six dependent vector instructions.  A shuffle goes through
// the LDS unit and takes a hundred cycles.  With shuffles an iteration at 32K tokens, six merges of two reductions each, took
// 71.5 us instead of 70.5, and one on 24 sequences of 1K..20K tokens, whose plan needs a dozen of them in a row, 367.5
// instead of 361.7.
template <typename T, typename F>
__device__ __forceinline__ T wave_reduce(T x, F op) {
  static_assert(sizeof(T) == 4, "one register");
  auto rotated = [](T v, auto ctrl) {
    return __builtin_bit_cast(T, __builtin_amdgcn_update_dpp(0, __builtin_bit_cast(int, v), decltype(ctrl)::value, 0xf, 0xf, true));
  };
  x = op(x, rotated(x, std::integral_constant<int, 0x121>{}));   // row_ror:1, 2, 4, 8
  x = op(x, rotated(x, std::integral_constant<int, 0x122>{}));
  x = op(x, rotated(x, std::integral_constant<int, 0x124>{}));
  x = op(x, rotated(x, std::integral_constant<int, 0x128>{}));
  // (the two results by way of variables: a bit cast of a vector's element yields element 0)
  uint32_t u = __builtin_bit_cast(uint32_t, x);
  const auto rows = __builtin_amdgcn_permlane16_swap(u, u, false, false);
  const uint32_t row0 = rows[0], row1 = rows[1];
  x = op(__builtin_bit_cast(T, row0), __builtin_bit_cast(T, row1));
  u = __builtin_bit_cast(uint32_t, x);
  const auto halves = __builtin_amdgcn_permlane32_swap(u, u, false, false);
  const uint32_t half0 = halves[0], half1 = halves[1];
  return op(__builtin_bit_cast(T, half0), __builtin_bit_cast(T, half1));
}
__device__ __forceinline__ float wave_max(float x) { return wave_reduce(x, [](float a, float b) { return fmaxf(a, b); }); }
__device__ __forceinline__ float wave_sum(float x) { return wave_reduce(x, [](float a, float b) { return a + b; }); }
__device__ __forceinline__ uint32_t wave_max(uint32_t x) { return wave_reduce(x, [](uint32_t a, uint32_t b) { return a > b ? a : b; }); }
__device__ __forceinline__ uint32_t wave_sum(uint32_t x) { return wave_reduce(x, [](uint32_t a, uint32_t b) { return a + b; }); }

// Inclusive prefix sum over the 64 lanes of a wave with DPP row shifts and row broadcasts (no LDS).
__device__ __forceinline__ uint32_t wave_prefix_sum(uint32_t x) {
  int v = static_cast<int>(x);
  v += __builtin_amdgcn_update_dpp(0, v, 0x111, 0xf, 0xf, false);   // row_shr:1
  v += __builtin_amdgcn_update_dpp(0, v, 0x112, 0xf, 0xf, false);   // row_shr:2
  v += __builtin_amdgcn_update_dpp(0, v, 0x114, 0xf, 0xf, false);   // row_shr:4
  v += __builtin_amdgcn_update_dpp(0, v, 0x118, 0xf, 0xf, false);   // row_shr:8
  v += __builtin_amdgcn_update_dpp(0, v, 0x142, 0xa, 0xf, false);   // row_bcast:15 into rows 1 and 3
  v += __builtin_amdgcn_update_dpp(0, v, 0x143, 0xc, 0xf, false);   // row_bcast:31 into rows 2 and 3
  return static_cast<uint32_t>(v);
}

// What the batch planner (balanced_slot) asks of the 64 lanes that run it together; a host program can put a class of its
// own in its place.
struct GpuWave {
  static __device__ __forceinline__ int lane() { return threadIdx.x & 63; }
  // (in a scalar register: what follows from them are the same branches for all lanes)
  static __device__ __forceinline__ uint32_t sum(uint32_t x) { return __builtin_amdgcn_readfirstlane(wave_sum(x)); }
  static __device__ __forceinline__ uint32_t max(uint32_t x) { return __builtin_amdgcn_readfirstlane(wave_max(x)); }
  static __device__ __forceinline__ uint32_t prefix_sum(uint32_t x) { return wave_prefix_sum(x); }   // inclusive
  static __device__ __forceinline__ uint64_t ballot(bool x) { return __builtin_amdgcn_ballot_w64(x); }
  static __device__ __forceinline__ uint32_t readlane(uint32_t x, int lane) { return __builtin_amdgcn_readlane(x, lane); }
  static __device__ __forceinline__ float rcp(float x) { return __builtin_amdgcn_rcpf(x); }          // within one ulp or so
};

// base + how many of the lanes below this one are set in mask.
__device__ __forceinline__ uint32_t lanes_below(uint64_t mask, uint32_t base) {
  return __builtin_amdgcn_mbcnt_hi(static_cast<uint32_t>(mask >> 32),
                                   __builtin_amdgcn_mbcnt_lo(static_cast<uint32_t>(mask), base));
}

// Orders LDS traffic between the lanes of ONE wave (a wave's LDS instructions execute in order,
// so only the compiler has to be kept from moving accesses across this point).
__device__ __forceinline__ void wave_lds_fence() {
  __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
  __builtin_amdgcn_wave_barrier();
  __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}

__device__ __forceinline__ float bf16_bits_to_float(uint16_t b) {
  return __uint_as_float(static_cast<uint32_t>(b) << 16);
}

// float -> bf16 bits, round to nearest even (finite values and infinities).
__device__ __forceinline__ uint16_t float_to_bf16_bits(float f) {
  uint32_t u = __float_as_uint(f);
  u += 0x7FFFu + ((u >> 16) & 1u);
  return static_cast<uint16_t>(u >> 16);
}

// Pins a wave-uniform pointer into scalar registers so that loads take the
// "scalar base + 32-bit lane offset" addressing form.
__device__ __forceinline__ const unsigned char* uniform_ptr(const unsigned char* ptr) {
  const uint64_t v = reinterpret_cast<uint64_t>(ptr);
  const uint32_t lo = __builtin_amdgcn_readfirstlane(static_cast<uint32_t>(v));
  const uint32_t hi = __builtin_amdgcn_readfirstlane(static_cast<uint32_t>(v >> 32));
  return reinterpret_cast<const unsigned char*>((static_cast<uint64_t>(hi) << 32) | lo);
}

__device__ __forceinline__ unsigned char* uniform_ptr_mut(unsigned char* ptr) {
  return const_cast<unsigned char*>(uniform_ptr(ptr));
}

// Global-memory load at (wave-uniform base) + (32-bit lane offset).  STREAMING marks data that is
// read once (the verification pass over the whole cache): the non-temporal hint keeps it from
// displacing useful lines and was worth 7-12 % of the kernel time.
template <typename T, bool STREAMING>
__device__ __forceinline__ T gload(const unsigned char* sbase, uint32_t voff) {
  typedef const __attribute__((address_space(1))) T* gp;
  gp ptr = (gp)((const __attribute__((address_space(1))) unsigned char*)sbase + voff);
  if constexpr (STREAMING) return __builtin_nontemporal_load(ptr);
  else return *ptr;
}

// The same from a per-lane address.
template <typename T, bool STREAMING>
__device__ __forceinline__ T gload_at(const __attribute__((address_space(1))) unsigned char* at) {
  typedef const __attribute__((address_space(1))) T* gp;
  if constexpr (STREAMING) return __builtin_nontemporal_load((gp)at);
  else return *(gp)at;
}

// 64 lanes x 16 bytes from (base + lane offset) to LDS [lds, lds + 1 KB), for N lane offsets and consecutive kilobytes.
// Nothing is returned in registers; the load counter counts one per kilobyte.  (Assembly, because the compiler makes every
// LDS read that follows the builtin wait for all such loads.  M0 cannot be declared as overwritten, it is a reserved
// register; the build report's test holds these kernels to no other use of it.)
// STREAMING: with the non-temporal hint (16 x 36864 tokens without collection 399 us against 446).
template <int N, bool STREAMING>
__device__ __forceinline__ void load_to_lds(uint32_t lds, const unsigned char* base, const uint32_t (&off)[N]) {
#pragma unroll
  for (int i = 0; i < N; ++i) {
    if constexpr (STREAMING)
      asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %1, %2 nt"
                   :: "s"(lds + 1024u * i), "v"(off[i]), "s"(base) : "memory");
    else
      asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %1, %2"
                   :: "s"(lds + 1024u * i), "v"(off[i]), "s"(base) : "memory");
  }
}
// Waits until at most N of this wave's loads and stores are under way.
template <int N>
__device__ __forceinline__ void wait_vm() {
  static_assert(N >= 0 && N < 64, "the counter has six bits");
  asm volatile("s_waitcnt vmcnt(%0)" :: "n"(N) : "memory");
}
// This wave's LDS reads are done: what follows may land on their source.
__device__ __forceinline__ void wait_lds() { asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory"); }

// Write-through store of 16 bytes (4-byte aligned) to base + off.
__device__ __forceinline__ void store_through(unsigned char* base, uint32_t off, f32x4 v) {
  asm volatile("global_store_dwordx4 %0, %1, %2 sc0 sc1\n\ts_nop 1" :: "v"(off), "v"(v), "s"(base) : "memory");
}
__device__ __forceinline__ void store_through(unsigned char* base, uint32_t off, float v) {
  asm volatile("global_store_dword %0, %1, %2 sc0 sc1\n\ts_nop 1" :: "v"(off), "v"(v), "s"(base) : "memory");
}

// A draft step: the drafted token's K/V rows enter the cache and the selection grows by it in the draft call's own launches
// (attn_draft16_kernel with APPEND, then the merge).
struct DraftStep {
  const uint16_t* k_new;      // bf16 [B, Hkv, D]
  const uint16_t* v_new;
  const int32_t* block_table; // [B, max_blocks]
  int32_t* sel_table;         // [B, table_stride]: SplitParams::table
  int2* grown;                // [B] (length of the sequence, of the selection) after the step, for the merge to store
  int32_t* sel_lens;          // [B] what the draft call reads, for the merge
  int32_t max_blocks, cap;    // a sequence of `cap` tokens takes no more
};
// Where the merge of a draft step stores the lengths (one thread per sequence; nobody else in the merge reads or writes them).
struct GrownLengths {
  const int2* grown;          // DraftStep::grown
  int32_t* seq_lens;
  int32_t* sel_seq_lens;
  __device__ __forceinline__ void store(int b) const {
    const int2 to = grown[b];
    seq_lens[b] = to.x;
    sel_seq_lens[b] = to.y;
  }
};
// (Both are an argument of their own, of the kernels of a draft step only: 64 bytes more for every kernel cost an iteration 0.5 us.)
__device__ __forceinline__ const DraftStep& the_one(const DraftStep& s) { return s; }

// Arguments of the KV-streaming attention kernel (verification and draft share it).
struct SplitParams {
  const uint16_t* q;        // verify [B, G, Hq, D]; draft [B, Hq, D] (G = 1)
  const uint16_t* k;
  const uint16_t* v;
  const int32_t* table;     // [B, table_stride] physical page of each logical page
  const int32_t* lens;      // [B] valid tokens
  float* part_o;            // [B, Hkv, nsplit, R, D] un-normalised partial outputs
  float2* part_ml;          // [B, Hkv, nsplit, R]    (running max in log2 units, partial sum)
  float* page_lse;          // [B, Hkv, lse_pages, Rc] log2-sum-exp2 of each page's scaled logits for the Rc collected
                            // rows of a KV head; or, for the logit metric, [B, Hkv, lse_pages] per-token sums of
                            // the collected rows' q . k
  int32_t table_stride;
  int32_t G, g, R, Hq, Hkv;
  int32_t chunk_tokens;     // tokens per chunk (a planned call's are the plan's: the batch, see the leading arguments below)
  int32_t nsplit, lse_pages, max_tokens;
  int32_t lds_q_off;        // byte offset of the query tile inside dynamic LDS
  int32_t row_blocks;       // row blocks of one KV head (32 rows; attn_pair_kernel: 64), one workgroup each
  int32_t collect_rows;     // which verification rows are collected (1: all, 2: first and last)
  int32_t Rc;               // collected rows per KV head (collected_count)
  int32_t window;           // > 0: local masking, a row at position pos sees keys pos - window + 1 .. pos (causal calls)
  uint16_t* out_direct;     // draft calls, and verification with a local mask, with one chunk per (sequence, KV head): the
                            // bf16 output [B, G, Hq, D], which the streaming kernel then normalises and writes itself
                            // (nullptr: partials for a merge kernel)
  int32_t park_tiles;       // attn_pair_kernel: tiles of collected values a wave holds back in LDS
  uint32_t epoch_mul;       // attn_pair_kernel: 2^32 / ticks of the wall-clock interval at whose end they leave
  int2* plan;               // balanced chunking (or nullptr): [B] (first partial slot, chunk tokens) per sequence,
                            // computed by every workgroup from the lengths and written here by workgroup 0
  int32_t batch;            // B (balanced chunking)
  int32_t slots_target;     // workgroups per KV head (and row block) of one launch wave
  int32_t slots_target2;    // j2: of two waves (= j1 where only one plan is wanted)
  int32_t share_margin;     // what cutting the batch into shares has to win, in units (-1: it is not cut)
  int32_t share_group;      // so many consecutive workgroups of a head start on as many shader engines (a power of two)
  int32_t chunk_cap_units;  // longest chunk the plan may produce, in units
  int32_t slots_total;      // slots per KV head the workspace holds
  int64_t page_stride, token_stride, head_stride, num_pages;
  float scale_log2e;
  unsigned long long* timeline;   // profiling builds: where the waves' phase stamps go (nullptr: nowhere)
};

// ---- per-wave phase timeline (builds with -DVEGAS_TIMELINE only: a profiling build, never the product) ----
// Every wave of a streaming kernel notes the wall clock (100 MHz, the same on all compute units) at a few fixed
// program points and stores the notes when it exits: [workgroup][wave][kTimelineEvents] 64-bit stamps in a buffer
// the caller registers with vegas_debug_set_timeline.  In ordinary builds the macros expand to nothing.
constexpr int kTimelineEvents = 8;
enum {
  kTlEntry = 0,        // first instruction of the wave
  kTlLength = 1,       // sequence length known (past the early exit)
  kTlLoadsIssued = 2,  // the first tile's K/V requests are out
  kTlQueries = 3,      // queries in LDS, workgroup past its first barrier
  kTlFirstTile = 4,    // first tile's arithmetic done
  kTlStreamed = 5,     // last tile's arithmetic done
  kTlMerged = 6,       // row maxima exchanged: past the merge's first barrier
  kTlExit = 7          // partial result stored
};
#ifdef VEGAS_TIMELINE
#define VEGAS_TL_DECL unsigned long long tl_stamps[kTimelineEvents] = {0, 0, 0, 0, 0, 0, 0, 0}
// (the empty asm statements keep the compiler from moving memory operations across a stamp)
#define VEGAS_TL(ev)                                       \
  do {                                                     \
    asm volatile("" ::: "memory");                         \
    tl_stamps[ev] = __builtin_amdgcn_s_memrealtime();      \
    asm volatile("" ::: "memory");                         \
  } while (0)
#define VEGAS_TL_FLUSH(buf, waves)                                                                              \
  do {                                                                                                          \
    if ((buf) != nullptr && (threadIdx.x & 63) == 0) {                                                          \
      const unsigned lin = blockIdx.x + gridDim.x * (blockIdx.y + gridDim.y * blockIdx.z);                      \
      unsigned long long* tl_dst = (buf) + (static_cast<size_t>(lin) * (waves) + (threadIdx.x >> 6)) * kTimelineEvents; \
      for (int tl_i = 0; tl_i < kTimelineEvents; ++tl_i) tl_dst[tl_i] = tl_stamps[tl_i];                        \
    }                                                                                                           \
  } while (0)
#else
#define VEGAS_TL_DECL
#define VEGAS_TL(ev)
#define VEGAS_TL_FLUSH(buf, waves)
#endif

// Leading kernel arguments of the streaming kernels: the fields of SplitParams that the first memory requests (page
// ids, sequence length, query rows) depend on (heads by way of the group size, which saves a division) -- 14 dwords, all that can be preloaded.  Leading scalar arguments are preloaded into scalar registers when a wave starts
// (the library is built with kernel-argument preloading); the copies inside SplitParams are then not read.  A planned call's
// first request is for the lengths, so it has the batch where others have the chunk length.
#define VEGAS_SPLIT_HOT_PARAMS                                                                                     \
  const int32_t *hot_table, const int32_t *hot_lens, int2 *hot_plan, const uint16_t *hot_q, int32_t hot_table_stride, \
      int32_t hot_chunk_tokens, int32_t hot_Hkv, int32_t hot_row_blocks, int32_t hot_G, int32_t hot_g
#define VEGAS_SPLIT_HOT_ASSIGN(p)            \
  do {                                       \
    (p).table = hot_table;                   \
    (p).lens = hot_lens;                     \
    (p).plan = hot_plan;                     \
    (p).q = hot_q;                           \
    (p).table_stride = hot_table_stride;     \
    (p).chunk_tokens = hot_chunk_tokens;     \
    if ((p).plan) (p).batch = hot_chunk_tokens; \
    (p).Hkv = hot_Hkv;                       \
    (p).row_blocks = hot_row_blocks;         \
    (p).G = hot_G;                           \
    (p).Hq = hot_Hkv * hot_g;                \
    (p).g = hot_g;                           \
    (p).R = hot_G * hot_g;                   \
  } while (0)
#define VEGAS_SPLIT_HOT_ARGS(sp)                                                                                   \
  (sp).table, (sp).lens, (sp).plan, (sp).q, (sp).table_stride, (sp).chunk_tokens, (sp).Hkv, (sp).row_blocks, (sp).G, \
      (sp).g

struct CombineParams {
  const float* part_o;
  const float2* part_ml;
  const int32_t* lens;
  uint16_t* out;            // bf16 [B, G, Hq, D]
  int32_t G, g, R, Hq, Hkv, chunk_tokens, nsplit, max_tokens;
  int32_t window;           // > 0: chunks wholly before token n - G - window + 1 were skipped and hold nothing
  int32_t D;                // head dimension (128 or 64) = threads per row
  const int2* plan;         // balanced chunking (or nullptr): [B] (first partial slot, chunk tokens)
  int32_t slots_total;      // balanced chunking: partial slots per KV head
};

// Arguments of the one-round-trip merge kernel, all of them preloaded.  shape: rows per KV head (<= 128), head dimension << 8,
// chunks per column (<= 64) << 16.
#define VEGAS_COMBINE_SMALL_PARAMS                                                                                  \
  const float *part_o, const float2 *part_ml, const int32_t *lens, uint16_t *out, int32_t shape, int32_t Hkv,       \
      int32_t chunk_tokens, int32_t max_tokens, int32_t g, int32_t window
#define VEGAS_COMBINE_SMALL_ARGS(cp)                                                                                \
  (cp).part_o, (cp).part_ml, (cp).lens, (cp).out, (cp).R | (cp).D << 8 | (cp).nsplit << 16, (cp).Hkv, (cp).chunk_tokens, \
      (cp).max_tokens, (cp).g, (cp).window

// The rows of one KV head (row = t * g + j for verification token t, head j of the group) whose page log-sum-exps
// are collected: all G g rows (Eq. 2), or the g rows of the first verification token and the g rows of the bonus
// token (Eq. 3; with G <= 2 that is every row).  Only these are written and read back.
__host__ __device__ __forceinline__ int collected_count(int collect_rows, int G, int g) {
  return (collect_rows == 1 || G <= 2) ? G * g : 2 * g;
}
__device__ __forceinline__ int collected_row(int ci, int collect_rows, int G, int g) {   // ci-th collected row
  return (collect_rows == 1 || G <= 2 || ci < g) ? ci : ci + (G - 2) * g;
}

// First chunk that any row of a (windowed) verification call can see.
__device__ __forceinline__ int first_live_chunk(int n, int G, int window, int chunk_tokens) {
  if (window <= 0) return 0;
  const int lo = n - G - window + 1;
  return lo > 0 ? lo / chunk_tokens : 0;
}

// Where the chunk partials of sequence b live and how long its chunks are.  Partial slot of (KV head h, chunk s):
// off + h * stride_h + s.  Uniform chunking: every (sequence, head) column owns nsplit slots of chunk_tokens
// tokens.  Balanced chunking: the slots of one head are shared by all sequences, sequence b starts at plan[b].x
// and its chunks are plan[b].y tokens long.  `last`: the largest s that still is a slot of the workspace (loads
// of slots past a column's chunks are clamped to it and discarded).
struct ColumnSlots {
  int64_t off;
  int32_t stride_h, chunk, last;
  int32_t count;               // chunks the column has, where they are not equal (0: they follow from `chunk`)
};
__host__ __device__ __forceinline__ ColumnSlots planned_slots(int2 e, int slots_total) {      // e: the plan's entry
  ColumnSlots c;
  c.off = e.x;
  c.stride_h = slots_total;
  c.chunk = e.y > 0 ? e.y : 1;
  c.last = slots_total - 1 - e.x;
  c.count = e.y < 0 ? -e.y : 0;
  return c;
}
__host__ __device__ __forceinline__ ColumnSlots column_slots(const int2* plan, int slots_total, int b, int Hkv, int nsplit,
                                                    int chunk_tokens) {
  if (plan) return planned_slots(plan[b], slots_total);
  ColumnSlots c;
  c.off = static_cast<int64_t>(b) * Hkv * nsplit;
  c.stride_h = nsplit;
  c.chunk = chunk_tokens;
  c.last = nsplit - 1;
  c.count = 0;
  return c;
}
// Chunks of n tokens in such a column, and the largest slot that a merge which knows n requests: its last chunk's; none
// (last < 0) for an empty sequence, which may own no slot at all: in a plan whose chunks fill every slot it starts one
// past the last of them.
struct ColumnChunks {
  int32_t ns, last;
};
__host__ __device__ __forceinline__ ColumnChunks column_chunks(const ColumnSlots& cs, int n) {
  ColumnChunks c;
  c.ns = cs.count > 0 ? (n > 0 ? cs.count : 0) : (n + cs.chunk - 1) / cs.chunk;
  c.last = cs.last < c.ns - 1 ? cs.last : c.ns - 1;
  return c;
}
// The slot that a merge requests for chunk s of a column whose slots 0 .. last (>= 0) may be read.
__host__ __device__ __forceinline__ uint32_t requested_slot(int s, int last) {
  const uint32_t a = static_cast<uint32_t>(s), b = static_cast<uint32_t>(last);
  return a < b ? a : b;
}

// Balanced chunking of a batch (B <= 64 sequences, lengths < 2^24), computed identically by every wave that
// calls it, from the lengths alone (the host does not know them).  Two plans:
//   * Equal chunks.  J workgroups per KV head are given to the sequences so that the longest chunk is as short as possible:
//     with C the smallest chunk length for which sum_b ceil(n_b / C) <= J, sequence b is cut into s_b = ceil(n_b / C) equal
//     chunks (multiples of `unit` tokens).  J is j1 (one launch wave) or j2 (two waves of half-size chunks, handed out longest
//     first; wants_second_wave).  Partial slot j = workgroup j, laid out by descending chunk length.
//   * Shares.  Where the longest equal chunk is well above the mean (least_shared_chunk), the sequences are laid end to end and cut
//     every S units, S = 1/J of the whole, whatever sequence that falls into.  A share that holds an end of a sequence is as
//     many pieces, each a workgroup of its own: whole shares start first, then the others by descending length, so that the
//     pieces of one share meet on a compute unit again (the shortest first piece ends first and is followed by the longest
//     second one).  A sequence's partial slots are consecutive: cuts before it + sequences before it, one per piece.
//     The hardware deals workgroups to the shader engines in turn, and none starts before its predecessor has: while every unit
//     is taken, workgroup J + i waits for a unit of the engine on which J - share_group + i started.  So the first J are
//     reversed in groups of share_group: of the last such group the shortest piece sits where the next workgroup, the longest
//     of the second pieces, will wait, and so on.  Verification with collection, 20 rows, us, two waves of equal chunks /
//     shares without / with the reversal: 8 sequences of 16384..131072 tokens 439 / 465 / 413; 16 of 8192..65536 424 / 444 / 407;
//     16 of 4000..16000 132 / 123 / 117; 24 of 1001..20011 205 / 197 / 194.  40 rows: 16 of 8192..65536 449 / 477 / 431.
// No chunk is longer than cap_units * unit tokens (what a workgroup can park in LDS), and a share that would be is not made; a
// batch too long for J2 chunks of that size simply takes more slots.
struct BalancedSlot {
  int32_t b;                    // sequence; < 0: workgroup j has nothing to do
  int32_t c0, chunk;            // its first token here, and how many follow (as far as the sequence reaches)
  int32_t slot;                 // partial slot of the KV head
  int32_t n;                    // the sequence's length
};
// floor and ceil of x / d (a float reciprocal and one correction step either way instead of an integer division, which is two dozen
// instructions).  The estimate is off by one at most where x and d are below 2^23, or where the quotient is below 2^20 whatever rounds (x, d and the
// reciprocal are off by 2^-23 or less of themselves, the product by four times that of the quotient); (q + 1) d has to fit 32 bits.
template <typename Wave>
__host__ __device__ __forceinline__ uint32_t floor_div_small(uint32_t x, uint32_t d) {
  uint32_t q = static_cast<uint32_t>(static_cast<float>(x) * Wave::rcp(static_cast<float>(d)));
  q = q * d > x ? q - 1u : q;                                   // (the estimate is off by one at most)
  return (q + 1u) * d <= x ? q + 1u : q;
}
template <typename Wave>
__host__ __device__ __forceinline__ uint32_t ceil_div_small(uint32_t x, uint32_t d) {
  const uint32_t q = floor_div_small<Wave>(x, d);
  return q * d < x ? q + 1u : q;
}
// Are chunks of c units, of sequences of nu units (this lane's), at most J?
template <typename Wave>
__host__ __device__ __forceinline__ bool chunks_fit(uint32_t nu, uint32_t c, uint32_t J) {
  return Wave::sum(ceil_div_small<Wave>(nu, c)) <= J;
}
// Smallest C >= 1 (in units) with sum over lanes of ceil(nu / C) <= J; nu is this lane's length in units (< 2^18),
// total their sum, longest their maximum (the condition always holds there when J >= number of sequences, and
// nothing changes beyond it).  No plan can beat ceil(total / J), and a batch of equal lengths meets it, so the
// search starts there (balanced_lower_bound) and, where that fails, widens its steps before it bisects; it ends at `most` units at the latest,
// which fit or are no less than the longest.
template <typename Wave>
__host__ __device__ __forceinline__ uint32_t balanced_lower_bound(uint32_t total, uint32_t J) {
  const uint32_t lo = ceil_div_small<Wave>(total, J);           // wave-uniform from here on
  return lo < 1u ? 1u : lo;
}
template <typename Wave>
__host__ __device__ __forceinline__ uint32_t balanced_search(uint32_t nu, uint32_t lo, uint32_t most, uint32_t J) {
  uint32_t step = (lo + 15u) / 16u, hi = lo + step;             // lo fails; find a length that fits
  while (hi < most && !chunks_fit<Wave>(nu, hi, J)) { lo = hi; step *= 2u; hi = lo + step; }
  hi = hi < most ? hi : most;
  ++lo;                                                         // invariant: everything below lo fails, hi fits (or is the end)
  while (lo < hi) {
    const uint32_t mid = (lo + hi) >> 1;
    if (chunks_fit<Wave>(nu, mid, J)) hi = mid; else lo = mid + 1u;
  }
  return lo;
}
template <typename Wave>
__host__ __device__ __forceinline__ uint32_t balanced_chunk_units(uint32_t nu, uint32_t total, uint32_t longest, uint32_t J) {
  const uint32_t lo = balanced_lower_bound<Wave>(total, J);
  if (lo >= longest || chunks_fit<Wave>(nu, lo, J)) return lo < longest ? lo : longest;
  return balanced_search<Wave>(nu, lo, longest, J);
}
// Would chunks of C units, the longest of a plan for j1 workgroups, leave more than a tenth of them idle after giving up
// second_cost units, what the alternative costs?  total / j1 is the lower bound of any plan.  second_cost is high where its workgroups cannot start beside the first's (64-row workgroups fill a
// compute unit's LDS).  There, us, one wave / two, by C / bound: 8 sequences of 500..2000 tokens, 40 rows, 3 / 2.6: 25.6 / 35.6;
// 12 of 2000..20000, 49 rows, 19 / 16.7: 80.2 / 92.0; 32 of 300..1500, 40 rows, 12 / 7.6: 52.9 / 60.8; 24 of 1000..8000,
// 44 / 27: 126.0 / 117.9; 12 of 2000..20000, 80 rows, 103 / 67: 244 / 197.
__host__ __device__ __forceinline__ bool wants_second_wave(uint32_t total, uint32_t j1, uint32_t C, uint32_t second_cost) {
  return C > second_cost && 10u * total < 9u * j1 * (C - second_cost);
}
// Is a batch cut into shares?  If it has no more sequences than workgroups and its longest equal chunk has this many units or more: more than
// a tenth above the mean share, with something for every sequence, and `margin` units above it.  priced: units of all sequences plus kShareCost
// for every one but the first, lives: sequences, J workgroups, S = priced / J rounded up.  The longest equal chunk has that many if one unit less
// does not fit, so a batch that is cut into shares needs two trial lengths and no search, which takes eight as a rule, each a division and a sum
// over the wave.
// us, equal chunks / shares, verification with collection, by C / (priced / J), C the longest equal chunk: 20 rows:
// 8 of 1001..20011 tokens, 25 / 22.4: 71.4 / 68.5; 16 of 4000..16000, 54 / 41: 131 / 117; 32 of 300..1500, 12 / 10.5: 38.5 /
// 39.3; without collection 34.2 / 39.4; 4 of 4096..32768, 21 / 19.6: 63.5 / 71.5.  40 rows: 12 of 2000..20000, 41 / 34.3: 120.7 /
// 114.6; 24 of 5000, 40 / 32.2: 107 / 110, at head dimension 64 78.6 / 74.2; 35 rows, 4 heads (J = 64): 48 of 300..3000,
// 17 / 12.2: 64.8 / 59.8; 32 of 2000..8000, 27 / 21.5: 95.6 / 91.2.  margin: 2 (2 of
// 3000..30000, 40 rows, head dimension 64, 4 / 3.6, no collection: 21 / 24.8), 4 with 64-row workgroups, which take longer to
// begin and to end (7 of 15501, 48 rows and token sums, 31 / 27.3: 215.9 / 218.9 for the iteration).
template <typename Wave>
__host__ __device__ __forceinline__ uint32_t least_shared_chunk(uint32_t priced, uint32_t lives, uint32_t J, uint32_t S, uint32_t margin) {
  const uint32_t more = floor_div_small<Wave>(11u * priced + 8u * lives, 10u * J) + 1u;      // (its least: 10 J C > 11 priced + 8 lives)
  return more > S + margin ? more : S + margin;
}

// slots: workgroups there are; share_margin: for least_shared_chunk, or -1 for no shares; second_cost: for wants_second_wave.
template <typename Wave = GpuWave>
__host__ __device__ __forceinline__ BalancedSlot balanced_slot(const int32_t* lens, int B, int max_tokens, int j1, int j2,
                                                               int share_group, int slots, int share_margin, int second_cost,
                                                               int cap_units, int unit, int j, int2* plan_out) {
  const int lane = Wave::lane();
  uint32_t n = 0u;
  if (lane < B) {
    const int v = lens[lane];
    n = static_cast<uint32_t>(v < 0 ? 0 : (v > max_tokens ? max_tokens : v));
  }
  const uint32_t nu = (n + unit - 1u) / unit;                   // length in units (a constant in the kernels)
  const uint32_t total = Wave::sum(nu);
  BalancedSlot r = {-1, 0, unit, 0, 0};
  if (total == 0u) {
    if (plan_out && lane < B) plan_out[lane] = make_int2(0, unit);
    return r;
  }
  const uint32_t longest = Wave::max(nu);
  const uint64_t live = Wave::ballot(nu > 0u);
  const uint32_t J = j1, lives = __builtin_popcountll(live);
  const uint32_t priced = total + kShareCost * (lives - 1u), S = ceil_div_small<Wave>(priced, J);
  const uint32_t bound = balanced_lower_bound<Wave>(total, J);
  const bool equal = bound >= longest || chunks_fit<Wave>(nu, bound, J);       // (the longest chunk is the bound: no shares)
  bool shares = false;
  uint32_t C = bound < longest ? bound : longest;
  if (!equal) {
    uint32_t most = longest;
    if (share_margin >= 0 && S <= static_cast<uint32_t>(cap_units) && J + lives <= static_cast<uint32_t>(slots) + 1u && lives <= J) {
      const uint32_t below = least_shared_chunk<Wave>(priced, lives, J, S, static_cast<uint32_t>(share_margin)) - 1u;
      if (below < longest) {
        shares = !chunks_fit<Wave>(nu, below, J);
        most = below;
      }
    }
    if (!shares) C = balanced_search<Wave>(nu, bound, most, J);
  }
  if (shares) {
    const uint32_t rank = __builtin_popcountll(live & ((1ull << lane) - 1ull));
    const uint32_t base = Wave::prefix_sum(nu) - nu + kShareCost * rank;       // where the sequence's first token lies
    const uint32_t q = floor_div_small<Wave>(base, S), count = nu > 0u ? floor_div_small<Wave>(base + nu - 1u, S) - q + 1u : 0u;
    if (plan_out && lane < B) plan_out[lane] = nu > 0u ? make_int2(q + rank, -static_cast<int>(count)) : make_int2(0, unit);
    const uint32_t head = min(nu, (q + 1u) * S - base);                       // first piece (0 if empty); last one, where there
    const uint32_t tail = count > 1u ? nu - head - (count - 2u) * S : 0u;     // are several; whole shares between them
    const uint32_t mid = count > 2u ? count - 2u : 0u;
    const uint32_t before = Wave::prefix_sum(mid) - mid;
    const uint32_t mids = Wave::readlane(before + mid, 63);
    const uint32_t at = static_cast<uint32_t>(j) < (J & -static_cast<uint32_t>(share_group)) ? j ^ (share_group - 1) : j;
    uint64_t hit;
    uint32_t piece;
    if (at < mids) {
      hit = Wave::ballot(at >= before && at - before < mid);
      piece = at - Wave::readlane(before, __builtin_ctzll(hit)) + 1u;
    } else {                                                    // the others, longest first
      uint32_t at_head = mids, at_tail = mids;
      for (int i0 = 0; i0 < B; i0 += 4) {                       // (lanes past the batch have nothing)
#pragma unroll
        for (int i = i0; i < i0 + 4; ++i) {
          const uint32_t hi = Wave::readlane(head, i), ti = Wave::readlane(tail, i);
          at_head += (hi + (i < lane ? 1u : 0u) > head ? 1u : 0u) + (ti > head ? 1u : 0u);
          at_tail += (hi >= tail ? 1u : 0u) + (ti + (i < lane ? 1u : 0u) > tail ? 1u : 0u);
        }
      }
      const uint64_t heads = Wave::ballot(head > 0u && at_head == at);
      const uint64_t tails = Wave::ballot(tail > 0u && at_tail == at);
      hit = heads | tails;
      if (hit == 0ull) return r;
      piece = heads ? 0u : Wave::readlane(count, __builtin_ctzll(hit)) - 1u;
    }
    r.b = __builtin_ctzll(hit);
    const uint32_t first = Wave::readlane(head, r.b);
    r.c0 = piece == 0u ? 0 : static_cast<int>((first + (piece - 1u) * S) * unit);
    r.chunk = static_cast<int>((piece == 0u ? first : S) * unit);
    r.slot = Wave::readlane(q + rank, r.b) + piece;
    r.n = Wave::readlane(n, r.b);
    return r;
  }
  if (j2 > j1 && wants_second_wave(total, static_cast<uint32_t>(j1), C, static_cast<uint32_t>(second_cost)))
    C = balanced_chunk_units<Wave>(nu, total, longest, static_cast<uint32_t>(j2));
  C = min(C, static_cast<uint32_t>(cap_units));
  const uint32_t s = ceil_div_small<Wave>(nu, C);               // chunks of this sequence (0 if empty)
  const int chunk = s > 0u ? static_cast<int>(ceil_div_small<Wave>(nu, s) * unit) : 0;   // equal chunks, at most C units
  int P = 0;                                                    // slots of the sequences with longer chunks
  for (int i0 = 0; i0 < B; i0 += 4) {                           // (lanes past the batch have none)
#pragma unroll
    for (int i = i0; i < i0 + 4; ++i) {
      const int ci = Wave::readlane(chunk, i);
      const int si = Wave::readlane(static_cast<int>(s), i);
      P += ci + (i < lane ? 1 : 0) > chunk ? si : 0;
    }
  }
  if (plan_out && lane < B) plan_out[lane] = make_int2(P, chunk > 0 ? chunk : unit);
  const uint64_t hit = Wave::ballot(lane < B && s > 0u && j >= P && j < P + static_cast<int>(s));
  if (hit == 0ull) return r;
  r.b = __builtin_ctzll(hit);
  r.chunk = Wave::readlane(chunk, r.b);
  r.c0 = (j - Wave::readlane(P, r.b)) * r.chunk;
  r.slot = j;
  r.n = Wave::readlane(n, r.b);
  return r;
}

struct FinalizeParams {
  const float* part_o;
  const float2* part_ml;
  const float* page_lse;
  const int32_t* lens;
  uint16_t* out;            // bf16 [B, G, Hq, D]
  float* block_scores;      // [B, max_blocks]
  int32_t G, g, R, Hq, Hkv, chunk_tokens, nsplit, max_tokens;
  int32_t max_blocks, lse_pages, collect_rows;
  int32_t Rc;               // collected rows per KV head (collected_count)
  int32_t D;                // head dimension (128 or 64)
  const int2* plan;         // balanced chunking (or nullptr): [B] (first partial slot, chunk tokens)
  int32_t slots_total;      // balanced chunking: partial slots per KV head
  int32_t nC;               // logit metric: workgroups that sum the token partials (1024 tokens each)
  float tok_norm;           // logit metric: softmax_scale / (collected rows * H_q)
  int32_t nA;               // workgroups that merge rows (two rows each); the rest score pages
  float inv_norm;
};

struct SelectParams {
  const float* block_scores;
  const int32_t* block_table;
  const int32_t* seq_lens;
  const int32_t* budgets;   // or nullptr
  int32_t* sel_table;
  int32_t* sel_seq_lens;
  int32_t budget_tokens, G, max_blocks, max_sel_blocks, max_tokens;
  int32_t key_cap;          // score keys that fit the kernel's dynamic LDS
  float budget_ratio;       // > 0: budget = ceil(ratio * seq_len) unless per-sequence budgets are given
};

// Token budget of one sequence: per-sequence value, or a sparsity ratio of its length (App. C), or the call's constant.
__device__ __forceinline__ int sequence_budget(const int32_t* budgets, float ratio, int constant, int b, int n) {
  int budget = budgets ? budgets[b] : (ratio > 0.f ? static_cast<int>(ceilf(ratio * static_cast<float>(n))) : constant);
  return budget < 0 ? 0 : budget;
}

struct ExtendParams {
  const int32_t* block_table;
  const int32_t* seq_lens;   // lengths after the append
  int32_t* sel_table;
  int32_t* sel_seq_lens;
  int32_t batch, num_new, max_blocks, max_sel_blocks, page_size;
};

}  // namespace vegas
