// Host side of the C ABI declared in include/vegas.h: argument validation, launch planning,
// workspace carving and kernel launches.  Nothing here allocates or synchronises.
#include "../../include/vegas.h"

#include <hip/hip_runtime.h>

#include <cmath>
#include <iterator>
#include <map>
#include <mutex>
#include <set>
#include <utility>

#include "attn_finalize.hpp"
#include "attn_draft.hpp"
#include "attn_pair.hpp"
#include "attn_split.hpp"
#include "debug_kernels.hpp"
#include "kv_append.hpp"
#include "plan_rules.hpp"
#include "select_blocks.hpp"
#include "select_tokens.hpp"
#include "vegas_common.hpp"

namespace {

using namespace vegas;

constexpr int kDefaultCU = 256;       // MI355X compute units: assumed where no device is visible
constexpr size_t kAlign = 256;
constexpr size_t kLoneLds = 81 * 1024;   // LDS of a workgroup that is to have a compute unit to itself (BatchPlan::alone)

// Compute units of the current device, asked once per device.  The launch plans aim at one or two workgroups per
// compute unit, and the workspace is sized from the same plans, so sizing and launching must see the same number:
// without a visible device (the pure-host sizing call on a machine that has none) it is the MI355X's 256.
int device_cu_count() {
  static std::mutex mu;
  static std::map<int, int> known;
  int dev = 0;
  if (hipGetDevice(&dev) != hipSuccess) {
    (void)hipGetLastError();
    return kDefaultCU;
  }
  std::lock_guard<std::mutex> lock(mu);
  const auto it = known.find(dev);
  if (it != known.end()) return it->second;
  int n = 0;
  if (hipDeviceGetAttribute(&n, hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess || n <= 0) {
    (void)hipGetLastError();
    n = kDefaultCU;
  }
  known[dev] = n;
  return n;
}
// Longest selection a draft call of more than kDraftRows rows per KV head streams with one workgroup per (sequence,
// KV head): 256 tokens at head dimension 128, 384 at 64 (tiles of half the bytes), each plus the two pages of slack a
// selection table carries.  (Smaller groups: lone_workgroup_tokens.)
constexpr int kFinishTokens128 = 288, kFinishTokens64 = 416;

inline size_t align_up(size_t x) { return (x + kAlign - 1) / kAlign * kAlign; }
inline bool aligned16(const void* p) { return (reinterpret_cast<uintptr_t>(p) & 15u) == 0; }

struct SplitPlan {
  int R = 0, Rc = 0, NB = 0, NW = 0, chunk = 0, nsplit = 0, lse_pages = 0;   // Rc: collected rows per KV head
  bool pair = false;                 // verification of more than 32 rows per KV head: 64-row workgroups (attn_pair_kernel)
  int pair_waves = kPairWaves;       // its waves
  bool balanced = false;             // chunk lengths per sequence, computed on the GPU from the lengths (ragged batches)
  BatchPlan bp;                      // balanced: numbers of workgroups, in units of kTile * NW tokens
  size_t off_plan = 0;               // balanced: [B] (first slot, chunk tokens)
  size_t off_part_o = 0, off_part_ml = 0, off_page_lse = 0, total = 0;
};

int check_common(const vegas_desc* d) {
  if (!d) return VEGAS_ERR_NULL;
  if (d->batch <= 0 || d->num_q_heads <= 0 || d->num_kv_heads <= 0 || d->max_blocks <= 0 ||
      d->max_seq_len <= 0 || d->num_pages <= 0)
    return VEGAS_ERR_SHAPE;
  if (d->num_q_heads % d->num_kv_heads != 0) return VEGAS_ERR_SHAPE;
  if (d->head_dim != 128 && d->head_dim != 64) return VEGAS_ERR_UNSUPPORTED;
  if (d->max_seq_len > (1 << 30)) return VEGAS_ERR_UNSUPPORTED;      // token counts and offsets are 32-bit in the kernels
  if (d->batch > 65535) return VEGAS_ERR_UNSUPPORTED;                // sequences are a grid's y or z dimension
  if (d->page_size != 1 && d->page_size != 2 && d->page_size != 4 && d->page_size != 8 && d->page_size != kPage)
    return VEGAS_ERR_UNSUPPORTED;
  if (d->kv_head_stride < d->head_dim || d->kv_token_stride < d->head_dim ||
      d->kv_page_stride < static_cast<int64_t>(d->page_size) * d->head_dim)
    return VEGAS_ERR_SHAPE;
  if ((d->kv_head_stride % 8) || (d->kv_token_stride % 8) || (d->kv_page_stride % 8)) return VEGAS_ERR_ALIGN;
  if (d->kv_chunk_tokens < 0 || (d->kv_chunk_tokens % kTile) != 0) return VEGAS_ERR_SHAPE;
  if (!(d->softmax_scale > 0.f)) return VEGAS_ERR_SHAPE;
  if (d->reserved != 0) return VEGAS_ERR_SHAPE;
  return VEGAS_OK;
}

// Verification and selection work on 16-token pages and a block table that covers max_seq_len.
int check_paged16(const vegas_desc* d) {
  if (d->page_size != kPage) return VEGAS_ERR_UNSUPPORTED;
  if (static_cast<int64_t>(d->max_seq_len) > static_cast<int64_t>(d->max_blocks) * kPage) return VEGAS_ERR_SHAPE;
  return VEGAS_OK;
}

// Rows stacked on one KV head decide the kernel variant; the chunk size decides the grid.
// max_len bounds the lengths the call may see; small problems get small workgroups.
// collect: 0 nothing, 1 page log-sum-exps [pages x rows], 2 token sums [padded tokens] per (sequence, KV head)
int plan_split(const vegas_desc* d, int rows_per_head, int max_len, int collect, int wg_per_cu, SplitPlan* pl,
               bool may_pair = false, bool may_finish = false, bool fine = false) {
  pl->R = rows_per_head;
  const int num_cu = device_cu_count();
  const int64_t heads = static_cast<int64_t>(d->batch) * d->num_kv_heads;
  if (rows_per_head > 128) return VEGAS_ERR_UNSUPPORTED;
  pl->NW = 4;                                        // measured: 4-wave groups match or beat 8-wave groups everywhere but in short bands (below)
  // Row blocks: 32 rows each, sibling workgroups that share an XCD's L2; verification of more than 32 rows (with the two
  // sum rows of the logit metric, which take a block's spare rows) has blocks of 64 served from one read of K/V, small
  // calls excepted (unless they bring a chunk length, whose collected values siblings might not park).  The sum rows may
  // have the last block to themselves.
  const int tile_rows = rows_per_head + (collect == 2 ? 2 : 0);
  const bool siblings = d->kv_chunk_tokens == 0 && rows_as_siblings(d->batch, d->num_kv_heads, max_len, rows_per_head,
                                                                    d->collect_rows, collect == 2, d->head_dim);
  pl->pair = may_pair && tile_rows > 32 && !siblings;
  pl->NB = (tile_rows + (pl->pair ? kPairRows : 32) - 1) / (pl->pair ? kPairRows : 32);
  // A draft call (may_finish) over a selection that one workgroup per (sequence, KV head) streams fast enough: it
  // writes the output rows itself, so no merge kernel is launched.  Groups of more than kDraftRows heads run the 32-row
  // kernel, whose workgroups take about 0.35 us per tile; at 4K context, five draft calls per iteration: 256 selected
  // tokens (eight tiles, two per wave) 54.7 us against 59.3 us with three chunks and a merge; 384 tokens 61.8 against
  // 59.4; 512 tokens 67.2 against 59.8.  At head dimension 64 (32K context, 64 query heads): 256 tokens 66.5 against
  // 73.0 us, 384 tokens 71.4 against 73.0, 512 tokens 75.1 against 73.3.
  const bool own_chunks = may_finish && d->kv_chunk_tokens == 0;
  const bool short_call = own_chunks && max_len <= (d->head_dim == 64 ? kFinishTokens64 : kFinishTokens128) &&
                          heads * pl->NB <= num_cu;
  const int unit = kTile * pl->NW;
  int chunk = d->kv_chunk_tokens;
  const int whole = (max_len + unit - 1) / unit * unit;
  if (short_call) chunk = whole;
  if (chunk == 0) {
    // Verification: one workgroup per CU when the batch is small (at 32K context 256 equal workgroups
    // beat 512); draft calls are latency-bound and like two small workgroups per CU.  With many
    // (sequence, head) columns, shorter chunks balance ragged lengths better.
    const int64_t columns = heads * pl->NB;
    int64_t splits = static_cast<int64_t>(num_cu) * wg_per_cu / columns;
    if (splits < 1) splits = 1;
    int64_t c = (max_len + splits - 1) / splits;
    {
      // Round to whole units: up, unless a bound a little above a multiple (a selection table with two pages of
      // slack) would then double every wave's tiles -- a few more workgroups than planned, of a tile per wave at most in
      // all, are the better price where two of them fit a compute unit.  (More than that are a second round of the chip:
      // one sequence, verification with collection, up to a quarter more workgroups / rounded up: 17000 tokens 26.1 / 20.8 us,
      // 45000 51.3 / 38.2, 100000 92.8 / 73.5, with 4 KV heads 61.8 / 44.1; draft calls, 16 x 4352 tokens 61.2 / 51.0, 1 x 8704
      // 17.5 / 12.4.  64-row workgroups fill a compute unit's LDS: 288 of them, 80 rows, 32749 tokens, took two rounds.)
      const int64_t up = (c + unit - 1) / unit * unit, down = c / unit * unit;
      c = up;
      if (!pl->pair && down >= unit && max_len - splits * down < unit &&
          ((max_len + down - 1) / down) * columns * 4 <= static_cast<int64_t>(num_cu) * wg_per_cu * 5) c = down;
    }
    // What a workgroup collects is parked in LDS until its chunk ends, so a chunk cannot be arbitrarily long.  A
    // chunk that gives every CU exactly one workgroup is taken as it is while its LDS fits (batch 4 x 64K tokens:
    // 256 chunks of 8192 tokens reach 78 % of the HBM peak, 512 chunks of 4096 tokens 75 %); otherwise chunks are
    // capped so that two workgroups fit a CU.  (64-row workgroups park no whole chunk: unplanned_pair_chunk.)
    const int64_t cap = (columns >= num_cu) ? 2048 : 4096;
    const int prows = rows_per_head < 32 ? rows_per_head : 32;
    const bool fits_alone = columns * splits >= num_cu / 2 &&
                            split_lds_bytes(pl->NW, prows, collect, static_cast<int>(c), d->head_dim) <= 150 * 1024;
    if (!pl->pair && c > cap && !(wg_per_cu == 1 && fits_alone)) c = cap;
    if (pl->pair && splits == 1) c = (unplanned_pair_chunk(rows_per_head, max_len) + unit - 1) / unit * unit;
    chunk = static_cast<int>(c);
  }
  // A batch of several sequences whose lengths the host does not know (only max_seq_len, which may be loose): every
  // workgroup derives the chunk length of each sequence from seq_lens on the GPU (balanced_slot), so that a fixed
  // number of workgroups stream about the same number of tokens each.  (A host-side chunk length cuts a ragged
  // batch into unequal numbers of equal chunks: 45 % of the HBM peak on 16 sequences of 8K..64K tokens, 40 rows,
  // against 68 % with the plan; and it sizes chunks for lengths that may never occur.)
  const int64_t per_head = static_cast<int64_t>(d->num_kv_heads) * pl->NB;   // workgroups per slot
  pl->balanced = may_pair && d->kv_chunk_tokens == 0 && d->batch >= 2 && d->batch <= 64 && max_len < (1 << 24) &&
                 per_head <= num_cu;
  // Smaller groups have a rule of their own, and so has verification with a local mask: no row sees more than
  // window + G - 1 tokens, and a workgroup begins where the first of them is (16 sequences of 8192..65536 tokens, 40 rows,
  // head dimension 64, window 128: 11.7 us with a merge, 5.5 without).
  const bool banded = !may_finish && d->window > 0 && d->kv_chunk_tokens == 0 &&
                      lone_workgroup_band(d->window, d->num_queries, max_len, chunk, lone_band_tokens(d->head_dim));
  const bool finish = banded || (own_chunks && rows_per_head <= kDraftRows && max_len <= lone_workgroup_tokens(heads, num_cu, d->head_dim));
  if (fine && own_chunks && !finish && rows_per_head <= kDraftRows && chunk == unit)
    chunk = draft_chunk_tokens(heads, num_cu, max_len, unit, rows_per_head * d->head_dim);
  // (A call that one workgroup per column finishes uses no partials; its workspace is sized for the chunked plan all
  //  the same, so that these rules move neither the sizes callers allocate nor what the built-in scratch takes.)
  size_t slots = static_cast<size_t>(heads) * ((max_len + chunk - 1) / chunk);   // chunk partials the workspace holds
  if (finish) chunk = whole;
  if (banded && eight_wave_band(heads, pl->NB, num_cu, std::min<int64_t>(static_cast<int64_t>(d->window) + d->num_queries - 1, max_len), d->head_dim,
                                rows_per_head))
    pl->NW = kBandWaves;
  pl->chunk = chunk;
  pl->nsplit = (max_len + chunk - 1) / chunk;
  if (pl->balanced) {
    // one workgroup per CU with chunks as long as its LDS can park (16 x 36864 tokens, 20 rows: 256 chunks of
    // 18432 tokens reach 80 % of the peak, 512 of 9216 75 %, 4096-token chunks 69 %), or shares of the batch when the
    // lengths are too ragged for equal chunks.  The same for 64-row workgroups, which park no whole chunk (4 x 65536 tokens, 40
    // rows: 256 chunks 196 us, 512 198, 1024 208; 2 x 8192: 18.5, 26.9, 36.1).
    int cap = 1 << 24;
    if (collect != 0 && !pl->pair) {
      const int prows = rows_per_head < 32 ? rows_per_head : 32;
      cap = unit;
      while (split_lds_bytes(pl->NW, prows, collect, cap + unit, d->head_dim) <= 150 * 1024 && cap < (1 << 24)) cap += unit;
    }
    pl->bp = batch_plan(num_cu, per_head, d->batch, max_len, unit, cap / unit, pl->pair,
                        pl->pair && pair_two_per_cu(d->head_dim, collect), collect != 0, d->head_dim);
    pl->chunk = collect != 0 && !pl->pair ? cap : unit;         // sizes the LDS that parks a chunk's collected values
    slots = static_cast<size_t>(d->num_kv_heads) * pl->bp.JS;   // (sibling row blocks share a slot)
  }
  if (pl->pair) pl->pair_waves = pair_waves(d->head_dim, collect, pl->NB, d->batch, max_len, static_cast<int64_t>(d->batch) * max_len * per_head / num_cu);
  pl->lse_pages = collect == 1 ? (max_len + kPage - 1) / kPage
                               : (collect == 2 ? (pl->balanced ? (max_len + unit - 1) / unit * unit : pl->nsplit * chunk) : 0);
  size_t off = 0;
  const size_t hs = static_cast<size_t>(heads);
  pl->off_part_o = off;  off += align_up(slots * pl->R * d->head_dim * sizeof(float));
  pl->off_part_ml = off; off += align_up(slots * pl->R * sizeof(float2));
  pl->off_page_lse = off;
  pl->Rc = collected_count(d->collect_rows, d->num_queries, d->num_q_heads / d->num_kv_heads);
  off += align_up(hs * static_cast<size_t>(pl->lse_pages) * (collect == 2 ? 1 : pl->Rc) * sizeof(float));
  pl->off_plan = off;
  if (pl->balanced) off += align_up(static_cast<size_t>(d->batch) * sizeof(int2));
  pl->total = off;
  return VEGAS_OK;
}

int plan_verify(const vegas_desc* d, SplitPlan* pl) {
  if (d->num_queries <= 0) return VEGAS_ERR_SHAPE;
  if (d->collect_rows < 0 || d->collect_rows > 2) return VEGAS_ERR_SHAPE;
  const int g = d->num_q_heads / d->num_kv_heads;
  if (d->score_metric != VEGAS_METRIC_PAGE_WEIGHTS && d->score_metric != VEGAS_METRIC_TOKEN_LOGITS)
    return VEGAS_ERR_SHAPE;
  const int R = d->num_queries * g;
  const int collect = d->collect_rows == 0 ? 0 : (d->score_metric == VEGAS_METRIC_TOKEN_LOGITS ? 2 : 1);
  return plan_split(d, R, d->max_seq_len, collect, 1, pl, d->window == 0, false);
}

// What a draft step keeps for its merge behind a draft call's partials: per sequence the grown lengths and the one it attends over.
size_t step_bytes(const vegas_desc* d) { return align_up(static_cast<size_t>(d->batch) * (sizeof(int2) + sizeof(int32_t))); }

// have: bytes of workspace there are.  (Chunks shorter than a unit need more slots: a workspace sized without them, for another
// descriptor, keeps the units.)
int plan_draft(const vegas_desc* d, SplitPlan* pl, size_t have = ~size_t(0)) {
  const int g = d->num_q_heads / d->num_kv_heads;
  const int rc = plan_split(d, g, d->max_seq_len, 0, 2, pl, false, true, true);
  if (rc != VEGAS_OK || pl->total <= have) return rc;
  return plan_split(d, g, d->max_seq_len, 0, 2, pl, false, true);
}

// A kernel whose static + dynamic LDS passes the default 64 KB limit needs its limit raised first: once
// per (device, kernel function).  The table is keyed by the function's address because every
// instantiation of the streaming kernel has the same C++ type.
// (vegas_init raises every kernel's limit up front; this lazy path serves callers that never call it.)
int ensure_dynamic_lds(const void* kern, size_t lds) {
  if (lds <= 32 * 1024) return VEGAS_OK;
  static std::mutex mu;
  static std::set<std::pair<int, const void*>> raised;
  int dev = 0;
  if (hipGetDevice(&dev) != hipSuccess) return VEGAS_ERR_LAUNCH;
  std::lock_guard<std::mutex> lock(mu);
  const std::pair<int, const void*> key(dev, kern);
  if (raised.count(key)) return VEGAS_OK;
  hipFuncAttributes attr;
  if (hipFuncGetAttributes(&attr, kern) != hipSuccess) return VEGAS_ERR_LAUNCH;
  const int room = 160 * 1024 - static_cast<int>(attr.sharedSizeBytes);   // the CU's LDS minus the kernel's static part
  if (hipFuncSetAttribute(kern, hipFuncAttributeMaxDynamicSharedMemorySize, room) != hipSuccess)
    return VEGAS_ERR_LAUNCH;
  raised.insert(key);
  return VEGAS_OK;
}

// Profiling builds (-DVEGAS_TIMELINE): the buffer that vegas_debug_set_timeline registered receives the phase stamps of
// the next streaming kernels (if it is large enough for the launch); ordinary builds have no such buffer.
unsigned long long* g_timeline = nullptr;
size_t g_timeline_bytes = 0;

template <typename Kern, typename... More>
int launch_one(Kern kern, dim3 grid, dim3 block, size_t lds, hipStream_t st, SplitParams sp, More... more) {
  if (int rc = ensure_dynamic_lds(reinterpret_cast<const void*>(kern), lds)) return rc;
  const size_t tl_need = static_cast<size_t>(grid.x) * grid.y * grid.z * (block.x / 64) * kTimelineEvents * sizeof(unsigned long long);
  sp.timeline = (g_timeline != nullptr && tl_need <= g_timeline_bytes) ? g_timeline : nullptr;
  hipLaunchKernelGGL(kern, grid, block, lds, st, VEGAS_SPLIT_HOT_ARGS(sp), sp, more...);
  return hipGetLastError() == hipSuccess ? VEGAS_OK : VEGAS_ERR_LAUNCH;
}

// May a draft call's selections be read past the last-level cache?  (The bound first: lengths that cannot get there are not looked at.)
bool draft_chooses(int batch, int max_tokens, int kv_heads, int head_dim) {
  return past_cache(static_cast<uint64_t>(batch) * ((static_cast<uint64_t>(max_tokens) + 15) / 16), kv_heads, head_dim);
}

// More workgroups per (KV head, sequence) than a grid dimension holds?  (32-row blocks; 64-row ones: launch_split_d)
bool exceeds_grid(const SplitPlan& pl) {
  return static_cast<int64_t>(pl.NB) * (pl.balanced ? pl.bp.JS : pl.nsplit) > 65535;
}

template <bool CAUSAL, int COLLECT, int D>
int launch_split_d(const SplitPlan& pl, SplitParams sp, int batch, hipStream_t st, int page_size, const DraftStep* step) {
  if constexpr (CAUSAL) {
    if (pl.pair) {
      const unsigned slots = pl.balanced ? pl.bp.JS : pl.nsplit, seqs = pl.balanced ? 1 : batch;
      const PairLds lds = pair_lds(pl.R, pl.Rc, pl.NB, COLLECT, D, pl.pair_waves);
      sp.row_blocks = pl.NB;
      sp.lds_q_off = static_cast<int32_t>(lds.off_max);
      sp.park_tiles = lds.park_tiles;
      if (lds.bytes > 160 * 1024 || (COLLECT != 0 && lds.park_tiles < 1)) return VEGAS_ERR_UNSUPPORTED;
      // A wave parks a tile every 2.7 us (1.35 at head dimension 64) where HBM bounds the stream; the interval ends when
      // its LDS is three quarters full, so that the faster compute units seldom have to write before it does (16 x 36864
      // tokens, 40 rows, 15 tiles: 60 % 434 us, 75 % 430, 95 % 440, 140 % 446; without collection 395).
      const double ticks = 0.75 * lds.park_tiles * (D == 128 ? 270 : 135) * pl.pair_waves / kPairWaves;
      sp.epoch_mul = static_cast<uint32_t>(4294967296.0 / (ticks < 256 ? 256 : ticks));
      dim3 pgrid(sp.Hkv, pl.NB * slots, seqs);
      // Chunks are a dimension of the grid, and the interface's limit on them (vegas.h, kv_chunk_tokens) counts 32-row
      // blocks.  33 to 64 rows with chunks of a multiple of 64 tokens are exempt from it: the grid is folded for them.
      const int tile_rows = pl.R + (COLLECT == 2 ? 2 : 0);
      const bool folds = pl.R > 32 && tile_rows <= kPairRows && pl.chunk % (2 * kTile) == 0;
      if (!folds && static_cast<uint64_t>((tile_rows + 31) / 32) * slots > 65535u) return VEGAS_ERR_UNSUPPORTED;
      if (pgrid.y > 65535u) {
        pgrid.z = seqs * ((pgrid.y + kPairFold - 1) / kPairFold);
        pgrid.y = kPairFold;
        if (pgrid.z > 65535u) return VEGAS_ERR_UNSUPPORTED;
      }
      const dim3 block(pl.pair_waves * 64);
      if constexpr (D == 64 && COLLECT == 1) {
        if (pl.pair_waves != kPairWaves) {
          if (pl.NB == 1) return launch_one(attn_pair_kernel<COLLECT, D, true, 2 * kPairWaves>, pgrid, block, lds.bytes, st, sp);
          return launch_one(attn_pair_kernel<COLLECT, D, false, 2 * kPairWaves>, pgrid, block, lds.bytes, st, sp);
        }
      }
      if (pl.NB == 1) return launch_one(attn_pair_kernel<COLLECT, D, true>, pgrid, block, lds.bytes, st, sp);
      return launch_one(attn_pair_kernel<COLLECT, D, false>, pgrid, block, lds.bytes, st, sp);
    }
  }
  // (KV head, row block + NB * chunk, sequence): the kernels read their indices off the grid without a division
  const dim3 grid = pl.balanced ? dim3(sp.Hkv, static_cast<unsigned>(pl.NB) * pl.bp.JS, 1)
                                : dim3(sp.Hkv, static_cast<unsigned>(pl.NB) * pl.nsplit, batch);
  if (exceeds_grid(pl)) return VEGAS_ERR_UNSUPPORTED;
  const int rows = pl.R < 32 ? pl.R : 32;
  size_t lds = split_lds_bytes(pl.NW, rows, COLLECT, pl.chunk, D);
  if (pl.balanced && pl.bp.alone && lds < kLoneLds) lds = kLoneLds;
  sp.lds_q_off = static_cast<int32_t>(lds - split_lds_tail_bytes(pl.NW, D));
  sp.row_blocks = pl.NB;
  if (lds > 160 * 1024) return VEGAS_ERR_UNSUPPORTED;
  if constexpr (!CAUSAL && COLLECT == 0) {
    // one draft token, a group of at most 16 heads, 16-token pages: the kernel written for exactly that
    if (pl.R <= kDraftRows && sp.G == 1 && pl.NB == 1) {
      const dim3 dblock(kDraftWaves * 64);
      const size_t dlds = draft16_lds_bytes(pl.R, D);
      const bool choose = draft_chooses(batch, sp.max_tokens, sp.Hkv, D);
      if (step != nullptr) return launch_one(attn_draft16_kernel<D, 4, false, false, DraftStep>, grid, dblock, dlds, st, sp, *step);
      const int64_t columns = static_cast<int64_t>(batch) * sp.Hkv;
      const bool lone = sp.out_direct != nullptr && !choose;       // one workgroup per column, or one per part of its V
      const int parts = lone ? draft_value_parts(columns, device_cu_count(), D) : 1;
      auto launch = [&](auto ps, auto ring, auto value_dims) {
        constexpr int PS = decltype(ps)::value, DV = decltype(value_dims)::value;
        constexpr bool RING = decltype(ring)::value;
        const size_t bytes = RING ? draft_ring_lds_bytes() : dlds;
        if constexpr (DV == D) return launch_one(attn_draft16_kernel<D, PS, false, RING>, grid, dblock, bytes, st, sp);
        else {
          SplitParams cut = sp;
          cut.row_blocks = column_rounds(static_cast<int>(columns), sp.Hkv);      // (a preloaded argument that no draft call needs)
          const unsigned width = part_grid_width(sp.Hkv);
          return launch_one(attn_draft16_parts_kernel<D, DV, PS, RING>, dim3(width, D / DV, static_cast<unsigned>((columns + width - 1) / width)), dblock,
                            bytes, st, cut);
        }
      };
      auto by_parts = [&](auto ps, auto ring) {
        if (parts == D / 32) return launch(ps, ring, std::integral_constant<int, 32>{});
        if constexpr (D == 128) {
          if (parts == 2) return launch(ps, ring, std::integral_constant<int, 64>{});
        }
        return launch(ps, ring, std::integral_constant<int, D>{});
      };
      if constexpr (D == 128) {
        if (page_size == kPage && lone && ring_draft(columns, device_cu_count(), pl.chunk))
          return by_parts(std::integral_constant<int, 4>{}, std::true_type{});
      }
      auto by_page = [&](auto ps) {
        if (choose) return launch_one(attn_draft16_kernel<D, decltype(ps)::value, true>, grid, dblock, dlds, st, sp);
        return by_parts(ps, std::false_type{});
      };
      switch (page_size) {                              // (draft calls may walk a table of smaller pages)
        case 1: return by_page(std::integral_constant<int, 0>{});
        case 2: return by_page(std::integral_constant<int, 1>{});
        case 4: return by_page(std::integral_constant<int, 2>{});
        case 8: return by_page(std::integral_constant<int, 3>{});
        default: return by_page(std::integral_constant<int, 4>{});
      }
    }
    switch (page_size) {                                // larger groups: the 32-row kernel, any page size
      case 1: return launch_one(attn_split_kernel<4, 2, false, 0, false, 0, false, D>, grid, dim3(256), lds, st, sp);
      case 2: return launch_one(attn_split_kernel<4, 2, false, 0, false, 1, false, D>, grid, dim3(256), lds, st, sp);
      case 4: return launch_one(attn_split_kernel<4, 2, false, 0, false, 2, false, D>, grid, dim3(256), lds, st, sp);
      case 8: return launch_one(attn_split_kernel<4, 2, false, 0, false, 3, false, D>, grid, dim3(256), lds, st, sp);
      default: break;
    }
  }
  if constexpr (CAUSAL && COLLECT == 0) {           // banded layer: local masking on top of the causal mask
    if (sp.window > 0) {
      if (pl.NW == kBandWaves) {
        if (pl.NB == 1) return launch_one(attn_split_kernel<kBandWaves, 2, true, 0, true, 4, true, D>, grid, dim3(kBandWaves * 64), lds, st, sp);
        return launch_one(attn_split_kernel<kBandWaves, 2, true, 0, false, 4, true, D>, grid, dim3(kBandWaves * 64), lds, st, sp);
      }
      if (pl.NB == 1) return launch_one(attn_split_kernel<4, 2, true, 0, true, 4, true, D>, grid, dim3(256), lds, st, sp);
      return launch_one(attn_split_kernel<4, 2, true, 0, false, 4, true, D>, grid, dim3(256), lds, st, sp);
    }
  }
  if constexpr (CAUSAL) {                           // sibling workgroups: the second reader of a line finds it in the L2
    if (pl.NB > 1) return launch_one(attn_split_kernel<4, 2, true, COLLECT, false, 4, false, D>, grid, dim3(256), lds, st, sp);
  }
  // verification of up to 32 rows: one reader per K/V line, read once: stream it
  return launch_one(attn_split_kernel<4, 2, CAUSAL, COLLECT, CAUSAL, 4, false, D>, grid, dim3(256), lds, st, sp);
}

template <bool CAUSAL, int COLLECT>
int launch_split(const SplitPlan& pl, const SplitParams& sp, int batch, hipStream_t st, int head_dim, int page_size = kPage,
                 const DraftStep* step = nullptr) {
  if (head_dim == 64) return launch_split_d<CAUSAL, COLLECT, 64>(pl, sp, batch, st, page_size, step);
  return launch_split_d<CAUSAL, COLLECT, 128>(pl, sp, batch, st, page_size, step);
}

void fill_split_params(const vegas_desc* d, const SplitPlan& pl, int G, const void* q, const void* k,
                       const void* v, const int32_t* table, int table_stride, const int32_t* lens,
                       unsigned char* ws, SplitParams* sp) {
  sp->q = static_cast<const uint16_t*>(q);
  sp->k = static_cast<const uint16_t*>(k);
  sp->v = static_cast<const uint16_t*>(v);
  sp->table = table;
  sp->lens = lens;
  sp->part_o = reinterpret_cast<float*>(ws + pl.off_part_o);
  sp->part_ml = reinterpret_cast<float2*>(ws + pl.off_part_ml);
  sp->page_lse = reinterpret_cast<float*>(ws + pl.off_page_lse);
  sp->table_stride = table_stride;
  sp->G = G;
  sp->g = d->num_q_heads / d->num_kv_heads;
  sp->R = pl.R;
  sp->Hq = d->num_q_heads;
  sp->Hkv = d->num_kv_heads;
  sp->chunk_tokens = pl.chunk;
  sp->nsplit = pl.nsplit;
  sp->lse_pages = pl.lse_pages;
  sp->collect_rows = d->collect_rows;
  sp->Rc = pl.Rc;
  sp->window = 0;
  sp->out_direct = nullptr;
  sp->park_tiles = 0;
  sp->epoch_mul = 0;
  sp->plan = pl.balanced ? reinterpret_cast<int2*>(ws + pl.off_plan) : nullptr;
  sp->batch = d->batch;
  sp->slots_target = pl.bp.J;
  sp->slots_target2 = pl.bp.J2;
  sp->share_margin = pl.bp.share_margin;
  sp->share_group = share_group(d->num_kv_heads * pl.NB);
  sp->chunk_cap_units = pl.bp.cap_units;
  sp->slots_total = pl.bp.JS;
  if (pl.balanced) sp->chunk_tokens = d->batch;                    // (VEGAS_SPLIT_HOT_ASSIGN)
  sp->max_tokens = d->max_seq_len;
  sp->page_stride = d->kv_page_stride;
  sp->token_stride = d->kv_token_stride;
  sp->head_stride = d->kv_head_stride;
  sp->num_pages = d->num_pages;
  sp->scale_log2e = d->softmax_scale * 1.4426950408889634f;
  sp->timeline = nullptr;
}

// Scratch of vegas_select_tokens: digit histograms [B, 4 passes, slices, 256].
int token_slices(const vegas_desc* d) {
  return static_cast<int>((static_cast<int64_t>(d->max_blocks) * kPage + kTokSlice - 1) / kTokSlice);
}
size_t token_select_bytes(const vegas_desc* d) {
  return align_up(static_cast<size_t>(d->batch) * 4 * token_slices(d) * 256 * sizeof(uint32_t));
}

// Largest token budget a selection call can meet when no per-sequence budgets are passed: the constant,
// or (budget_ratio > 0) the ratio applied to the longest allowed sequence, in the kernels' fp32 arithmetic.
int64_t ratio_or_constant_budget(const vegas_desc* d, int32_t budget_tokens) {
  if (d->budget_ratio > 0.f) return static_cast<int64_t>(std::ceil(d->budget_ratio * static_cast<float>(d->max_seq_len)));
  return budget_tokens;
}

template <typename... Lengths>                       // (GrownLengths: the merge of a draft step)
int launch_combine(const vegas_desc* d, const SplitPlan& pl, const SplitParams& sp, void* out, hipStream_t st, Lengths... lengths) {
  CombineParams cp;
  cp.part_o = sp.part_o;
  cp.part_ml = sp.part_ml;
  cp.lens = sp.lens;
  cp.out = static_cast<uint16_t*>(out);
  cp.G = sp.G; cp.g = sp.g; cp.R = sp.R; cp.Hq = sp.Hq; cp.Hkv = sp.Hkv;
  cp.chunk_tokens = pl.chunk; cp.nsplit = pl.nsplit; cp.max_tokens = d->max_seq_len;
  cp.window = sp.window;
  cp.D = d->head_dim;
  cp.plan = sp.plan;
  cp.slots_total = sp.slots_total;
  const dim3 grid(pl.R, sp.Hkv, d->batch);
  auto any = [&] { hipLaunchKernelGGL((attn_combine_kernel<Lengths...>), grid, dim3(cp.D), 0, st, cp, lengths...); };
  auto small = [&](auto maxs) {
    hipLaunchKernelGGL((attn_combine_small_kernel<decltype(maxs)::value, Lengths...>), grid, dim3(cp.D), 0, st, VEGAS_COMBINE_SMALL_ARGS(cp), lengths...);
  };
  auto by_steps = [&](auto self, auto at) {
    constexpr size_t I = decltype(at)::value;
    if constexpr (I == std::size(kSmallMerges)) any();
    else if (pl.nsplit <= kSmallMerges[I]) small(std::integral_constant<int, kSmallMerges[I]>{});
    else self(self, std::integral_constant<size_t, I + 1>{});
  };
  if (pl.balanced) any();
  else by_steps(by_steps, std::integral_constant<size_t, 0>{});
  return hipGetLastError() == hipSuccess ? VEGAS_OK : VEGAS_ERR_LAUNCH;
}

// Scratch of vegas_draft_attention_static: the chunk partials of one draft call, in the library's own device image
// instead of a caller's workspace.  Every device the library runs on holds its own copy of the array at its own
// address until the process ends.  In host code the array's name is only a handle for hipGetSymbolAddress: the
// device address it yields (per device, asked once with that device current) is what kernels and copies get.
constexpr size_t kStaticScratchBytes = size_t(8) << 20;
static __device__ __align__(256) unsigned char scratch[kStaticScratchBytes];

int static_scratch_address(void** out) {
  static std::mutex mu;
  static std::map<int, void*> known;
  int dev = 0;
  if (hipGetDevice(&dev) != hipSuccess) {
    (void)hipGetLastError();
    return VEGAS_ERR_LAUNCH;
  }
  std::lock_guard<std::mutex> lock(mu);
  const auto it = known.find(dev);
  if (it != known.end()) {
    *out = it->second;
    return VEGAS_OK;
  }
  void* ptr = nullptr;
  if (hipGetSymbolAddress(&ptr, HIP_SYMBOL(scratch)) != hipSuccess || ptr == nullptr) {
    (void)hipGetLastError();
    return VEGAS_ERR_LAUNCH;
  }
  known[dev] = ptr;
  *out = ptr;
  return VEGAS_OK;
}

// Every kernel that is launched with dynamic LDS, for vegas_init: f(kernel address).
template <typename F>
int for_each_lds_kernel(F f) {
  int rc = VEGAS_OK;
  auto one = [&](auto kern) { if (rc == VEGAS_OK) rc = f(reinterpret_cast<const void*>(kern)); };
  auto per_dim = [&](auto dtag) {
    constexpr int D = decltype(dtag)::value;
    one(attn_split_kernel<4, 2, false, 0, false, 0, false, D>);      // draft calls, page sizes 1, 2, 4, 8, 16
    one(attn_split_kernel<4, 2, false, 0, false, 1, false, D>);
    one(attn_split_kernel<4, 2, false, 0, false, 2, false, D>);
    one(attn_split_kernel<4, 2, false, 0, false, 3, false, D>);
    one(attn_split_kernel<4, 2, false, 0, false, 4, false, D>);
    one(attn_split_kernel<4, 2, true, 0, true, 4, true, D>);         // verification of a banded layer
    one(attn_split_kernel<4, 2, true, 0, false, 4, true, D>);
    one(attn_split_kernel<kBandWaves, 2, true, 0, true, 4, true, D>); one(attn_split_kernel<kBandWaves, 2, true, 0, false, 4, true, D>);
    one(attn_split_kernel<4, 2, true, 0, true, 4, false, D>);        // verification: no collection / page weights / logits
    one(attn_split_kernel<4, 2, true, 1, true, 4, false, D>);
    one(attn_split_kernel<4, 2, true, 0, false, 4, false, D>);       // ... as sibling row blocks
    one(attn_split_kernel<4, 2, true, 1, false, 4, false, D>);
    one(attn_split_kernel<4, 2, true, 2, false, 4, false, D>);
    one(attn_split_kernel<4, 2, true, 2, true, 4, false, D>);
    auto draft16 = [&](auto ps) {
      constexpr int PS = decltype(ps)::value;
      one(attn_draft16_kernel<D, PS, false>); one(attn_draft16_kernel<D, PS, true>);
      one(attn_draft16_parts_kernel<D, 32, PS, false>);
      if constexpr (D == 128) one(attn_draft16_parts_kernel<D, 64, PS, false>);
    };
    draft16(std::integral_constant<int, 0>{}); draft16(std::integral_constant<int, 1>{}); draft16(std::integral_constant<int, 2>{});
    draft16(std::integral_constant<int, 3>{}); draft16(std::integral_constant<int, 4>{});
    one(attn_draft16_kernel<D, 4, false, false, DraftStep>);
    one(attn_pair_kernel<0, D, true>); one(attn_pair_kernel<0, D, false>);
    one(attn_pair_kernel<1, D, true>); one(attn_pair_kernel<1, D, false>);
    one(attn_pair_kernel<2, D, true>); one(attn_pair_kernel<2, D, false>);
  };
  one(attn_pair_kernel<1, 64, true, 2 * kPairWaves>); one(attn_pair_kernel<1, 64, false, 2 * kPairWaves>);
  one(attn_draft16_kernel<128, 4, false, true>); one(attn_draft16_parts_kernel<128, 64, 4, true>); one(attn_draft16_parts_kernel<128, 32, 4, true>);
  per_dim(std::integral_constant<int, 128>{});
  per_dim(std::integral_constant<int, 64>{});
  one(verify_finalize_kernel<16, 0>); one(verify_finalize_kernel<32, 0>);
  one(verify_finalize_kernel<64, 0>); one(verify_finalize_kernel<0, 0>);
  one(verify_finalize_kernel<16, 0, kFinWideRounds>); one(verify_finalize_kernel<32, 0, kFinWideRounds>);
  one(verify_finalize_kernel<16, 1>); one(verify_finalize_kernel<32, 1>);
  one(verify_finalize_kernel<64, 1>); one(verify_finalize_kernel<0, 1>);
  one(verify_finalize_kernel<kFinPlanned, 0>); one(verify_finalize_kernel<kFinPlanned, 1>);
  one(verify_finalize_kernel<kFinPlannedSmall, 0>); one(verify_finalize_kernel<kFinPlannedSmall, 1>);
  one(select_blocks_kernel<kSelectThreads>);
  return rc;
}

}  // namespace

extern "C" {

int vegas_init(void) {
  int dev = 0;
  if (hipGetDevice(&dev) != hipSuccess) {
    (void)hipGetLastError();
    return VEGAS_ERR_LAUNCH;
  }
  (void)device_cu_count();
  void* ptr = nullptr;
  if (int rc = static_scratch_address(&ptr)) return rc;
  return for_each_lds_kernel([](const void* kern) { return ensure_dynamic_lds(kern, 160 * 1024); });
}

size_t vegas_static_scratch_bytes(void) { return kStaticScratchBytes; }

size_t vegas_workspace_bytes(const vegas_desc* desc) {
  if (check_common(desc) != VEGAS_OK) return 0;
  SplitPlan pv, pd;
  size_t need = kAlign;
  if (desc->num_queries > 0 && check_paged16(desc) == VEGAS_OK && plan_verify(desc, &pv) == VEGAS_OK)
    need = pv.total > need ? pv.total : need;
  if (plan_draft(desc, &pd) == VEGAS_OK) {
    const size_t draft = pd.total + step_bytes(desc);
    need = draft > need ? draft : need;
  }
  if (check_paged16(desc) == VEGAS_OK) {
    const size_t ts = token_select_bytes(desc);
    need = ts > need ? ts : need;
  }
  return need;
}

static int verify_impl(const vegas_desc* desc, const void* q, const void* k_cache, const void* v_cache,
                       const int32_t* block_table, const int32_t* seq_lens, void* out, float* block_scores,
                       void* workspace, size_t workspace_bytes, void* hip_stream, int32_t stages) {
  if (stages < 0 || stages > (VEGAS_STAGE_STREAM | VEGAS_STAGE_MERGE)) return VEGAS_ERR_SHAPE;
  int rc = check_common(desc);
  if (rc == VEGAS_OK) rc = check_paged16(desc);
  if (rc != VEGAS_OK) return rc;
  if (!q || !k_cache || !v_cache || !block_table || !seq_lens || !out) return VEGAS_ERR_NULL;
  SplitPlan pl;
  rc = plan_verify(desc, &pl);
  if (rc != VEGAS_OK) return rc;
  const bool collect = desc->collect_rows != VEGAS_COLLECT_NONE;
  const bool logits = collect && desc->score_metric == VEGAS_METRIC_TOKEN_LOGITS;
  if (collect && !block_scores) return VEGAS_ERR_NULL;
  if (!aligned16(q) || !aligned16(k_cache) || !aligned16(v_cache) || !aligned16(out) || !aligned16(block_table) ||
      (block_scores && !aligned16(block_scores)))
    return VEGAS_ERR_ALIGN;
  if (!workspace || workspace_bytes < pl.total) return VEGAS_ERR_WORKSPACE;
  if (reinterpret_cast<uintptr_t>(workspace) % kAlign) return VEGAS_ERR_ALIGN;
  hipStream_t st = static_cast<hipStream_t>(hip_stream);
  unsigned char* ws = static_cast<unsigned char*>(workspace);

  SplitParams sp;
  fill_split_params(desc, pl, desc->num_queries, q, k_cache, v_cache, block_table, desc->max_blocks, seq_lens, ws, &sp);
  if (desc->window < 0) return VEGAS_ERR_SHAPE;
  if (desc->window > 0 && collect) return VEGAS_ERR_UNSUPPORTED;   // banded layers are not sparsified: nothing to score
  sp.window = desc->window;
  const bool direct = desc->window > 0 && pl.nsplit == 1;          // the streaming kernel writes the output rows itself
  if (direct) sp.out_direct = static_cast<uint16_t*>(out);
  const bool do_stream = stages == 0 || (stages & VEGAS_STAGE_STREAM);
  const bool do_merge = stages == 0 || (stages & VEGAS_STAGE_MERGE);
  if (do_stream) {
    const int hd = desc->head_dim;
    rc = !collect ? launch_split<true, 0>(pl, sp, desc->batch, st, hd)
                  : (logits ? launch_split<true, 2>(pl, sp, desc->batch, st, hd)
                            : launch_split<true, 1>(pl, sp, desc->batch, st, hd));
    if (rc != VEGAS_OK) return rc;
  }
  if (!do_merge || direct) return VEGAS_OK;
  if (!collect) return launch_combine(desc, pl, sp, out, st);
  FinalizeParams fp;
  fp.part_o = sp.part_o;
  fp.part_ml = sp.part_ml;
  fp.page_lse = sp.page_lse;
  fp.lens = seq_lens;
  fp.out = static_cast<uint16_t*>(out);
  fp.block_scores = block_scores;
  fp.G = desc->num_queries; fp.g = sp.g; fp.R = pl.R; fp.Hq = sp.Hq; fp.Hkv = sp.Hkv;
  fp.chunk_tokens = pl.chunk; fp.nsplit = pl.nsplit; fp.max_tokens = desc->max_seq_len;
  fp.max_blocks = desc->max_blocks; fp.lse_pages = pl.lse_pages; fp.collect_rows = desc->collect_rows;
  fp.Rc = pl.Rc;
  fp.D = desc->head_dim;
  fp.plan = sp.plan;
  fp.slots_total = sp.slots_total;
  const bool small = planned_merge_is_small(desc->batch, sp.Hkv * pl.R, fp.D);
  const int rows_per_wg = (pl.balanced && !small ? 1024 : 256) / fp.D;   // merge workgroups: 256 threads, D per row, or D / 4
  fp.nA = (sp.Hkv * pl.R + rows_per_wg - 1) / rows_per_wg;
  const int nrows = (desc->collect_rows == VEGAS_COLLECT_ALL_ROWS) ? desc->num_queries
                                                                   : (desc->num_queries > 1 ? 2 : 1);
  fp.inv_norm = 1.0f / (static_cast<float>(nrows) * static_cast<float>(desc->num_q_heads));
  // Every score workgroup (32 pages) rebuilds the row log-sum-exps from the (rows x chunks) table of
  // (max, sum) pairs; giving a workgroup more pages to amortise that was measured slower.
  const size_t hr = static_cast<size_t>(sp.Hkv) * pl.R;
  int nB = (desc->max_blocks + 31) / 32;
  // An upper bound of what the roles lay out (at most 13 x rows + 262 floats of collected rows, up to hr; verify_finalize_kernel), by which a
  // call of more than 2394 rows is refused.
  size_t shm = (hr + 256 + 16 * hr) * sizeof(float);
  fp.nC = 0;
  fp.tok_norm = 0.f;
  if (logits) {                                        // token sums instead of page scores: 1024 tokens per workgroup
    fp.nC = static_cast<int>((static_cast<int64_t>(desc->max_blocks) * kPage + 1023) / 1024);
    fp.tok_norm = desc->softmax_scale / (static_cast<float>(nrows) * static_cast<float>(desc->num_q_heads));
    nB = fp.nC;
    shm = 272 * sizeof(float);
  }
  if (shm > 160 * 1024) return VEGAS_ERR_UNSUPPORTED;
  const dim3 fgrid(fp.nA + nB, desc->batch);
  auto launch_finalize = [&](auto kern) -> int {
    if (int lrc = ensure_dynamic_lds(reinterpret_cast<const void*>(kern), shm)) return lrc;
    hipLaunchKernelGGL(kern, fgrid, dim3(256), shm, st, fp);
    return VEGAS_OK;
  };
  if (logits) {
    if (pl.balanced && small) rc = launch_finalize(verify_finalize_kernel<kFinPlannedSmall, 1>);
    else if (pl.balanced) rc = launch_finalize(verify_finalize_kernel<kFinPlanned, 1>);
    else if (pl.nsplit <= 16) rc = launch_finalize(verify_finalize_kernel<16, 1>);
    else if (pl.nsplit <= 32) rc = launch_finalize(verify_finalize_kernel<32, 1>);
    else if (pl.nsplit <= 64) rc = launch_finalize(verify_finalize_kernel<64, 1>);
    else rc = launch_finalize(verify_finalize_kernel<0, 1>);
  } else {
    if (pl.balanced && small) rc = launch_finalize(verify_finalize_kernel<kFinPlannedSmall>);
    else if (pl.balanced) rc = launch_finalize(verify_finalize_kernel<kFinPlanned>);
    else if (finalize_is_wide(sp.Hkv * pl.Rc, desc->batch, pl.nsplit)) {
      if (pl.nsplit <= 16) rc = launch_finalize(verify_finalize_kernel<16, 0, kFinWideRounds>);
      else rc = launch_finalize(verify_finalize_kernel<32, 0, kFinWideRounds>);
    } else if (pl.nsplit <= 16) rc = launch_finalize(verify_finalize_kernel<16>);
    else if (pl.nsplit <= 32) rc = launch_finalize(verify_finalize_kernel<32>);
    else if (pl.nsplit <= 64) rc = launch_finalize(verify_finalize_kernel<64>);
    else rc = launch_finalize(verify_finalize_kernel<0>);
  }
  if (rc != VEGAS_OK) return rc;
  if (hipGetLastError() != hipSuccess) return VEGAS_ERR_LAUNCH;
  return VEGAS_OK;
}

int vegas_select_blocks(const vegas_desc* desc, const float* block_scores, const int32_t* block_table,
                        const int32_t* seq_lens, int32_t budget_tokens, const int32_t* budgets,
                        int32_t* sel_table, int32_t* sel_seq_lens, void* workspace, size_t workspace_bytes,
                        void* hip_stream) {
  (void)workspace;
  (void)workspace_bytes;
  int rc = check_common(desc);
  if (rc == VEGAS_OK) rc = check_paged16(desc);
  if (rc != VEGAS_OK) return rc;
  if (!block_scores || !block_table || !seq_lens || !sel_table || !sel_seq_lens) return VEGAS_ERR_NULL;
  if (desc->num_queries <= 0 || desc->max_sel_blocks <= 0) return VEGAS_ERR_SHAPE;
  if (!budgets) {
    const int64_t bt = ratio_or_constant_budget(desc, budget_tokens);
    if (bt <= 0) return VEGAS_ERR_SHAPE;
    const int64_t max_pages = (static_cast<int64_t>(desc->max_seq_len) + kPage - 1) / kPage;
    int64_t kmax = (bt + kPage - 1) / kPage;
    const int64_t forced = (desc->num_queries + kPage - 2) / kPage + 1;   // pages G positions can touch
    if (kmax < forced) kmax = forced;
    if (kmax > max_pages) kmax = max_pages;
    if (desc->max_sel_blocks < kmax) return VEGAS_ERR_SHAPE;
  }
  SelectParams sp;
  sp.block_scores = block_scores;
  sp.block_table = block_table;
  sp.seq_lens = seq_lens;
  sp.budgets = budgets;
  sp.sel_table = sel_table;
  sp.sel_seq_lens = sel_seq_lens;
  sp.budget_tokens = budget_tokens;
  sp.G = desc->num_queries;
  sp.max_blocks = desc->max_blocks;
  sp.max_sel_blocks = desc->max_sel_blocks;
  sp.max_tokens = desc->max_seq_len;
  sp.budget_ratio = desc->budget_ratio;
  const int64_t max_pages = (static_cast<int64_t>(desc->max_seq_len) + kPage - 1) / kPage;
  sp.key_cap = static_cast<int32_t>(max_pages < kSelectKeyCap ? max_pages : kSelectKeyCap);
  const size_t shm = static_cast<size_t>(sp.key_cap) * sizeof(uint32_t);
  const hipStream_t stream = static_cast<hipStream_t>(hip_stream);
  if (max_pages <= kSelectRegRows * kSelectFewThreads) {
    hipLaunchKernelGGL(select_blocks_kernel<kSelectFewThreads>, dim3(desc->batch), dim3(kSelectFewThreads), 0, stream, sp);
  } else {
    if (int rc = ensure_dynamic_lds(reinterpret_cast<const void*>(select_blocks_kernel<kSelectThreads>), shm)) return rc;
    hipLaunchKernelGGL(select_blocks_kernel<kSelectThreads>, dim3(desc->batch), dim3(kSelectThreads), shm, stream, sp);
  }
  return hipGetLastError() == hipSuccess ? VEGAS_OK : VEGAS_ERR_LAUNCH;
}

int vegas_select_tokens(const vegas_desc* desc, const float* token_scores, const int32_t* block_table,
                        const int32_t* seq_lens, int32_t budget_tokens, const int32_t* budgets,
                        int32_t* sel_table, int32_t* sel_seq_lens, void* workspace, size_t workspace_bytes,
                        void* hip_stream) {
  int rc = check_common(desc);
  if (rc == VEGAS_OK) rc = check_paged16(desc);
  if (rc != VEGAS_OK) return rc;
  if (!token_scores || !block_table || !seq_lens || !sel_table || !sel_seq_lens) return VEGAS_ERR_NULL;
  if (desc->num_queries <= 0 || desc->max_sel_blocks <= 0) return VEGAS_ERR_SHAPE;
  if (!budgets) {
    const int64_t bt = ratio_or_constant_budget(desc, budget_tokens);
    if (bt <= 0) return VEGAS_ERR_SHAPE;
    int64_t kmax = bt < desc->max_seq_len ? bt : desc->max_seq_len;
    const int64_t tail = desc->num_queries < desc->max_seq_len ? desc->num_queries : desc->max_seq_len;
    if (kmax < tail) kmax = tail;
    if (desc->max_sel_blocks < kmax) return VEGAS_ERR_SHAPE;
  }
  const size_t need = token_select_bytes(desc);
  if (!workspace || workspace_bytes < need) return VEGAS_ERR_WORKSPACE;
  if (reinterpret_cast<uintptr_t>(workspace) % kAlign) return VEGAS_ERR_ALIGN;
  hipStream_t st = static_cast<hipStream_t>(hip_stream);
  unsigned char* ws = static_cast<unsigned char*>(workspace);
  TokenSelectParams tp;
  tp.scores = token_scores;
  tp.block_table = block_table;
  tp.seq_lens = seq_lens;
  tp.budgets = budgets;
  tp.sel_table = sel_table;
  tp.sel_seq_lens = sel_seq_lens;
  tp.hist = reinterpret_cast<uint32_t*>(ws);
  tp.budget_tokens = budget_tokens;
  tp.G = desc->num_queries;
  tp.max_blocks = desc->max_blocks;
  tp.max_sel = desc->max_sel_blocks;
  tp.max_tokens = desc->max_seq_len;
  tp.slices = token_slices(desc);
  tp.budget_ratio = desc->budget_ratio;
  // Up to 32768 tokens one workgroup per sequence (9.8 us there, five launches 21; beyond, 22.8 us at 65536, where a thread would have to
  // hold 64 scores), built for the fewest rows of 4096 that the bound on the lengths allows: a row that is not there costs its tests and
  // requests.
  auto launch_one_wg = [&](auto rows) {
    hipLaunchKernelGGL(token_select_one_kernel<decltype(rows)::value>, dim3(desc->batch), dim3(kTokThreads), 0, st, tp);
  };
  if (desc->max_seq_len <= 4 * kTokThreads) {
    launch_one_wg(std::integral_constant<int, 1>{});
  } else if (desc->max_seq_len <= 8 * kTokThreads) {
    launch_one_wg(std::integral_constant<int, 2>{});
  } else if (desc->max_seq_len <= 16 * kTokThreads) {
    launch_one_wg(std::integral_constant<int, 4>{});
  } else if (desc->max_seq_len <= 32 * kTokThreads) {
    launch_one_wg(std::integral_constant<int, 8>{});
  } else {
    const dim3 grid(tp.slices, desc->batch);
    for (int pass = 0; pass < 4; ++pass)
      hipLaunchKernelGGL(token_select_hist, grid, dim3(kTokThreads), 0, st, tp, pass);
    hipLaunchKernelGGL(token_select_write, grid, dim3(kTokThreads), 0, st, tp);
  }
  return hipGetLastError() == hipSuccess ? VEGAS_OK : VEGAS_ERR_LAUNCH;
}

static int check_append(const vegas_desc* desc, const void* k_new, const void* v_new, int32_t num_new,
                        const int32_t* block_table, const int32_t* seq_lens, const void* k_cache, const void* v_cache) {
  int rc = check_common(desc);
  if (rc == VEGAS_OK) rc = check_paged16(desc);
  if (rc != VEGAS_OK) return rc;
  if (!k_new || !v_new || !block_table || !seq_lens || !k_cache || !v_cache) return VEGAS_ERR_NULL;
  if (num_new <= 0 || num_new > 4096) return VEGAS_ERR_SHAPE;
  if (!aligned16(k_new) || !aligned16(v_new) || !aligned16(k_cache) || !aligned16(v_cache)) return VEGAS_ERR_ALIGN;
  return VEGAS_OK;
}

static int append_impl(const vegas_desc* desc, const void* k_new, const void* v_new, int32_t num_new,
                       const int32_t* block_table, int32_t* seq_lens, void* k_cache, void* v_cache, int32_t* sel_table,
                       int32_t* sel_seq_lens, int32_t sel_page_size, void* hip_stream) {
  if (int rc = check_append(desc, k_new, v_new, num_new, block_table, seq_lens, k_cache, v_cache)) return rc;
  AppendParams ap;
  ap.k_new = static_cast<const uint16_t*>(k_new);
  ap.v_new = static_cast<const uint16_t*>(v_new);
  ap.k_cache = static_cast<uint16_t*>(k_cache);
  ap.v_cache = static_cast<uint16_t*>(v_cache);
  ap.block_table = block_table;
  ap.seq_lens = seq_lens;
  ap.T = num_new;
  ap.Hkv = desc->num_kv_heads;
  ap.D = desc->head_dim;
  ap.max_blocks = desc->max_blocks;
  ap.max_tokens = desc->max_seq_len;
  ap.page_stride = desc->kv_page_stride;
  ap.token_stride = desc->kv_token_stride;
  ap.head_stride = desc->kv_head_stride;
  ap.num_pages = desc->num_pages;
  ap.grow.block_table = block_table;
  ap.grow.seq_lens = seq_lens;
  ap.grow.sel_table = sel_table;
  ap.grow.sel_seq_lens = sel_seq_lens;
  ap.grow.batch = desc->batch;
  ap.grow.num_new = num_new;
  ap.grow.max_blocks = desc->max_blocks;
  ap.grow.max_sel_blocks = desc->max_sel_blocks;
  ap.grow.page_size = sel_page_size;
  hipLaunchKernelGGL(append_kv_kernel, dim3(desc->batch), dim3(256), 0, static_cast<hipStream_t>(hip_stream), ap);
  return hipGetLastError() == hipSuccess ? VEGAS_OK : VEGAS_ERR_LAUNCH;
}

int vegas_append_kv(const vegas_desc* desc, const void* k_new, const void* v_new, int32_t num_new,
                    const int32_t* block_table, int32_t* seq_lens, void* k_cache, void* v_cache, void* hip_stream) {
  return append_impl(desc, k_new, v_new, num_new, block_table, seq_lens, k_cache, v_cache, nullptr, nullptr, kPage,
                     hip_stream);
}

int vegas_append_kv_extend(const vegas_desc* desc, const void* k_new, const void* v_new, int32_t num_new,
                           const int32_t* block_table, int32_t* seq_lens, void* k_cache, void* v_cache,
                           int32_t* sel_table, int32_t* sel_seq_lens, int32_t sel_page_size, void* hip_stream) {
  if (!sel_table || !sel_seq_lens) return VEGAS_ERR_NULL;
  if (sel_page_size != kPage && sel_page_size != 1) return VEGAS_ERR_UNSUPPORTED;
  if (!desc || desc->max_sel_blocks <= 0) return desc ? VEGAS_ERR_SHAPE : VEGAS_ERR_NULL;
  return append_impl(desc, k_new, v_new, num_new, block_table, seq_lens, k_cache, v_cache, sel_table, sel_seq_lens,
                     sel_page_size, hip_stream);
}

int vegas_extend_selection(const vegas_desc* desc, const int32_t* block_table, const int32_t* seq_lens,
                           int32_t num_new, int32_t* sel_table, int32_t* sel_seq_lens, void* hip_stream) {
  int rc = check_common(desc);
  if (rc != VEGAS_OK) return rc;
  if (desc->page_size != kPage && desc->page_size != 1) return VEGAS_ERR_UNSUPPORTED;
  if (!block_table || !seq_lens || !sel_table || !sel_seq_lens) return VEGAS_ERR_NULL;
  if (num_new <= 0 || desc->max_sel_blocks <= 0) return VEGAS_ERR_SHAPE;
  ExtendParams ep;
  ep.block_table = block_table;
  ep.seq_lens = seq_lens;
  ep.sel_table = sel_table;
  ep.sel_seq_lens = sel_seq_lens;
  ep.batch = desc->batch;
  ep.num_new = num_new;
  ep.max_blocks = desc->max_blocks;
  ep.max_sel_blocks = desc->max_sel_blocks;
  ep.page_size = desc->page_size;
  hipLaunchKernelGGL(extend_selection_kernel, dim3((desc->batch + 63) / 64), dim3(64), 0,
                     static_cast<hipStream_t>(hip_stream), ep);
  return hipGetLastError() == hipSuccess ? VEGAS_OK : VEGAS_ERR_LAUNCH;
}

static int check_draft(const vegas_desc* desc, const void* q, const void* k_cache, const void* v_cache,
                       const int32_t* sel_table, const int32_t* sel_seq_lens, const void* out, const void* workspace,
                       size_t workspace_bytes, SplitPlan* pl) {
  int rc = check_common(desc);
  if (rc != VEGAS_OK) return rc;
  if (!q || !k_cache || !v_cache || !sel_table || !sel_seq_lens || !out) return VEGAS_ERR_NULL;
  if (desc->max_sel_blocks <= 0) return VEGAS_ERR_SHAPE;
  if (static_cast<int64_t>(desc->max_seq_len) > static_cast<int64_t>(desc->max_sel_blocks) * desc->page_size)
    return VEGAS_ERR_SHAPE;
  rc = plan_draft(desc, pl, workspace_bytes);
  if (rc != VEGAS_OK) return rc;
  if (!aligned16(q) || !aligned16(k_cache) || !aligned16(v_cache) || !aligned16(out) || !aligned16(sel_table))
    return VEGAS_ERR_ALIGN;
  if (!workspace || workspace_bytes < pl->total) return VEGAS_ERR_WORKSPACE;
  if (reinterpret_cast<uintptr_t>(workspace) % kAlign) return VEGAS_ERR_ALIGN;
  return VEGAS_OK;
}

static int draft_impl(const vegas_desc* desc, const void* q, const void* k_cache, const void* v_cache,
                      const int32_t* sel_table, const int32_t* sel_seq_lens, void* out, void* workspace,
                      size_t workspace_bytes, void* hip_stream, int32_t stages) {
  if (stages < 0 || stages > (VEGAS_STAGE_STREAM | VEGAS_STAGE_MERGE)) return VEGAS_ERR_SHAPE;
  SplitPlan pl;
  int rc = check_draft(desc, q, k_cache, v_cache, sel_table, sel_seq_lens, out, workspace, workspace_bytes, &pl);
  if (rc != VEGAS_OK) return rc;
  hipStream_t st = static_cast<hipStream_t>(hip_stream);
  unsigned char* ws = static_cast<unsigned char*>(workspace);
  SplitParams sp;
  fill_split_params(desc, pl, 1, q, k_cache, v_cache, sel_table, desc->max_sel_blocks, sel_seq_lens, ws, &sp);
  // One chunk per (sequence, KV head): the streaming kernel finishes the rows itself and no merge kernel is launched.
  const bool direct = pl.nsplit == 1;
  if (direct) sp.out_direct = static_cast<uint16_t*>(out);
  if (stages == 0 || (stages & VEGAS_STAGE_STREAM)) {
    rc = launch_split<false, 0>(pl, sp, desc->batch, st, desc->head_dim, desc->page_size);
    if (rc != VEGAS_OK) return rc;
  }
  if (direct || (stages != 0 && !(stages & VEGAS_STAGE_MERGE))) return VEGAS_OK;
  return launch_combine(desc, pl, sp, out, st);
}

int vegas_draft_step(const vegas_desc* cache_desc, const vegas_desc* desc, const void* q, const void* k_new, const void* v_new,
                     const int32_t* block_table, int32_t* seq_lens, void* k_cache, void* v_cache, int32_t* sel_table,
                     int32_t* sel_seq_lens, void* out, void* workspace, size_t workspace_bytes, void* hip_stream) {
  if (int rc = check_append(cache_desc, k_new, v_new, 1, block_table, seq_lens, k_cache, v_cache)) return rc;
  SplitPlan pl;
  if (int rc = check_draft(desc, q, k_cache, v_cache, sel_table, sel_seq_lens, out, workspace, workspace_bytes, &pl)) return rc;
  const vegas_desc& c = *cache_desc;
  const vegas_desc& d = *desc;
  if (d.page_size != kPage && d.page_size != 1) return VEGAS_ERR_UNSUPPORTED;
  if (c.batch != d.batch || c.num_kv_heads != d.num_kv_heads || c.head_dim != d.head_dim || c.max_sel_blocks != d.max_sel_blocks ||
      c.kv_token_stride != d.kv_token_stride || c.kv_head_stride != d.kv_head_stride)
    return VEGAS_ERR_SHAPE;
  if (exceeds_grid(pl)) return VEGAS_ERR_UNSUPPORTED;              // (before the append: the draft call would refuse after it)
  // Where a second launch merges chunks of 16-token pages it stores the lengths too, and the append needs no launch of its own: an
  // iteration of one sequence of 32749 tokens, 2048 selected, five steps, 86.9 -> 76.5 us.  A call that one workgroup per column
  // finishes has no second launch, and nothing in it could tell when the last of the columns has read the old lengths.
  const bool one_pass = d.page_size == kPage && pl.nsplit > 1 && pl.R <= kDraftRows && pl.NB == 1 && c.kv_page_stride == d.kv_page_stride &&
                        c.num_pages == d.num_pages && workspace_bytes >= pl.total + step_bytes(desc) &&
                        !draft_chooses(d.batch, d.max_seq_len, d.num_kv_heads, d.head_dim);
  if (!one_pass) {
    if (int rc = append_impl(cache_desc, k_new, v_new, 1, block_table, seq_lens, k_cache, v_cache, sel_table, sel_seq_lens, d.page_size, hip_stream))
      return rc;
    return draft_impl(desc, q, k_cache, v_cache, sel_table, sel_seq_lens, out, workspace, workspace_bytes, hip_stream, 0);
  }
  hipStream_t st = static_cast<hipStream_t>(hip_stream);
  unsigned char* ws = static_cast<unsigned char*>(workspace);
  SplitParams sp;
  fill_split_params(desc, pl, 1, q, k_cache, v_cache, sel_table, d.max_sel_blocks, sel_seq_lens, ws, &sp);
  sp.plan = reinterpret_cast<int2*>(seq_lens);                     // (a draft call has no plan: attn_draft16_kernel)
  DraftStep step;
  step.k_new = static_cast<const uint16_t*>(k_new);
  step.v_new = static_cast<const uint16_t*>(v_new);
  step.block_table = block_table;
  step.sel_table = sel_table;
  step.grown = reinterpret_cast<int2*>(ws + pl.total);
  step.sel_lens = reinterpret_cast<int32_t*>(step.grown + d.batch);
  step.max_blocks = c.max_blocks;
  const int64_t table_tokens = static_cast<int64_t>(c.max_blocks) * kPage;
  step.cap = static_cast<int32_t>(table_tokens < c.max_seq_len ? table_tokens : c.max_seq_len);
  if (int rc = launch_split<false, 0>(pl, sp, d.batch, st, d.head_dim, d.page_size, &step)) return rc;
  sp.plan = nullptr;
  sp.lens = step.sel_lens;
  return launch_combine(desc, pl, sp, out, st, GrownLengths{step.grown, seq_lens, sel_seq_lens});
}

int vegas_verify_attention(const vegas_desc* desc, const void* q, const void* k_cache, const void* v_cache,
                           const int32_t* block_table, const int32_t* seq_lens, void* out, float* block_scores,
                           void* workspace, size_t workspace_bytes, void* hip_stream) {
  return verify_impl(desc, q, k_cache, v_cache, block_table, seq_lens, out, block_scores, workspace, workspace_bytes,
                     hip_stream, 0);
}

int vegas_draft_attention(const vegas_desc* desc, const void* q, const void* k_cache, const void* v_cache,
                          const int32_t* sel_table, const int32_t* sel_seq_lens, void* out, void* workspace,
                          size_t workspace_bytes, void* hip_stream) {
  return draft_impl(desc, q, k_cache, v_cache, sel_table, sel_seq_lens, out, workspace, workspace_bytes, hip_stream, 0);
}

int vegas_draft_attention_static(const vegas_desc* desc, const void* q, const void* k_cache, const void* v_cache,
                                 const int32_t* sel_table, const int32_t* sel_seq_lens, void* out, void* hip_stream) {
  const int rc = check_common(desc);
  if (rc != VEGAS_OK) return rc;
  SplitPlan pl;
  if (int prc = plan_draft(desc, &pl, kStaticScratchBytes)) return prc;
  if (pl.total > kStaticScratchBytes) return VEGAS_ERR_WORKSPACE;      // the call needs more than the built-in scratch
  void* ptr = nullptr;
  if (int src = static_scratch_address(&ptr)) return src;
  return draft_impl(desc, q, k_cache, v_cache, sel_table, sel_seq_lens, out, ptr, kStaticScratchBytes, hip_stream, 0);
}

int vegas_debug_verify_attention_stages(const vegas_desc* desc, const void* q, const void* k_cache,
                                        const void* v_cache, const int32_t* block_table, const int32_t* seq_lens,
                                        void* out, float* block_scores, void* workspace, size_t workspace_bytes,
                                        void* hip_stream, int32_t stages) {
  return verify_impl(desc, q, k_cache, v_cache, block_table, seq_lens, out, block_scores, workspace, workspace_bytes,
                     hip_stream, stages);
}

int vegas_debug_draft_attention_stages(const vegas_desc* desc, const void* q, const void* k_cache, const void* v_cache,
                                       const int32_t* sel_table, const int32_t* sel_seq_lens, void* out,
                                       void* workspace, size_t workspace_bytes, void* hip_stream, int32_t stages) {
  return draft_impl(desc, q, k_cache, v_cache, sel_table, sel_seq_lens, out, workspace, workspace_bytes, hip_stream,
                    stages);
}

int vegas_debug_stream_read(const void* a, const void* b, size_t bytes_each, int32_t workgroups, int32_t non_temporal,
                            void* sink, void* hip_stream) {
  if (!a || !b || !sink) return VEGAS_ERR_NULL;
  if (bytes_each < 16 || (bytes_each % 16) != 0 || workgroups <= 0 || workgroups > (1 << 20)) return VEGAS_ERR_SHAPE;
  if (!aligned16(a) || !aligned16(b) || !aligned16(sink)) return VEGAS_ERR_ALIGN;
  StreamReadParams rp;
  rp.a = static_cast<const u32x4*>(a);
  rp.b = static_cast<const u32x4*>(b);
  rp.vecs = bytes_each / 16;
  rp.sink = static_cast<uint32_t*>(sink);
  hipStream_t st = static_cast<hipStream_t>(hip_stream);
  if (non_temporal) hipLaunchKernelGGL(stream_read_kernel<true>, dim3(workgroups), dim3(256), 0, st, rp);
  else hipLaunchKernelGGL(stream_read_kernel<false>, dim3(workgroups), dim3(256), 0, st, rp);
  return hipGetLastError() == hipSuccess ? VEGAS_OK : VEGAS_ERR_LAUNCH;
}

int vegas_debug_check_tables(const vegas_desc* desc, int32_t which, const int32_t* table, const int32_t* lens,
                             int32_t* error_word, void* hip_stream) {
  const int rc = check_common(desc);
  if (rc != VEGAS_OK) return rc;
  if (!table || !lens || !error_word) return VEGAS_ERR_NULL;
  if (which != VEGAS_TABLE_BLOCKS && which != VEGAS_TABLE_SELECTION) return VEGAS_ERR_SHAPE;
  CheckParams cp;
  cp.table = table;
  cp.lens = lens;
  cp.error_word = error_word;
  cp.batch = desc->batch;
  cp.max_tokens = desc->max_seq_len;
  cp.num_pages = desc->num_pages;
  if (which == VEGAS_TABLE_BLOCKS) {
    cp.stride = desc->max_blocks;
    cp.page_size = kPage;
    cp.num_queries = desc->num_queries;
  } else {
    if (desc->max_sel_blocks <= 0) return VEGAS_ERR_SHAPE;
    cp.stride = desc->max_sel_blocks;
    cp.page_size = desc->page_size;
    cp.num_queries = 0;
  }
  hipLaunchKernelGGL(check_tables_kernel, dim3(desc->batch), dim3(256), 0, static_cast<hipStream_t>(hip_stream), cp);
  return hipGetLastError() == hipSuccess ? VEGAS_OK : VEGAS_ERR_LAUNCH;
}

int vegas_debug_set_timeline(void* buffer, size_t bytes) {
#ifdef VEGAS_TIMELINE
  g_timeline = static_cast<unsigned long long*>(buffer);
  g_timeline_bytes = buffer ? bytes : 0;
  return VEGAS_OK;
#else
  (void)buffer;
  (void)bytes;
  return VEGAS_ERR_UNSUPPORTED;
#endif
}

int vegas_debug_verify_waves(const vegas_desc* desc) {
  int rc = check_common(desc);
  if (rc == VEGAS_OK) rc = check_paged16(desc);
  SplitPlan pl;
  if (rc == VEGAS_OK) rc = plan_verify(desc, &pl);
  if (rc != VEGAS_OK) return rc;
  return pl.pair ? pl.pair_waves : pl.NW;
}

const char* vegas_strerror(int status) {
  switch (status) {
    case VEGAS_OK: return "ok";
    case VEGAS_ERR_NULL: return "a required pointer is NULL";
    case VEGAS_ERR_SHAPE: return "a size is non-positive or inconsistent";
    case VEGAS_ERR_UNSUPPORTED:
      return "shape not supported by this build (head_dim 128 or 64; page_size 16, in draft calls also 1, 2, 4, 8; "
             "<= 128 rows per KV head; max_seq_len <= 2^30; batch <= 65535)";
    case VEGAS_ERR_ALIGN: return "pointer or stride alignment";
    case VEGAS_ERR_WORKSPACE: return "workspace missing or too small";
    case VEGAS_ERR_LAUNCH: return "the HIP runtime refused a kernel launch";
    default: return "unknown status";
  }
}

}  // extern "C"
