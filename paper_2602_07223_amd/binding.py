"""ctypes binding of libvegas.so: the three calls of include/vegas.h under the same names.

Argument marshalling only -- every step of the path runs in the HIP kernels.  Tensors may be
torch tensors on the GPU (their ``data_ptr()`` is passed) or raw integer device addresses.  The
library is loaded on first use and a missing build is an error, never a fallback.
"""
from __future__ import annotations

import ctypes
import os
from typing import Optional

_HERE = os.path.dirname(os.path.abspath(__file__))
LIB_PATH = os.path.join(_HERE, "libvegas.so")

VEGAS_OK = 0
VEGAS_ERR_NULL = -1
VEGAS_ERR_SHAPE = -2
VEGAS_ERR_UNSUPPORTED = -3
VEGAS_ERR_ALIGN = -4
VEGAS_ERR_WORKSPACE = -5
VEGAS_ERR_LAUNCH = -6

COLLECT_NONE = 0
COLLECT_ALL_ROWS = 1
COLLECT_FIRST_LAST = 2

METRIC_PAGE_WEIGHTS = 0
METRIC_TOKEN_LOGITS = 1

TABLE_BLOCKS = 0
TABLE_SELECTION = 1
CHECK_LENGTH_RANGE = 1
CHECK_LENGTH_EXCEEDS_TABLE = 2
CHECK_PAGE_ID = 4
CHECK_SHORTER_THAN_QUERIES = 8

STAGE_STREAM = 1
STAGE_MERGE = 2

EXPORTS = ("vegas_init", "vegas_workspace_bytes", "vegas_verify_attention", "vegas_select_blocks",
           "vegas_select_tokens", "vegas_append_kv", "vegas_append_kv_extend", "vegas_extend_selection", "vegas_draft_attention",
           "vegas_draft_step", "vegas_draft_attention_static", "vegas_static_scratch_bytes",
           "vegas_debug_verify_attention_stages", "vegas_debug_draft_attention_stages", "vegas_debug_stream_read",
           "vegas_debug_check_tables", "vegas_debug_set_timeline", "vegas_debug_verify_waves", "vegas_strerror")


class VegasDesc(ctypes.Structure):
    """Mirror of ``vegas_desc`` (include/vegas.h)."""
    _fields_ = [
        ("batch", ctypes.c_int32),
        ("num_q_heads", ctypes.c_int32),
        ("num_kv_heads", ctypes.c_int32),
        ("head_dim", ctypes.c_int32),
        ("page_size", ctypes.c_int32),
        ("num_queries", ctypes.c_int32),
        ("max_blocks", ctypes.c_int32),
        ("max_sel_blocks", ctypes.c_int32),
        ("max_seq_len", ctypes.c_int32),
        ("collect_rows", ctypes.c_int32),
        ("kv_chunk_tokens", ctypes.c_int32),
        ("reserved", ctypes.c_int32),
        ("softmax_scale", ctypes.c_float),
        ("score_metric", ctypes.c_int32),
        ("window", ctypes.c_int32),
        ("budget_ratio", ctypes.c_float),
        ("num_pages", ctypes.c_int64),
        ("kv_page_stride", ctypes.c_int64),
        ("kv_token_stride", ctypes.c_int64),
        ("kv_head_stride", ctypes.c_int64),
    ]


class VegasError(RuntimeError):
    def __init__(self, status: int, where: str):
        self.status = status
        super().__init__(f"{where}: {strerror(status)} (status {status})")


_lib = None
_byref = ctypes.byref


def load_library(path: Optional[str] = None):
    """Load libvegas.so (once).  Raises if it has not been built."""
    global _lib
    if _lib is not None:
        return _lib
    path = path or os.environ.get("VEGAS_LIB", LIB_PATH)
    if not os.path.exists(path):
        raise RuntimeError(f"{path} is missing: build it first (python -m paper_2602_07223_amd.build, "
                           "or __graft_entry__.build()); there is no fallback path")
    lib = ctypes.CDLL(path)
    P = ctypes.c_void_p
    D = ctypes.POINTER(VegasDesc)
    lib.vegas_init.restype = ctypes.c_int
    lib.vegas_init.argtypes = []
    lib.vegas_workspace_bytes.restype = ctypes.c_size_t
    lib.vegas_workspace_bytes.argtypes = [D]
    lib.vegas_verify_attention.restype = ctypes.c_int
    lib.vegas_verify_attention.argtypes = [D, P, P, P, P, P, P, P, P, ctypes.c_size_t, P]
    lib.vegas_select_blocks.restype = ctypes.c_int
    lib.vegas_select_blocks.argtypes = [D, P, P, P, ctypes.c_int32, P, P, P, P, ctypes.c_size_t, P]
    lib.vegas_select_tokens.restype = ctypes.c_int
    lib.vegas_select_tokens.argtypes = [D, P, P, P, ctypes.c_int32, P, P, P, P, ctypes.c_size_t, P]
    lib.vegas_append_kv.restype = ctypes.c_int
    lib.vegas_append_kv.argtypes = [D, P, P, ctypes.c_int32, P, P, P, P, P]
    lib.vegas_append_kv_extend.restype = ctypes.c_int
    lib.vegas_append_kv_extend.argtypes = [D, P, P, ctypes.c_int32, P, P, P, P, P, P, ctypes.c_int32, P]
    lib.vegas_extend_selection.restype = ctypes.c_int
    lib.vegas_extend_selection.argtypes = [D, P, P, ctypes.c_int32, P, P, P]
    lib.vegas_draft_attention.restype = ctypes.c_int
    lib.vegas_draft_attention.argtypes = [D, P, P, P, P, P, P, P, ctypes.c_size_t, P]
    lib.vegas_draft_step.restype = ctypes.c_int
    lib.vegas_draft_step.argtypes = [D, D, P, P, P, P, P, P, P, P, P, P, P, ctypes.c_size_t, P]
    lib.vegas_draft_attention_static.restype = ctypes.c_int
    lib.vegas_draft_attention_static.argtypes = [D, P, P, P, P, P, P, P]
    lib.vegas_static_scratch_bytes.restype = ctypes.c_size_t
    lib.vegas_static_scratch_bytes.argtypes = []
    lib.vegas_debug_verify_attention_stages.restype = ctypes.c_int
    lib.vegas_debug_verify_attention_stages.argtypes = [D, P, P, P, P, P, P, P, P, ctypes.c_size_t, P, ctypes.c_int32]
    lib.vegas_debug_draft_attention_stages.restype = ctypes.c_int
    lib.vegas_debug_draft_attention_stages.argtypes = [D, P, P, P, P, P, P, P, ctypes.c_size_t, P, ctypes.c_int32]
    lib.vegas_debug_stream_read.restype = ctypes.c_int
    lib.vegas_debug_stream_read.argtypes = [P, P, ctypes.c_size_t, ctypes.c_int32, ctypes.c_int32, P, P]
    lib.vegas_debug_check_tables.restype = ctypes.c_int
    lib.vegas_debug_check_tables.argtypes = [D, ctypes.c_int32, P, P, P, P]
    lib.vegas_debug_set_timeline.restype = ctypes.c_int
    lib.vegas_debug_set_timeline.argtypes = [P, ctypes.c_size_t]
    lib.vegas_debug_verify_waves.restype = ctypes.c_int
    lib.vegas_debug_verify_waves.argtypes = [D]
    lib.vegas_strerror.restype = ctypes.c_char_p
    lib.vegas_strerror.argtypes = [ctypes.c_int]
    _lib = lib
    return lib


# A kernel launch takes the host three microseconds, and small calls are over on the GPU in five, so Python's share counts: addresses
# and streams that are plain integers already are not passed through _ptr and _stream.  Host us, before / with that and the raw stream
# handle (harness): an iteration of 4096 tokens 42.6 / 33.8 (GPU 38), of 32768 56 / 43, a verification of one launch 6.8 / 4.5 (7.3 ->
# 6.4 a call).
def _ptr(x) -> Optional[int]:
    if x is None:
        return None
    if isinstance(x, int):
        return x
    return int(x.data_ptr())


def _nbytes(x) -> int:
    return int(x.nbytes)


def _avail_bytes(x) -> int:
    """Bytes from a tensor's first element to the end of its storage (what a kernel may address through it)."""
    have, first = x.untyped_storage().nbytes(), x.storage_offset()
    return have - first * x.element_size() if first else have


def cache_extent_bytes(desc: "VegasDesc") -> int:
    """Bytes a K or V cache must span under the descriptor's strides: the kernels clamp page ids to
    [0, num_pages) and address every token slot and KV head of such a page."""
    last = ((desc.num_pages - 1) * desc.kv_page_stride + (desc.page_size - 1) * desc.kv_token_stride +
            (desc.num_kv_heads - 1) * desc.kv_head_stride + desc.head_dim)
    return 2 * int(last)


def _fits(where: str, name: str, x, nbytes: int) -> Optional[int]:
    """The C ABI takes bare pointers and cannot see allocation sizes; where tensors (not raw addresses) are
    passed, refuse any that is smaller than what the descriptor lets the kernels touch.  Returns the address."""
    if x is None or isinstance(x, int):
        return x
    have = _avail_bytes(x)                          # (the storage's: it may have been resized under a tensor that still has its shape)
    if have < nbytes:
        raise ValueError(f"{where}: {name} spans {have} bytes, the descriptor needs {nbytes}")
    return x.data_ptr()


def _stream(stream) -> Optional[int]:
    if stream is None:
        return None
    if isinstance(stream, int):
        return stream
    return int(stream.cuda_stream)


def strerror(status: int) -> str:
    return load_library().vegas_strerror(int(status)).decode()


def make_desc(*, batch: int, num_q_heads: int, num_kv_heads: int, num_queries: int, max_blocks: int,
              max_sel_blocks: int, max_seq_len: int, num_pages: int, softmax_scale: float,
              collect_rows: int = COLLECT_ALL_ROWS, head_dim: int = 128, page_size: int = 16,
              kv_chunk_tokens: int = 0, kv_page_stride: int = 0, kv_token_stride: int = 0,
              kv_head_stride: int = 0, score_metric: int = METRIC_PAGE_WEIGHTS,
              budget_ratio: float = 0.0, window: int = 0) -> VegasDesc:
    """Descriptor for a contiguous NHD cache unless strides are given (elements)."""
    d = VegasDesc()
    d.batch, d.num_q_heads, d.num_kv_heads = batch, num_q_heads, num_kv_heads
    d.head_dim, d.page_size, d.num_queries = head_dim, page_size, num_queries
    d.max_blocks, d.max_sel_blocks, d.max_seq_len = max_blocks, max_sel_blocks, max_seq_len
    d.collect_rows, d.kv_chunk_tokens, d.softmax_scale = collect_rows, kv_chunk_tokens, softmax_scale
    d.reserved = 0
    d.score_metric = score_metric
    d.budget_ratio = budget_ratio
    d.window = window
    d.num_pages = num_pages
    d.kv_head_stride = kv_head_stride or head_dim
    d.kv_token_stride = kv_token_stride or num_kv_heads * head_dim
    d.kv_page_stride = kv_page_stride or page_size * num_kv_heads * head_dim
    return d


def vegas_workspace_bytes(desc: VegasDesc) -> int:
    return int((_lib or load_library()).vegas_workspace_bytes(_byref(desc)))


def vegas_init() -> None:
    """One-time set-up for the current device (see include/vegas.h); optional, the calls do it lazily otherwise."""
    rc = (_lib or load_library()).vegas_init()
    if rc != VEGAS_OK:
        raise VegasError(rc, "vegas_init")


def vegas_verify_attention(desc: VegasDesc, q, k_cache, v_cache, block_table, seq_lens, out, block_scores,
                           workspace, stream=None, workspace_bytes: Optional[int] = None, stages: int = 0) -> None:
    """stages != 0: vegas_debug_verify_attention_stages (a profiling aid: only those kernels of the call)."""
    wb = workspace_bytes if workspace_bytes is not None else (_nbytes(workspace) if workspace is not None else 0)
    q_at, k_cache_at, v_cache_at, block_table_at, seq_lens_at = q, k_cache, v_cache, block_table, seq_lens
    out_at, block_scores_at, workspace_at, stream_at = out, block_scores, workspace, stream
    if not (isinstance(q, int) and isinstance(k_cache, int)):      # raw addresses: the caller has checked (harness)
        d = desc
        rows = d.batch * d.num_queries * d.num_q_heads * d.head_dim * 2
        extent = cache_extent_bytes(d)
        per_page = 16 if d.score_metric == METRIC_TOKEN_LOGITS else 1
        q_at = _fits("vegas_verify_attention", "q", q, rows)
        out_at = _fits("vegas_verify_attention", "out", out, rows)
        k_cache_at = _fits("vegas_verify_attention", "k_cache", k_cache, extent)
        v_cache_at = _fits("vegas_verify_attention", "v_cache", v_cache, extent)
        block_table_at = _fits("vegas_verify_attention", "block_table", block_table, d.batch * d.max_blocks * 4)
        seq_lens_at = _fits("vegas_verify_attention", "seq_lens", seq_lens, d.batch * 4)
        if d.collect_rows != COLLECT_NONE:
            block_scores_at = _fits("vegas_verify_attention", "block_scores", block_scores, d.batch * d.max_blocks * per_page * 4)
    if type(q_at) is not int: q_at = _ptr(q_at)
    if type(k_cache_at) is not int: k_cache_at = _ptr(k_cache_at)
    if type(v_cache_at) is not int: v_cache_at = _ptr(v_cache_at)
    if type(block_table_at) is not int: block_table_at = _ptr(block_table_at)
    if type(seq_lens_at) is not int: seq_lens_at = _ptr(seq_lens_at)
    if type(out_at) is not int: out_at = _ptr(out_at)
    if type(block_scores_at) is not int: block_scores_at = _ptr(block_scores_at)
    if type(workspace_at) is not int: workspace_at = _ptr(workspace_at)
    if type(stream_at) is not int: stream_at = _stream(stream_at)
    args = (_byref(desc), q_at, k_cache_at, v_cache_at, block_table_at, seq_lens_at, out_at, block_scores_at, workspace_at, wb, stream_at)
    if stages:
        rc = (_lib or load_library()).vegas_debug_verify_attention_stages(*args, int(stages))
    else:
        rc = (_lib or load_library()).vegas_verify_attention(*args)
    if rc != VEGAS_OK:
        raise VegasError(rc, "vegas_verify_attention")


def vegas_select_blocks(desc: VegasDesc, block_scores, block_table, seq_lens, budget_tokens: int, sel_table,
                        sel_seq_lens, budgets=None, workspace=None, stream=None) -> None:
    wb = _nbytes(workspace) if workspace is not None and not isinstance(workspace, int) else 0
    block_scores_at, block_table_at, seq_lens_at, budgets_at = block_scores, block_table, seq_lens, budgets
    sel_table_at, sel_seq_lens_at, workspace_at, stream_at = sel_table, sel_seq_lens, workspace, stream
    if not (isinstance(block_scores, int) and isinstance(sel_table, int)):
        d = desc
        block_scores_at = _fits("vegas_select_blocks", "block_scores", block_scores, d.batch * d.max_blocks * 4)
        block_table_at = _fits("vegas_select_blocks", "block_table", block_table, d.batch * d.max_blocks * 4)
        seq_lens_at = _fits("vegas_select_blocks", "seq_lens", seq_lens, d.batch * 4)
        budgets_at = _fits("vegas_select_blocks", "budgets", budgets, d.batch * 4)
        sel_table_at = _fits("vegas_select_blocks", "sel_table", sel_table, d.batch * d.max_sel_blocks * 4)
        sel_seq_lens_at = _fits("vegas_select_blocks", "sel_seq_lens", sel_seq_lens, d.batch * 4)
    if type(block_scores_at) is not int: block_scores_at = _ptr(block_scores_at)
    if type(block_table_at) is not int: block_table_at = _ptr(block_table_at)
    if type(seq_lens_at) is not int: seq_lens_at = _ptr(seq_lens_at)
    if type(budgets_at) is not int: budgets_at = _ptr(budgets_at)
    if type(sel_table_at) is not int: sel_table_at = _ptr(sel_table_at)
    if type(sel_seq_lens_at) is not int: sel_seq_lens_at = _ptr(sel_seq_lens_at)
    if type(workspace_at) is not int: workspace_at = _ptr(workspace_at)
    if type(stream_at) is not int: stream_at = _stream(stream_at)
    rc = (_lib or load_library()).vegas_select_blocks(_byref(desc), block_scores_at, block_table_at, seq_lens_at, int(budget_tokens), budgets_at, sel_table_at,
        sel_seq_lens_at, workspace_at, wb, stream_at)
    if rc != VEGAS_OK:
        raise VegasError(rc, "vegas_select_blocks")


def vegas_select_tokens(desc: VegasDesc, token_scores, block_table, seq_lens, budget_tokens: int, sel_table,
                        sel_seq_lens, workspace, budgets=None, stream=None, workspace_bytes: Optional[int] = None) -> None:
    wb = workspace_bytes if workspace_bytes is not None else (_nbytes(workspace) if workspace is not None else 0)
    token_scores_at, block_table_at, seq_lens_at, budgets_at = token_scores, block_table, seq_lens, budgets
    sel_table_at, sel_seq_lens_at, workspace_at, stream_at = sel_table, sel_seq_lens, workspace, stream
    if not (isinstance(token_scores, int) and isinstance(sel_table, int)):
        d = desc
        token_scores_at = _fits("vegas_select_tokens", "token_scores", token_scores, d.batch * d.max_blocks * 16 * 4)
        block_table_at = _fits("vegas_select_tokens", "block_table", block_table, d.batch * d.max_blocks * 4)
        seq_lens_at = _fits("vegas_select_tokens", "seq_lens", seq_lens, d.batch * 4)
        budgets_at = _fits("vegas_select_tokens", "budgets", budgets, d.batch * 4)
        sel_table_at = _fits("vegas_select_tokens", "sel_table", sel_table, d.batch * d.max_sel_blocks * 4)
        sel_seq_lens_at = _fits("vegas_select_tokens", "sel_seq_lens", sel_seq_lens, d.batch * 4)
    if type(token_scores_at) is not int: token_scores_at = _ptr(token_scores_at)
    if type(block_table_at) is not int: block_table_at = _ptr(block_table_at)
    if type(seq_lens_at) is not int: seq_lens_at = _ptr(seq_lens_at)
    if type(budgets_at) is not int: budgets_at = _ptr(budgets_at)
    if type(sel_table_at) is not int: sel_table_at = _ptr(sel_table_at)
    if type(sel_seq_lens_at) is not int: sel_seq_lens_at = _ptr(sel_seq_lens_at)
    if type(workspace_at) is not int: workspace_at = _ptr(workspace_at)
    if type(stream_at) is not int: stream_at = _stream(stream_at)
    rc = (_lib or load_library()).vegas_select_tokens(_byref(desc), token_scores_at, block_table_at, seq_lens_at, int(budget_tokens), budgets_at, sel_table_at,
        sel_seq_lens_at, workspace_at, wb, stream_at)
    if rc != VEGAS_OK:
        raise VegasError(rc, "vegas_select_tokens")


def vegas_append_kv(desc: VegasDesc, k_new, v_new, num_new: int, block_table, seq_lens, k_cache, v_cache,
                    stream=None) -> None:
    k_new_at, v_new_at, block_table_at, seq_lens_at = k_new, v_new, block_table, seq_lens
    k_cache_at, v_cache_at, stream_at = k_cache, v_cache, stream
    if not (isinstance(k_new, int) and isinstance(k_cache, int)):
        d = desc
        rows = d.batch * int(num_new) * d.num_kv_heads * d.head_dim * 2
        extent = cache_extent_bytes(d)
        k_new_at = _fits("vegas_append_kv", "k_new", k_new, rows)
        v_new_at = _fits("vegas_append_kv", "v_new", v_new, rows)
        k_cache_at = _fits("vegas_append_kv", "k_cache", k_cache, extent)
        v_cache_at = _fits("vegas_append_kv", "v_cache", v_cache, extent)
        block_table_at = _fits("vegas_append_kv", "block_table", block_table, d.batch * d.max_blocks * 4)
        seq_lens_at = _fits("vegas_append_kv", "seq_lens", seq_lens, d.batch * 4)
    if type(k_new_at) is not int: k_new_at = _ptr(k_new_at)
    if type(v_new_at) is not int: v_new_at = _ptr(v_new_at)
    if type(block_table_at) is not int: block_table_at = _ptr(block_table_at)
    if type(seq_lens_at) is not int: seq_lens_at = _ptr(seq_lens_at)
    if type(k_cache_at) is not int: k_cache_at = _ptr(k_cache_at)
    if type(v_cache_at) is not int: v_cache_at = _ptr(v_cache_at)
    if type(stream_at) is not int: stream_at = _stream(stream_at)
    rc = (_lib or load_library()).vegas_append_kv(_byref(desc), k_new_at, v_new_at, int(num_new), block_table_at, seq_lens_at, k_cache_at, v_cache_at, stream_at)
    if rc != VEGAS_OK:
        raise VegasError(rc, "vegas_append_kv")


def vegas_append_kv_extend(desc: VegasDesc, k_new, v_new, num_new: int, block_table, seq_lens, k_cache, v_cache,
                           sel_table, sel_seq_lens, sel_page_size: int, stream=None) -> None:
    k_new_at, v_new_at, block_table_at, seq_lens_at, k_cache_at = k_new, v_new, block_table, seq_lens, k_cache
    v_cache_at, sel_table_at, sel_seq_lens_at, stream_at = v_cache, sel_table, sel_seq_lens, stream
    if not (isinstance(k_new, int) and isinstance(k_cache, int)):
        d = desc
        rows = d.batch * int(num_new) * d.num_kv_heads * d.head_dim * 2
        extent = cache_extent_bytes(d)
        k_new_at = _fits("vegas_append_kv_extend", "k_new", k_new, rows)
        v_new_at = _fits("vegas_append_kv_extend", "v_new", v_new, rows)
        k_cache_at = _fits("vegas_append_kv_extend", "k_cache", k_cache, extent)
        v_cache_at = _fits("vegas_append_kv_extend", "v_cache", v_cache, extent)
        block_table_at = _fits("vegas_append_kv_extend", "block_table", block_table, d.batch * d.max_blocks * 4)
        seq_lens_at = _fits("vegas_append_kv_extend", "seq_lens", seq_lens, d.batch * 4)
        sel_table_at = _fits("vegas_append_kv_extend", "sel_table", sel_table, d.batch * d.max_sel_blocks * 4)
        sel_seq_lens_at = _fits("vegas_append_kv_extend", "sel_seq_lens", sel_seq_lens, d.batch * 4)
    if type(k_new_at) is not int: k_new_at = _ptr(k_new_at)
    if type(v_new_at) is not int: v_new_at = _ptr(v_new_at)
    if type(block_table_at) is not int: block_table_at = _ptr(block_table_at)
    if type(seq_lens_at) is not int: seq_lens_at = _ptr(seq_lens_at)
    if type(k_cache_at) is not int: k_cache_at = _ptr(k_cache_at)
    if type(v_cache_at) is not int: v_cache_at = _ptr(v_cache_at)
    if type(sel_table_at) is not int: sel_table_at = _ptr(sel_table_at)
    if type(sel_seq_lens_at) is not int: sel_seq_lens_at = _ptr(sel_seq_lens_at)
    if type(stream_at) is not int: stream_at = _stream(stream_at)
    rc = (_lib or load_library()).vegas_append_kv_extend(
        _byref(desc), k_new_at, v_new_at, int(num_new), block_table_at, seq_lens_at, k_cache_at, v_cache_at, sel_table_at, sel_seq_lens_at, int(sel_page_size), stream_at)
    if rc != VEGAS_OK:
        raise VegasError(rc, "vegas_append_kv_extend")


def vegas_extend_selection(desc: VegasDesc, block_table, seq_lens, num_new: int, sel_table, sel_seq_lens,
                           stream=None) -> None:
    block_table_at, seq_lens_at, sel_table_at, sel_seq_lens_at, stream_at = block_table, seq_lens, sel_table, sel_seq_lens, stream
    if not (isinstance(block_table, int) and isinstance(sel_table, int)):
        d = desc
        block_table_at = _fits("vegas_extend_selection", "block_table", block_table, d.batch * d.max_blocks * 4)
        seq_lens_at = _fits("vegas_extend_selection", "seq_lens", seq_lens, d.batch * 4)
        sel_table_at = _fits("vegas_extend_selection", "sel_table", sel_table, d.batch * d.max_sel_blocks * 4)
        sel_seq_lens_at = _fits("vegas_extend_selection", "sel_seq_lens", sel_seq_lens, d.batch * 4)
    if type(block_table_at) is not int: block_table_at = _ptr(block_table_at)
    if type(seq_lens_at) is not int: seq_lens_at = _ptr(seq_lens_at)
    if type(sel_table_at) is not int: sel_table_at = _ptr(sel_table_at)
    if type(sel_seq_lens_at) is not int: sel_seq_lens_at = _ptr(sel_seq_lens_at)
    if type(stream_at) is not int: stream_at = _stream(stream_at)
    rc = (_lib or load_library()).vegas_extend_selection(_byref(desc), block_table_at, seq_lens_at, int(num_new), sel_table_at, sel_seq_lens_at, stream_at)
    if rc != VEGAS_OK:
        raise VegasError(rc, "vegas_extend_selection")


def vegas_draft_attention(desc: VegasDesc, q, k_cache, v_cache, sel_table, sel_seq_lens, out, workspace,
                          stream=None, workspace_bytes: Optional[int] = None, stages: int = 0) -> None:
    """stages != 0: vegas_debug_draft_attention_stages (a profiling aid: only those kernels of the call)."""
    wb = workspace_bytes if workspace_bytes is not None else (_nbytes(workspace) if workspace is not None else 0)
    q_at, k_cache_at, v_cache_at, sel_table_at = q, k_cache, v_cache, sel_table
    sel_seq_lens_at, out_at, workspace_at, stream_at = sel_seq_lens, out, workspace, stream
    if not (isinstance(q, int) and isinstance(k_cache, int)):
        d = desc
        rows = d.batch * d.num_q_heads * d.head_dim * 2
        extent = cache_extent_bytes(d)
        q_at = _fits("vegas_draft_attention", "q", q, rows)
        out_at = _fits("vegas_draft_attention", "out", out, rows)
        k_cache_at = _fits("vegas_draft_attention", "k_cache", k_cache, extent)
        v_cache_at = _fits("vegas_draft_attention", "v_cache", v_cache, extent)
        sel_table_at = _fits("vegas_draft_attention", "sel_table", sel_table, d.batch * d.max_sel_blocks * 4)
        sel_seq_lens_at = _fits("vegas_draft_attention", "sel_seq_lens", sel_seq_lens, d.batch * 4)
    if type(q_at) is not int: q_at = _ptr(q_at)
    if type(k_cache_at) is not int: k_cache_at = _ptr(k_cache_at)
    if type(v_cache_at) is not int: v_cache_at = _ptr(v_cache_at)
    if type(sel_table_at) is not int: sel_table_at = _ptr(sel_table_at)
    if type(sel_seq_lens_at) is not int: sel_seq_lens_at = _ptr(sel_seq_lens_at)
    if type(out_at) is not int: out_at = _ptr(out_at)
    if type(workspace_at) is not int: workspace_at = _ptr(workspace_at)
    if type(stream_at) is not int: stream_at = _stream(stream_at)
    args = (_byref(desc), q_at, k_cache_at, v_cache_at, sel_table_at, sel_seq_lens_at, out_at, workspace_at, wb, stream_at)
    if stages:
        rc = (_lib or load_library()).vegas_debug_draft_attention_stages(*args, int(stages))
    else:
        rc = (_lib or load_library()).vegas_draft_attention(*args)
    if rc != VEGAS_OK:
        raise VegasError(rc, "vegas_draft_attention")


def vegas_draft_step(cache_desc: VegasDesc, desc: VegasDesc, q, k_new, v_new, block_table, seq_lens, k_cache, v_cache, sel_table,
                     sel_seq_lens, out, workspace, stream=None, workspace_bytes: Optional[int] = None) -> None:
    """vegas_append_kv_extend of one token (cache_desc) and vegas_draft_attention (desc) in one call (see include/vegas.h)."""
    wb = workspace_bytes if workspace_bytes is not None else (_nbytes(workspace) if workspace is not None else 0)
    q_at, k_new_at, v_new_at, block_table_at, seq_lens_at, k_cache_at = q, k_new, v_new, block_table, seq_lens, k_cache
    v_cache_at, sel_table_at, sel_seq_lens_at, out_at, workspace_at, stream_at = v_cache, sel_table, sel_seq_lens, out, workspace, stream
    if not (isinstance(q, int) and isinstance(k_cache, int)):
        d, c = desc, cache_desc
        rows, new = d.batch * d.num_q_heads * d.head_dim * 2, c.batch * c.num_kv_heads * c.head_dim * 2
        extent = max(cache_extent_bytes(d), cache_extent_bytes(c))
        q_at = _fits("vegas_draft_step", "q", q, rows)
        out_at = _fits("vegas_draft_step", "out", out, rows)
        k_new_at = _fits("vegas_draft_step", "k_new", k_new, new)
        v_new_at = _fits("vegas_draft_step", "v_new", v_new, new)
        k_cache_at = _fits("vegas_draft_step", "k_cache", k_cache, extent)
        v_cache_at = _fits("vegas_draft_step", "v_cache", v_cache, extent)
        block_table_at = _fits("vegas_draft_step", "block_table", block_table, c.batch * c.max_blocks * 4)
        seq_lens_at = _fits("vegas_draft_step", "seq_lens", seq_lens, c.batch * 4)
        sel_table_at = _fits("vegas_draft_step", "sel_table", sel_table, d.batch * d.max_sel_blocks * 4)
        sel_seq_lens_at = _fits("vegas_draft_step", "sel_seq_lens", sel_seq_lens, d.batch * 4)
    if type(q_at) is not int: q_at = _ptr(q_at)
    if type(k_new_at) is not int: k_new_at = _ptr(k_new_at)
    if type(v_new_at) is not int: v_new_at = _ptr(v_new_at)
    if type(block_table_at) is not int: block_table_at = _ptr(block_table_at)
    if type(seq_lens_at) is not int: seq_lens_at = _ptr(seq_lens_at)
    if type(k_cache_at) is not int: k_cache_at = _ptr(k_cache_at)
    if type(v_cache_at) is not int: v_cache_at = _ptr(v_cache_at)
    if type(sel_table_at) is not int: sel_table_at = _ptr(sel_table_at)
    if type(sel_seq_lens_at) is not int: sel_seq_lens_at = _ptr(sel_seq_lens_at)
    if type(out_at) is not int: out_at = _ptr(out_at)
    if type(workspace_at) is not int: workspace_at = _ptr(workspace_at)
    if type(stream_at) is not int: stream_at = _stream(stream_at)
    rc = (_lib or load_library()).vegas_draft_step(
        _byref(cache_desc), _byref(desc), q_at, k_new_at, v_new_at, block_table_at, seq_lens_at, k_cache_at, v_cache_at, sel_table_at, sel_seq_lens_at,
        out_at, workspace_at, wb, stream_at)
    if rc != VEGAS_OK:
        raise VegasError(rc, "vegas_draft_step")


def vegas_static_scratch_bytes() -> int:
    return int(load_library().vegas_static_scratch_bytes())


def vegas_draft_attention_static(desc: VegasDesc, q, k_cache, v_cache, sel_table, sel_seq_lens, out, stream=None) -> None:
    """vegas_draft_attention without a workspace argument: the library's built-in scratch array is used."""
    q_at, out_at, k_cache_at, v_cache_at, sel_table_at, sel_seq_lens_at = q, out, k_cache, v_cache, sel_table, sel_seq_lens
    if not (isinstance(q, int) and isinstance(k_cache, int)):
        d = desc
        rows = d.batch * d.num_q_heads * d.head_dim * 2
        extent = cache_extent_bytes(d)
        q_at = _fits("vegas_draft_attention_static", "q", q, rows)
        out_at = _fits("vegas_draft_attention_static", "out", out, rows)
        k_cache_at = _fits("vegas_draft_attention_static", "k_cache", k_cache, extent)
        v_cache_at = _fits("vegas_draft_attention_static", "v_cache", v_cache, extent)
        sel_table_at = _fits("vegas_draft_attention_static", "sel_table", sel_table, d.batch * d.max_sel_blocks * 4)
        sel_seq_lens_at = _fits("vegas_draft_attention_static", "sel_seq_lens", sel_seq_lens, d.batch * 4)
    rc = load_library().vegas_draft_attention_static(ctypes.byref(desc), _ptr(q_at), _ptr(k_cache_at), _ptr(v_cache_at),
                                                     _ptr(sel_table_at), _ptr(sel_seq_lens_at), _ptr(out_at), _stream(stream))
    if rc != VEGAS_OK:
        raise VegasError(rc, "vegas_draft_attention_static")


def vegas_debug_check_tables(desc: VegasDesc, which: int, table, lens, error_word, stream=None) -> None:
    """ORs VEGAS_CHECK_* bits for out-of-range lengths and page ids into the device word (see include/vegas.h)."""
    table_at, lens_at, error_word_at = table, lens, error_word
    if not isinstance(table, int):
        stride = desc.max_blocks if which == TABLE_BLOCKS else desc.max_sel_blocks
        table_at = _fits("vegas_debug_check_tables", "table", table, desc.batch * stride * 4)
        lens_at = _fits("vegas_debug_check_tables", "lens", lens, desc.batch * 4)
        error_word_at = _fits("vegas_debug_check_tables", "error_word", error_word, 4)
    rc = load_library().vegas_debug_check_tables(ctypes.byref(desc), int(which), _ptr(table_at), _ptr(lens_at),
                                                 _ptr(error_word_at), _stream(stream))
    if rc != VEGAS_OK:
        raise VegasError(rc, "vegas_debug_check_tables")


def vegas_debug_set_timeline(buffer, nbytes: Optional[int] = None) -> None:
    """Profiling builds only: register (or, with None, drop) the buffer for the streaming kernels' phase stamps."""
    nb = 0 if buffer is None else (nbytes if nbytes is not None else _nbytes(buffer))
    rc = load_library().vegas_debug_set_timeline(_ptr(buffer), nb)
    if rc != VEGAS_OK:
        raise VegasError(rc, "vegas_debug_set_timeline")


def vegas_debug_verify_waves(desc: VegasDesc) -> int:
    """Waves per workgroup of the KV-streaming kernel of vegas_verify_attention for this descriptor."""
    rc = int(load_library().vegas_debug_verify_waves(ctypes.byref(desc)))
    if rc < 0:
        raise VegasError(rc, "vegas_debug_verify_waves")
    return rc


def vegas_debug_stream_read(a, b, bytes_each: int, workgroups: int, non_temporal: bool, sink, stream=None) -> None:
    """The plain streaming read the benchmark uses as its yardstick (see include/vegas.h)."""
    a_at, b_at, sink_at = a, b, sink
    if not isinstance(a, int):
        a_at = _fits("vegas_debug_stream_read", "a", a, bytes_each)
        b_at = _fits("vegas_debug_stream_read", "b", b, bytes_each)
        sink_at = _fits("vegas_debug_stream_read", "sink", sink, workgroups * 256 * 4)
    rc = load_library().vegas_debug_stream_read(_ptr(a_at), _ptr(b_at), int(bytes_each), int(workgroups), int(bool(non_temporal)),
                                                _ptr(sink_at), _stream(stream))
    if rc != VEGAS_OK:
        raise VegasError(rc, "vegas_debug_stream_read")


# ---------------------------------------------------------------------------------------------
# HIP events on a raw stream (timing plumbing for the benchmark)
# ---------------------------------------------------------------------------------------------

_hip = None


def _hip_runtime():
    global _hip
    if _hip is None:
        for name in ("libamdhip64.so", "libamdhip64.so.7", "libamdhip64.so.6", "/opt/rocm/lib/libamdhip64.so"):
            try:
                _hip = ctypes.CDLL(name)
                break
            except OSError:
                continue
        if _hip is None:
            raise RuntimeError("libamdhip64.so not found")
        _hip.hipEventCreate.argtypes = [ctypes.POINTER(ctypes.c_void_p)]
        _hip.hipEventDestroy.argtypes = [ctypes.c_void_p]
        _hip.hipEventSynchronize.argtypes = [ctypes.c_void_p]
        _hip.hipEventRecord.argtypes = [ctypes.c_void_p, ctypes.c_void_p]
        _hip.hipEventElapsedTime.argtypes = [ctypes.POINTER(ctypes.c_float), ctypes.c_void_p, ctypes.c_void_p]
    return _hip


class HipEvent:
    """A hipEvent_t recorded on a raw stream handle (the stream the library's kernels are launched on)."""

    def __init__(self):
        self.handle = ctypes.c_void_p()
        rc = _hip_runtime().hipEventCreate(ctypes.byref(self.handle))
        if rc != 0:
            raise RuntimeError(f"hipEventCreate failed ({rc})")

    def record(self, stream=None) -> None:
        rc = _hip_runtime().hipEventRecord(self.handle, _stream(stream))
        if rc != 0:
            raise RuntimeError(f"hipEventRecord failed ({rc})")

    def synchronize(self) -> None:
        rc = _hip_runtime().hipEventSynchronize(self.handle)
        if rc != 0:
            raise RuntimeError(f"hipEventSynchronize failed ({rc})")

    def elapsed_ms(self, end: "HipEvent") -> float:
        ms = ctypes.c_float()
        rc = _hip_runtime().hipEventElapsedTime(ctypes.byref(ms), self.handle, end.handle)
        if rc != 0:
            raise RuntimeError(f"hipEventElapsedTime failed ({rc})")
        return float(ms.value)

    def __del__(self):
        try:
            if self.handle:
                _hip_runtime().hipEventDestroy(self.handle)
        except Exception:
            pass
