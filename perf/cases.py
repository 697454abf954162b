"""The work a user of this library has it do, as timed cases.

A case is one layer's attention work of a Vegas decoding iteration, issued through the package's public entry points
(`harness.VegasPath` for the path a serving loop keeps per layer, `binding.vegas_draft_attention` for a bare draft
call).  The kinds:

  iterate   verify -> select -> gamma + 1 draft calls on a static cache (Sec. 2.3, Sec. 3)
  live      the same with the drafted token's K/V appended and the selection grown before every draft call
  token     the paper's own granularity: token logits, single-token selection, drafting over one-token pages (Sec. 3.3)
  verify    a verification call alone (other row counts, collection modes, the local mask of a banded layer)
  draft     a draft call alone over random token positions (App. D)

Sizes are the repository's own workloads (paper_2602_07223_amd/synth.py, bench.py) and generic ragged batches.  Keys
and queries have unit-variance elements, so scaled logits have standard deviation 1; on top of that every page has an
importance that all heads agree on (a normally distributed shift of its tokens' logits, along a direction the queries
carry) and the first four tokens of a sequence are attention sinks.  That is the shape sparse drafting relies on: a
minority of pages carries most of the weight.
"""
from __future__ import annotations

import math
from typing import Dict, List

import torch

from paper_2602_07223_amd import binding as vb
from paper_2602_07223_amd import harness

PAGE = 16
DEVICE = "cuda:0"


def _case(name: str, kind: str, batch: int, heads: int, kv_heads: int, dim: int, queries: int, lo: int, hi: int,
          budget: int, collect: int = vb.COLLECT_ALL_ROWS, window: int = 0, page: int = PAGE) -> Dict[str, object]:
    return dict(name=name, kind=kind, batch=batch, heads=heads, kv_heads=kv_heads, dim=dim, queries=queries, lo=lo,
                hi=hi, budget=budget, collect=collect, window=window, page=page)


def listed() -> List[Dict[str, object]]:
    return [
        # A short context, one sequence: everything is launches and round trips (workload ctx4k).
        _case("iterate_4k", "iterate", 1, 32, 8, 128, 5, 4096, 4096, 256),
        # Reasoning outputs in flight: a batch of sequences that are all at another length (Sec. 5's short-input
        # setting: short prompts, outputs of up to about 20K tokens, many sequences), seven drafted tokens.
        _case("iterate_batch24_1k_20k", "iterate", 24, 32, 8, 128, 8, 1001, 20011, 1024),
        # The headline: one sequence of 32K tokens (workload ctx32k).
        _case("iterate_32k", "iterate", 1, 32, 8, 128, 5, 32768, 32768, 2048),
        # One very long sequence (workload ctx128k_drift).
        _case("iterate_128k", "iterate", 1, 32, 8, 128, 7, 131072, 131072, 4096),
        # A serving batch of ragged long contexts with eight query heads per KV head: 40 rows (workload ragged16).
        _case("iterate_ragged16_8k_64k", "iterate", 16, 64, 8, 128, 5, 8192, 65536, 2048),
        # One layer of the 32-layer stack: four sequences of 64K tokens (workload stack32).
        _case("iterate_batch4_64k", "iterate", 4, 32, 8, 128, 5, 65536, 65536, 4096),
        # The 2-KB-per-token attention shape of App. D: head dimension 64, 40 rows (workload hd64_ctx32k).
        _case("iterate_hd64_32k", "iterate", 1, 64, 8, 64, 5, 32768, 32768, 2048),
        # Live drafting as a decoding loop runs it, at a length that ends inside a page.
        _case("live_32k", "live", 1, 32, 8, 128, 5, 32749, 32749, 2048),
        # The paper's own variant: single tokens chosen by averaged logits, one-token pages.
        _case("token_32k", "token", 1, 32, 8, 128, 5, 32768, 32768, 2048),
        # The largest row count of the collection sweep with the two-row collection of Eq. 3: 48 rows.
        _case("verify_two_rows_32k", "verify", 1, 32, 8, 128, 12, 32749, 32749, 0, collect=vb.COLLECT_FIRST_LAST),
        # A banded layer between the full-attention ones: a local mask of 128 tokens, nothing collected.
        _case("verify_window_batch16", "verify", 16, 64, 8, 64, 5, 8192, 65536, 0, collect=vb.COLLECT_NONE, window=128),
        # App. D's comparison: 16 requests of 8192 selected tokens at random positions, one-token pages (Table 5).
        _case("draft_tokens_16x8k", "draft", 16, 32, 8, 128, 1, 131072, 131072, 8192, page=1),
    ]


def _lengths(case) -> List[int]:
    """Lengths of the batch: spread over [lo, hi] in an order without pattern, fixed by the case alone."""
    lo, hi, n = case["lo"], case["hi"], case["batch"]
    return [lo + int((hi - lo) * math.fmod((i + 1) * 0.6180339887498949, 1.0)) for i in range(n)]


def _selected(case) -> List[int]:
    """Tokens a draft call reads per sequence."""
    if case["kind"] == "draft":
        return [case["budget"]] * case["batch"]
    if case["kind"] == "token":
        return [min(max(case["budget"], case["queries"]), n) for n in _lengths(case)]
    out = []
    for n in _lengths(case):
        pages = -(-n // PAGE)
        forced = pages - max(n - case["queries"], 0) // PAGE
        k = max(min(-(-case["budget"] // PAGE), pages), forced)
        out.append(PAGE * (k - 1) + n - PAGE * (pages - 1))
    return out


def _bytes_per_token(case) -> int:
    return 2 * case["kv_heads"] * case["dim"] * 2


# The largest listed case (iterate_ragged16_8k_64k) streams about 2.4 GB in its verification and 0.7 GB in its draft calls.
_MOST_BYTES = 2.9e9


def draw(rng) -> Dict[str, object]:
    """Another case of the same ranges: 1 to 32 sequences, 500 to 131072 tokens, both head dimensions, 1 to 12
    verification rows, groups of 1 to 8 heads."""
    def log_int(lo, hi):
        return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))

    while True:
        kind = rng.choice(["iterate", "iterate", "iterate", "live", "token", "verify", "draft"])
        heads, kv_heads = rng.choice([(32, 8), (32, 8), (64, 8), (16, 8), (28, 4), (40, 8), (8, 8)])
        dim = rng.choice([128, 128, 64])
        batch = log_int(1, 32)
        hi = log_int(500, 131072)
        lo = max(300, int(hi * rng.choice([1.0, 0.7, 0.25, 0.1])))
        lo = min(lo, hi)
        queries = rng.randint(1, 12)
        if queries * (heads // kv_heads) > 96:
            continue
        budget = max(64, int(hi * rng.uniform(0.03, 0.12)))
        c = _case("", kind, batch, heads, kv_heads, dim, queries, lo, hi, budget)
        if kind == "verify":
            c["budget"] = 0
            if rng.random() < 0.3:
                c["collect"], c["window"] = vb.COLLECT_NONE, log_int(64, 4096)
            else:
                c["collect"] = rng.choice([vb.COLLECT_NONE, vb.COLLECT_ALL_ROWS, vb.COLLECT_FIRST_LAST])
        if kind == "draft":
            c["queries"], c["lo"] = 1, hi
            c["page"] = rng.choice([1, 1, 2, 4, 8, 16])
        del c["name"]
        pool = sum(_lengths(c)) * _bytes_per_token(c)
        if pool > 2.5e9 or work(c)["bytes"] > _MOST_BYTES:
            continue
        return c


def _normal(shape, gen) -> torch.Tensor:
    return torch.randn(shape, generator=gen, device=DEVICE, dtype=torch.float32)


def _pool(pages: int, kv_heads: int, dim: int, gen, importance=None, direction=None) -> torch.Tensor:
    """bf16 [pages, 16, kv_heads, dim] of unit normals, plus importance[page] * direction[kv_head] where given."""
    out = torch.empty((pages, PAGE, kv_heads, dim), dtype=torch.bfloat16, device=DEVICE)
    step = max(1, (1 << 26) // (PAGE * kv_heads * dim))
    for p0 in range(0, pages, step):
        x = _normal((min(step, pages - p0), PAGE, kv_heads, dim), gen)
        if importance is not None:
            x += importance[p0:p0 + step].view(-1, 1, 1, 1) * direction
        out[p0:p0 + step] = x
    return out


def prepare(case, seed: int):
    gen = torch.Generator(device=DEVICE)
    gen.manual_seed(int(seed))
    B, Hq, Hkv, D, G = case["batch"], case["heads"], case["kv_heads"], case["dim"], case["queries"]
    lens = _lengths(case)
    kind = case["kind"]
    growth = G if kind == "live" else 0
    # A shared pool whose pages are handed out in random order, as a serving engine's allocator does.
    counts = [-(-(n + growth) // PAGE) for n in lens]
    pages = sum(counts)
    order = torch.randperm(pages, generator=gen, device=DEVICE).to(torch.int32)
    max_blocks = max(counts)
    table = torch.full((B, max_blocks), -1, dtype=torch.int32, device=DEVICE)
    first = 0
    for b, c in enumerate(counts):
        table[b, :c] = order[first:first + c]
        first += c
    # Per KV head a unit direction; queries carry a quarter of sqrt(D) along it, so a key shifted by 4 a along it
    # gets a scaled logit a higher.
    direction = _normal((Hkv, D), gen)
    direction /= direction.norm(dim=-1, keepdim=True)
    importance = 4.0 * _normal((pages,), gen)
    k = _pool(pages, Hkv, D, gen, importance, direction)
    v = _pool(pages, Hkv, D, gen)
    sink = table[:, 0].long()
    k[sink, :4] += (16.0 * direction).to(torch.bfloat16)
    along = 0.25 * math.sqrt(D) * direction.repeat_interleave(Hq // Hkv, dim=0)
    q_base = _normal((B, G, Hq, D), gen)
    q_verify = (q_base + along).to(torch.bfloat16)
    q_draft = (q_base.transpose(0, 1) + 0.1 * _normal((G, B, Hq, D), gen) + along).to(torch.bfloat16).contiguous()
    seq_lens = torch.tensor(lens, dtype=torch.int32, device=DEVICE)
    scale = 1.0 / math.sqrt(D)

    if kind == "draft":
        ps, n_sel = case["page"], case["budget"]
        per = -(-n_sel // ps)
        # `per` distinct pages of ps tokens out of each sequence's own, in ascending order; the last may be partial.
        sel = torch.empty((B, per), dtype=torch.int32, device=DEVICE)
        for b, n in enumerate(lens):
            small = n // ps
            pick = torch.randperm(small, generator=gen, device=DEVICE)[:per].sort().values
            pos = pick * ps
            sel[b] = table[b, pos // PAGE] * (PAGE // ps) + ((pos % PAGE) // ps).to(torch.int32)
        desc = vb.make_desc(batch=B, num_q_heads=Hq, num_kv_heads=Hkv, num_queries=1, max_blocks=max_blocks,
                            max_sel_blocks=per, max_seq_len=n_sel, num_pages=pages * (PAGE // ps), softmax_scale=scale,
                            collect_rows=vb.COLLECT_NONE, head_dim=D, page_size=ps)
        return dict(kind=kind, desc=desc, q=q_draft[0], k=k, v=v, sel=sel,
                    sel_lens=torch.full((B,), n_sel, dtype=torch.int32, device=DEVICE),
                    out=torch.empty((B, Hq, D), dtype=torch.bfloat16, device=DEVICE),
                    workspace=torch.empty(vb.vegas_workspace_bytes(desc), dtype=torch.uint8, device=DEVICE))

    layer = harness.DeviceLayer(q_verify=q_verify, q_draft=q_draft, k_cache=k, v_cache=v, block_table=table,
                                seq_lens=seq_lens)
    if kind == "live":
        layer.k_new = _normal((G, B, 1, Hkv, D), gen).to(torch.bfloat16)
        layer.v_new = _normal((G, B, 1, Hkv, D), gen).to(torch.bfloat16)
        layer.seq_lens_live = seq_lens.clone()
    path = harness.VegasPath(batch=B, num_q_heads=Hq, num_kv_heads=Hkv, num_queries=G, max_blocks=max_blocks,
                             max_seq_len=max(lens), num_pages=pages, budget_tokens=max(case["budget"], 1),
                             softmax_scale=scale, collect_rows=case["collect"], head_dim=D, device=DEVICE,
                             token_granular=kind == "token", window=case["window"], growth=growth)
    return dict(kind=kind, path=path, layer=layer, scores=case["collect"] != vb.COLLECT_NONE)


def run(state):
    kind = state["kind"]
    if kind == "draft":
        vb.vegas_draft_attention(state["desc"], state["q"], state["k"], state["v"], state["sel"], state["sel_lens"],
                                 state["out"], state["workspace"], stream=torch.cuda.current_stream())
        return state["out"]
    path, layer = state["path"], state["layer"]
    if kind == "verify":
        path.verify(layer)
        return (path.out_verify, path.block_scores) if state["scores"] else path.out_verify
    if kind == "live":
        path.live_iteration(layer)
        return (path.out_verify, path.block_scores, path.sel_table, path.sel_seq_lens, path.out_draft,
                layer.seq_lens_live)
    path.iteration(layer)
    return path.out_verify, path.block_scores, path.sel_table, path.sel_seq_lens, path.out_draft


def work(case) -> Dict[str, float]:
    """Per call: its K/V tokens, queries, tables and outputs once.  (A draft call is a call of its own: the pages it
    reads count although verification has read them before.)"""
    B, Hq, D, G = case["batch"], case["heads"], case["dim"], case["queries"]
    bpt = _bytes_per_token(case)
    per_token_flops = 4.0 * Hq * D
    nbytes = flops = 0.0
    if case["kind"] != "draft":
        lens = _lengths(case)
        seen = [min(n, case["window"] + G - 1) if case["window"] else n for n in lens]
        nbytes += sum(seen) * bpt + 2 * B * G * Hq * D * 2 + sum(4 * -(-n // PAGE) for n in seen)
        flops += sum(seen) * per_token_flops * G
        if case["collect"] != vb.COLLECT_NONE:
            per = 4 if case["kind"] == "token" else 4 / PAGE
            nbytes += sum(lens) * per
    if case["kind"] in ("iterate", "live", "token"):
        nbytes += sum(_lengths(case)) * (4 if case["kind"] == "token" else 4 / PAGE)      # the selection reads the scores
    if case["kind"] != "verify":
        steps = 1 if case["kind"] == "draft" else G
        grown = sum(range(1, G + 1)) if case["kind"] == "live" else 0
        sel = sum(_selected(case))
        nbytes += (steps * sel + B * grown) * bpt + steps * 2 * B * Hq * D * 2
        flops += (steps * sel + B * grown) * per_token_flops
        if case["kind"] == "live":
            nbytes += steps * B * 2 * bpt
    return {"bytes": nbytes, "flops": flops}


def tolerance(case):
    """bf16 outputs formed from bf16-rounded softmax weights: against a float64 reference of the same inputs the
    2-norm of the error is 1.8e-3 to 2.0e-3 of the result's (rounding the exact result to bf16 alone gives 1.6e-3) and
    the largest error 0.006 to 0.010 of its root mean square; four times that is stated.  The fp32 page scores are off
    by 3e-7 at most (2-norm), so a page exchanged for another at the end of the budget is rare: "differ" leaves room
    for one."""
    return {"rel": 8e-3, "max": 0.04, "differ": 0.01}
