"""vegas_draft_step against vegas_append_kv_extend followed by vegas_draft_attention, bit for bit (those two have their oracle
tests in test_gpu_live_iteration.py): lengths, selection, cache and output after each of a few steps, with NaN in every slot that
has no token yet."""
import numpy as np
import pytest
import torch

from oracle import vegas_oracle as O
from paper_2602_07223_amd import binding as vb

pytestmark = pytest.mark.gpu
PAGE = 16
DEV = "cuda:0"

# name, query heads, KV heads, head dim, lengths, selected pages (None: all), entries of a selection row, chunk, bound of the call
CASES = [
    ("merged", 32, 8, 128, [2045], 100, 104, 0, None),                    # crosses into a new page, 18 chunks of 96 tokens
    ("page_starts_a_chunk", 32, 8, 128, [4096], 128, 132, 128, None),     # the selection ends with a whole chunk of 128 tokens
    ("page_starts_a_fine_chunk", 32, 8, 128, [4096], 126, 132, 0, None),  # ... of 96: the next has one tile and three idle waves
    ("row_fills_up", 32, 8, 128, [3198, 3200], 128, 128, 0, None),        # no new page fits: at the third step, at the first
    ("no_room", 32, 8, 128, [3215, 3216, 1000], 128, 140, 0, None),       # at the end of the table: refused
    ("bound_ends_it", 32, 8, 128, [3000], 128, 140, 0, 2042),             # 2040 tokens, then the draft call's own bound lies before the new one
    ("empty_and_short", 16, 4, 64, [0, 5, 3100], None, 256, 0, None),
    ("many_chunks", 8, 8, 128, [3333], None, 220, 32, None),              # more than 64 chunks: the general merge
    ("one_tile_chunks", 28, 4, 64, [700, 31, 16], None, 50, 32, None),
    ("group16", 32, 2, 128, [2100, 900], None, 140, 0, None),
    ("one_workgroup", 32, 8, 128, [200, 300], None, 22, 0, None),         # the streaming kernel writes the rows: two calls
    ("group32", 64, 2, 128, [1500], None, 100, 0, None),                  # more rows than the 16-row kernel takes: two calls
    ("past_the_cache", 64, 16, 128, [3000] * 16, None, 194, 0, None),     # 402 MB under the bound: two calls
]


CALLS = [(P, *c) for P in (16, 1) for c in CASES if P == 16 or c[0] not in ("past_the_cache", "row_fills_up")]   # (those: 16-token pages)


@pytest.mark.parametrize("P,name,Hq,Hkv,D,lens,pages,row,chunk,bound", CALLS, ids=[f"{c[1]}-{c[0]}" for c in CALLS])
def test_one_call_is_the_two_calls(P, name, Hq, Hkv, D, lens, pages, row, chunk, bound):
    B, steps, max_blocks = len(lens), 4, 201 if name == "no_room" else 300
    gen = torch.Generator(device=DEV).manual_seed(71000 + sum(lens) + D + Hq)
    rng = np.random.default_rng(71000 + sum(lens))
    need = [min(max_blocks, -(-(n + steps) // PAGE)) for n in lens]
    pool = sum(need) + 3
    order = rng.permutation(pool).astype(np.int32)
    table = np.full((B, max_blocks), -1, dtype=np.int32)
    at = 0
    for b, c in enumerate(need):
        table[b, :c] = order[at:at + c]
        at += c
    k = torch.randn((pool, PAGE, Hkv, D), generator=gen, device=DEV).to(torch.bfloat16)
    v = torch.randn((pool, PAGE, Hkv, D), generator=gen, device=DEV).to(torch.bfloat16)
    for b, n in enumerate(lens):                                          # slots without a token
        for pos in range(n, need[b] * PAGE):
            k[int(table[b, pos // PAGE]), pos % PAGE] = float("nan")
            v[int(table[b, pos // PAGE]), pos % PAGE] = float("nan")
    budget = 10 ** 6 if pages is None else pages * PAGE
    n32 = np.array(lens, dtype=np.int32)
    entries = row if P == 16 else row * PAGE
    if P == 16:
        sel, ssl, _ = O.select_blocks(rng.random((B, max_blocks)).astype(np.float32), table, n32, 1, budget, entries)
    else:
        sel, ssl, _ = O.select_tokens(rng.random((B, max_blocks * PAGE)).astype(np.float32), table, n32, 1, min(budget, entries), entries)
    common = dict(batch=B, num_q_heads=Hq, num_kv_heads=Hkv, num_queries=1, max_sel_blocks=entries, softmax_scale=D ** -0.5, head_dim=D,
                  collect_rows=vb.COLLECT_NONE)
    cache = vb.make_desc(max_blocks=max_blocks, max_seq_len=max_blocks * PAGE, num_pages=pool, **common)
    draft = vb.make_desc(max_blocks=max_blocks if P == 16 else entries, max_seq_len=bound or entries * P, num_pages=pool * (PAGE // P),
                         page_size=P, kv_chunk_tokens=chunk, **common)
    print(f"[case] draft step {name} P={P} lens={lens[:4]} selected={ssl[:4].tolist()}", flush=True)

    def state():
        return dict(k=k.clone(), v=v.clone(), table=torch.from_numpy(table).to(DEV), n=torch.from_numpy(n32).to(DEV),
                    sel=torch.from_numpy(sel.copy()).to(DEV), ssl=torch.from_numpy(ssl.copy()).to(DEV),
                    out=torch.full((B, Hq, D), float("nan"), dtype=torch.bfloat16, device=DEV),
                    ws=torch.full((vb.vegas_workspace_bytes(draft),), 0xFF, dtype=torch.uint8, device=DEV))

    one, two = state(), state()
    kept = set()                                                          # sequences that took a token and did not select it
    for step in range(steps):
        before = {x: one[x].clone() for x in ("n", "ssl")}
        q, kn, vn = (torch.randn((B, h, D), generator=gen, device=DEV).to(torch.bfloat16) for h in (Hq, Hkv, Hkv))
        vb.vegas_draft_step(cache, draft, q, kn, vn, one["table"], one["n"], one["k"], one["v"], one["sel"], one["ssl"], one["out"], one["ws"])
        vb.vegas_append_kv_extend(cache, kn, vn, 1, two["table"], two["n"], two["k"], two["v"], two["sel"], two["ssl"], P)
        vb.vegas_draft_attention(draft, q, two["k"], two["v"], two["sel"], two["ssl"], two["out"], two["ws"])
        torch.cuda.synchronize()
        for name_, a in one.items():
            if name_ == "ws":
                continue
            b_ = two[name_]
            if a.dtype == torch.bfloat16:
                a, b_ = a.view(torch.int16), b_.view(torch.int16)
            assert torch.equal(a, b_), f"{name} P={P} step {step}: {name_}"
        assert bool(torch.isfinite(one["out"].float()).all()), f"{name} P={P} step {step}"
        kept |= set(torch.nonzero((one["n"] > before["n"]) & (one["ssl"] == before["ssl"]) & (before["ssl"] > 0)).flatten().tolist())
    grown = one["n"].cpu().numpy()
    assert [int(x) for x in grown] == [min(n + steps, max_blocks * PAGE) for n in lens]
    assert kept == ({0, 1} if name == "row_fills_up" else set())          # (the named edge is the one that was met)
    if name == "bound_ends_it":
        assert int(one["ssl"].max()) > draft.max_seq_len


def test_refused_steps_launch_nothing():
    common = dict(batch=1, num_q_heads=8, num_kv_heads=8, num_queries=1, softmax_scale=0.1, collect_rows=vb.COLLECT_NONE)
    cache = vb.make_desc(max_blocks=64, max_sel_blocks=64, max_seq_len=1024, num_pages=64, **common)
    draft = vb.make_desc(max_blocks=64, max_sel_blocks=64, max_seq_len=1024, num_pages=64, **common)
    other = vb.make_desc(max_blocks=64, max_sel_blocks=63, max_seq_len=1008, num_pages=64, **common)
    eight = vb.make_desc(max_blocks=64, max_sel_blocks=64, max_seq_len=512, num_pages=128, page_size=8, **common)
    t = {n: torch.zeros(s, dtype=d, device=DEV) for n, s, d in (
        ("q", (1, 8, 128), torch.bfloat16), ("kn", (1, 8, 128), torch.bfloat16), ("k", (64, 16, 8, 128), torch.bfloat16),
        ("table", (1, 64), torch.int32), ("n", (1,), torch.int32), ("sel", (1, 64), torch.int32), ("ssl", (1,), torch.int32),
        ("out", (1, 8, 128), torch.bfloat16), ("ws", (vb.vegas_workspace_bytes(draft),), torch.uint8))}
    def step(desc, wsn=None):
        vb.vegas_draft_step(cache, desc, t["q"], t["kn"], t["kn"], t["table"], t["n"], t["k"], t["k"], t["sel"], t["ssl"], t["out"], t["ws"],
                            workspace_bytes=wsn)
    for bad in (lambda: step(other), lambda: step(eight), lambda: step(draft, 16)):
        with pytest.raises(vb.VegasError):
            bad()
    torch.cuda.synchronize()
    assert int(t["n"].item()) == 0
    step(draft)
    torch.cuda.synchronize()
    assert int(t["n"].item()) == 1 and int(t["ssl"].item()) == 0           # appended to; an empty selection stays empty
