"""Selection among keys in registers (select_blocks.hpp, find_last_key) where scores do not spread over the digits: waves that
count a few digits or runs of lanes by themselves, bins that hold an eighth of the keys and set the range of the next pass, at the edges of
the rows of 4096 tokens (or 1024 pages) and of the launch variants, against the oracle, bit for bit."""
import numpy as np
import pytest
import torch

from oracle import vegas_oracle as O
from paper_2602_07223_amd import binding as vb
from tests.test_gpu_token_variant import gpu_select_tokens

pytestmark = pytest.mark.gpu
PAGE = 16
INF, NAN = np.float32(np.inf), np.float32(np.nan)


def percent(n, rng):
    return ((1 + 0.01 * rng.random(n)) / n).astype(np.float32)


def make_scores(kind, n, rng):
    x = rng.random(n).astype(np.float32)
    some = rng.random(n)
    if kind == "four_values":
        return (rng.integers(0, 4, size=n) * np.float32(0.125)).astype(np.float32)
    if kind == "forty_values":
        return (rng.integers(0, 40, size=n) * np.float32(0.125) - 2).astype(np.float32)
    if kind == "half_zero":
        return np.where(some < 0.5, np.float32(0), x)
    if kind == "few_nonzero":
        return np.where(some < 0.95, np.float32(0), x - np.float32(0.5)).astype(np.float32)
    if kind == "masked":                   # -infinity and NaN beside scores that agree to a percent
        return np.where(some < 0.04, -INF, np.where(some < 0.05, NAN, percent(n, rng))).astype(np.float32)
    if kind == "outliers":                 # a cluster of a few ulps, a neighbour of it, far ones at both ends
        x = (np.uint32(0x3F800000) + rng.integers(0, 16, size=n).astype(np.uint32)).view(np.float32).copy()
        x[rng.integers(0, n, size=max(n // 5, 1))] = np.float32(1.25)
        x[n // 2], x[n // 3], x[n // 4] = np.float32(-3e38), INF, NAN
        return x
    if kind == "ascending":
        return np.sort(x)
    return np.repeat(x[:n // 97 + 1], 97)[:n].copy()      # runs of equal scores


KINDS = ["four_values", "forty_values", "half_zero", "few_nonzero", "masked", "outliers", "runs", "ascending"]


# longest sequence, queries: prefixes of whole rows of 4096 tokens and one token more, both sides of every launch variant
@pytest.mark.parametrize("longest,G", [(4096, 1), (4097, 1), (4098, 1), (8192, 1), (8193, 1), (16384, 1), (16385, 1), (28677, 5),
                                       (32768, 1), (32769, 1)])
@pytest.mark.parametrize("kind", KINDS)
def test_tokens(kind, longest, G):
    rng = np.random.default_rng(longest * 11 + len(kind))
    lens = np.array([longest, max(longest // 2, 1), min(4096 + G, longest), min(8192 + G, longest), 1 + G], dtype=np.int32)
    B, mb = len(lens), (longest + PAGE - 1) // PAGE
    scores = np.stack([make_scores(kind, mb * PAGE, rng) for _ in range(B)])
    table = np.stack([rng.permutation(mb + 5)[:mb] for _ in range(B)]).astype(np.int32)
    for budgets in (None, np.array([longest - G, 300, 4095, 1 + G, 2], dtype=np.int32)):
        max_sel = longest + 2
        print(f"[case] crowded tokens {kind} longest={longest} per_sequence={budgets is not None}", flush=True)
        sel, ssl = gpu_select_tokens(scores, table, lens, G, longest // 14 + 1, max_sel, budgets)
        with np.errstate(invalid="ignore"):
            ref_sel, ref_ssl, _ = O.select_tokens(scores, table, lens, G, longest // 14 + 1, max_sel, budgets)
        assert np.array_equal(ssl, ref_ssl)
        assert np.array_equal(sel, ref_sel)


def bordering(n, above):
    """Keys (as bits of scores in [1, 2)): an eighth of them and more within one bin of 4096 from its second key to its last,
    which `above` keys, before it by position, follow at once; the last one taken is the bin's last.  Its exact range, cut by
    11-bit digits, ends half a digit after it."""
    rng = np.random.default_rng(n)
    off = 10 * 4096 + rng.integers(0, 2**23 - 10 * 4096, size=n)
    off[::3] = 5 * 4096 + 1
    off[1::7] = 0
    off[-1] = 2**23 - 1
    off[-2] = 5 * 4096 + 4095
    off[2:2 + 3 * above:3] = 6 * 4096
    return (np.uint32(0x3F800000) + off.astype(np.uint32)).view(np.float32), int((off >= 5 * 4096 + 4095).sum())


@pytest.mark.parametrize("above", [0, 1, 20])
@pytest.mark.parametrize("longest", [4096, 8192, 32768])
def test_tokens_above_the_last_bin_of_an_exact_range(longest, above):
    G = 5
    x, take = bordering(longest - G, above)
    scores = np.zeros((1, longest), dtype=np.float32)
    scores[0, :longest - G] = x
    table = np.arange(longest // PAGE, dtype=np.int32)[None]
    lens = np.array([longest], dtype=np.int32)
    for k in (take, take - 1, take + 1):
        sel, ssl = gpu_select_tokens(scores, table, lens, G, k + G, longest, None)
        ref_sel, ref_ssl, _ = O.select_tokens(scores, table, lens, G, k + G, longest, None)
        assert np.array_equal(ssl, ref_ssl)
        assert np.array_equal(sel, ref_sel)


@pytest.mark.parametrize("pages", [100, 1025, 2049, 3072, 3073, 4097, 8192])
@pytest.mark.parametrize("kind", KINDS)
def test_pages(kind, pages):
    rng = np.random.default_rng(pages * 13 + len(kind))
    G = 5
    lens = np.array([pages * PAGE, pages * PAGE - 12, min(1024 * PAGE + G, pages * PAGE), 900], dtype=np.int32)
    B = len(lens)
    scores = np.stack([make_scores(kind, pages, rng) for _ in range(B)])
    table = np.stack([rng.permutation(pages + 5)[:pages] for _ in range(B)]).astype(np.int32)
    dev = torch.device("cuda:0")
    for budget in (48, pages * PAGE // 14 + 64, pages * PAGE - 40):
        msb = pages + 2
        print(f"[case] crowded pages {kind} pages={pages} budget={budget}", flush=True)
        desc = vb.make_desc(batch=B, num_q_heads=32, num_kv_heads=8, num_queries=G, max_blocks=pages, max_sel_blocks=msb,
                            max_seq_len=pages * PAGE, num_pages=pages + 5, softmax_scale=0.1)
        sel = torch.full((B, msb), -7, dtype=torch.int32, device=dev)
        ssl = torch.full((B,), -7, dtype=torch.int32, device=dev)
        vb.vegas_select_blocks(desc, torch.from_numpy(scores).to(dev), torch.from_numpy(table).to(dev),
                               torch.from_numpy(lens).to(dev), budget, sel, ssl)
        torch.cuda.synchronize()
        with np.errstate(invalid="ignore"):
            ref_sel, ref_ssl, _ = O.select_blocks(scores, table, lens, G, budget, msb)
        assert np.array_equal(ssl.cpu().numpy(), ref_ssl)
        assert np.array_equal(sel.cpu().numpy(), ref_sel)
