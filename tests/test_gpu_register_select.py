"""Token selection by one workgroup per sequence (prefixes of at most 32768 tokens) against the oracle, bit for bit, at
lengths inside its rows of 4096 tokens and at the edges of its digit passes (whole rows: test_gpu_select_crowded.py)."""
import numpy as np
import pytest

from oracle import vegas_oracle as O
from tests.test_gpu_token_variant import gpu_select_tokens

pytestmark = pytest.mark.gpu
PAGE = 16


def make_scores(kind, n, rng):
    if kind == "any_bits":                 # every exponent, both signs, NaNs, infinities, denormals
        return rng.integers(0, 1 << 32, size=n, dtype=np.uint64).astype(np.uint32).view(np.float32)
    if kind == "mostly_nan":
        x = np.full(n, np.nan, dtype=np.float32)
        x[rng.integers(0, n, size=n // 40 + 1)] = rng.standard_normal(n // 40 + 1).astype(np.float32)
        return x
    if kind == "one_bin":                  # neighbours of one number: all differences in the lowest bits
        return (np.uint32(0x3F800000) + rng.integers(0, 3000, size=n).astype(np.uint32)).view(np.float32)
    if kind == "equal":
        return np.full(n, -0.5, dtype=np.float32)
    if kind == "far_outlier":              # the rest falls into one bin of the first pass, and of the second
        x = (np.float32(1.0) + rng.random(n).astype(np.float32) * np.float32(1e-6)).astype(np.float32)
        x[n // 2] = -3e38
        return x
    return rng.standard_normal(n).astype(np.float32)


@pytest.mark.parametrize("longest", [9, 1029, 8192, 8193, 32768])
@pytest.mark.parametrize("kind", ["normal", "any_bits", "mostly_nan", "one_bin", "equal", "far_outlier"])
def test_one_workgroup_token_select_is_bit_exact(kind, longest):
    rng = np.random.default_rng(longest * 7 + len(kind))
    G = 5 if longest != 32768 else 1
    lens = np.array([longest, max(longest // 2 + 3, 1), min(longest, 1024 + G), min(longest, 1025 + G), 0], dtype=np.int32)
    B, mb = len(lens), (longest + PAGE - 1) // PAGE + 2
    scores = np.zeros((B, mb * PAGE), dtype=np.float32)
    for b in range(B):
        scores[b] = make_scores(kind, mb * PAGE, rng)          # (what lies past the prefix must not matter)
    table = np.stack([rng.permutation(mb + 5)[:mb] for _ in range(B)]).astype(np.int32)
    for budget, budgets in ((max(longest // 16, 6), None),
                            (64, np.array([longest - 1, longest // 3 + 1, 1, 1024 + G - 1, 50], dtype=np.int32)),
                            (64, np.array([longest, 6, 700, 1025 + G, 0], dtype=np.int32))):
        max_sel = max(longest, 1100) + 3
        print(f"[case] token select {kind} longest={longest} budget={budget} per_sequence={budgets is not None}", flush=True)
        sel, ssl = gpu_select_tokens(scores, table, lens, G, budget, max_sel, budgets)
        with np.errstate(invalid="ignore"):
            ref_sel, ref_ssl, _ = O.select_tokens(scores, table, lens, G, budget, max_sel, budgets)
        assert np.array_equal(ssl, ref_ssl)
        assert np.array_equal(sel, ref_sel)
