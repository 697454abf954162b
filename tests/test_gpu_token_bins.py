"""Selection of up to 32768 tokens by bins of equal width (select_tokens.hpp, take_by_bins): ties inside the last bin, more of them than are
ranked, scores that nearly fill or leave the range in which bins are formed, NaNs that floating-point maxima lose, and shares of the sequence
at which another bound holds, against the oracle, bit for bit."""
import numpy as np
import pytest

from oracle import vegas_oracle as O
from tests.test_gpu_token_variant import gpu_select_tokens

pytestmark = pytest.mark.gpu
PAGE = 16


def make_scores(kind, n, rng):
    x = rng.standard_normal(n).astype(np.float32)
    if kind == "rounded":                  # a few hundred values: every bin holds ties
        return (np.round(x * 64) / 64).astype(np.float32)
    if kind == "cluster":                  # a sixteenth of the scores within one bin, at the selection's end
        x[::16] = 1.3 + 1e-5 * rng.random(x[::16].shape).astype(np.float32)
        return x
    if kind == "signs":                    # zeros of both signs around the end
        return np.where(rng.random(n) < 0.3, np.where(rng.random(n) < 0.5, np.float32(0), np.float32(-0.0)), -np.abs(x) + np.float32(x > 1.7)).astype(np.float32)
    if kind == "tiny":
        return (x * np.float32(1e-41)).astype(np.float32)
    if kind == "huge":
        return (x * np.float32(3e37)).astype(np.float32)
    if kind == "offset":                   # far from 0 for their spread
        return (np.float32(4096) + x).astype(np.float32)
    if kind == "nans":                     # quiet and signalling ones among the largest scores
        x[rng.integers(0, n, size=max(n // 50, 1))] = np.nan
        bits = x.view(np.uint32).copy()
        bits[rng.integers(0, n, size=max(n // 50, 1))] = 0x7FA00000
        x = bits.view(np.float32)
        x[rng.integers(0, n, size=3)] = 9.0
        return x
    if kind == "nearly_all_nan":
        x[rng.random(n) < 0.97] = np.nan
        return x
    return x


@pytest.mark.parametrize("longest,G", [(64, 1), (4097, 1), (4100, 5), (8193, 5), (16385, 1), (32768, 5)])
@pytest.mark.parametrize("kind", ["normal", "rounded", "cluster", "signs", "tiny", "huge", "offset", "nans", "nearly_all_nan"])
def test_token_bins(kind, longest, G):
    rng = np.random.default_rng(longest * 7 + len(kind))
    lens = np.array([longest, max(longest - 4095, G + 1), max(longest // 3, G + 1)], dtype=np.int32)
    B, mb = len(lens), (longest + PAGE - 1) // PAGE
    scores = np.stack([make_scores(kind, mb * PAGE, rng) for _ in range(B)])
    table = np.stack([rng.permutation(mb + 5)[:mb] for _ in range(B)]).astype(np.int32)
    for share in (16, 8, 4, 3):                # on both sides of the groups' sizes, a token more and a token fewer
        for extra in (-1, 0, 1):
            budgets = np.maximum((lens - G) // share + G + extra, 1).astype(np.int32)
            print(f"[case] token bins {kind} longest={longest} G={G} share={share} extra={extra}", flush=True)
            sel, ssl = gpu_select_tokens(scores, table, lens, G, 1, longest + 2, budgets)
            ref_sel, ref_ssl, _ = O.select_tokens(scores, table, lens, G, 1, longest + 2, budgets)
            assert np.array_equal(ssl, ref_ssl)
            assert np.array_equal(sel, ref_sel)


def crowded_scores(kind, n, rng):
    x = rng.standard_normal(n).astype(np.float32)
    if kind == "four_values":
        return rng.integers(0, 4, n).astype(np.float32)
    if kind == "hundred_values":           # bins hold them, the last one more than are ranked
        return rng.integers(0, 100, n).astype(np.float32)
    if kind == "mostly_zero":
        return np.where(rng.random(n) < 1 / 16, np.abs(x), 0).astype(np.float32)
    if kind == "half_zero":                # what occurs twice lies below the selection's end
        return np.where(rng.random(n) < 0.5, np.abs(x), 0).astype(np.float32)
    if kind == "one_far":
        x[n // 3] = 3e38
        return x
    if kind == "exponentials":
        return np.exp(5 * x).astype(np.float32)
    if kind == "masked_but_few":           # equal scores in the sample that are no scores
        x[rng.random(n) < 0.8] = -np.inf
        return x
    return x


@pytest.mark.parametrize("longest,G", [(20, 1), (64, 1), (1023, 5), (4096, 1), (8192, 5), (9000, 1), (32768, 5)])
@pytest.mark.parametrize("kind", ["four_values", "hundred_values", "mostly_zero", "half_zero", "one_far", "exponentials", "masked_but_few"])
def test_scores_that_bins_do_not_tell_apart(kind, longest, G):
    """The ways past the bins: few values seen in the sample, many scores of a wave in one bin, too many in the last one; and the tokens of a last
    bin that is not taken whole, kept by position, for shares on both sides of what bins are tried for."""
    rng = np.random.default_rng(longest * 11 + len(kind))
    lens = np.array([longest, max(longest - 4095, G + 1), max(longest // 3, G + 1)], dtype=np.int32)
    B, mb = len(lens), (longest + PAGE - 1) // PAGE
    scores = np.stack([crowded_scores(kind, mb * PAGE, rng) for _ in range(B)])
    table = np.stack([rng.permutation(mb + 5)[:mb] for _ in range(B)]).astype(np.int32)
    for share in (64, 16, 4, 2):
        for extra in (0, 1):
            budgets = np.maximum((lens - G) // share + G + extra, 1).astype(np.int32)
            print(f"[case] token selection {kind} longest={longest} G={G} share={share} extra={extra}", flush=True)
            sel, ssl = gpu_select_tokens(scores, table, lens, G, 1, longest + 2, budgets)
            ref_sel, ref_ssl, _ = O.select_tokens(scores, table, lens, G, 1, longest + 2, budgets)
            assert np.array_equal(ssl, ref_ssl)
            assert np.array_equal(sel, ref_sel)
