"""Verification with a local mask where eight waves take a workgroup's band and where four do (bands of 97 and 98 tokens, 256 and 264
workgroups), at the edges of a wave's tiles, behind the first batch of page ids, and at both ends of the one-workgroup rule, against the
float64 oracle."""
import pytest
import torch

from oracle import vegas_oracle as O
from paper_2602_07223_amd import binding as vb
from paper_2602_07223_amd import harness, synth
from tests import parity_util as U

pytestmark = pytest.mark.gpu

LENGTHS = {1: [1031], 2: [9000, 16400], 4: [0, 1, 130, 8301], 33: [7 * i + 1 for i in range(33)]}


ROWS = [(32, 8, 5), (16, 2, 5), (8, 8, 1)]
BANDS = [(1, 93), (1, 94), (1, 444), (1, 636), (2, 129), (2, 256), (2, 444), (2, 643), (4, 93), (4, 94), (4, 225),
         (4, 500), (4, 8300), (33, 20), (33, 120), (33, 250), (1, 137), (4, 130)]


@pytest.mark.parametrize("D", [128, 64])
@pytest.mark.parametrize("Hq,Hkv,G", ROWS, ids=["20_rows", "40_rows", "1_row"])
@pytest.mark.parametrize("batch,window", BANDS)
def test_band_by_four_and_by_eight_waves(batch, window, Hq, Hkv, G, D):
    lens = LENGTHS[batch]
    L = synth.make_random_case(seed=8100 + window + Hq + D, batch=batch, num_q_heads=Hq, num_kv_heads=Hkv, num_queries=G, seq_lens=lens,
                               head_dim=D, logit_std=2.0, value_std=1.0)
    print(f"[case] band batch={batch} W={window} Hq={Hq} Hkv={Hkv} G={G} D={D}", flush=True)
    dl = harness.DeviceLayer.upload(L)
    path = harness.VegasPath.for_layer(L, budget_tokens=64, collect_rows=vb.COLLECT_NONE, window=window)
    path.workspace.fill_(0xFF)                    # NaN partials where nothing was written
    path.out_verify.fill_(float("nan"))
    path.verify(dl)
    torch.cuda.synchronize()
    ref_out, _ = O.verify_attention(L.q_verify, L.k_cache, L.v_cache, L.block_table, L.seq_lens, L.softmax_scale, 0, window=window)
    U.check_out(f"band.{batch}.{window}.{Hq}.{D}", path.out_verify, ref_out, U.vmax_visible(L))


@pytest.mark.parametrize("over,waves", [
    (dict(window=93), 4), (dict(window=94), 8), (dict(window=400), 8), (dict(batch=33, window=128), 4), (dict(batch=32, window=128), 8),
    (dict(batch=32, window=256), 4), (dict(batch=16, window=400, num_queries=10), 8)])
def test_waves_of_a_band(over, waves):
    args = dict(batch=1, num_q_heads=32, num_kv_heads=8, num_queries=5, max_blocks=512, max_sel_blocks=8, max_seq_len=8192, num_pages=4096,
                softmax_scale=0.1, collect_rows=vb.COLLECT_NONE)
    assert vb.vegas_debug_verify_waves(vb.make_desc(**{**args, **over})) == waves


@pytest.mark.parametrize("Hq,Hkv,G", ROWS, ids=["20_rows", "40_rows", "1_row"])
@pytest.mark.parametrize("D", [128, 64])
def test_bands_above_are_taken_by_four_and_by_eight_waves(D, Hq, Hkv, G):
    seen = {}
    for batch, window in BANDS:
        longest = max(LENGTHS[batch])
        desc = vb.make_desc(batch=batch, num_q_heads=Hq, num_kv_heads=Hkv, num_queries=G, max_blocks=-(-longest // 16), max_sel_blocks=8,
                            max_seq_len=longest, num_pages=4096, softmax_scale=0.1, collect_rows=vb.COLLECT_NONE, head_dim=D, window=window)
        seen.setdefault(vb.vegas_debug_verify_waves(desc), []).append((batch, window))
    assert sorted(seen) == [4, 8] and min(map(len, seen.values())) >= 3, seen
