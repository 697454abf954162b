"""Merge and page scores of a planned batch (balanced chunking) by row counts: page values read as runs of 16-byte quads, in one
batch per workgroup or several, or row by row where the collected rows are no multiple of four; groups of 32 pages that end
anywhere; both collection modes; against the oracle."""
import pytest
import torch

from oracle import vegas_oracle as O
from paper_2602_07223_amd import binding as vb
from paper_2602_07223_amd import harness, synth
from tests import parity_util as U

pytestmark = pytest.mark.gpu

# KV heads, group, queries: 4, 6, 12, 20, 32, 40, 48 (two batches of quads) and 96 rows; 3, 8, 16 and 1 KV heads
SHAPES = [(8, 4, 1), (3, 2, 3), (8, 4, 3), (16, 4, 5), (8, 4, 8), (8, 8, 5), (8, 8, 6), (8, 8, 12), (1, 12, 4)]


@pytest.mark.parametrize("D", [128, 64])
@pytest.mark.parametrize("Hkv,group,queries", SHAPES)
def test_planned_scores_by_row_count(Hkv, group, queries, D):
    lens = [33 * 16 + 1, 5, 0, 32 * 16, 1203, 31 * 16 - 2]
    L = synth.make_random_case(seed=52000 + 100 * Hkv + group * queries, batch=len(lens), num_q_heads=Hkv * group,
                               num_kv_heads=Hkv, num_queries=queries, seq_lens=lens, head_dim=D, logit_std=2.0, value_std=1.0,
                               outliers=2, outlier_logit=25.0)
    print(f"[case] planned scores, {Hkv} heads, {group * queries} rows, D={D}", flush=True)
    dl = harness.DeviceLayer.upload(L)
    for collect in (vb.COLLECT_ALL_ROWS, vb.COLLECT_FIRST_LAST):
        ref_out, ref_scores = O.verify_attention(L.q_verify, L.k_cache, L.v_cache, L.block_table, L.seq_lens, L.softmax_scale,
                                                 collect)
        path = harness.VegasPath.for_layer(L, budget_tokens=256, collect_rows=collect)
        path.workspace.fill_(0xFF)               # NaN where nothing was written
        path.out_verify.fill_(float("nan"))
        path.block_scores.fill_(float("nan"))
        path.verify(dl)
        torch.cuda.synchronize()
        U.check_out(f"planned_scores.{collect}", path.out_verify, ref_out, U.vmax_visible(L))
        U.check_scores(f"planned_scores.{collect}", path.block_scores, ref_scores)


@pytest.mark.parametrize("D", [128, 64])
@pytest.mark.parametrize("Hkv,group", [(64, 1), (40, 2), (29, 3), (16, 4), (17, 5)])
def test_planned_scores_of_short_runs(Hkv, group, D):
    """Large enough for pages scored by quads, with 4, 8, 12, 16 and 20 rows a head: runs of half a request to two of them, and just above, in groups of
    heads that the last one fills or not."""
    lens = [33 * 16 + 1, 5, 0, 32 * 16, 603, 31 * 16 - 2] * 4
    assert len(lens) * Hkv * group * 4 * D >= 1024 * 256
    L = synth.make_random_case(seed=53000 + Hkv + D, batch=len(lens), num_q_heads=Hkv * group, num_kv_heads=Hkv, num_queries=4, seq_lens=lens,
                               head_dim=D, logit_std=2.0, value_std=1.0)
    print(f"[case] planned scores, {Hkv} heads, {4 * group} rows, D={D}", flush=True)
    dl = harness.DeviceLayer.upload(L)
    ref_out, ref_scores = O.verify_attention(L.q_verify, L.k_cache, L.v_cache, L.block_table, L.seq_lens, L.softmax_scale, vb.COLLECT_ALL_ROWS)
    path = harness.VegasPath.for_layer(L, budget_tokens=256, collect_rows=vb.COLLECT_ALL_ROWS)
    path.workspace.fill_(0xFF)                   # NaN where nothing was written
    path.out_verify.fill_(float("nan"))
    path.block_scores.fill_(float("nan"))
    path.verify(dl)
    torch.cuda.synchronize()
    U.check_out(f"planned_runs.{Hkv}", path.out_verify, ref_out, U.vmax_visible(L))
    U.check_scores(f"planned_runs.{Hkv}", path.block_scores, ref_scores)
