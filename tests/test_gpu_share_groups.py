"""Batches cut into shares where consecutive workgroups of a head start on 2, 4 or 32 shader engines, so that the first wave's
workgroups are reversed in groups (vegas_common.hpp, balanced_slot; 16, 8 and 5 KV heads: the last group of 51 workgroups is
not whole), in both verification kernels, against the oracle.  (Groups of one: test_gpu_batch_shares.py; every group on the CPU:
test_batch_plan.py.)"""
import pytest
import torch

from oracle import vegas_oracle as O
from paper_2602_07223_amd import binding as vb
from paper_2602_07223_amd import harness, synth
from tests import parity_util as U
from tests.test_batch_plan import UNIT, plans, program, wanted

# KV heads, query heads per KV head, units of 128 tokens per sequence
BATCHES = [
    (16, 2, [8] * 9),
    (16, 7, [13, 13, 13, 25, 13, 13, 14, 13]),
    (8, 2, [10, 8, 8, 8, 10, 8, 8, 15, 10, 8, 10, 8, 8, 8, 8, 8]),
    (8, 7, [12, 12, 14, 13, 12, 12, 13, 12, 12, 13, 12, 12, 14, 12, 23, 13]),
    (5, 2, [17, 19, 17, 26, 18, 19, 17, 18, 18, 17, 17, 17, 17, 17, 18, 17, 17]),
    (5, 7, [31, 49, 31, 32, 31, 31, 31, 31, 31, 32, 32, 31, 31, 31, 32, 32, 31]),
]
QUERIES = 5


def lengths(units):
    return [u * UNIT - 37 * i % UNIT for i, u in enumerate(units)]       # last units of any length


def planned(batch, D):
    heads, group, units = BATCHES[batch]
    return heads, D, group * QUERIES, 1, max(lengths(units)), lengths(units)


def test_these_batches_are_cut_into_shares(tmp_path_factory):
    calls = [planned(b, D) for b in range(len(BATCHES)) for D in (128, 64)]
    for c, d in zip(calls, plans(program(tmp_path_factory), calls)):
        assert wanted(c, d) and d["shares"] and d["group"] == {16: 2, 8: 4, 5: 32}[c[0]], c


@pytest.mark.gpu
@pytest.mark.parametrize("D", [128, 64])
@pytest.mark.parametrize("batch", range(len(BATCHES)))
def test_reversed_groups(batch, D):
    heads, group, units = BATCHES[batch]
    lens = lengths(units)
    L = synth.make_random_case(seed=54000 + 10 * batch + D, batch=len(lens), num_q_heads=heads * group, num_kv_heads=heads,
                               num_queries=QUERIES, seq_lens=lens, head_dim=D, logit_std=2.0, value_std=1.0, outliers=2,
                               outlier_logit=25.0)
    print(f"[case] share groups, batch {batch}, {heads} heads, {group * QUERIES} rows, D={D}", flush=True)
    dl = harness.DeviceLayer.upload(L)
    for collect in (vb.COLLECT_ALL_ROWS, vb.COLLECT_FIRST_LAST, vb.COLLECT_NONE):
        ref_out, ref_scores = O.verify_attention(L.q_verify, L.k_cache, L.v_cache, L.block_table, L.seq_lens, L.softmax_scale,
                                                 collect or vb.COLLECT_ALL_ROWS)
        path = harness.VegasPath.for_layer(L, budget_tokens=256, collect_rows=collect)
        path.workspace.fill_(0xFF)               # NaN partials where nothing was written
        path.out_verify.fill_(float("nan"))
        path.block_scores.fill_(float("nan"))
        path.verify(dl)
        torch.cuda.synchronize()
        U.check_out(f"share_groups.{batch}.{collect}", path.out_verify, ref_out, U.vmax_visible(L))
        if collect:
            U.check_scores(f"share_groups.{batch}.{collect}", path.block_scores, ref_scores)
