"""Merge and page scores of planned batches on both sides of the rule that tells small calls from others (plan_rules.hpp,
planned_merge_is_small): row counts that are and are not multiples of four and of eight, sequences of one chunk and of more than
eight, empty ones, both collection modes and token sums, against the oracle."""
import pytest
import torch

from oracle import vegas_oracle as O
from paper_2602_07223_amd import binding as vb
from paper_2602_07223_amd import harness, synth
from tests import parity_util as U

pytestmark = pytest.mark.gpu


def lengths(batch):
    return [(7 + 331 * i) % 700 + 1 if i % 7 else 0 for i in range(batch - 2)] + [33 * 16 + 1, 1500]


def smallest_large(heads, rows, D):
    return -(-1024 * 256 // (heads * rows * D))


# KV heads, group, queries; rows 4, 12, 20, 21, 35, 36, 42, 77
@pytest.mark.parametrize("D", [128, 64])
@pytest.mark.parametrize("heads,group,queries", [(8, 4, 1), (8, 4, 3), (8, 4, 5), (8, 7, 3), (4, 7, 5), (4, 6, 6), (4, 6, 7), (2, 7, 11)])
def test_rows_on_both_sides(heads, group, queries, D):
    edge = smallest_large(heads, group * queries, D)
    for batch in {min(max(edge - 1, 3), 64), min(max(edge, 3), 64)}:
        lens = lengths(batch)
        L = synth.make_random_case(seed=53000 + 10 * batch + queries, batch=batch, num_q_heads=heads * group, num_kv_heads=heads,
                                   num_queries=queries, seq_lens=lens, head_dim=D, logit_std=2.0, value_std=1.0, outliers=2,
                                   outlier_logit=25.0)
        print(f"[case] planned rows, {heads} heads, {group * queries} rows, D={D}, {batch} sequences", flush=True)
        dl = harness.DeviceLayer.upload(L)
        for collect in (vb.COLLECT_ALL_ROWS, vb.COLLECT_FIRST_LAST):
            ref_out, ref_scores = O.verify_attention(L.q_verify, L.k_cache, L.v_cache, L.block_table, L.seq_lens,
                                                     L.softmax_scale, collect)
            path = harness.VegasPath.for_layer(L, budget_tokens=256, collect_rows=collect)
            path.workspace.fill_(0xFF)               # NaN where nothing was written
            path.out_verify.fill_(float("nan"))
            path.block_scores.fill_(float("nan"))
            path.verify(dl)
            torch.cuda.synchronize()
            U.check_out(f"planned_rows.{batch}.{collect}", path.out_verify, ref_out, U.vmax_visible(L))
            U.check_scores(f"planned_rows.{batch}.{collect}", path.block_scores, ref_scores)
        path = harness.VegasPath.for_layer(L, budget_tokens=256, token_granular=True)
        path.workspace.fill_(0xFF)
        path.out_verify.fill_(float("nan"))
        path.verify(dl)
        torch.cuda.synchronize()
        U.check_out(f"planned_rows.{batch}.tokens", path.out_verify, ref_out, U.vmax_visible(L))
