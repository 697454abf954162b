"""Balanced chunking by shares: batches whose sequences are laid end to end and cut every S units of 128 tokens, against the
oracle -- a sequence that is many whole shares, one that begins or ends exactly at a cut, several sequences inside one share,
empty ones between them, last pieces of one token -- in both verification kernels, for every collection mode."""
import numpy as np
import pytest
import torch

from oracle import vegas_oracle as O
from paper_2602_07223_amd import binding as vb
from paper_2602_07223_amd import harness, synth
from tests import parity_util as U

pytestmark = pytest.mark.gpu
UNIT, COST = 128, 3


def cuts(lens, J):
    """(S, taken): the share length in units, and whether the plan is by shares (J workgroups per KV head)."""
    nu = [-(-n // UNIT) for n in lens]
    live = sum(1 for x in nu if x)
    longest = next(c for c in range(1, max(nu) + 1) if c == max(nu) or sum(-(-x // c) for x in nu) <= J)
    priced = sum(nu) + COST * (live - 1)
    return -(-priced // J), live <= J and 10 * J * longest > 11 * priced + 8 * live and longest >= -(-priced // J) + 4


# 64 KV heads leave 4 workgroups per head on 256 compute units, 32 leave 8
BATCHES = [
    (64, [3840, 1, 128, 77]),                    # many whole shares; a share with three sequences
    (64, [1, 3840, 5, 2]),                       # the long one in the middle of a share
    (64, [0, 3841, 640, 0, 129, 64]),            # empty ones; a last unit of one token
    (64, [14 * 128, 30 * 128, 128, 128]),        # ends at a cut
    (64, [10 * 128, 30 * 128, 100, 5]),          # begins at a cut
    (32, [26 * 128, 17, 26 * 128 + 1, 300, 128, 1, 640]),
    (32, [300, 0, 50 * 128, 3 * 128, 1, 12 * 128 - 1, 2 * 128, 130]),
]


@pytest.mark.parametrize("group,queries,D", [(2, 5, 64), (2, 5, 128), (7, 5, 64), (7, 5, 128)],
                         ids=["10_rows_64", "10_rows_128", "35_rows_64", "35_rows_128"])
@pytest.mark.parametrize("batch", range(len(BATCHES)))
def test_batches_cut_into_shares(batch, group, queries, D):
    Hkv, lens = BATCHES[batch]
    J = torch.cuda.get_device_properties(0).multi_processor_count // Hkv
    S, taken = cuts(lens, J)
    assert taken, (S, lens)
    L = synth.make_random_case(seed=47000 + 10 * batch + group, batch=len(lens), num_q_heads=Hkv * group, num_kv_heads=Hkv,
                               num_queries=queries, seq_lens=lens, head_dim=D, logit_std=2.0, value_std=1.0, outliers=2,
                               outlier_logit=25.0)
    print(f"[case] shares of {S} units, batch {batch}, {group * queries} rows, D={D}", flush=True)
    dl = harness.DeviceLayer.upload(L)
    ref = {}
    for collect in (vb.COLLECT_ALL_ROWS, vb.COLLECT_FIRST_LAST):
        ref[collect] = O.verify_attention(L.q_verify, L.k_cache, L.v_cache, L.block_table, L.seq_lens, L.softmax_scale, collect)
    for collect in (vb.COLLECT_NONE, vb.COLLECT_ALL_ROWS, vb.COLLECT_FIRST_LAST):
        path = harness.VegasPath.for_layer(L, budget_tokens=256, collect_rows=collect)
        path.workspace.fill_(0xFF)               # NaN partials where nothing was written
        path.out_verify.fill_(float("nan"))
        path.block_scores.fill_(float("nan"))
        path.verify(dl)
        torch.cuda.synchronize()
        ref_out, ref_scores = ref[collect or vb.COLLECT_ALL_ROWS]
        U.check_out(f"shares.{batch}.{collect}", path.out_verify, ref_out, U.vmax_visible(L))
        if collect:
            U.check_scores(f"shares.{batch}.{collect}", path.block_scores, ref_scores)
        for b, n in enumerate(lens):
            assert n or not path.out_verify[b].any()
