"""Balanced chunking's merge and page scores over every number of chunks the merge distinguishes: a batch in which one
sequence gets 1, 4, 5, 8, 9, 16, 17, 31 or 57 chunks (the shortest chunk is 128 tokens) and the others one each, with
and without collection, in calls of few rows and (57 chunks) of many, against the oracle."""
import pytest
import torch

from oracle import vegas_oracle as O
from paper_2602_07223_amd import binding as vb
from paper_2602_07223_amd import harness, synth
from tests import parity_util as U
from tests.test_batch_plan import plans, program


def batch_of(chunks):
    """KV heads and lengths: 8 heads leave 32 workgroups per head, which 57 chunks do not fit; 4 leave 64."""
    return (8, [128 * chunks - 3, 16]) if chunks < 32 else (4, [128 * chunks - 3] + [16] * 3)


MANY = (2, [128 * 57 - 3] + [16] * 25)       # 26 sequences x 80 rows: a merge of many rows

CHUNKS = [1, 4, 5, 8, 9, 16, 17, 31, 57]


def test_the_batches_have_so_many_chunks(tmp_path_factory):
    calls = [(heads, 128, rows, c, max(lens), lens) for rows in (20, 40) for c in (0, 1)
             for heads, lens in [batch_of(n) for n in CHUNKS] + [MANY]]
    for c, d in zip(calls, plans(program(tmp_path_factory), calls)):
        assert not d["shares"] and d["columns"][0][1] == -(-c[5][0] // 128), c


@pytest.mark.gpu
@pytest.mark.parametrize("Hq", [32, 64], ids=["20_rows", "40_rows"])
@pytest.mark.parametrize("chunks", CHUNKS + ["many_rows"])
def test_planned_sequences_with_every_chunk_count(chunks, Hq):
    heads, lens = MANY if chunks == "many_rows" else batch_of(chunks)
    L = synth.make_random_case(seed=41000 + lens[0] // 128 + Hq, batch=len(lens), num_q_heads=Hq // 8 * heads, num_kv_heads=heads, num_queries=5,
                               seq_lens=lens, logit_std=2.0, value_std=1.0, outliers=2, outlier_logit=25.0)
    print(f"[case] planned merge, {chunks} chunks, Hq={Hq}", flush=True)
    dl = harness.DeviceLayer.upload(L)
    ref_out, ref_scores = O.verify_attention(L.q_verify, L.k_cache, L.v_cache, L.block_table, L.seq_lens,
                                             L.softmax_scale, vb.COLLECT_ALL_ROWS)
    for collect in (vb.COLLECT_ALL_ROWS, vb.COLLECT_NONE):
        path = harness.VegasPath.for_layer(L, budget_tokens=256, collect_rows=collect)
        path.workspace.fill_(0xFF)                # NaN partials where nothing was written
        path.out_verify.fill_(float("nan"))
        path.block_scores.fill_(float("nan"))
        path.verify(dl)
        torch.cuda.synchronize()
        U.check_out(f"planned.{chunks}.{collect}", path.out_verify, ref_out, U.vmax_visible(L))
        if collect:
            U.check_scores(f"planned.{chunks}", path.block_scores, ref_scores)


@pytest.mark.gpu
@pytest.mark.parametrize("collect", [vb.COLLECT_NONE, vb.COLLECT_ALL_ROWS], ids=["none", "all_rows"])
@pytest.mark.parametrize("lens", [[4096, 0], [0, 4096, 0], [0, 0]], ids=str)
def test_empty_members_of_a_plan_that_fills_every_slot(lens, collect):
    """32 chunks of 128 tokens are all the slots a head has (8 KV heads, 256 compute units): an empty sequence owns none,
    and its rows are zeros whatever the workspace holds."""
    L = synth.make_random_case(seed=41200 + len(lens), batch=len(lens), num_q_heads=64, num_kv_heads=8, num_queries=5,
                               seq_lens=lens, logit_std=2.0, value_std=1.0)
    print(f"[case] planned merge, lengths {lens}, collect={collect}", flush=True)
    dl = harness.DeviceLayer.upload(L)
    path = harness.VegasPath.for_layer(L, budget_tokens=256, collect_rows=collect)
    path.workspace.fill_(0xFF)
    path.out_verify.fill_(float("nan"))
    path.verify(dl)
    torch.cuda.synchronize()
    ref_out, _ = O.verify_attention(L.q_verify, L.k_cache, L.v_cache, L.block_table, L.seq_lens, L.softmax_scale,
                                    vb.COLLECT_ALL_ROWS)
    U.check_out(f"planned.empty.{lens}.{collect}", path.out_verify, ref_out, U.vmax_visible(L))
    for b, n in enumerate(lens):
        assert n or not path.out_verify[b].any()
