"""Verification of more than 32 rows per KV head where its kernel can go wrong: chunks of less than a tile to more than a
wave parks or its ring holds, row counts at the edges of the two row blocks and of a second workgroup, both collection
modes and none, against the float64 oracle."""
import numpy as np
import pytest
import torch

from oracle import vegas_oracle as O
from paper_2602_07223_amd import binding as vb
from paper_2602_07223_amd import harness, synth
from tests import parity_util as U

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("D", [128, 64])
@pytest.mark.parametrize("Hq,Hkv,G", [(33, 1, 1), (16, 2, 5), (64, 4, 4), (26, 2, 5), (64, 2, 4)],
                         ids=["33_rows", "40_rows", "64_rows", "65_rows", "128_rows"])
@pytest.mark.parametrize("n,chunk", [(1, 0), (31, 32), (97, 0), (129, 128), (1025, 416), (4133, 4160), (9000, 9024)])
def test_chunks_of_every_length(n, chunk, Hq, Hkv, G, D):
    lens = [n] if chunk else [n, max(n - 17, 0), 2 * n]          # (no chunk length: also the balanced plan)
    L = synth.make_random_case(seed=6100 + n + Hq + D, batch=len(lens), num_q_heads=Hq, num_kv_heads=Hkv, num_queries=G,
                               seq_lens=lens, head_dim=D, logit_std=2.0, value_std=1.0, outliers=min(2, n // 2),
                               outlier_logit=25.0)
    print(f"[case] wide rows n={n} chunk={chunk} Hq={Hq} Hkv={Hkv} G={G} D={D}", flush=True)
    dl = harness.DeviceLayer.upload(L)
    for collect in (vb.COLLECT_ALL_ROWS, vb.COLLECT_FIRST_LAST, vb.COLLECT_NONE):
        path = harness.VegasPath.for_layer(L, budget_tokens=256, collect_rows=collect, verify_chunk=chunk)
        path.workspace.fill_(0xFF)                # NaN partials where nothing was written
        path.out_verify.fill_(float("nan"))
        path.block_scores.fill_(float("nan"))
        path.verify(dl)
        torch.cuda.synchronize()
        ref_out, ref_scores = O.verify_attention(L.q_verify, L.k_cache, L.v_cache, L.block_table, L.seq_lens,
                                                 L.softmax_scale, collect or vb.COLLECT_ALL_ROWS)
        U.check_out(f"wide.{n}.{Hq}.{collect}", path.out_verify, ref_out, U.vmax_visible(L))
        if collect:
            U.check_scores(f"wide.{n}.{Hq}.{collect}", path.block_scores, ref_scores)


@pytest.mark.parametrize("D", [128, 64])
@pytest.mark.parametrize("Hq,Hkv,G", [(26, 2, 5), (32, 4, 10), (64, 4, 8)], ids=["65_rows", "80_rows", "128_rows"])
@pytest.mark.parametrize("lens", [[1025], [4133], [30011], [517, 0, 2049], [97, 0, 16, 1300, 640, 33, 1, 900]], ids=str)
def test_more_than_64_rows_on_both_sides_of_the_sibling_rule(lens, Hq, Hkv, G, D):
    """Small calls run as 32-row siblings, larger ones and batches of eight that collect as 64-row workgroups."""
    L = synth.make_random_case(seed=6500 + sum(lens) + Hq + D, batch=len(lens), num_q_heads=Hq, num_kv_heads=Hkv, num_queries=G,
                               seq_lens=lens, head_dim=D, logit_std=2.0, value_std=1.0, outliers=2, outlier_logit=25.0)
    print(f"[case] siblings lens={lens} Hq={Hq} Hkv={Hkv} G={G} D={D}", flush=True)
    dl = harness.DeviceLayer.upload(L)
    for collect in (vb.COLLECT_ALL_ROWS, vb.COLLECT_FIRST_LAST, vb.COLLECT_NONE):
        path = harness.VegasPath.for_layer(L, budget_tokens=256, collect_rows=collect)
        path.workspace.fill_(0xFF)
        path.out_verify.fill_(float("nan"))
        path.block_scores.fill_(float("nan"))
        path.verify(dl)
        torch.cuda.synchronize()
        ref_out, ref_scores = O.verify_attention(L.q_verify, L.k_cache, L.v_cache, L.block_table, L.seq_lens,
                                                 L.softmax_scale, collect or vb.COLLECT_ALL_ROWS)
        U.check_out(f"sib.{sum(lens)}.{Hq}.{collect}", path.out_verify, ref_out, U.vmax_visible(L))
        if collect:
            U.check_scores(f"sib.{sum(lens)}.{Hq}.{collect}", path.block_scores, ref_scores)


@pytest.mark.parametrize("D", [128, 64])
@pytest.mark.parametrize("Hq,Hkv,G", [(28, 4, 7), (37, 1, 1), (61, 1, 1)], ids=["49_rows", "37_rows", "61_rows"])
def test_odd_numbers_of_collected_rows(Hq, Hkv, G, D):
    """Row counts with which an odd number of parked tiles would leave waves 1 and 3 between two 16-byte pieces of the LDS:
    one chunk long enough that every wave writes out what it has parked more than once."""
    L = synth.make_random_case(seed=6200 + Hq + D, batch=1, num_q_heads=Hq, num_kv_heads=Hkv, num_queries=G,
                               seq_lens=[4133], head_dim=D, logit_std=2.0, value_std=1.0, outliers=2, outlier_logit=25.0)
    print(f"[case] odd collected rows Hq={Hq} Hkv={Hkv} G={G} D={D}", flush=True)
    dl = harness.DeviceLayer.upload(L)
    path = harness.VegasPath.for_layer(L, budget_tokens=256, verify_chunk=4160)
    path.workspace.fill_(0xFF)
    path.out_verify.fill_(float("nan"))
    path.block_scores.fill_(float("nan"))
    path.verify(dl)
    torch.cuda.synchronize()
    ref_out, ref_scores = O.verify_attention(L.q_verify, L.k_cache, L.v_cache, L.block_table, L.seq_lens, L.softmax_scale,
                                             vb.COLLECT_ALL_ROWS)
    U.check_out(f"odd.{Hq}.{D}", path.out_verify, ref_out, U.vmax_visible(L))
    U.check_scores(f"odd.{Hq}.{D}", path.block_scores, ref_scores)


@pytest.mark.parametrize("Hq,Hkv,D", [(16, 2, 64), (8, 2, 128), (96, 96, 128)], ids=["40_rows", "20_rows", "96_columns"])
@pytest.mark.parametrize("window", [1, 128, 411, 412, 507, 508, 539, 540, 1083, 1084, 2171, 2172, 9600])
def test_local_mask_on_both_sides_of_the_one_workgroup_rule(window, Hq, Hkv, D):
    """The rule changes at a band of 416 tokens, or of a chunk where that is longer (256 compute units: 512 tokens with
    40 rows, 2176 with 96 columns); 9000 tokens make a workgroup begin behind its first batch of page ids.
    A window longer than the context is a band of the context: 400 tokens are left to one workgroup."""
    lens = [9000, 0, 1, 4100] if Hkv == 2 else [4500]
    if window > 9000:
        lens = [400, 0, 1, 137] if Hkv == 2 else [400]
    L = synth.make_random_case(seed=6300 + window + Hq, batch=len(lens), num_q_heads=Hq, num_kv_heads=Hkv, num_queries=5,
                               seq_lens=lens, head_dim=D, logit_std=1.5, value_std=1.0)
    print(f"[case] local mask W={window} Hq={Hq} Hkv={Hkv} D={D}", flush=True)
    dl = harness.DeviceLayer.upload(L)
    path = harness.VegasPath.for_layer(L, budget_tokens=64, collect_rows=vb.COLLECT_NONE, window=window)
    path.workspace.fill_(0xFF)
    path.out_verify.fill_(float("nan"))
    path.verify(dl)
    torch.cuda.synchronize()
    ref_out, _ = O.verify_attention(L.q_verify, L.k_cache, L.v_cache, L.block_table, L.seq_lens, L.softmax_scale, 0,
                                    window=window)
    U.check_out(f"local.{window}.{Hq}", path.out_verify, ref_out, U.vmax_visible(L))


@pytest.mark.parametrize("D", [128, 64])
@pytest.mark.parametrize("Hq,G", [(32, 5), (32, 10)], ids=["40_rows", "80_rows"])
def test_one_long_sequence_among_more_than_64(Hq, G, D):
    """No plan (more than 64 sequences): the long one is cut into chunks that the short ones have nothing in."""
    lens = [int(n) for n in np.random.default_rng(65 + G).integers(0, 40, size=65)]
    lens[21] = 8209
    L = synth.make_random_case(seed=6700 + G + D, batch=65, num_q_heads=Hq, num_kv_heads=4, num_queries=G, seq_lens=lens,
                               head_dim=D, logit_std=2.0, value_std=1.0, outliers=1, outlier_logit=25.0)
    print(f"[case] one long among 65 Hq={Hq} G={G} D={D}", flush=True)
    dl = harness.DeviceLayer.upload(L)
    for collect in (vb.COLLECT_ALL_ROWS, vb.COLLECT_NONE):
        path = harness.VegasPath.for_layer(L, budget_tokens=256, collect_rows=collect)
        path.workspace.fill_(0xFF)
        path.out_verify.fill_(float("nan"))
        path.block_scores.fill_(float("nan"))
        path.verify(dl)
        torch.cuda.synchronize()
        ref_out, ref_scores = O.verify_attention(L.q_verify, L.k_cache, L.v_cache, L.block_table, L.seq_lens,
                                                 L.softmax_scale, vb.COLLECT_ALL_ROWS)
        U.check_out(f"one_long.{Hq}.{G}.{collect}", path.out_verify, ref_out, U.vmax_visible(L))
        if collect:
            U.check_scores(f"one_long.{Hq}.{G}.{collect}", path.block_scores, ref_scores)


def folded_call(G, chunk):
    max_len = chunk * 65537
    L = synth.make_random_case(seed=6400 + G, batch=2, num_q_heads=11, num_kv_heads=1, num_queries=G, seq_lens=[200, 77],
                               head_dim=64, logit_std=1.5, value_std=1.0)
    dl = harness.DeviceLayer.upload(L)
    blocks = max_len // 16
    table = torch.zeros((2, blocks), dtype=torch.int32, device=dl.block_table.device)
    table[:, :dl.block_table.shape[1]] = dl.block_table
    dl.block_table = table
    path = harness.VegasPath(batch=2, num_q_heads=11, num_kv_heads=1, num_queries=G, max_blocks=blocks, max_seq_len=max_len,
                             num_pages=L.num_pages, budget_tokens=64, softmax_scale=L.softmax_scale, head_dim=64,
                             verify_chunk=chunk)
    return L, dl, path


def test_more_chunks_than_a_grid_dimension_holds():
    """max_seq_len of 65537 chunks of 64 tokens (the lengths themselves are short), 33 rows: the grid is folded."""
    L, dl, path = folded_call(3, 64)
    print("[case] folded grid", flush=True)
    path.verify(dl)
    torch.cuda.synchronize()
    ref_out, ref_scores = O.verify_attention(L.q_verify, L.k_cache, L.v_cache, L.block_table, L.seq_lens, L.softmax_scale,
                                             vb.COLLECT_ALL_ROWS)
    U.check_out("folded", path.out_verify, ref_out, U.vmax_visible(L))
    U.check_scores("folded", path.block_scores[:, :ref_scores.shape[1]], ref_scores)
    assert not path.block_scores[:, ref_scores.shape[1]:].any()


@pytest.mark.parametrize("G,chunk", [(3, 32), (6, 64)], ids=["33_rows_odd_chunk", "66_rows"])
def test_too_many_chunks_are_refused(G, chunk):
    _, dl, path = folded_call(G, chunk)
    with pytest.raises(vb.VegasError, match="not supported"):
        path.verify(dl)
