"""Page scores around what finalize_is_wide decides (five rounds of (max, sum) pairs in flight instead of three: up to 320 collected
rows in up to 32 chunks that the host cuts, four sequences or more than 16 chunks), below and beyond that many rows, for up to 16, 32, 64 and more chunks, for
one sequence, more than a plan takes (64) and several in chunks of the caller's, against the oracle."""
import pytest
import torch

from oracle import vegas_oracle as O
from paper_2602_07223_amd import harness, synth
from tests import parity_util as U

# KV heads, query heads per KV head, queries: 208, 210, 216, 256, 320 and 330 rows
SHAPES = [(8, 2, 13), (5, 7, 6), (8, 3, 9), (16, 2, 8), (8, 8, 5), (10, 3, 11)]
# tokens, and in chunks of how many (0: the plan's own)
LENGTHS = [(2000, 128), (4003, 128), (8192, 128), (9001, 128), (6000, 0)]


@pytest.mark.gpu
@pytest.mark.parametrize("D", [128, 64])
@pytest.mark.parametrize("shape", range(len(SHAPES)))
def test_page_scores(shape, D):
    heads, group, queries = SHAPES[shape]
    for tokens, chunk in LENGTHS:
        print(f"[case] wide finalize, {heads * group * queries} rows, D={D}, {tokens} tokens in chunks of {chunk}", flush=True)
        L = synth.make_random_case(seed=61000 + 100 * shape + tokens % 97 + D, batch=1, num_q_heads=heads * group, num_kv_heads=heads,
                                   num_queries=queries, seq_lens=[tokens], head_dim=D, logit_std=2.0, value_std=1.0, outliers=2,
                                   outlier_logit=25.0)
        ref_out, ref_scores = O.verify_attention(L.q_verify, L.k_cache, L.v_cache, L.block_table, L.seq_lens, L.softmax_scale)
        path = harness.VegasPath.for_layer(L, budget_tokens=256, verify_chunk=chunk)
        path.workspace.fill_(0xFF)               # NaN partials where nothing was written
        path.out_verify.fill_(float("nan"))
        path.block_scores.fill_(float("nan"))
        path.verify(harness.DeviceLayer.upload(L))
        torch.cuda.synchronize()
        U.check_out(f"wide_finalize.{shape}.{tokens}", path.out_verify, ref_out, U.vmax_visible(L))
        U.check_scores(f"wide_finalize.{shape}.{tokens}", path.block_scores, ref_scores)


# sequences and their lengths (ragged, an empty one and one shorter than the queries among them), chunk of the caller's
BATCHES = [([(37 * b * b) % 400 for b in range(65)], 0), ([3, 0, 1500, 2000, 129], 128), ([2049, 700, 4100], 64)]


@pytest.mark.gpu
@pytest.mark.parametrize("D", [128, 64])
@pytest.mark.parametrize("lens,chunk", BATCHES, ids=["65_sequences", "chunks_of_128", "chunks_of_64"])
def test_page_scores_of_batches(lens, chunk, D):
    for heads, group, queries in ((8, 4, 8), (8, 8, 5), (5, 7, 6)):
        print(f"[case] wide finalize, {heads * group * queries} rows, D={D}, {len(lens)} sequences in chunks of {chunk}", flush=True)
        L = synth.make_random_case(seed=62000 + heads * group + len(lens) + D, batch=len(lens), num_q_heads=heads * group, num_kv_heads=heads,
                                   num_queries=queries, seq_lens=lens, head_dim=D, logit_std=2.0, value_std=1.0, outliers=2, outlier_logit=25.0)
        ref_out, ref_scores = O.verify_attention(L.q_verify, L.k_cache, L.v_cache, L.block_table, L.seq_lens, L.softmax_scale)
        path = harness.VegasPath.for_layer(L, budget_tokens=256, verify_chunk=chunk)
        path.workspace.fill_(0xFF)               # NaN partials where nothing was written
        path.out_verify.fill_(float("nan"))
        path.block_scores.fill_(float("nan"))
        path.verify(harness.DeviceLayer.upload(L))
        torch.cuda.synchronize()
        U.check_out(f"wide_finalize.batch.{len(lens)}.{chunk}", path.out_verify, ref_out, U.vmax_visible(L))
        U.check_scores(f"wide_finalize.batch.{len(lens)}.{chunk}", path.block_scores, ref_scores)
