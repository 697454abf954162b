"""Page scores of chunks that the host cuts (score_pages): a wave has a quarter of 16, 32 or 64 chunks, or of every 32 where there are more, and
a lane a row of 64; chunk counts at the ends of quarters and windows, rows at the ends of rounds, lengths under a looser bound, both
collection modes, against the oracle."""
import pytest
import torch

from oracle import vegas_oracle as O
from paper_2602_07223_amd import binding as vb
from paper_2602_07223_amd import harness, synth
from tests import parity_util as U

pytestmark = pytest.mark.gpu

# KV heads, group, queries: 1, 7, 64, 160, 192 and 200 rows
SHAPES = [(1, 1, 1), (7, 1, 1), (8, 2, 4), (8, 4, 5), (8, 4, 6), (5, 8, 5)]
CHUNKS = [1, 4, 5, 16, 17, 31, 32, 33, 48, 64, 65, 96, 97, 130]


@pytest.mark.parametrize("heads,group,queries", SHAPES)
def test_scores_by_chunk_count(heads, group, queries):
    chunk, D = 32, 64
    for chunks in CHUNKS:
        tokens = chunk * (chunks - 1) + 1 + 7 * chunks % chunk
        for bound in (tokens, max(CHUNKS) * chunk):                # (the kernel goes by the bound's number of chunks)
            print(f"[case] score windows, {heads * group * queries} rows, {chunks} chunks, bound {bound}", flush=True)
            L = synth.make_random_case(seed=64000 + 100 * heads + chunks, batch=1, num_q_heads=heads * group, num_kv_heads=heads,
                                       num_queries=queries, seq_lens=[tokens], head_dim=D, logit_std=2.0, value_std=1.0, outliers=2,
                                       outlier_logit=25.0)
            dl = harness.DeviceLayer.upload(L)
            pages = -(-bound // 16)
            if pages > L.block_table.shape[1]:
                dl.block_table = torch.nn.functional.pad(dl.block_table, (0, pages - L.block_table.shape[1]), value=-1)
            for collect in (vb.COLLECT_ALL_ROWS, vb.COLLECT_FIRST_LAST):
                ref_out, ref_scores = O.verify_attention(L.q_verify, L.k_cache, L.v_cache, L.block_table, L.seq_lens, L.softmax_scale, collect)
                path = harness.VegasPath(batch=1, num_q_heads=heads * group, num_kv_heads=heads, num_queries=queries, max_blocks=dl.block_table.shape[1],
                                         max_seq_len=bound, num_pages=L.num_pages, budget_tokens=64, softmax_scale=L.softmax_scale, head_dim=D,
                                         collect_rows=collect, verify_chunk=chunk)
                path.workspace.fill_(0xFF)           # NaN where nothing was written
                path.out_verify.fill_(float("nan"))
                path.block_scores.fill_(float("nan"))
                path.verify(dl)
                torch.cuda.synchronize()
                U.check_out(f"score_windows.{chunks}", path.out_verify, ref_out, U.vmax_visible(L))
                U.check_scores(f"score_windows.{chunks}", path.block_scores[:, :ref_scores.shape[1]], ref_scores)
                assert not bool(path.block_scores[:, ref_scores.shape[1]:].any())
