"""An infinite value of the last chunk's through the merges of chunk partials (RowMerge): slots past the row's chunks are requested as the last
one once more, and their weight, 0, must not meet it (0 times an infinity is NaN).  Every other head dim keeps its bits."""
import pytest
import torch

from paper_2602_07223_amd import binding as vb
from paper_2602_07223_amd import harness, synth

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("collect", [None, vb.COLLECT_NONE, vb.COLLECT_ALL_ROWS], ids=["draft", "verify", "verify_collect"])
@pytest.mark.parametrize("chunks", [2, 3, 5, 9, 13, 17, 22, 25, 33, 41, 49, 64])
def test_infinite_value_in_the_last_chunk(chunks, collect):
    chunk, D, heads, kv_heads = 32, 64, 8, 2
    tokens = chunk * chunks - 3
    for bound in (tokens, tokens + 2 * chunk):                # (the kernels go by the bound's number of chunks)
        L = synth.make_random_case(seed=67000 + chunks, batch=1, num_q_heads=heads, num_kv_heads=kv_heads, num_queries=1, seq_lens=[tokens], head_dim=D)
        dl = harness.DeviceLayer.upload(L)
        per = -(-bound // 16)
        table = torch.nn.functional.pad(dl.block_table, (0, per - dl.block_table.shape[1]), value=-1)
        desc = vb.make_desc(batch=1, num_q_heads=heads, num_kv_heads=kv_heads, num_queries=1, max_blocks=per, max_sel_blocks=per, max_seq_len=bound,
                            num_pages=L.num_pages, softmax_scale=L.softmax_scale, collect_rows=vb.COLLECT_NONE if collect is None else collect,
                            head_dim=D, kv_chunk_tokens=chunk)
        outs = []
        for value in (1.0, float("inf")):
            v = dl.v_cache.clone()
            v[int(L.block_table[0, (tokens - 1) // 16]), (tokens - 1) % 16, :, 7] = value
            out = torch.full((1, 1, heads, D), float("nan"), dtype=torch.bfloat16, device="cuda:0")
            scores = torch.empty((1, per), dtype=torch.float32, device="cuda:0")
            ws = torch.full((vb.vegas_workspace_bytes(desc),), 0xFF, dtype=torch.uint8, device="cuda:0")
            print(f"[case] infinite value, {chunks} chunks, bound {bound}, collect {collect}, {value}", flush=True)
            if collect is None:
                vb.vegas_draft_attention(desc, dl.q_verify.reshape(1, heads, D), dl.k_cache, v, table, dl.seq_lens, out, ws)
            else:
                vb.vegas_verify_attention(desc, dl.q_verify, dl.k_cache, v, table, dl.seq_lens, out, scores, ws)
            torch.cuda.synchronize()
            outs.append(out.view(heads, D))
        assert bool(torch.isposinf(outs[1][:, 7]).all()), outs[1][:, 7]
        others = [i for i in range(D) if i != 7]
        assert torch.equal(outs[0][:, others], outs[1][:, others])
