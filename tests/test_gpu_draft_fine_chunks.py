"""Draft calls in chunks of 64 and 96 tokens (draft_chunk_tokens: a wave or two of every workgroup without a tile), at the ends of the range
and one token past them, for every page size, against the oracle; and in a workspace that holds the chunks of 128 tokens only.
Of the bits: any workspace of the size asked for and the built-in scratch give the same."""
import pytest
import torch

from oracle import vegas_oracle as O
from paper_2602_07223_amd import binding as vb
from paper_2602_07223_amd import harness, synth
from tests import parity_util as U

# sequences, KV heads, query heads per KV head, selected tokens (bound), head dim, page size
CALLS = [
    (1, 8, 4, 465, 128, 16), (1, 8, 4, 1536, 128, 16), (1, 8, 8, 1537, 128, 16), (1, 8, 4, 2304, 128, 16), (1, 8, 4, 2305, 128, 16),
    (1, 8, 16, 1280, 128, 16), (1, 8, 16, 1281, 128, 16), (1, 8, 16, 1920, 128, 16), (1, 8, 16, 1921, 128, 16),   # the bound on the partials
    (2, 16, 2, 481, 128, 16), (1, 4, 7, 1000, 64, 16), (3, 2, 16, 1700, 64, 16), (1, 8, 4, 2048, 128, 1), (1, 8, 4, 1003, 64, 4),
]


@pytest.mark.gpu
@pytest.mark.parametrize("call", range(len(CALLS)))
def test_fine_chunks(call):
    batch, heads, group, tokens, D, page = CALLS[call]
    lens = [tokens - 211 * b for b in range(batch)]
    print(f"[case] fine chunks {CALLS[call]}", flush=True)
    L = synth.make_random_case(seed=71000 + call, batch=batch, num_q_heads=heads * group, num_kv_heads=heads, num_queries=1,
                               seq_lens=lens, head_dim=D, logit_std=2.0, value_std=1.0, outliers=2, outlier_logit=25.0)
    dl = harness.DeviceLayer.upload(L)
    pages = -(-tokens // page)
    table = torch.zeros((batch, pages), dtype=torch.int32, device="cuda:0")
    for b, n in enumerate(lens):
        pos = torch.arange(-(-n // page), device="cuda:0") * page
        table[b, :len(pos)] = dl.block_table[b, pos // 16] * (16 // page) + ((pos % 16) // page).to(torch.int32)
    desc = vb.make_desc(batch=batch, num_q_heads=heads * group, num_kv_heads=heads, num_queries=1, max_blocks=dl.block_table.shape[1],
                        max_sel_blocks=pages, max_seq_len=tokens, num_pages=dl.k_cache.shape[0] * (16 // page),
                        softmax_scale=L.softmax_scale, head_dim=D, page_size=page)
    ref, _ = O.verify_attention(L.q_draft[:1].transpose(1, 0, 2, 3), L.k_cache, L.v_cache, L.block_table, L.seq_lens, L.softmax_scale, 0)
    slots = heads * batch * -(-tokens // 128)                        # of chunks of 128 tokens
    coarse = -(-slots * group * D * 4 // 256) * 256 + -(-slots * group * 8 // 256) * 256
    asked = vb.vegas_workspace_bytes(desc)
    outs = {}
    for size in (asked, asked + 4096, coarse):
        ws = torch.full((size,), 0xFF, dtype=torch.uint8, device="cuda:0")   # NaN partials where nothing was written
        out = outs[size] = torch.full((batch, heads * group, D), float("nan"), dtype=torch.bfloat16, device="cuda:0")
        vb.vegas_draft_attention(desc, dl.q_draft[0], dl.k_cache, dl.v_cache, table, dl.seq_lens, out, ws)
        torch.cuda.synchronize()
        U.check_out(f"fine_chunks.{call}.{size}", out[:, None], ref, U.vmax_visible(L))
    static = torch.full_like(out, float("nan"))
    vb.vegas_draft_attention_static(desc, dl.q_draft[0], dl.k_cache, dl.v_cache, table, dl.seq_lens, static)
    torch.cuda.synchronize()
    for name, other in (("static", static), ("larger", outs[asked + 4096])):
        assert torch.equal(other.view(torch.int16), outs[asked].view(torch.int16)), name
