"""Draft calls whose bound on the selected K and V exceeds the last-level cache: the 16-row kernel that chooses by the lengths
(attn_draft.hpp, past_cache).  Short selections under a large bound: ends inside a page, a tile and on one, every page size,
both head dimensions, chunk lengths from the planner and of one tile per wave, against the oracle.  (Selections that are read past
the cache: test_gpu_draft_lengths.py.)"""
import numpy as np
import pytest
import torch

from oracle import vegas_oracle as O
from paper_2602_07223_amd import binding as vb
from paper_2602_07223_amd import harness, synth
from tests import parity_util as U
from tests.test_gpu_small_pages import random_selection

pytestmark = pytest.mark.gpu
PAGE = 16


@pytest.mark.parametrize("P", [16, 1, 2, 4, 8])
@pytest.mark.parametrize("D", [128, 64])
@pytest.mark.parametrize("g", [1, 5, 16])
def test_large_bounds(g, D, P):
    Hkv = 2
    lens = [1999, 0, 512, 33, 16, 1]
    bound = (352 << 20) // (len(lens) * Hkv * D * 4) // PAGE * PAGE + PAGE
    assert len(lens) * Hkv * bound * D * 4 >= 352 << 20
    L = synth.make_random_case(seed=48000 + g + D, batch=len(lens), num_q_heads=Hkv * g, num_kv_heads=Hkv, num_queries=2,
                               seq_lens=lens, head_dim=D, logit_std=1.5, value_std=1.0, outliers=2, outlier_logit=25.0)
    sel, ssl = random_selection(L, P, np.random.default_rng(g), keep_fraction=0.7)
    print(f"[case] streamed draft g={g} D={D} P={P} sel_lens={ssl.tolist()}", flush=True)
    ref = O.draft_attention(L.q_draft[0], L.k_cache.reshape(-1, P, Hkv, D), L.v_cache.reshape(-1, P, Hkv, D), sel, ssl, L.softmax_scale)
    wide = np.full((len(lens), bound // P), -1, dtype=np.int32)
    wide[:, :sel.shape[1]] = sel
    dev = torch.device("cuda:0")
    args = (harness.bf16_to_device(L.q_draft[0], dev), harness.bf16_to_device(L.k_cache, dev),
            harness.bf16_to_device(L.v_cache, dev), torch.from_numpy(wide).to(dev), torch.from_numpy(ssl).to(dev))
    for chunk in (0, 128):                      # the planner's chunks; one tile per wave
        desc = vb.make_desc(batch=len(lens), num_q_heads=Hkv * g, num_kv_heads=Hkv, num_queries=1, max_blocks=bound // P,
                            max_sel_blocks=bound // P, max_seq_len=bound, num_pages=L.num_pages * (PAGE // P),
                            softmax_scale=L.softmax_scale, page_size=P, kv_chunk_tokens=chunk, head_dim=D)
        ws = torch.empty(vb.vegas_workspace_bytes(desc), dtype=torch.uint8, device=dev)
        ws.fill_(0xFF)
        out = torch.full((len(lens), Hkv * g, D), float("nan"), dtype=torch.bfloat16, device=dev)
        vb.vegas_draft_attention(desc, *args, out, ws)
        torch.cuda.synchronize()
        U.check_out(f"streamed.g{g}.D{D}.P{P}.chunk{chunk}", out, ref, U.vmax_visible(L))
