"""Draft calls whose columns are split by parts of V (draft_value_parts): four, two and one workgroup per column, through rings and
through registers, every page size and head dimension, selections at the ends of tiles and of the wave's ring, an empty sequence, rows of a group that do
and do not fill the tile, padded strides; against the oracle and, cut into chunks, against the merged call."""
import numpy as np
import pytest
import torch

from oracle import vegas_oracle as O
from paper_2602_07223_amd import binding as vb
from tests import parity_util as U

pytestmark = pytest.mark.gpu
DEV = "cuda:0"
LENGTHS = [1, 31, 32, 33, 127, 129, 160, 255, 257, 289, 383, 448]


def bf16(x):
    return x.view(torch.int16).cpu().numpy().view(np.uint16)


@pytest.mark.parametrize("D", [128, 64])
@pytest.mark.parametrize("P", [16, 8, 4, 2, 1])
@pytest.mark.parametrize("B,Hq,Hkv", [(1, 8, 8), (4, 28, 4), (8, 32, 8), (9, 40, 8), (16, 64, 8), (17, 8, 8), (33, 32, 2)])
def test_parts(B, Hq, Hkv, P, D):
    gen = torch.Generator(device=DEV).manual_seed(66000 + B * 10 + P + D)
    rng = np.random.default_rng(B + P)
    pool, pad = 600, 8
    per_slot = Hkv * D + pad                                     # (a token's row is longer than its heads)
    K = torch.randn((pool, 16, per_slot), generator=gen, device=DEV).to(torch.bfloat16)
    V = torch.randn((pool, 16, per_slot), generator=gen, device=DEV).to(torch.bfloat16)
    k_np, v_np = bf16(K)[:, :, :Hkv * D].reshape(pool, 16, Hkv, D), bf16(V)[:, :, :Hkv * D].reshape(pool, 16, Hkv, D)
    small = pool * (16 // P)
    for bound in (100, 448):
        lens = np.array([min(LENGTHS[(7 * i + B) % len(LENGTHS)], bound) for i in range(B)], dtype=np.int32)
        lens[0] = bound
        if B > 1:
            lens[1] = 0
        per = -(-bound // P) + 2
        sel = np.full((B, per), -1, dtype=np.int32)
        for b in range(B):
            need = -(-int(lens[b]) // P)
            sel[b, :need] = np.sort(rng.permutation(small)[:need])
        q = torch.randn((B, Hq, D), generator=gen, device=DEV).to(torch.bfloat16)
        kw = dict(batch=B, num_q_heads=Hq, num_kv_heads=Hkv, num_queries=1, max_blocks=per, max_sel_blocks=per, max_seq_len=bound,
                  num_pages=small, softmax_scale=D ** -0.5, collect_rows=vb.COLLECT_NONE, head_dim=D, page_size=P,
                  kv_token_stride=per_slot, kv_page_stride=P * per_slot, kv_head_stride=D)
        outs = []
        for chunk in (0, 32):
            desc = vb.make_desc(kv_chunk_tokens=chunk, **kw)
            out = torch.full((B, Hq, D), float("nan"), dtype=torch.bfloat16, device=DEV)
            ws = torch.full((vb.vegas_workspace_bytes(desc),), 0xFF, dtype=torch.uint8, device=DEV)
            print(f"[case] draft parts {B}x{Hkv} columns, D={D}, pages of {P}, bound {bound}, chunk {chunk}", flush=True)
            vb.vegas_draft_attention(desc, q, K, V, torch.from_numpy(sel).to(DEV), torch.from_numpy(lens).to(DEV), out, ws)
            torch.cuda.synchronize()
            outs.append(out)
        ref = O.draft_attention(bf16(q), k_np.reshape(small, P, Hkv, D), v_np.reshape(small, P, Hkv, D), sel, lens, D ** -0.5)
        vmax = float(V.float().abs().max())
        for out in outs:
            U.check_out(f"draft_parts.{B}.{P}.{D}.{bound}", out, ref, vmax)


@pytest.mark.parametrize("D,P", [(128, 16), (128, 1), (64, 16), (64, 4)])
@pytest.mark.parametrize("B,Hq,Hkv", [(1, 4, 1), (65, 2, 1), (5, 21, 3), (3, 35, 7), (18, 7, 7), (11, 10, 10), (5, 24, 24)])
def test_parts_by_rounds_of_columns(B, Hq, Hkv, P, D):
    """Numbers of KV heads that are not whole rounds of the XCDs (part_grid_width): the last round of columns is full or not, a sequence's heads lie
    in one or in two."""
    test_parts(B, Hq, Hkv, P, D)
