"""Draft calls that one workgroup per column streams through rings in LDS (plan_rules.hpp, ring_draft), where they can go wrong: a wave
with no tile, fewer tiles than its ring holds, as many and one more; the selection's end at every place of a page; more tiles than
one register of page ids covers; every group size class; and both sides of the rule.  Against the float64 oracle, with NaN in the
slots past the end."""
import re

import numpy as np
import pytest
import torch

from oracle import vegas_oracle as O
from paper_2602_07223_amd import binding as vb
from paper_2602_07223_amd import build, harness

PAGE = 16
DEV = "cuda:0"


def run(lens, Hq, Hkv, chunk=0, D=128, seed=0):
    B, gen = len(lens), torch.Generator(device=DEV).manual_seed(91000 + seed)
    rng = np.random.default_rng(91000 + seed)
    per = max(-(-n // PAGE) for n in lens) + 2
    pool = B * per + 3
    order = rng.permutation(pool).astype(np.int32)
    table = np.full((B, per), -1, dtype=np.int32)
    k = torch.randn((pool, PAGE, Hkv, D), generator=gen, device=DEV).to(torch.bfloat16)
    v = torch.randn((pool, PAGE, Hkv, D), generator=gen, device=DEV).to(torch.bfloat16)
    for b, n in enumerate(lens):
        pages = -(-n // PAGE)
        table[b, :pages] = order[b * per:b * per + pages]
        if n % PAGE:
            k[int(table[b, pages - 1]), n % PAGE:] = float("nan")
            v[int(table[b, pages - 1]), n % PAGE:] = float("nan")
    q = (2.0 * torch.randn((B, Hq, D), generator=gen, device=DEV)).to(torch.bfloat16)
    scale = D ** -0.5
    desc = vb.make_desc(batch=B, num_q_heads=Hq, num_kv_heads=Hkv, num_queries=1, max_blocks=per, max_sel_blocks=per,
                        max_seq_len=max(max(lens), 1), num_pages=pool, softmax_scale=scale, head_dim=D, collect_rows=vb.COLLECT_NONE,
                        kv_chunk_tokens=chunk)
    out = torch.full((B, Hq, D), float("nan"), dtype=torch.bfloat16, device=DEV)
    ws = torch.full((vb.vegas_workspace_bytes(desc),), 0xFF, dtype=torch.uint8, device=DEV)
    n32 = np.array(lens, dtype=np.int32)
    print(f"[case] draft rings lens={lens[:6]} Hq={Hq} Hkv={Hkv} chunk={chunk}", flush=True)
    vb.vegas_draft_attention(desc, q, k, v, torch.from_numpy(table).to(DEV), torch.from_numpy(n32).to(DEV), out, ws)
    torch.cuda.synchronize()

    def bits(t):
        return t.contiguous().view(torch.int16).cpu().numpy().view(np.uint16)

    ref = O.draft_attention(bits(q), bits(k), bits(v), table, n32, scale)
    got = harness.bf16_to_host_f64(out)
    assert np.all(np.isfinite(got))
    vmax = float(np.nanmax(np.abs(v.float().cpu().numpy())))
    # (the bar of tests/parity_util.py: half the worst case of rounding the weights to bf16)
    assert np.abs(got - ref).max() <= max(2e-3, vmax / 256.0)
    assert np.sqrt(((got - ref) ** 2).sum()) <= 1e-2 * np.sqrt((ref ** 2).sum()) + 1e-12


@pytest.mark.gpu
@pytest.mark.parametrize("n", [1, 31, 97, 128, 129, 160, 161, 255, 256, 257, 289, 384, 385, 417, 448])
@pytest.mark.parametrize("Hq,Hkv", [(8, 8), (32, 8), (28, 4), (32, 2)], ids=["group1", "group4", "group7", "group16"])
def test_lengths_at_the_edges_of_rings(n, Hq, Hkv):
    run([n, max(n - 18, 0), 448, 0], Hq, Hkv, seed=n + Hq)


@pytest.mark.gpu
@pytest.mark.parametrize("lens,chunk", [([3200, 1, 2049] * 10, 0), ([4097, 8200], 8320), ([4224], 4224), ([700] * 12, 0), ([700] * 31, 0), ([700] * 32, 0)],
                         ids=["long", "page_ids_reloaded", "one_over_32_tiles", "96_columns", "248_columns", "256_columns"])
def test_long_selections_and_both_sides_of_the_rule(lens, chunk):
    run(lens, 32, 8, chunk=chunk, seed=len(lens) + chunk)


def test_m0_belongs_to_the_loads_into_lds(tmp_path):
    """The loads write M0 in inline assembly and cannot say so (a reserved register): nothing else in this kernel may use it."""
    path = tmp_path / "device.s"
    build.kernel_resource_usage(str(path))
    bodies = [b for name, b in re.findall(r"^(_ZN5vegas19attn_draft16_kernel\w*):(.*?)^\.Lfunc_end", path.read_text(), flags=re.M | re.S)
              if "global_load_lds" in b]
    assert len(bodies) == 1
    body = re.sub(r"[ \t]*;.*", "", bodies[0])
    own = re.compile(r"s_mov_b32 m0, s\d+\s+s_nop 0\s+global_load_lds_dwordx4 v\d+, s\[\d+:\d+\]")
    foreign = [line.strip() for line in own.sub("", body).splitlines() if re.search(r"\bm0\b|global_load_lds", line)]
    assert len(own.findall(body)) >= 48 and not foreign, foreign[:4]
