"""Workgroups of eight waves of 64 rows (attn_pair.hpp, pair_waves: head dimension 64, page values collected), where they can go
wrong: fewer tiles than waves, one more than a round of them, more than a wave's ring holds or than it parks; row counts at the
edges of a row block and of a second workgroup; both sides of the rule's two lines; against the float64 oracle."""
import pytest
import torch

from oracle import vegas_oracle as O
from paper_2602_07223_amd import binding as vb
from paper_2602_07223_amd import harness, synth
from tests import parity_util as U

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("Hq,Hkv,G", [(88, 8, 3), (64, 8, 5), (64, 8, 8), (104, 8, 5), (64, 8, 12)],
                         ids=["33_rows", "40_rows", "64_rows", "65_rows", "96_rows"])
@pytest.mark.parametrize("lens,chunk", [([4127], 0), ([4128], 0), ([4128], 32), ([4129], 288), ([8192], 0), ([9000], 9024),
                                        ([4133, 0, 517], 0), ([700, 1300, 33, 2048, 1, 900, 1029, 500], 0),
                                        ([1100], 0), ([2065], 0), ([128, 37, 5, 120], 0)], ids=str)
def test_eight_waves(lens, chunk, Hq, Hkv, G):
    L = synth.make_random_case(seed=6700 + sum(lens) + Hq + G, batch=len(lens), num_q_heads=Hq, num_kv_heads=Hkv, num_queries=G,
                               seq_lens=lens, head_dim=64, logit_std=2.0, value_std=1.0, outliers=2,
                               outlier_logit=25.0)
    print(f"[case] eight waves lens={lens} chunk={chunk} Hq={Hq} G={G}", flush=True)
    dl = harness.DeviceLayer.upload(L)
    for collect in (vb.COLLECT_ALL_ROWS, vb.COLLECT_FIRST_LAST):
        ref_out, ref_scores = O.verify_attention(L.q_verify, L.k_cache, L.v_cache, L.block_table, L.seq_lens, L.softmax_scale,
                                                 collect)
        path = harness.VegasPath.for_layer(L, budget_tokens=256, collect_rows=collect, verify_chunk=chunk)
        path.workspace.fill_(0xFF)                # NaN partials where nothing was written
        path.out_verify.fill_(float("nan"))
        path.block_scores.fill_(float("nan"))
        path.verify(dl)
        torch.cuda.synchronize()
        U.check_out(f"eight.{sum(lens)}.{Hq}.{collect}", path.out_verify, ref_out, U.vmax_visible(L))
        U.check_scores(f"eight.{sum(lens)}.{Hq}.{collect}", path.block_scores, ref_scores)
