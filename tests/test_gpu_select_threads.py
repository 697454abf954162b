"""Page selection at the edges of its thread counts and rows (512 pages a row up to 4096 pages, 1024 a row beyond) against the
oracle, bit for bit; the table is also wider than the longest sequence needs, and holds scores there that must not matter."""
import numpy as np
import pytest
import torch

from oracle import vegas_oracle as O
from paper_2602_07223_amd import binding as vb
from tests.test_gpu_register_select import make_scores

pytestmark = pytest.mark.gpu
PAGE = 16


@pytest.mark.parametrize("spare", [0, 5000])
@pytest.mark.parametrize("pages", [2, 512, 513, 514, 2048, 2049, 2050, 3585, 4096, 4097])
@pytest.mark.parametrize("kind", ["normal", "any_bits", "equal", "far_outlier"])
def test_page_select_by_threads(kind, pages, spare):
    rng = np.random.default_rng(pages * 5 + len(kind) + spare)
    G, mb = 5, pages + spare
    lens = np.array([pages * PAGE, pages * PAGE - 12, min(511 * PAGE + G, pages * PAGE), min(512 * PAGE + G, pages * PAGE), 20, 0],
                    dtype=np.int32)
    B = len(lens)
    scores = np.stack([make_scores(kind, mb, rng) for _ in range(B)])
    table = np.stack([rng.permutation(mb + 5)[:mb] for _ in range(B)]).astype(np.int32)
    dev = torch.device("cuda:0")
    for budget in (48, pages * PAGE // 14 + 64, max(pages * PAGE - 40, 16)):
        msb = pages + 2
        print(f"[case] page select {kind} pages={pages} spare={spare} budget={budget}", flush=True)
        desc = vb.make_desc(batch=B, num_q_heads=32, num_kv_heads=8, num_queries=G, max_blocks=mb, max_sel_blocks=msb,
                            max_seq_len=pages * PAGE, num_pages=mb + 5, softmax_scale=0.1)
        sel = torch.full((B, msb), -7, dtype=torch.int32, device=dev)
        ssl = torch.full((B,), -7, dtype=torch.int32, device=dev)
        vb.vegas_select_blocks(desc, torch.from_numpy(scores).to(dev), torch.from_numpy(table).to(dev),
                               torch.from_numpy(lens).to(dev), budget, sel, ssl)
        torch.cuda.synchronize()
        with np.errstate(invalid="ignore"):
            ref_sel, ref_ssl, _ = O.select_blocks(scores, table, lens, G, budget, msb)
        assert np.array_equal(ssl.cpu().numpy(), ref_ssl)
        assert np.array_equal(sel.cpu().numpy(), ref_sel)
