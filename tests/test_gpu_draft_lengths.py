"""Draft calls whose bound allows more selected K and V than the last-level cache keeps (attn_draft.hpp, past_cache): the lengths on
the GPU say whether they are read past it, in whole 128-byte lines whose pieces lanes exchange, or through it.  On the CPU the
rule; on the GPU both kinds of calls under the same bound, every page size and head dimension, against the oracle."""
import numpy as np
import pytest
import torch

from oracle import vegas_oracle as O
from paper_2602_07223_amd import binding as vb
from paper_2602_07223_amd import harness, synth
from tests import parity_util as U
from tests.test_host_layout import run_host_program

PAGE = 16
EDGE = 352 << 20                       # bytes of selected K and V

RULE = r'''
#include <cstdio>
#include <vector>
#include "attn_draft.hpp"
int main() {                       // lines of: KV heads, head dimension, longest, sequences, lengths
  int heads, D, longest, batch;
  while (std::scanf("%d %d %d %d", &heads, &D, &longest, &batch) == 4) {
    std::vector<int> lens(batch);
    for (int& n : lens) if (std::scanf("%d", &n) != 1) return 1;
    uint64_t sixteens = 0;
    for (int lane = 0; lane < 64; ++lane) sixteens += vegas::lane_sixteens(lens[lane < batch ? lane : batch - 1], lens.data(), batch, longest, lane);
    std::printf("%llu %d\n", static_cast<unsigned long long>(sixteens), vegas::past_cache(sixteens, heads, D) ? 1 : 0);
  }
}
'''


def test_selections_are_judged_by_their_lengths(tmp_path):
    """Not by the bound: a long one beside short ones, a loose bound, unequal lengths stay below the edge."""
    calls = [(8, 128, 8192, [8192] + [400] * 15, 0), (8, 128, 16384, [2048] * 8, 0), (8, 128, 8192, [8192] * 16, 1),
             (8, 128, 1 << 20, [300] * 32, 0), (8, 64, 8192, [8192] * 16, 0), (8, 64, 8192, [8192] * 24, 1),
             (8, 128, 5632, [5632] * 16, 1), (8, 128, 5632, [5632] * 15 + [5616], 0), (8, 128, 4000, [1 << 30] * 22, 0),
             (8, 128, 4096, [1 << 30] * 22, 1), (8, 128, 100, [-5, 0, 3], 0), (1, 64, 1 << 30, [1 << 30] * 3000, 1),
             (8, 128, 700, [699] * 129, 1), (8, 128, 700, [699] * 127, 0)]
    ask = "\n".join(" ".join(map(str, (h, D, longest, len(lens), *lens))) for h, D, longest, lens, _ in calls)
    for call, line in zip(calls, run_host_program(tmp_path, RULE, ask).strip().split("\n"), strict=True):
        h, D, longest, lens, past = call
        sixteens, got = map(int, line.split())
        whole = sum(-(-min(max(n, 0), longest) // 16) for n in lens)
        assert sixteens == whole or sixteens >= 1 << 30
        assert got == past == (whole * 64 * h * D >= EDGE), (h, D, longest, lens[:4])


@pytest.mark.gpu
@pytest.mark.parametrize("P", [16, 1, 2, 4, 8])
@pytest.mark.parametrize("D", [128, 64])
@pytest.mark.parametrize("g", [1, 5, 16])
def test_long_and_short_selections_under_one_bound(g, D, P):
    """One selection as long as the edge needs beside others that end inside a page, a tile and on one; then the short ones
    without it.  (Long: its pages are the pool's over and over.)"""
    Hkv = 16
    short = [1999, 0, 512, 33, 16, 1]
    long = EDGE // (Hkv * D * 4) + 5
    B = len(short) + 1
    L = synth.make_random_case(seed=48500 + g + D, batch=B, num_q_heads=Hkv * g, num_kv_heads=Hkv, num_queries=2,
                               seq_lens=[2048] + [16] * len(short), head_dim=D, logit_std=1.5, value_std=1.0, outliers=2, outlier_logit=25.0)
    rng = np.random.default_rng(g + P)
    dev = torch.device("cuda:0")
    bound = -(-long // PAGE) * PAGE
    q = L.q_draft[0]
    k, v = L.k_cache.reshape(-1, P, Hkv, D), L.v_cache.reshape(-1, P, Hkv, D)
    pages = np.concatenate([np.arange(int(t) * (PAGE // P), (int(t) + 1) * (PAGE // P)) for t in L.block_table[0][:2048 // PAGE]])
    for lens in ([long] + short, [7] + short):
        sel = np.full((B, bound // P), -1, dtype=np.int32)
        for b, n in enumerate(lens):
            need = -(-n // P)
            sel[b, :need] = np.concatenate([rng.permutation(pages) for _ in range(-(-need // len(pages)))] or [pages])[:need]
        ssl = np.array(lens, dtype=np.int32)
        print(f"[case] draft lengths g={g} D={D} P={P} longest={max(lens)}", flush=True)
        ref = O.draft_attention(q, k, v, sel, ssl, L.softmax_scale)
        desc = vb.make_desc(batch=B, num_q_heads=Hkv * g, num_kv_heads=Hkv, num_queries=1, max_blocks=bound // P,
                            max_sel_blocks=bound // P, max_seq_len=bound, num_pages=L.num_pages * (PAGE // P),
                            softmax_scale=L.softmax_scale, page_size=P, head_dim=D)
        ws = torch.empty(vb.vegas_workspace_bytes(desc), dtype=torch.uint8, device=dev)
        ws.fill_(0xFF)
        out = torch.full((B, Hkv * g, D), float("nan"), dtype=torch.bfloat16, device=dev)
        vb.vegas_draft_attention(desc, harness.bf16_to_device(q, dev), harness.bf16_to_device(L.k_cache, dev),
                                 harness.bf16_to_device(L.v_cache, dev), torch.from_numpy(sel).to(dev),
                                 torch.from_numpy(ssl).to(dev), out, ws)
        torch.cuda.synchronize()
        U.check_out(f"draft_lengths.g{g}.D{D}.P{P}.{max(lens)}", out, ref, U.vmax_visible(L))
