"""Index arithmetic that kernels and host code share, checked on the CPU: the headers' host-callable functions are compiled
into a small program and compared with the rules written out here."""
import bisect
import subprocess

import numpy as np
import pytest

from paper_2602_07223_amd import binding as vb
from paper_2602_07223_amd import build


def run_host_program(tmp_path, body: str, stdin: str = "") -> str:
    """Compiles `body` (a main() that may include the library's headers) for the host only and runs it."""
    src, exe = tmp_path / "probe.hip", tmp_path / "probe"
    src.write_text(body)
    cmd = [build.hipcc_path(), "--cuda-host-only", "-std=c++17", "-O1", "-I", build.CSRC, str(src), "-o", str(exe)]
    r = subprocess.run(cmd, capture_output=True, text=True)
    assert r.returncode == 0, r.stderr
    r = subprocess.run([str(exe)], input=stdin, capture_output=True, text=True, timeout=120)
    assert r.returncode == 0, r.stderr
    return r.stdout


def balanced_plan(lens, j1, j2, unit):
    """Balanced chunking by its definition: (first slot, chunk tokens) per sequence, chunks per sequence."""
    nu = [-(-n // unit) for n in lens]

    def smallest(J):
        return next(c for c in range(1, max(nu) + 1) if c == max(nu) or sum(-(-x // c) for x in nu) <= J)

    if sum(nu) == 0:
        return [(0, unit)] * len(lens), [0] * len(lens)
    C = smallest(j1)
    if j2 > j1 and 10 * sum(nu) < 9 * j1 * C:
        C = smallest(j2)
    s = [-(-x // C) for x in nu]
    chunk = [(-(-x // k)) * unit if k else 0 for x, k in zip(nu, s)]
    first = [sum(s[i] for i in range(len(lens)) if chunk[i] > chunk[b] or (chunk[i] == chunk[b] and i < b))
             for b in range(len(lens))]
    return [(f, c or unit) for f, c in zip(first, chunk)], s


SLOTS = r'''
#include <cstdio>
#include "vegas_common.hpp"
int main() {                       // lines of: slots of a head, number of KV heads, first slot, chunk tokens, tokens
  int slots, heads, first, chunk, n;
  while (std::scanf("%d %d %d %d %d", &slots, &heads, &first, &chunk, &n) == 5) {
    const int2 plan = {first, chunk};
    const vegas::ColumnSlots cs = vegas::column_slots(&plan, slots, 0, heads, 0, 0);
    const vegas::ColumnChunks cc = vegas::column_chunks(cs, n);
    long long most = -1;           // largest slot the merge of this column requests (lane s asks for chunk s)
    if (cc.last >= 0)
      for (int s = 0; s < 64; ++s) most = cs.off + vegas::requested_slot(s, cc.last);
    std::printf("%lld %d %d %lld\n", static_cast<long long>(cs.off), cs.stride_h, cc.ns, most);
  }
}
'''


def test_planned_merges_request_a_sequences_own_slots_only(tmp_path):
    """Batches whose chunks fill every slot of a head, some with empty members (which start one past the last slot and own
    none): a merge requests slots of its own column and none of an empty one's."""
    unit, heads = 128, 8
    rng = np.random.default_rng(7)
    batches = [[4096, 0], [0, 4096], [4096, 0, 0, 0], [0, 0, 12288], [0, 0], [1, 0], [2048, 2048], [2048, 0, 2048],
               [36864] * 7 + [0], [65536, 0] * 8, [128] * 16 + [0] * 16]
    batches += [[int(n) for n in rng.integers(0, 6000, size=b) * rng.integers(0, 2, size=b)]
                for b in rng.integers(2, 33, size=60)]
    cases = []
    for lens in batches:
        j1 = 32
        j2 = 64 if len(lens) >= 8 else 32
        slots = max(j2, len(lens))
        plan, s = balanced_plan(lens, j1, j2, unit)
        assert sum(s) <= slots
        cases += [(slots, heads, *plan[b], lens[b], s[b]) for b in range(len(lens))]
    # the case this is about is among them: an empty sequence that starts one past the last slot of its head
    assert any(first == slots and n == 0 for slots, _, first, _, n, _ in cases)
    out = run_host_program(tmp_path, SLOTS, "\n".join(" ".join(map(str, c[:5])) for c in cases))
    for (slots, _, first, chunk, n, s), line in zip(cases, out.strip().split("\n"), strict=True):
        off, stride, ns, most = map(int, line.split())
        assert (off, stride, ns) == (first, slots, s), (first, chunk, n)
        assert most == (first + min(64, s) - 1 if s else -1), (slots, first, chunk, n, most)
        assert most < slots


PARKS = r'''
#include <cstdio>
#include "attn_pair.hpp"
int main() {                       // lines of: query rows, collected rows, collection mode, head dimension
  int R, Rc, collect, D;
  while (std::scanf("%d %d %d %d", &R, &Rc, &collect, &D) == 4) {
    const int tile_rows = R + (collect == 2 ? 2 : 0), blocks = (tile_rows + vegas::kPairRows - 1) / vegas::kPairRows;
    const vegas::PairLds lds = vegas::pair_lds(R, Rc, blocks, collect, D);
    const int queries = (blocks == 1 ? tile_rows : vegas::kPairRows) * vegas::row_pitch(D);
    std::printf("%d %d %zu %zu %zu\n", lds.park_tiles, vegas::pair_park_floats(lds.park_tiles, Rc, collect),
                static_cast<size_t>(vegas::kPairWaves * vegas::pair_ring(D, collect) + queries), lds.off_max, lds.bytes);
  }
}
'''


def test_parked_values_of_every_wave_are_aligned(tmp_path):
    """64-row workgroups: a wave reads what it has parked in 16-byte pieces, so its part of the LDS starts on a multiple of
    16 bytes and ends before the row maxima, for every row count, collection mode and head dimension."""
    cases = [(R, R, 0, D) for D in (128, 64) for R in range(33, 129)]
    cases += [(R, Rc, collect, D) for D in (128, 64) for R in range(31, 129)
             for collect, rcs in ((1, {R} | {2 * g for g in range(1, 43) if R % g == 0 and R // g > 2}), (2, {R}))
             for Rc in sorted(rcs) if R + (2 if collect == 2 else 0) > 32]
    out = run_host_program(tmp_path, PARKS, "\n".join(" ".join(map(str, c)) for c in cases))
    for case, line in zip(cases, out.strip().split("\n"), strict=True):
        tiles, floats, parks, off_max, total = map(int, line.split())
        R, Rc, collect, D = case
        # at head dimension 64, unless page values are parked, two workgroups fit a compute unit
        assert total <= (80 if D == 64 and collect != 1 else 160) * 1024, (case, total)
        if collect == 0:
            assert tiles == 0
            continue
        assert tiles >= 2 and floats >= tiles * 2 * (32 if collect == 2 else min(Rc, 64)), case
        assert parks % 16 == 0 and floats % 4 == 0, case
        assert parks + 4 * floats * 4 <= off_max, case


RULES = r'''
#include <cstdio>
#include "plan_rules.hpp"
int main() {                       // lines of: columns, head dimension, window, longest sequence, chunk tokens (256 compute units)
  int columns, D, window, longest, chunk;
  while (std::scanf("%d %d %d %d %d", &columns, &D, &window, &longest, &chunk) == 5)
    std::printf("%d %d\n", vegas::lone_workgroup_tokens(columns, 256, D),
                vegas::lone_workgroup_band(window, 5, longest, chunk, vegas::lone_band_tokens(D)) ? 1 : 0);
}
'''


def test_rules_for_calls_without_a_merge(tmp_path):
    """A column is left to one workgroup where that was measured faster, for selections of unequal length too (or within a
    microsecond): never the longer the fewer columns there are, and not beyond 3200 tokens however many."""
    measured = [(8, 128, 416, True), (8, 128, 544, False), (80, 128, 544, True), (64, 128, 800, False),
                (8, 64, 608, True), (32, 64, 608, True), (16, 64, 800, False), (64, 64, 1056, False), (16, 64, 1056, False),
                (96, 128, 800, True), (96, 128, 1056, False), (80, 64, 928, True), (96, 64, 928, True), (96, 64, 2080, False),
                (128, 128, 1312, True), (128, 128, 2080, False), (128, 64, 2080, True), (128, 64, 3104, False),
                (136, 64, 3104, True), (136, 128, 2080, False), (144, 128, 2080, True), (144, 64, 3104, True), (192, 128, 3200, True), (192, 128, 6176, False),
                (256, 64, 3200, True), (256, 64, 6176, False), (320, 128, 4128, False), (512, 64, 2080, True)]
    every = [(c, D) for D in (128, 64) for c in (1, 8, 24, 71, 72, 95, 96, 127, 128, 135, 136, 143, 144, 191, 192, 256, 1000)]
    bands = [(128, 384, 4096, 128, True), (128, 512, 4096, 128, False), (128, 512, 4096, 256, False), (128, 1024, 32768, 1024, False),
             (128, 1024, 14591, 1792, True), (128, 2048, 14591, 1792, False), (128, 4096, 15699, 15744, True), (128, 3223, 400, 128, True),
             (128, 3223, 637, 128, False), (128, (1 << 31) - 1, 400, 128, True),   # a window beyond the context
             (128, 443, 4096, 128, True), (128, 444, 4096, 128, False), (64, 444, 4096, 128, True), (64, 635, 4096, 128, True),
             (64, 636, 4096, 128, False), (64, 636, 4096, 768, True)]              # both sides of the line, which is the head dimension's
    ask = ([(c, D, 1, 1, 1) for c, D, _, _ in measured] + [(c, D, 1, 1, 1) for c, D in every] +
           [(8, D, w, n, c) for D, w, n, c, _ in bands])
    out = [tuple(map(int, line.split()))
           for line in run_host_program(tmp_path, RULES, "\n".join(" ".join(map(str, a)) for a in ask)).strip().split("\n")]
    assert len(out) == len(ask)
    for (c, D, n, alone), (limit, _) in zip(measured, out):
        assert (n <= limit) == alone, (c, D, n, limit)
    limits = dict(zip(every, (o[0] for o in out[len(measured):])))
    for D in (128, 64):
        per = [limits[(c, D)] for c, d in every if d == D]
        assert per == sorted(per) and per[-1] == 3200
    for (D, window, longest, chunk, alone), (_, got) in zip(bands, out[-len(bands):]):
        assert bool(got) == alone, (D, window, longest, chunk)


@pytest.mark.parametrize("rows,n,chunks", [(40, 8192, 1), (40, 8193, 2), (64, 16384, 2), (80, 4096, 1), (80, 65536, 16), (128, 16384, 4),
                                           (128, (1 << 24) - 16, 4096), (128, 1 << 26, 4096)])
def test_many_sequences_are_not_left_to_a_workgroup_each(rows, n, chunks):
    """More than 64 sequences have no plan: a long one is cut all the same."""
    assert chunk_slots(65, rows, 8, n) == 65 * 8 * chunks


def chunk_slots(batch, rows, kv_heads, max_len, head_dim=128, group=8):
    """Chunk partials (sequence, KV head, chunk) a verification call without collection holds, from what its workspace takes."""
    desc = vb.make_desc(batch=batch, num_q_heads=group * kv_heads, num_kv_heads=kv_heads, num_queries=rows // group,
                        max_blocks=-(-max_len // 16), max_sel_blocks=1, max_seq_len=max_len, num_pages=1 << 20,
                        softmax_scale=0.1, collect_rows=vb.COLLECT_NONE, head_dim=head_dim, page_size=16)
    total, up = vb.vegas_workspace_bytes(desc), lambda x: -(-x // 256) * 256
    return bisect.bisect_right(range(1, 1 << 26), total, key=lambda s: up(s * rows * head_dim * 4) + up(s * rows * 8))


@pytest.mark.parametrize("rows,n", [(40, 4097), (64, 12345), (40, 32749), (64, 65521), (72, 32749), (96, 65521), (128, 32749)])
def test_one_long_sequence_takes_one_round_of_64_row_workgroups(n, rows):
    """They fill a compute unit's LDS: more workgroups than the 256 compute units would take a second round."""
    blocks = -(-rows // 64)
    assert chunk_slots(1, rows, 8, n) * blocks <= 256


@pytest.mark.parametrize("n,chunks", [(9000, 24), (16384, 32), (16385, 33), (16511, 33), (16512, 26), (17000, 27), (45000, 32), (100000, 32)])
def test_one_sequence_of_any_length_takes_one_round(n, chunks):
    """24 rows, 8 KV heads: 32 chunks per head are one workgroup per compute unit; more only where all that lies beyond 32
    of them is less than a unit of 128 tokens."""
    assert chunk_slots(1, 24, 8, n) == 8 * chunks


WAVES = r'''
#include <cstdio>
#include "attn_pair.hpp"
int main() {                       // lines of: units of all sequences, workgroups of one wave, chunk units of its plan
  unsigned total, j1, C;
  while (std::scanf("%u %u %u", &total, &j1, &C) == 3)
    std::printf("%d %d\n", vegas::wants_second_wave(total, j1, C, 0), vegas::wants_second_wave(total, j1, C, vegas::pair_second_cost(128, 1)));
}
'''


def test_second_wave_of_64_row_workgroups(tmp_path):
    """Ragged batches, for which chunks half as long were measured faster (True) or slower although the first wave is not
    full: (units of 128 tokens, workgroups of one wave, longest chunk of its plan)."""
    measured = [((84, 32, 3), False), ((1067, 64, 19), False), ((244, 32, 12), False), ((100, 32, 4), False),
                ((320, 32, 17), False), ((640, 32, 23), False), ((1066, 32, 41), False), ((1293, 64, 32), False),
                ((877, 32, 44), True), ((1066, 16, 103), True), ((1263, 16, 120), True), ((4608, 32, 190), True)]
    out = run_host_program(tmp_path, WAVES, "\n".join(" ".join(map(str, m)) for m, _ in measured)).strip().split("\n")
    for (m, two), line in zip(measured, out, strict=True):
        anywhere, here = map(int, line.split())
        assert anywhere == 1, m                   # less than nine tenths of the wave is busy in all of them
        assert here == two, m


SIBLINGS = r'''
#include <cstdio>
#include "plan_rules.hpp"
int main() {                       // lines of: sequences, KV heads, longest, rows, collected rows, token sums, head dimension
  int B, H, n, R, c, tokens, D;
  while (std::scanf("%d %d %d %d %d %d %d", &B, &H, &n, &R, &c, &tokens, &D) == 7)
    std::printf("%d\n", vegas::rows_as_siblings(B, H, n, R, c, tokens, D) ? 1 : 0);
}
'''


def test_wide_rows_as_siblings_where_that_is_faster(tmp_path):
    """(sequences, KV heads, longest, rows, collected rows, token sums, head dimension): siblings measured faster, or not."""
    measured = [((1, 8, 4096, 128, 0, 0, 128), 1), ((8, 8, 2000, 80, 0, 0, 128), 1), ((16, 8, 1200, 80, 0, 0, 128), 1),
                ((1, 4, 32768, 80, 0, 0, 64), 1), ((1, 8, 32768, 128, 0, 0, 64), 0), ((4, 8, 16384, 80, 0, 0, 64), 0),
                ((1, 4, 4096, 80, 1, 0, 128), 1), ((1, 8, 12345, 80, 1, 0, 128), 1), ((1, 8, 12345, 128, 1, 0, 128), 0),
                ((2, 8, 8192, 80, 1, 0, 128), 0), ((8, 8, 2000, 80, 1, 0, 128), 0), ((2, 8, 8192, 80, 2, 0, 128), 1),
                ((1, 4, 32768, 80, 2, 0, 64), 1), ((1, 8, 32768, 128, 2, 0, 128), 0), ((16, 8, 1200, 80, 2, 0, 64), 0),
                ((4, 8, 16384, 80, 2, 0, 128), 0), ((1, 8, 4096, 40, 1, 0, 128), 0), ((1, 8, 4096, 64, 0, 0, 128), 0),
                ((1, 8, 12345, 32, 1, 1, 64), 1), ((1, 8, 32749, 32, 1, 1, 64), 0), ((1, 8, 12345, 40, 1, 1, 64), 0),
                ((1, 8, 4096, 96, 2, 1, 128), 1), ((1, 8, 32749, 96, 1, 1, 128), 0), ((1, 8, 32749, 80, 1, 1, 64), 1),
                ((1, 8, 32749, 64, 2, 1, 128), 1), ((1, 8, 32749, 64, 1, 1, 128), 0), ((4, 8, 16384, 80, 1, 1, 64), 0),
                ((16, 8, 1200, 64, 1, 1, 128), 0), ((65, 8, 16384, 80, 1, 0, 64), 1), ((65, 8, 65536, 80, 2, 0, 128), 1),
                ((65, 8, 65536, 80, 0, 0, 128), 0), ((65, 8, 65536, 40, 1, 0, 128), 0), ((64, 8, 65536, 80, 1, 0, 128), 0),
                ((65, 8, 1 << 24, 80, 1, 0, 128), 0), ((65, 1, 1 << 30, 128, 2, 0, 64), 0),
                ((1, 8, 4096, 31, 1, 1, 128), 1), ((1, 8, 4096, 30, 1, 1, 128), 0)]
    out = run_host_program(tmp_path, SIBLINGS, "\n".join(" ".join(map(str, m)) for m, _ in measured)).split()
    assert [int(x) for x in out] == [s for _, s in measured]


SHARES = r'''
#include <cstdio>
#include "vegas_common.hpp"
struct Host { static float rcp(float x) { return 1.f / x; } };
int main() {                       // lines of: units of all sequences with what further pieces cost, sequences, workgroups, margin
  unsigned priced, lives, J, margin;
  while (std::scanf("%u %u %u %u", &priced, &lives, &J, &margin) == 4)
    std::printf("%u\n", vegas::least_shared_chunk<Host>(priced, lives, J, (priced + J - 1u) / J, margin));
}
'''


def test_batches_are_cut_into_shares_where_that_is_faster(tmp_path):
    """(units of all sequences + 3 for every one but the first, sequences, workgroups, longest equal chunk, margin: 2, or 4 of
    64-row workgroups): shares measured faster, or not; and the shortest such chunk by its definition, for batches up to the longest there are."""
    measured = [((718, 8, 32, 25, 2), 1), ((1312, 16, 32, 54, 2), 1), ((1099, 12, 32, 41, 4), 1), ((2110, 24, 32, 105, 4), 1),
                ((781, 48, 64, 17, 4), 1), ((1375, 32, 64, 27, 4), 1), ((336, 32, 32, 12, 2), 0), ((627, 4, 32, 21, 2), 0),
                ((145, 16, 32, 4, 2), 0), ((105, 8, 32, 3, 2), 0), ((230, 2, 64, 4, 4), 0), ((872, 7, 32, 31, 4), 0),
                ((778, 48, 32, 23, 2), 0), ((778, 48, 32, 500, 2), 0)]
    rng = np.random.default_rng(5)
    drawn = [(int(np.exp(rng.uniform(0, np.log((1 << 23) + 189)))), int(rng.integers(1, 65)), int(rng.integers(1, 257)), int(rng.choice([2, 4]))) for _ in range(4000)]
    drawn += [((1 << 23) + 189, 64, J, 2) for J in range(1, 257)] + [(10 * J * c // 11 + k, 1, J, 2) for J in (1, 7, 32, 256) for c in (11, 1000, 30000) for k in (-1, 0, 1)]
    out = [int(x) for x in run_host_program(tmp_path, SHARES, "\n".join(" ".join(map(str, c)) for c in [m[:3] + m[4:] for m, _ in measured] + drawn)).split()]
    for ((_, lives, J, C, _), shares), least in zip(measured, out):
        assert (lives <= J and C >= least) == shares, (C, least)
    for (priced, lives, J, margin), least in zip(drawn, out[len(measured):], strict=True):
        def holds(C):
            return 10 * J * C > 11 * priced + 8 * lives and C >= -(-priced // J) + margin
        assert holds(least) and not holds(least - 1), (priced, lives, J, margin, least)


ALONE = r'''
#include <cstdio>
#include "plan_rules.hpp"
int main() {                       // lines of: sequences, longest, head dimension (20 rows, 8 KV heads, no collection, 256 compute units)
  int batch, longest, D;
  while (std::scanf("%d %d %d", &batch, &longest, &D) == 3) {
    const vegas::BatchPlan p = vegas::batch_plan(256, 8, batch, longest, 128, 1 << 17, false, false, false, D);
    std::printf("%d\n", p.alone && p.share_margin == vegas::kShareMargin ? 1 : p.alone || p.share_margin >= 0 ? 2 : 0);
  }
}
'''


def test_workgroups_alone_on_a_compute_unit_where_that_is_faster(tmp_path):
    """Measured faster alone (and cut into shares), or not; never with more sequences than workgroups, whose bound says nothing
    about their lengths."""
    measured = [((16, 1200, 128), 0), ((18, 2500, 128), 0), ((8, 6000, 128), 0), ((20, 2600, 128), 1), ((30, 2000, 128), 1),
                ((24, 2500, 128), 1), ((28, 2200, 128), 1), ((32, 1900, 128), 1), ((24, 20011, 128), 1), ((12, 65536, 128), 1),
                ((20, 2600, 64), 0), ((30, 2000, 64), 0), ((32, 1900, 64), 0), ((24, 20011, 64), 1), ((12, 65536, 64), 1),
                ((64, 800, 128), 0), ((64, 131072, 128), 0), ((33, 1 << 20, 128), 0)]
    out = run_host_program(tmp_path, ALONE, "\n".join(" ".join(map(str, m)) for m, _ in measured)).split()
    assert [int(x) for x in out] == [s for _, s in measured]


BAND_WAVES = r'''
#include <cstdio>
#include "plan_rules.hpp"
int main() {                       // lines of: columns, row blocks, tokens of the band, head dimension, rows (256 compute units)
  int columns, blocks, seen, D, rows;
  while (std::scanf("%d %d %d %d %d", &columns, &blocks, &seen, &D, &rows) == 5)
    std::printf("%d\n", vegas::eight_wave_band(columns, blocks, 256, seen, D, rows) ? 1 : 0);
}
'''


def test_eight_waves_take_a_band_where_that_is_faster(tmp_path):
    """(columns, row blocks, tokens of the band, head dimension, rows): eight waves measured faster than four, or not; with one row block of
    head dimension 128 or of few rows they are slower than four from seven to eleven tiles, and where the call reads much."""
    measured = [((8, 1, 97, 128, 20), 0), ((8, 1, 98, 128, 20), 1), ((8, 1, 132, 128, 20), 1), ((128, 1, 128, 64, 8), 1), ((8, 1, 204, 128, 20), 0),
                ((8, 1, 260, 128, 20), 0), ((8, 1, 324, 128, 20), 0), ((8, 1, 388, 128, 20), 1), ((32, 1, 388, 128, 20), 1), ((32, 1, 444, 128, 20), 0),
                ((16, 1, 634, 128, 20), 1), ((16, 1, 1004, 128, 20), 0), ((32, 1, 516, 128, 20), 0), ((16, 1, 630, 128, 8), 0), ((64, 1, 256, 128, 4), 0),
                ((8, 1, 204, 64, 20), 1), ((8, 1, 324, 64, 20), 1), ((8, 1, 201, 64, 16), 0), ((32, 1, 440, 64, 4), 1), ((8, 1, 1004, 64, 20), 1),
                ((24, 1, 1004, 64, 20), 0), ((8, 2, 204, 128, 40), 1), ((64, 2, 1004, 128, 40), 1), ((128, 2, 132, 64, 40), 1), ((129, 2, 132, 64, 40), 0),
                ((256, 1, 132, 64, 20), 1), ((264, 1, 132, 64, 20), 0)]
    out = run_host_program(tmp_path, BAND_WAVES, "\n".join(" ".join(map(str, m)) for m, _ in measured)).split()
    assert [int(x) for x in out] == [w for _, w in measured]


PARTS = r'''
#include <cstdio>
#include "plan_rules.hpp"
int main() {                       // lines of: columns, head dimension, KV heads
  int columns, D, heads;
  while (std::scanf("%d %d %d", &columns, &D, &heads) == 3) {
    const int32_t rounds = vegas::column_rounds(columns, heads);
    int right = vegas::round_columns(rounds) == static_cast<uint32_t>(columns);
    for (int c = 0; c < columns; ++c) right &= vegas::round_sequence(rounds, c) == static_cast<uint32_t>(c / heads);
    std::printf("%d %d %d\n", vegas::draft_value_parts(columns, 256, D), vegas::part_grid_width(heads), right);
  }
}
'''


def test_parts_of_a_column_meet_on_one_xcd(tmp_path):
    """Draft calls split by parts of V: how many (four, two or one workgroup per column while there are compute units for them), and the grid
    (width, part, columns / width): every column once, by a rule that needs no division where the width is the number of heads, and all parts of a
    column on one of the 8 XCDs, round which workgroups go in the order of the grid; and a column's sequence without a division."""
    edges = [((1, 128, 8), 4), ((64, 128, 8), 4), ((65, 128, 8), 2), ((128, 128, 8), 2), ((129, 128, 8), 1), ((64, 64, 8), 2), ((128, 64, 8), 2),
             ((129, 64, 8), 1), ((1, 64, 8), 2)]
    shapes = [(batch * heads, 128, heads) for heads in range(1, 34) for batch in (1, 2, 3, 5, 16, 31) if batch * heads <= 128]
    out = [tuple(map(int, line.split()))
           for line in run_host_program(tmp_path, PARTS, "\n".join(" ".join(map(str, a)) for a in [e for e, _ in edges] + shapes)).strip().split("\n")]
    assert [parts for parts, _, _ in out[:len(edges)]] == [p for _, p in edges]
    assert all(right for _, _, right in out)
    for (columns, _, heads), (parts, width, _) in zip(shapes, out[len(edges):], strict=True):
        assert width == heads or heads % 8, (heads, width)
        place = {}
        for z in range(-(-columns // width)):
            for y in range(parts):
                for x in range(width):
                    if x + width * z < columns:
                        place.setdefault(x + width * z, []).append((x + width * (y + parts * z)) % 8)
        assert sorted(place) == list(range(columns)), (columns, heads)
        assert all(len(p) == parts and len(set(p)) == 1 for p in place.values()), (columns, heads, width)


WIDE = r'''
#include <cstdio>
#include "plan_rules.hpp"
int main() {                       // lines of: collected rows, sequences, chunks
  int rows, batch, chunks;
  while (std::scanf("%d %d %d", &rows, &batch, &chunks) == 3) std::printf("%d\n", vegas::finalize_is_wide(rows, batch, chunks) ? 1 : 0);
}
'''


def test_score_workgroups_are_wide_where_that_is_faster(tmp_path):
    """(collected rows, sequences, chunks): five rounds of pairs in flight measured faster than three, or not."""
    measured = [((192, 1, 32), 0), ((196, 1, 32), 1), ((208, 1, 12), 1), ((320, 1, 16), 1), ((384, 1, 32), 0), ((256, 1, 96), 0), ((224, 1, 48), 0),
                ((256, 2, 16), 1), ((320, 4, 16), 1), ((256, 8, 4), 0), ((320, 8, 4), 0), ((256, 16, 16), 0), ((256, 65, 2), 0), ((256, 65, 32), 1), ((280, 65, 17), 1), ((320, 128, 8), 0)]
    out = run_host_program(tmp_path, WIDE, "\n".join(" ".join(map(str, m)) for m, _ in measured)).split()
    assert [int(x) for x in out] == [w for _, w in measured]


STEPS = r'''
#include <cstdio>
#include "attn_finalize.hpp"
int main() {
  for (int step : vegas::kSmallMerges) std::printf("%d %d\n", step, vegas::small_merge_below(step));
}
'''


def test_merges_by_number_of_chunks_share_one_ladder(tmp_path):
    """What a merge kernel takes for sure is the step below the one it is built for, of the steps that the launch goes through."""
    steps = [tuple(map(int, line.split())) for line in run_host_program(tmp_path, STEPS).strip().split("\n")]
    assert [b for _, b in steps] == [0] + [s for s, _ in steps[:-1]] and steps[-1][0] == 64
