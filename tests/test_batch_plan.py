"""The plan of a batch whose chunk lengths are computed on the GPU, run on the CPU: balanced_slot is compiled for the host with
64 lanes that take turns (the same code, another class in place of the wave's instructions), for the numbers that
batch_plan gives the launch.  Every workgroup's piece is asked for; together they have to cover every sequence once, in distinct
slots that the workspace holds, in the order in which the merge reads them."""
import heapq
import math
import random
import subprocess

import pytest

from paper_2602_07223_amd import build

UNIT, CU = 128, 256
BUILT = {}

PLANS = r'''
#include <setjmp.h>
#include <ucontext.h>
#include <cstdio>
#include <vector>
#include "attn_pair.hpp"
#include "attn_split.hpp"
#include "plan_rules.hpp"
using namespace vegas;

// 64 lanes as coroutines: a lane that comes to an exchange notes its value and lets the next one run; when it runs again all
// have noted theirs.  (Two sets of values: a lane may be one exchange ahead of the last.)
struct Lanes {
  static constexpr int N = 64;
  static inline uint32_t in[2][N], total[2], top[2], prefix[2][N];
  static inline uint64_t set[2];
  static inline int cur, op[N];
  static inline bool started[N], done[N];
  static inline jmp_buf at[N], back;
  static int exchange(uint32_t x) {
    const int k = op[cur]++ & 1;
    in[k][cur] = x;
    if (!_setjmp(at[cur])) _longjmp(back, 1);
    if (cur == 0) {
      total[k] = top[k] = 0u;
      set[k] = 0ull;
      for (int i = 0; i < N; ++i) {
        prefix[k][i] = total[k] += in[k][i];
        top[k] = in[k][i] > top[k] ? in[k][i] : top[k];
        set[k] |= static_cast<uint64_t>(in[k][i] != 0u) << i;
      }
    }
    return k;
  }
  static int lane() { return cur; }
  static uint32_t sum(uint32_t x) { return total[exchange(x)]; }
  static uint32_t max(uint32_t x) { return top[exchange(x)]; }
  static uint32_t prefix_sum(uint32_t x) { const int k = exchange(x); return prefix[k][cur]; }
  static uint64_t ballot(bool x) { return set[exchange(x ? 1u : 0u)]; }
  static uint32_t readlane(uint32_t x, int lane) { return in[exchange(x)][lane & 63]; }
  static float rcp(float x) { return 1.f / x; }
};

struct Call {
  const int* lens;
  int batch, max_len, second, group, slot;
  BatchPlan bp;
  int2* plan;
  BalancedSlot out[64];
};
static Call call;
static ucontext_t fresh[64], home;
static char stack[64][1 << 16];
static void body() {
  const int lane = Lanes::cur;
  const BatchPlan& p = call.bp;
  call.out[lane] = balanced_slot<Lanes>(call.lens, call.batch, call.max_len, p.J, p.J2, call.group, p.JS,
                                        p.share_margin, call.second, p.cap_units, 128, call.slot, call.plan);
  Lanes::done[lane] = true;
  _longjmp(Lanes::back, 1);
}
static BalancedSlot run() {
  for (int i = 0; i < 64; ++i) {
    Lanes::op[i] = 0;
    Lanes::started[i] = Lanes::done[i] = false;
    getcontext(&fresh[i]);
    fresh[i].uc_stack.ss_sp = stack[i];
    fresh[i].uc_stack.ss_size = sizeof stack[i];
    fresh[i].uc_link = nullptr;
    makecontext(&fresh[i], body, 0);
  }
  static volatile int i;
  static volatile bool left;
  do {
    left = false;
    for (i = 0; i < 64; i = i + 1) {
      if (Lanes::done[i]) continue;
      left = true;
      if (_setjmp(Lanes::back)) continue;
      Lanes::cur = i;
      if (Lanes::started[i]) _longjmp(Lanes::at[i], 1);
      Lanes::started[i] = true;
      setcontext(&fresh[i]);
    }
  } while (left);
  for (int l = 1; l < 64; ++l)
    if (call.out[l].b != call.out[0].b || (call.out[0].b >= 0 && (call.out[l].c0 != call.out[0].c0 || call.out[l].chunk != call.out[0].chunk ||
                                                                call.out[l].slot != call.out[0].slot))) {
      std::printf("lanes differ\n");
      std::exit(1);
    }
  return call.out[0];
}

int main() {             // lines of: KV heads, head dimension, rows, collection (0, 1 pages, 2 tokens), longest, sequences, lengths
  int heads, D, rows, collect, max_len, batch;
  while (std::scanf("%d %d %d %d %d %d", &heads, &D, &rows, &collect, &max_len, &batch) == 6) {
    std::vector<int> lens(batch);
    for (int& n : lens) if (std::scanf("%d", &n) != 1) return 1;
    const int tile_rows = rows + (collect == 2 ? 2 : 0);
    const bool pair = tile_rows > 32, two_per_cu = pair && pair_two_per_cu(D, collect);
    const int blocks = (tile_rows + (pair ? kPairRows : 32) - 1) / (pair ? kPairRows : 32);
    int cap = 1 << 24;
    if (collect != 0 && !pair)
      for (cap = 128; split_lds_bytes(4, rows, collect, cap + 128, D) <= 150 * 1024 && cap < (1 << 24);) cap += 128;
    std::vector<int2> plan(batch, int2{-1, 0});
    call.lens = lens.data();
    call.batch = batch;
    call.max_len = max_len;
    call.second = pair ? pair_second_cost(D, collect) : 2;
    call.group = share_group(heads * blocks);
    call.bp = batch_plan(256, heads * blocks, batch, max_len, 128, cap / 128, pair, two_per_cu, collect != 0, D);
    call.plan = plan.data();
    const BatchPlan& p = call.bp;
    std::printf("%d %d %d %d %d", p.J, p.J2, p.JS, p.cap_units, call.group);
    for (int j = 0; j < p.JS; ++j) {
      call.slot = j;
      const BalancedSlot s = run();
      call.plan = nullptr;
      if (s.b >= 0) std::printf(" | %d %d %d %d %d", j, s.b, s.c0, s.chunk, s.slot);
    }
    for (int b = 0; b < batch; ++b) {
      const ColumnSlots cs = column_slots(plan.data(), p.JS, b, heads, 0, 0);
      const ColumnChunks cc = column_chunks(cs, lens[b]);
      std::printf(" ; %lld %d %d %d", static_cast<long long>(cs.off), cc.ns, cc.last, plan[b].y);
    }
    std::printf("\n");
  }
}
'''


def program(tmp_path_factory):
    if "exe" not in BUILT:
        d = tmp_path_factory.mktemp("plans")
        (d / "plans.hip").write_text("#include <cstdlib>\n" + PLANS)
        cmd = [build.hipcc_path(), "--cuda-host-only", "-std=c++17", "-O1", "-U_FORTIFY_SOURCE", "-I", build.CSRC,
               str(d / "plans.hip"), "-o", str(d / "plans")]
        r = subprocess.run(cmd, capture_output=True, text=True)
        assert r.returncode == 0, r.stderr
        BUILT["exe"] = str(d / "plans")
    return BUILT["exe"]


def plans(exe, calls):
    """calls: (KV heads, head dimension, rows, collection, longest, lengths).  One dict per call: the plan's numbers, its pieces
    (workgroup, sequence, first token, tokens, slot) in launch order, and per sequence (first slot, chunks, last slot - first,
    plan entry)."""
    text = "\n".join(" ".join(map(str, (h, D, rows, c, longest, len(lens), *lens))) for h, D, rows, c, longest, lens in calls)
    r = subprocess.run([exe], input=text, capture_output=True, text=True, timeout=600)
    assert r.returncode == 0, r.stdout[-300:] + r.stderr
    out = []
    for line in r.stdout.strip().split("\n"):
        head, *columns = line.split(" ; ")
        nums, *pieces = head.split(" | ")
        d = dict(zip(("J", "J2", "JS", "cap", "group"), map(int, nums.split())))
        d["pieces"] = [tuple(map(int, p.split())) for p in pieces]
        d["columns"] = [tuple(map(int, c.split())) for c in columns]
        d["shares"] = any(c[3] < 0 for c in d["columns"])
        out.append(d)
    assert len(out) == len(calls)
    return out


def check(call, d):
    heads, D, rows, collect, longest, lens = call
    covered, slots = {b: [] for b in range(len(lens))}, set()
    for j, b, c0, chunk, slot in d["pieces"]:
        assert 0 <= b < len(lens) and 0 <= j < d["JS"] and 0 <= slot < d["JS"], (call, j)
        assert chunk > 0 and chunk % UNIT == 0 and c0 % UNIT == 0 and chunk <= d["cap"] * UNIT, (call, j)
        assert slot not in slots, (call, j)
        slots.add(slot)
        covered[b].append((c0, min(c0 + chunk, lens[b]), slot))
    for b, n in enumerate(lens):
        off, ns, last, _ = d["columns"][b]
        got = sorted(covered[b])
        assert ns == len(got) and (n > 0) == (ns > 0), (call, b)
        at = 0
        for i, (lo, hi, slot) in enumerate(got):
            assert lo == at and hi > lo and slot == off + i, (call, b, i)
            at = hi
        assert at == n, (call, b)
        assert last == ns - 1, (call, b)


def wanted(c, d):
    """Would the lengths be cut into shares (by the definition that least_shared_chunk turns round), had the call the slots?"""
    nu = [-(-n // UNIT) for n in c[5]]
    live, J = sum(1 for x in nu if x), d["J"]
    tile_rows = c[2] + (2 if c[3] == 2 else 0)
    if not live or (tile_rows > 32 and c[1] == 64 and c[3] != 1):     # (two workgroups per compute unit)
        return False
    if tile_rows <= 32 and c[3] == 0 and (len(nu) > J or len(nu) * c[4] < (16 if c[1] == 64 else 12) * J * UNIT):
        return False                                                  # (workgroups that park nothing run side by side)
    longest = next(x for x in range(1, max(nu) + 1) if x == max(nu) or sum(-(-u // x) for u in nu) <= J)
    priced, margin = sum(nu) + 3 * (live - 1), 4 if tile_rows > 32 else 2
    S = -(-priced // J)
    return S <= d["cap"] and live <= J and 10 * J * longest > 11 * priced + 8 * live and longest >= S + margin


def load(d, begin=3):
    """The longest a compute unit is busy over the mean, in units of 128 tokens, with `begin` of them for every piece."""
    free = [0] * d["J"]
    total = 0
    for _, _, _, chunk, _ in d["pieces"]:
        t = heapq.heappop(free) + chunk // UNIT + begin
        total += chunk // UNIT
        heapq.heappush(free, t)
    return max(free) / (total / d["J"])


def spread(n, lo, hi):
    return [lo + int((hi - lo) * math.fmod((i + 1) * 0.6180339887498949, 1.0)) for i in range(n)]


def draw(rng):
    heads = rng.choice([1, 2, 3, 4, 5, 6, 8, 8, 16, 32, 64, 128])
    D, collect = rng.choice([128, 64]), rng.choice([0, 1, 1, 2])
    rows = rng.choice([4, 10, 16, 20, 24, 31, 32, 35, 40, 48, 64, 77, 96])
    n = rng.choice([2, 3, 5, 7, 8, 9, 16, 17, 24, 31, 32, 33, 64])
    hi = round(math.exp(rng.uniform(math.log(1), math.log(150000))))
    lo = int(hi * rng.choice([1, 0.9, 0.3, 0.1, 0]))
    lens = [rng.randint(lo, hi) for _ in range(n)]
    for _ in range(rng.choice([0, 0, 1, n // 2])):
        lens[rng.randrange(n)] = rng.choice([0, 1, lo, UNIT, min(UNIT * rng.randint(1, 40), hi)])
    longest = max(max(lens), 1) if rng.random() < 0.6 else 1 << 17
    return heads, D, rows, collect, max(longest, max(lens)), lens


def test_every_plan_covers_every_sequence_once(tmp_path_factory):
    rng = random.Random(20)
    calls = []
    while len(calls) < 500:
        c = draw(rng)
        blocks = -(-(c[2] + (2 if c[3] == 2 else 0)) // (64 if c[2] + (2 if c[3] == 2 else 0) > 32 else 32))
        if c[0] * blocks <= CU:
            calls.append(c)
    seen = set()
    for c, d in zip(calls, plans(program(tmp_path_factory), calls)):
        check(c, d)
        assert d["shares"] == wanted(c, d), c
        if d["shares"]:
            seen.add((d["group"], d["J"] % d["group"] != 0))
    # shares were met with every length of the reversed groups, and where the last group of the first wave is not whole
    assert {g for g, _ in seen} == {1, 2, 4, 8, 16, 32} and {part for _, part in seen} == {False, True}


# KV heads, head dimension, rows, collection, lengths: the mean of a compute unit is longer than a workgroup can park
LONG = [(8, 128, 24, 1, spread(16, 8192, 65536)), (8, 128, 28, 1, spread(16, 8192, 65536)), (8, 128, 32, 1, spread(16, 8192, 65536)),
        (8, 128, 20, 2, spread(16, 8192, 65536)), (8, 128, 28, 1, spread(8, 16384, 131072)), (8, 128, 32, 1, spread(8, 10000, 100000)),
        (8, 64, 32, 1, spread(16, 8192, 65536)), (8, 64, 32, 1, spread(9, 13107, 131072)), (8, 128, 4, 2, [51202] * 9),
        (8, 64, 24, 1, [40945] * 20), (8, 64, 12, 2, [44366] + [31056] * 18), (4, 128, 20, 1, [33248] * 41)]


def test_batches_beyond_the_parking_lds_are_spread_evenly(tmp_path_factory):
    """No compute unit is given more than a fifth above the mean (one wave of the longest chunks, and a few more of them
    behind it, gave 1.25 to 1.77 of it)."""
    calls = [(h, D, rows, c, max(lens), lens) for h, D, rows, c, lens in LONG]
    for c, d in zip(calls, plans(program(tmp_path_factory), calls)):
        check(c, d)
        assert sum(-(-n // UNIT) for n in c[5]) > d["J"] * d["cap"] * 0.9 and not d["shares"], c[:4]
        assert load(d) < 1.2, (c[:4], load(d), len(d["pieces"]))


def test_no_slots_for_shares_that_cannot_be(tmp_path_factory):
    """A workgroup that finds nothing to do waits for a compute unit all the same: where the bound on the lengths rules shares
    out, a call has one per compute unit; where they are possible they are found, down to the shortest such bound."""
    calls = [(8, 128, 20, 1, max(lens), lens) for lens in
             (spread(3, 900, 1500), spread(4, 300, 3000), spread(6, 900, 1500), spread(2, 1000, 10000), spread(16, 400, 500))]
    for c, d in zip(calls, plans(program(tmp_path_factory), calls)):
        assert d["JS"] == d["J"] == 32, c
    rng = random.Random(7)
    calls = []
    for _ in range(1200):                        # few sequences of few units, lengths of every shape
        n, most = rng.randint(2, 12), rng.choice([3, 8, 15, 30, 60, 130])
        lens = [rng.choice([most, rng.randint(1, most), rng.randint(1, most), 1]) * UNIT for _ in range(n)]
        calls.append((rng.choice([8, 16, 32, 64]), 128, rng.choice([20, 40]), rng.choice([0, 1]), max(lens), lens))
    answers = plans(program(tmp_path_factory), calls)
    for c, d in zip(calls, answers):
        check(c, d)
        assert d["shares"] == wanted(c, d), c
    assert sum(d["shares"] for d in answers) > 50
