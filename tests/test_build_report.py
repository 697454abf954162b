"""The compiler's own resource report for the device code (CPU only: hipcc cross-compiles without a GPU): no kernel
of the library may use scratch memory -- a register spill in a KV-streaming kernel costs it the very loads it is
built to keep in flight -- and the streaming kernels must fit two waves per SIMD (256 registers per lane)."""
import re

import pytest

from paper_2602_07223_amd import build


@pytest.fixture(scope="module")
def report(tmp_path_factory):
    path = tmp_path_factory.mktemp("asm") / "device.s"
    u = build.kernel_resource_usage(str(path))
    assert u, "the compiler printed no resource report"
    return u, path.read_text()


@pytest.fixture(scope="module")
def usage(report):
    return report[0]


def test_no_kernel_spills_registers(usage):
    spilled = {k: v["scratch_bytes_per_lane"] for k, v in usage.items() if v.get("scratch_bytes_per_lane", 0) != 0}
    assert not spilled, f"kernels with scratch (bytes per lane): {spilled}"


def test_streaming_kernels_fit_two_waves_per_simd(usage):
    streaming = {k: v for k, v in usage.items() if "attn_split_kernel" in k or "attn_pair_kernel" in k or "attn_draft16" in k}
    assert len(streaming) >= 32                      # every instantiation the launch code can pick is in the report
    # (workgroups of a part of V: three splits of five page sizes, and two of them through rings)
    assert len([k for k in streaming if "attn_draft16_parts_kernel" in k]) == 3 * 5 + 2, sorted(streaming)
    for name, v in streaming.items():
        assert v["vgprs"] + v.get("agprs", 0) <= 256, (name, v)
        assert v["occupancy"] >= 2, (name, v)


def foreign_m0_lines(asm: str):
    """Lines of each attn_pair_kernel in the assembly that mention M0, other than the three-instruction loads into LDS of
    its inline assembly; and the number of those loads."""
    loads, foreign = 0, []
    for body in re.findall(r"^_ZN5vegas16attn_pair_kernel\w*:(.*?)^\.Lfunc_end", asm, flags=re.M | re.S):
        body = re.sub(r"[ \t]*;.*", "", body)
        own = re.compile(r"s_mov_b32 m0, s\d+\s+s_nop 0\s+global_load_lds_dwordx4 v\d+, s\[\d+:\d+\]")
        loads += len(own.findall(body))
        foreign += [line.strip() for line in own.sub("", body).splitlines() if re.search(r"\bm0\b|global_load_lds", line)]
    return loads, foreign


def test_m0_belongs_to_the_loads_into_lds(report):
    """attn_pair_kernel writes M0 in inline assembly and cannot say so (a reserved register): the compiler must not use it
    in these kernels."""
    loads, foreign = foreign_m0_lines(report[1])
    assert loads >= 12 * 16 and not foreign, (loads, foreign[:4])
    planted = report[1].replace("s_nop 0\n\tglobal_load_lds", "v_readlane_b32 s0, v1, m0\n\ts_nop 0\n\tglobal_load_lds", 1)
    assert foreign_m0_lines(planted)[1]


WHOLE = r"^_ZN5vegas19attn_draft16_kernelILi(\d+)E()Li([0-3])ELb0ELb0EJEEE\w*:(.*?)^\.Lfunc_end"
PARTS = r"^_ZN5vegas25attn_draft16_parts_kernelILi(\d+)ELi(\d+)ELi([0-3])ELb0EEE\w*:(.*?)^\.Lfunc_end"


def small_page_kernels(asm: str):
    """Code of the draft kernels of pages of 1, 2, 4 or 8 tokens that do not choose by length, by head dimension, head dims of V (those of
    workgroups of a part of V) and log2 of the page size."""
    return {(int(D), int(DV or D), int(page)): body
            for form in (WHOLE, PARTS) for D, DV, page, body in re.findall(form, asm, flags=re.M | re.S)}


def drained_waits(asm: str):
    """Waits for all of a wave's loads, per kernel of small_page_kernels."""
    return {k: len(re.findall(r"s_waitcnt vmcnt\(0\)", body)) for k, body in small_page_kernels(asm).items()}


def test_small_page_draft_kernels_keep_their_prefetch(report):
    """The streaming loops request a tile ahead and wait for the tile at hand only.  Five or six waits for everything are at the
    kernel's ends and in the last tiles (a part of V: six); one or two more are in the loop, where they cost a call of several tiles per wave 6 to 10 %."""
    waits = drained_waits(report[1])
    assert len(waits) == 8 + 12 and max(waits.values()) <= 6, waits


def waits_before_the_stream(asm: str):
    """Loads left under way by the waits before the first contraction, per kernel of small_page_kernels."""
    return {k: [int(n) for n in re.findall(r"s_waitcnt vmcnt\((\d+)\)", body[:body.index("v_mfma")])] for k, body in small_page_kernels(asm).items()}


def test_small_page_draft_kernels_start_without_draining(report):
    """Before a wave's first contraction only what it uses is waited for: the length and the page ids, then its keys' first load.  A
    wait for everything (the next tile's page ids brought into the pool at once, stores of an empty sequence's rows that may be under
    way as far as the compiler knows) cost a call of one tile per wave 0.2 to 0.3 us."""
    waits = waits_before_the_stream(report[1])
    assert len(waits) == 8 + 12 and all(0 not in w for w in waits.values()), waits


def test_m0_belongs_to_the_loads_into_lds_of_draft_parts(report):
    """As above for the workgroups of a part of V each, whose K and V go through rings: 8 loads of K and 2 or 4 of V a tile."""
    rings = [b for b in re.findall(r"^_ZN5vegas25attn_draft16_parts_kernel\w*:(.*?)^\.Lfunc_end", report[1], flags=re.M | re.S) if "global_load_lds" in b]
    assert len(rings) == 2
    for body in rings:
        body = re.sub(r"[ \t]*;.*", "", body)
        own = re.compile(r"s_mov_b32 m0, s\d+\s+s_nop 0\s+global_load_lds_dwordx4 v\d+, s\[\d+:\d+\]")
        foreign = [line.strip() for line in own.sub("", body).splitlines() if re.search(r"\bm0\b|global_load_lds", line)]
        assert len(own.findall(body)) >= 16 and not foreign, foreign[:4]
