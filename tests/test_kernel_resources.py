"""Blocks per CU that the launch rules count on, from the built library's kernel metadata."""
import re
import shutil
import subprocess

import pytest

from paper_2412_01447_amd.build import LIB

TOOLS = "/opt/rocm/llvm/bin/"
VGPRS = 512         # per lane and SIMD of a CU, given out in eights
LDS = 160 * 1024    # bytes per CU


@pytest.fixture(scope="module")
def kernels(tmp_path_factory):
    """{name: (vgprs, spilled, static LDS bytes, threads per block)} of every kernel."""
    d = tmp_path_factory.mktemp("code")
    so = shutil.copy(LIB, d)
    subprocess.run([TOOLS + "llvm-objdump", "--offloading", so], check=True, cwd=d,
                   capture_output=True)
    out = {}
    for f in sorted(d.glob("*gfx950*")):
        text = subprocess.run([TOOLS + "llvm-readelf", "--notes", str(f)], check=True,
                              capture_output=True, text=True).stdout
        # one list item per kernel; its own keys are sorted and indented by four
        for k in re.split(r"\n  - (?=\.)", text)[1:]:
            get = lambda key: re.search(r"^ *(?:- )?\.%s: +(\S+)" % key, k, re.M).group(1)
            name = re.sub(r"^_ZN3pld\d+(\w+?)E+v?N.*$", r"\1", get("name"))
            out[name] = tuple(int(get(x)) for x in (
                "vgpr_count", "vgpr_spill_count", "group_segment_fixed_size",
                "max_flat_workgroup_size"))
    return out


def waves_per_simd(k):
    return min(8, VGPRS // ((k[0] + 7) // 8 * 8))


def blocks_per_cu(k):
    return min(waves_per_simd(k) * 4 // (k[3] // 64), LDS // max(1, k[2]))


def test_no_kernel_spills(kernels):
    assert len(kernels) > 50
    assert {n: k for n, k in kernels.items() if k[1]} == {}


def test_waves_per_simd_of_the_row_forms(kernels):
    """Four waves per SIMD wherever hidden rows are scored, but for the ranking kernels'
    widest whole-row forms."""
    rows = {n: waves_per_simd(k) for n, k in kernels.items()
            if re.match("draft_kernel|draft_part_kernel|rank_hidden|rank_both", n)}
    assert len(rows) > 80
    assert {n: w for n, w in rows.items() if w < 4} == {
        "rank_hidden_kernelILi1ELi12ELi4": 3, "rank_both_kernelILi1ELi11": 3,
        "rank_both_kernelILi1ELi12": 3}


def test_prompt_lookup_blocks_per_cu(kernels):
    """Large batches: two blocks of the 1024- and four of the 512-thread selection per CU,
    eight of the 256-thread one; two of the one-launch drafting of up to 8192 tokens."""
    sel = {k[3]: blocks_per_cu(k) for n, k in kernels.items() if "select_prefix_kernel" in n}
    assert sel == {1024: 2, 512: 4, 256: 8}
    one = [blocks_per_cu(k) for n, k in kernels.items() if "draft_prefix_kernel" in n]
    assert sorted(one) == [1, 2]
