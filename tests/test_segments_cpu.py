"""How the marches are cut into segments: the rule's own code, compiled for the
host, and the registers of the built kernels that it assumes."""
import os
import shutil
import subprocess

import pytest

from kernel_resources import kernels
from paper_2203_13760_amd import build

HERE = os.path.dirname(os.path.abspath(__file__))


@pytest.fixture(scope="module")
def cut(tmp_path_factory):
    hipcc = shutil.which("hipcc") or "/opt/rocm/bin/hipcc"
    if not os.path.exists(hipcc):
        pytest.skip("hipcc not available")
    exe = str(tmp_path_factory.mktemp("segments") / "segment_check")
    src = os.path.join(HERE, "native", "segment_check.cpp")
    subprocess.run([hipcc, "-O1", "-std=c++17", "--offload-arch=gfx950", "-Xclang", "-target-feature", "-Xclang",
                    "-packed-fp32-ops", "-x", "hip", "-o", exe, src], check=True, capture_output=True)

    def run(mode, *grids):
        args = [str(x) for g in grids for x in g]
        out = subprocess.run([exe, mode, *args], check=True, capture_output=True, text=True).stdout
        return [tuple(map(int, line.split())) for line in out.splitlines()]
    return run


@pytest.mark.parametrize("n,phys", [((128, 3, 1024), "e"), ((128, 3, 1024), "ns")])
def test_a_flat_box_marches_z_in_segments_of_its_own(cut, n, phys):
    """The z march of a cell-centred 3D step does not take the length of the y axis,
    which no march of its own runs along (two steps at 128 x 3 x 1024: 1077 -> 998 us)."""
    (seg, _, _, _), = cut("solo", (*n, "js", phys))
    assert seg > n[1]


def test_a_full_batch_and_a_lone_grid_take_different_segments(cut):
    """What the batch's test of long segments against each grid alone rests on: both
    its z marches and its marches with x faces are cut differently."""
    grid = (192, 192, 192, "js", "ns")
    (seg, segx), = cut("batch", *[grid] * 8)
    (seg1, segx1), = cut("batch", grid)
    assert (seg, segx) == (64, 64) and seg1 < seg and segx1 < segx


SCHEMES = {"js": 0, "z": 1, "roe": 2, "w3": 3, "jsrus": 4, "w3rus": 5, "nn": 6}
PHYS = {"e": 1, "ns": 2, "v": 0}


@pytest.mark.parametrize("scheme,phys", [(s, p) for s in SCHEMES for p in PHYS])
def test_residencies_of_the_rule_are_those_of_the_kernels(cut, scheme, phys):
    """march_waves and mx_waves against the registers of k_sweep_march and k_sweep_mx
    as built: the 3D grid's two sweeps (above and below the size that stores halo
    images) and the 2D grid's one."""
    if not os.path.exists(build.LIB):
        pytest.skip("libcfd.so is not built")
    found = kernels(build.LIB)
    sch, ph = SCHEMES[scheme], PHYS[phys] if scheme in ("js", "z", "roe") else (1 if phys == "e" else 0)

    def waves(*parts):
        regs = [r for n, (r, _) in found.items() if any(p in n for p in parts)]
        assert regs, parts
        return min(min(512 // (-(-r // 8) * 8) for r in regs), 8)

    small, big, flat = cut("solo", *((*n, scheme, phys) for n in ((40, 40, 40), (96, 96, 96), (128, 128, 1))))
    if scheme == "roe":  # y, z marches
        got = waves(f"k_sweep_marchILi1ELi0ELb0ELi2ELi{ph}EE", f"k_sweep_marchILi2ELi1ELb0ELi2ELi{ph}EE")
        assert small[2] == big[2] == flat[2] == got
        return
    z = waves(f"k_sweep_marchILi2ELi0ELb0ELi{sch}ELi{ph}EE")
    assert small[2] == big[2] == z
    for cell, mode, img in ((small, 2, 1), (big, 2, 0), (flat, 3, 1)):
        assert cell[3] == waves(f"k_sweep_mxILi1ELi{mode}ELb1ELi{sch}ELi{ph}ELb{img}EE"), (mode, img)
