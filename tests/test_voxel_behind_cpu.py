"""Index of the voxel behind a face (the patient step's prefetch) on the CPU:
for voxels on every face of grids up to the limit of 2^31 - 1 voxels it is the
exact sum, so the density read there stays inside the array and the nx * ny
readable entries on either side of it."""
import itertools
import os
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
HIPCC = "/opt/rocm/bin/hipcc"
DRIVER = r"""
#include <stdio.h>
#include "paper_2307_01416_amd/csrc/vpmc_internal.hpp"
int main() {
    unsigned v;
    int stride, up;
    while (scanf("%u %d %d", &v, &stride, &up) == 3)
        printf("%lld\n", (long long)vpmc::voxel_behind(v, stride, up != 0));
}
"""
GRIDS = [(3, 3, 3), (256, 256, 160), (1290, 1290, 1290), (46340, 46340, 1), (1, 46340, 46340), (2**31 - 1, 1, 1),
         (1, 1, 2**31 - 1), (2047, 1024, 1024)]


@pytest.mark.skipif(not os.path.exists(HIPCC), reason="hipcc not installed")
def test_prefetch_index_stays_in_the_margins(tmp_path):
    src, exe = tmp_path / "driver.cpp", tmp_path / "driver"
    src.write_text(DRIVER)
    subprocess.run([HIPCC, "-O1", "-std=c++17", "-I" + ROOT, "-o", str(exe), str(src)], check=True, timeout=300)
    asked, want = [], []
    for nx, ny, nz in GRIDS:
        nvox, margin = nx * ny * nz, nx * ny
        assert nvox < 2**31
        for i, j, k in itertools.product(*({0, n // 2, n - 1} for n in (nx, ny, nz))):
            v = i + nx * (j + ny * k)
            for stride, up in itertools.product((1, nx, nx * ny), (0, 1)):
                asked.append(f"{v} {stride} {up}")
                want.append(v + stride if up else v - stride)
                assert -margin <= want[-1] < nvox + margin   # what is readable
    r = subprocess.run([str(exe)], input="\n".join(asked), capture_output=True, text=True, check=True, timeout=60)
    assert [int(x) for x in r.stdout.split()] == want
