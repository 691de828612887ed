"""The library's host code on the CPU: tests/hoststub/driver.cpp runs it over a
HIP runtime of its own (memory from calloc, kernels that do nothing, allocations
refused and launches timed as a case says) and compares return codes and
launches with the documented ones: device allocations that fail, and the shapes
that tuning picks."""
import os
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
PKG = os.path.join(ROOT, "paper_2307_01416_amd")
CASES = ["geometry", "aperture", "slots", "fallback", "next_call", "autotune", "blocks", "many_histories",
         "counted"]


@pytest.fixture(scope="module")
def driver(tmp_path_factory):
    from paper_2307_01416_amd import build
    if not os.path.exists(build.LIB):
        build.build()
    exe = str(tmp_path_factory.mktemp("hoststub") / "driver")
    # -rdynamic: the library's HIP calls resolve to the program's
    subprocess.run(["g++", "-O1", "-g", "-std=c++17", "-rdynamic", "-o", exe,
                    os.path.join(ROOT, "tests", "hoststub", "driver.cpp"), "-L" + PKG, "-l:libvpmc.so",
                    "-Wl,-rpath," + PKG], check=True, timeout=300)
    return exe


@pytest.mark.parametrize("case", CASES)
def test_host_code(driver, case):
    r = subprocess.run([driver, case], capture_output=True, text=True, timeout=120)
    assert r.returncode == 0, f"{r.returncode}\n{r.stdout}\n{r.stderr}"
