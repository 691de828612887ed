"""The library's host code on the CPU: tests/hoststub/driver.cpp runs it over a
HIP runtime of its own (memory from calloc, kernels that do nothing, allocations
refused and launches timed as a case says) and compares return codes and
launches with the documented ones, under the address and undefined-behaviour
sanitizers: device allocations that fail, and the shapes
that tuning picks."""
import os
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
HIPCC = "/opt/rocm/bin/hipcc"
PKG = os.path.join(ROOT, "paper_2307_01416_amd")
ENV = dict(os.environ, ASAN_OPTIONS="detect_leaks=0", UBSAN_OPTIONS="halt_on_error=1:print_stacktrace=1")
CASES = ["geometry", "aperture", "slots", "fallback", "next_call", "autotune", "blocks", "many_histories",
         "counted", "outputs", "few", "many_spots"]


@pytest.fixture(scope="module")
def driver(tmp_path_factory):
    from paper_2307_01416_amd import build
    if not os.path.exists(build.LIB):
        build.build()
    exe = str(tmp_path_factory.mktemp("hoststub") / "driver")
    san = ["-Xarch_host", "-fsanitize=address", "-Xarch_host", "-fsanitize=undefined",
           "-Xarch_host", "-fno-omit-frame-pointer"]
    srcs = [os.path.join(ROOT, "tests", "hoststub", "driver.cpp")]
    srcs += [os.path.join(PKG, "csrc", s) for s in ("vpmc_api.cpp", "tables.cpp")]
    # the host code under the sanitizers, the kernels' launchers from the
    # library; -rdynamic: the library's HIP calls resolve to the program's
    subprocess.run([HIPCC, "--offload-arch=gfx950", "-O1", "-g", "-std=c++17"] + san +
                   ["-rdynamic", "-o", exe] + srcs + ["-L" + PKG, "-l:libvpmc.so", "-Wl,-rpath," + PKG],
                   check=True, timeout=600)
    return exe


@pytest.mark.skipif(not os.path.exists(HIPCC), reason="hipcc not installed")
@pytest.mark.parametrize("case", CASES)
def test_host_code(driver, case):
    r = subprocess.run([driver, case], capture_output=True, text=True, timeout=120, env=ENV)
    assert r.returncode == 0, f"{r.returncode}\n{r.stdout}\n{r.stderr}"
