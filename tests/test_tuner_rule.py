"""Which stage kernels the launch-shape tuner times (no GPU needed): built with
g++ from the library's header.  On 256 compute units FP32 times exactly one
kernel, on any other number, and in FP64, all of them."""

import os
import shutil
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CSRC = os.path.join(ROOT, "paper_2205_11052_amd", "csrc")

PROGRAM = """
#include <cstdio>
#include <cstdlib>
#include "tuner_rule.h"
int main(int, char **v) {
  for (int k = 0; k < 3; ++k)
    if (dgw::tuner_times(k, atoi(v[1]), atoi(v[2]), atoi(v[3]), atoll(v[4]), atoi(v[5])))
      std::printf("%d", k);
}
"""


@pytest.fixture(scope="module")
def timed(tmp_path_factory):
    if shutil.which("g++") is None:
        pytest.skip("needs g++")
    d = tmp_path_factory.mktemp("tuner")
    (d / "t.cpp").write_text(PROGRAM)
    exe = str(d / "t")
    subprocess.run(["g++", "-std=c++17", "-Wall", "-Werror", "-I" + CSRC, "-o", exe,
                    str(d / "t.cpp")], check=True, timeout=120)
    return lambda *a: subprocess.run([exe] + [str(int(x)) for x in a], check=True,
                                     capture_output=True, text=True, timeout=10).stdout


@pytest.mark.parametrize("N", [1, 2, 3, 4, 5, 6])
def test_kernels_timed(timed, N):
    for aniso in (False, True):
        for elems in (1, 384, 2000, 6000, 24576, 82944, 32 * 82944):
            assert timed(N, 32, aniso, elems, 256) in ("0", "1")
            for ncu in (32, 64, 128, 304):
                assert timed(N, 32, aniso, elems, ncu) == "012"
            assert timed(N, 64, aniso, elems, 256) == "012"


@pytest.mark.parametrize("N,elems,kernel", [(1, 5099, 1), (1, 5100, 0), (4, 999, 0), (4, 1000, 1),
                                            (4, 1650, 0), (4, 3700, 1), (6, 28999, 0),
                                            (6, 29000, 1)])
def test_edges_of_the_ranges(timed, N, elems, kernel):
    assert timed(N, 32, False, elems, 256) == str(kernel)
