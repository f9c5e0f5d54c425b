"""The split of Stage A's Gram matrices over workgroups (host arithmetic of csrc/sdfp_fit_plan.h), compiled on its own:
every column of every matrix belongs to exactly one slice, their number stays within its bound, and no slice is longer than
its share of the columns makes it (the scores' error grows with a slice's length)."""
import ctypes
import os
import subprocess

import pytest

CSRC = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "paper_2602_05499_amd", "csrc")
SHIM = """
#include "sdfp_fit_plan.h"
extern "C" void slices(const int* w, int n, int* out) {
    const sdfp::FitGramSlices s = sdfp::fit_gram_slices(w, n);
    for (int i = 0; i < n; ++i) out[i] = s.k_per[i];
    for (int i = 0; i <= n; ++i) out[n + i] = s.slice0[i];
}
"""


@pytest.fixture(scope="module")
def slices(tmp_path_factory):
    d = tmp_path_factory.mktemp("fit_plan")
    (d / "shim.cpp").write_text(SHIM)
    subprocess.run(["g++", "-O1", "-std=c++17", "-shared", "-fPIC", "-I", CSRC, "-o", str(d / "shim.so"), str(d / "shim.cpp")],
                   check=True)
    lib = ctypes.CDLL(str(d / "shim.so"))

    def call(widths):
        out = (ctypes.c_int * 7)()
        lib.slices((ctypes.c_int * len(widths))(*widths), len(widths), out)
        return list(out[:len(widths)]), list(out[len(widths):2 * len(widths) + 1])
    return call


@pytest.mark.parametrize("widths", [[32], [64], [128], [192], [256], [992], [4096], [11008], [32, 32], [11008, 11008],
                                    [28672, 28672], [32, 32, 32], [4096, 1024, 1024], [8192, 64, 64], [32, 4096, 32]])
def test_gram_slices_cover_the_columns_within_their_bounds(slices, widths):
    k_per, first = slices(widths)
    assert first[0] == 0
    for i, w in enumerate(widths):
        n = first[i + 1] - first[i]
        assert k_per[i] >= 16 and k_per[i] % 16 == 0
        assert 1 <= n <= 32 and (n - 1) * k_per[i] < w <= n * k_per[i]
        # 128 columns, or a 32nd of them, and less than twice that where they are no whole number of slices
        assert k_per[i] <= max(256, -(-w // 32) + 15)
