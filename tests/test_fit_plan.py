"""The split of Stage A's Gram matrices over workgroups (host arithmetic of csrc/sdfp_fit_plan.h), compiled on its own:
every column of every matrix belongs to exactly one slice, the number of slices stays within its bound, and the rule has
an answer on every device size, also where one slice alone is more workgroups than there are compute units."""
import ctypes
import os
import subprocess

import pytest

CSRC = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "paper_2602_05499_amd", "csrc")
SHIM = """
#include "sdfp_fit_plan.h"
extern "C" void slices(int T, const int* w, int n, int n_cu, int* out) {
    const sdfp::FitGramSlices s = sdfp::fit_gram_slices(T, w, n, n_cu);
    out[0] = s.k_per;
    for (int i = 0; i <= sdfp::FIT_GRAM_PARTS; ++i) out[1 + i] = s.slice0[i];
}
"""


@pytest.fixture(scope="module")
def slices(tmp_path_factory):
    d = tmp_path_factory.mktemp("fit_plan")
    (d / "shim.cpp").write_text(SHIM)
    subprocess.run(["g++", "-O1", "-std=c++17", "-shared", "-fPIC", "-I", CSRC, "-o", str(d / "shim.so"), str(d / "shim.cpp")],
                   check=True)
    lib = ctypes.CDLL(str(d / "shim.so"))

    def call(T, widths, n_cu):
        out = (ctypes.c_int * 5)()
        lib.slices(T, (ctypes.c_int * len(widths))(*widths), len(widths), n_cu, out)
        return out[0], list(out[1:2 + len(widths)])
    return call


@pytest.mark.parametrize("n_cu", [32, 64, 128, 256, 304])
def test_gram_slices_cover_the_columns_within_their_bound(slices, n_cu):
    widths = [[32], [64], [128], [192], [256], [992], [4096], [11008], [32, 32], [11008, 11008], [28672, 28672], [32, 32, 32],
              [4096, 1024, 1024], [8192, 64, 64], [32, 4096, 32]]
    for T in [2, 64, 128, 129, 512, 513, 777, 1024, 1500, 2048]:
        for w in widths:
            k_per, first = slices(T, w, n_cu)
            assert k_per >= 16 and k_per % 16 == 0, (T, w)
            assert first[0] == 0
            for i, wi in enumerate(w):
                n = first[i + 1] - first[i]
                assert n >= 1 and (n - 1) * k_per < wi <= n * k_per, (T, w)
            assert first[-1] <= max(32, len(w)), (T, w)
            tb = (T + 127) // 128
            blocks = tb * (tb + 1) // 2
            rounds = max(1, min(32, sum(w) // 128)) * blocks // n_cu
            if rounds > 0:      # whole rounds of the compute units, as long as a slice is no more than that
                assert first[-1] * blocks <= rounds * n_cu or first[-1] <= len(w), (T, w)
