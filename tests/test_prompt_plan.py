"""The choice between the two kernels of the prompt's attention (host arithmetic of csrc/sdfp_prefill_plan.h), compiled on
its own, against times of both kernels measured on an MI355X: the chosen one is never more than 12 % above the other."""
import ctypes
import os
import subprocess

import pytest

CSRC = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "paper_2602_05499_amd", "csrc")
SHIM = """
#include "sdfp_prefill_plan.h"
extern "C" int on_matrix_cores(int hd, int Hkv, int grp, int M, int pos0, int n_cu, int wg_valu, int wg_mx) {
    return sdfp::pf_attn_on_matrix_cores(sdfp::PfAttnPanel{hd, Hkv, grp, M, pos0, n_cu, wg_valu, wg_mx});
}
extern "C" int panels_hold(int hd, int n) { return sdfp::pf_panels_hold(hd, n); }
extern "C" int queries_in_lds(int lds_bytes, int n_splits) { return sdfp::pf_mx_queries_in_lds(lds_bytes, n_splits); }
"""
# head_dim, KV heads, query heads per KV head, first position of the panel: [(rows, us of k_pf_attn, us of k_pf_attn_mx)]
MEASURED = [
    (128, 4, 1, 0, [(5, 10, 24), (16, 22, 28), (17, 22, 24), (64, 23, 31), (129, 24, 32), (160, 36, 39), (256, 38, 41),
                    (257, 38, 46), (384, 52, 59), (512, 67, 68)]),
    (128, 4, 1, 512, [(1, 23, 71), (8, 45, 76), (16, 76, 79), (64, 77, 85), (512, 124, 121)]),
    (128, 4, 1, 1024, [(1, 47, 123), (8, 84, 127), (16, 135, 130), (512, 183, 176)]),
    (128, 32, 1, 0, [(64, 25, 32), (129, 26, 32), (224, 43, 42), (288, 74, 56), (384, 76, 60), (512, 121, 69)]),
    (128, 40, 1, 0, [(144, 40, 38), (224, 57, 43), (320, 84, 60), (512, 140, 75)]),
    (128, 8, 2, 0, [(5, 17, 26), (8, 24, 27), (12, 33, 29), (16, 43, 30), (129, 44, 33), (136, 44, 36), (512, 124, 69)]),
    (128, 8, 4, 0, [(5, 31, 28), (8, 46, 30), (16, 87, 31), (257, 138, 52), (512, 241, 69)]),
    (128, 8, 4, 512, [(1, 33, 76), (4, 79, 78), (8, 148, 80), (16, 285, 83)]),
    (128, 8, 4, 1536, [(1, 96, 184), (4, 205, 186), (16, 698, 191)]),
    (64, 4, 1, 0, [(5, 8, 16), (12, 15, 17), (16, 17, 17), (17, 17, 14), (64, 18, 19), (128, 18, 19), (129, 18, 19), (160, 28, 23),
                   (256, 30, 24), (512, 52, 38)]),
    (64, 4, 1, 512, [(1, 18, 43), (8, 34, 45), (12, 50, 46), (16, 62, 47)]),
    (64, 4, 1, 1536, [(1, 43, 100), (8, 88, 103), (16, 151, 104)]),
    (64, 32, 2, 0, [(5, 14, 18), (8, 19, 17), (16, 33, 17), (256, 62, 25), (512, 181, 59)]),
    (64, 8, 8, 512, [(1, 36, 45), (4, 117, 46), (16, 462, 48)]),
]


@pytest.fixture(scope="module")
def plan(tmp_path_factory):
    d = tmp_path_factory.mktemp("prompt_plan")
    (d / "shim.cpp").write_text(SHIM)
    subprocess.run(["g++", "-O1", "-std=c++17", "-shared", "-fPIC", "-I", CSRC, "-o", str(d / "shim.so"), str(d / "shim.cpp")],
                   check=True)
    return ctypes.CDLL(str(d / "shim.so"))


@pytest.fixture(scope="module")
def on_matrix_cores(plan):
    return plan.on_matrix_cores


@pytest.mark.parametrize("hd,n_kv,grp,pos0,times", MEASURED)
def test_the_quicker_attention_kernel_is_chosen(on_matrix_cores, hd, n_kv, grp, pos0, times):
    for rows, valu, mx in times:
        chosen = mx if on_matrix_cores(hd, n_kv, grp, rows, pos0, 256, 512, 512) else valu
        assert chosen <= 1.12 * min(valu, mx), (rows, valu, mx)


def test_the_choice_has_an_answer_at_the_limits(on_matrix_cores):
    for hd in (64, 128):
        for rows in (1, 15, 16, 17, 512):
            for n_kv, grp in ((1, 1), (64, 1), (1, 8), (3, 5)):
                for pos0 in (0, 512, 131072):
                    for n_cu in (32, 256):
                        for wg_valu, wg_mx in ((1, 1), (8, 2), (512, 1), (512, 4096)):
                            assert on_matrix_cores(hd, n_kv, grp, rows, pos0, n_cu, wg_valu, wg_mx) in (0, 1)
                assert on_matrix_cores(hd, n_kv, grp, rows, 2560 * 128, 256, 512, 512) == 1   # no room for the other's merge
                assert on_matrix_cores(hd, n_kv, grp, rows, 0, 256, 512, 0) == 0


@pytest.mark.parametrize("lds_bytes", [64 * 1024, 128 * 1024])      # head_dim 64, 128
def test_the_merge_statistics_never_exceed_the_lds(plan, lds_bytes):
    """Also beyond a million positions, where those of a single query do not fit and none are staged."""
    for n in list(range(1, 2000)) + [8191, 8192, 8193, 16383, 16384, 16385, 1 << 20]:
        q = plan.queries_in_lds(lds_bytes, n)
        assert 0 <= q <= 64 and q * n * 8 <= lds_bytes
        assert q == 64 or (q + 1) * n * 8 > lds_bytes


def test_prompts_longer_than_the_vector_kernels_merge_leave_the_panels(plan):
    """A workgroup of k_pf_attn has 20 KB of LDS at head_dim 16 and 32, 8 bytes per split: 2560 splits of 128 positions."""
    for hd in (16, 32):
        assert plan.panels_hold(hd, 5) and plan.panels_hold(hd, 2560 * 128) and not plan.panels_hold(hd, 2560 * 128 + 1)
    for hd in (64, 128):
        assert plan.panels_hold(hd, 1 << 24)
