"""The cut of a prompt into panels (host arithmetic of csrc/sdfp_prefill_plan.h), compiled on its own: every cut covers the
prompt with panels of at most the workspace's size, and is by the plan's own measure never worse than full panels and a rest."""
import ctypes
import os
import subprocess

import pytest

CSRC = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "paper_2602_05499_amd", "csrc")
SHIM = """
#include "sdfp_prefill_plan.h"
extern "C" int next_panel(int d, int hq, int hkv, int F, int n_cu, int rows, int max_tiles) {
    return sdfp::pf_next_panel(sdfp::PfModel{d, hq, hkv, F, n_cu}, rows, max_tiles);
}
extern "C" double units(int d, int hq, int hkv, int F, int n_cu, int tiles) {
    return sdfp::pf_panel_units(sdfp::PfModel{d, hq, hkv, F, n_cu}, tiles);
}
extern "C" int groups(int wgs, int n_cu) { return sdfp::pf_narrow_groups(wgs, n_cu); }
extern "C" int wide(int n_tiles, int my, int n_cu) { return sdfp::pf_wide_tiles(n_tiles, my, n_cu); }
"""
MODELS = {"7b": (4096, 4096, 4096, 11008), "13b": (5120, 5120, 5120, 13824), "l3-8b": (4096, 4096, 1024, 14336),
          "70b": (8192, 8192, 1024, 28672), "small": (1024, 1024, 256, 2816), "least": (32, 16, 16, 32)}


@pytest.fixture(scope="module")
def plan(tmp_path_factory):
    d = tmp_path_factory.mktemp("plan")
    (d / "shim.cpp").write_text(SHIM)
    subprocess.run(["g++", "-O1", "-std=c++17", "-shared", "-fPIC", "-I", CSRC, "-o", str(d / "shim.so"), str(d / "shim.cpp")], check=True)
    lib = ctypes.CDLL(str(d / "shim.so"))
    lib.units.restype = ctypes.c_double
    return lib


@pytest.mark.parametrize("model", MODELS)
@pytest.mark.parametrize("n_cu,max_tiles", [(256, 8), (256, 1), (256, 3), (64, 8)])
def test_cuts_cover_the_prompt(plan, model, n_cu, max_tiles):
    m = (*MODELS[model], n_cu)
    for n in (1, 5, 63, 64, 65, 127, 129, 511, 512, 513, 576, 777, 900, 1024, 1100, 2000, 4001, 4096, 4097, 5000, 9001):
        left, cost, last = n, 0.0, max_tiles
        while left > 0:
            t = plan.next_panel(*m, left, max_tiles)
            assert 1 <= t <= max_tiles and t <= -(-left // 64), (n, left, t)
            cost += plan.units(*m, t)
            left -= 64 * t
            last = t
        tiles = -(-n // 64)
        plain = tiles // max_tiles * plan.units(*m, max_tiles) + (plan.units(*m, tiles % max_tiles) if tiles % max_tiles else 0.0)
        assert cost <= plain * 1.03 and last >= 1


def test_tiles_and_groups(plan):
    # one workgroup per compute unit: four share groups of 64 workgroups; 80 are quicker in three rounds of one share
    assert [plan.groups(w, 256) for w in (64, 80, 128, 256, 1, 32)] == [4, 8, 2, 1, 8, 8]
    # gate/up of 512 rows: 7B three tiles, Llama-3-8B two, 13B two; one of a short prompt
    assert [plan.wide(t, 8, 256) for t in (1376, 1792, 1728)] == [3, 2, 2] and plan.wide(1376, 1, 256) == 1
