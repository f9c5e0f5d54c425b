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


def compile_plan(folder):
    (folder / "shim.cpp").write_text(SHIM)
    subprocess.run(["g++", "-O1", "-std=c++17", "-shared", "-fPIC", "-I", CSRC, "-o", str(folder / "shim.so"), str(folder / "shim.cpp")],
                   check=True)
    lib = ctypes.CDLL(str(folder / "shim.so"))
    lib.units.restype = ctypes.c_double
    return lib


@pytest.fixture(scope="module")
def plan(tmp_path_factory):
    return compile_plan(tmp_path_factory.mktemp("plan"))


def cut(plan, m, n, n_cu=256, max_tiles=8):
    """Row tiles of the panels of an n-row prompt."""
    tiles, left = [], n
    while left > 0:
        t = plan.next_panel(*m, n_cu, left, max_tiles)
        assert 1 <= t <= max_tiles and t <= -(-left // 64), (n, left, t)
        tiles.append(t)
        left -= 64 * t
    return tiles


def full_panels_and_a_rest(n, max_tiles=8):
    tiles = -(-n // 64)
    return [max_tiles] * (tiles // max_tiles) + [tiles % max_tiles] * (tiles % max_tiles > 0)


def _units(plan, m, n_cu, n, tiles):
    """The plan's measure of a cut; a last panel of one tile multiplies only the column tiles that it has."""
    rest = n % 64 or 64
    few = 0.8 if rest <= 16 else 0.9 if rest <= 32 else 1.0
    return sum(plan.units(*m, n_cu, t) for t in tiles) - (1 - few) * (plan.units(*m, n_cu, 1) if tiles[-1] == 1 else 0.0)


@pytest.mark.parametrize("model", MODELS)
@pytest.mark.parametrize("n_cu,max_tiles", [(256, 8), (256, 1), (256, 3), (64, 8)])
def test_cuts_cover_the_prompt(plan, model, n_cu, max_tiles):
    m = MODELS[model]
    for n in (1, 5, 63, 64, 65, 127, 129, 511, 512, 513, 576, 600, 777, 900, 1024, 1100, 2000, 4001, 4096, 4097, 5000, 9001):
        tiles = cut(plan, m, n, n_cu, max_tiles)
        plain = full_panels_and_a_rest(n, max_tiles)
        assert sum(tiles) == sum(plain)
        assert _units(plan, m, n_cu, n, tiles) <= _units(plan, m, n_cu, n, plain) + 1e-9, (n, tiles)


def test_cuts_that_are_not_full_panels_and_a_rest(plan):
    # where another cut is chosen it is better by 3 % or more
    for model, n, tiles in (("13b", 513, [6, 3]), ("13b", 777, [7, 6]), ("13b", 2000, [6, 6, 6, 8, 6]), ("small", 600, [5, 5]),
                            ("l3-8b", 576, [6, 3])):
        m = MODELS[model]
        assert cut(plan, m, n) == tiles, (model, n)
        assert _units(plan, m, 256, n, tiles) <= 0.97 * _units(plan, m, 256, n, full_panels_and_a_rest(n))
    for model, n in (("7b", 512), ("7b", 777), ("l3-8b", 1100), ("70b", 1300), ("13b", 512)):
        assert cut(plan, MODELS[model], n) == full_panels_and_a_rest(n), (model, n)


def test_tiles_and_groups(plan):
    # one workgroup per compute unit: four share groups of 64 workgroups; 80 are quicker in three rounds of one share
    assert [plan.groups(w, 256) for w in (64, 80, 128, 256, 1, 32)] == [4, 8, 2, 1, 8, 8]
    # gate/up of 512 rows: 7B three tiles, Llama-3-8B two, 13B two; one of a short prompt
    assert [plan.wide(t, 8, 256) for t in (1376, 1792, 1728)] == [3, 2, 2] and plan.wide(1376, 1, 256) == 1
