"""The cut of a prompt into panels (host arithmetic of csrc/sdfp_prefill_plan.h), compiled on its own: every cut covers the
prompt with panels of at most the workspace's size, is by the plan's own measure never worse than full panels and a rest, and
against cuts that were timed on an MI355X it is never slower than those and never more than 3.5 % above the quickest (another cut
is chosen from 2.5 % on, and the times have 1 % of noise)."""
import ctypes
import os
import subprocess

import pytest

CSRC = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "paper_2602_05499_amd", "csrc")
SHIM = """
#include "sdfp_prefill_plan.h"
using namespace sdfp;
static PfModel model(const int* v) { return PfModel{v[0], v[1], v[2], v[3], v[4], v[5], v[6], v[7], (size_t)v[8] * 1024}; }
extern "C" int cut(const int* v, int rows, int pos0, int* tiles) {
    const PfCut c = pf_cut(model(v), rows, pos0);
    for (int i = 0; i < c.n; ++i) tiles[i] = c.tiles[i];
    return c.n;
}
extern "C" double panel_us(const int* v, int rows, int pos0) {
    return pf_panel_us(model(v), rows, pos0, pf_gemms_us(model(v), (rows + PF_ROWS - 1) / PF_ROWS));
}
extern "C" double rounds(int columns, int my, int n_cu) { return pf_rounds(columns, my, n_cu); }
extern "C" int groups(int n_nt, int my, int n_cu) { return pf_narrow_groups(n_nt, my, n_cu); }
extern "C" int wide(int n_tiles, int my, int n_cu) { return pf_wide_tiles(n_tiles, my, n_cu); }
"""
# d_model, query heads, KV heads, head_dim, d_ffn
MODELS = {"7b": (4096, 32, 32, 128, 11008), "13b": (5120, 40, 40, 128, 13824), "l3-8b": (4096, 32, 8, 128, 14336),
          "70b": (8192, 64, 8, 128, 28672), "small": (1024, 16, 4, 64, 2816), "least": (32, 1, 1, 16, 32),
          "d1536": (1536, 12, 2, 128, 8960), "d2560": (2560, 20, 20, 128, 6912), "d2560-gqa": (2560, 32, 8, 128, 9728),
          "d3072": (3072, 24, 8, 128, 8192), "d4608": (4608, 36, 4, 128, 18432), "hd32": (512, 16, 8, 32, 1376)}
# us of a prompt's forward by its cut (8 layers up to d 3072, 4 beyond)
MEASURED = [
    ("small", 640, {(8, 2): 2005, (5, 5): 2050, (2, 8): 1854}),
    ("small", 1100, {(8, 8, 2): 3556, (8, 5, 5): 3608, (2, 8, 8): 3266}),
    ("small", 1300, {(8, 8, 5): 3901, (5, 8, 8): 3825}),
    ("d1536", 700, {(8, 3): 4227, (7, 4): 4177, (4, 7): 3979}),
    ("d1536", 1300, {(8, 8, 5): 7802, (7, 7, 7): 7509}),
    ("d2560", 513, {(8, 1): 3877, (6, 3): 4319}),
    ("d2560", 1100, {(8, 8, 2): 8719, (6, 6, 6): 7816}),
    ("d2560", 1536, {(8, 8, 8): 10437, (6, 6, 6, 6): 11075}),
    ("d2560", 3500, {(8, 8, 8, 8, 8, 8, 7): 30264, (7, 6, 6, 6, 6, 6, 6, 6, 6): 33698}),
    ("d2560-gqa", 900, {(8, 7): 7429, (5, 5, 5): 8162}),
    ("d2560-gqa", 2000, {(8, 8, 8, 8): 16802, (6, 6, 5, 5, 5, 5): 19704}),
    ("d2560-gqa", 3500, {(8, 8, 8, 8, 8, 8, 7): 33997, (5,) * 11: 41930}),
    ("d3072", 513, {(8, 1): 4142, (5, 4): 4438}),
    ("d3072", 900, {(8, 7): 6592, (5, 5, 5): 7257}),
    ("d3072", 3000, {(8, 8, 8, 8, 8, 7): 25425, (8, 8, 8, 8, 5, 5, 5): 27829}),
    ("7b", 640, {(8, 2): 3756, (2, 8): 3600}),
    ("7b", 1100, {(8, 8, 2): 6645, (2, 8, 8): 6284}),
    ("7b", 3000, {(8, 8, 8, 8, 8, 7): 20251, (8, 8, 8, 8, 4, 6, 5): 19648}),
    ("l3-8b", 576, {(8, 1): 3785, (6, 3): 3788, (1, 8): 3626}),
    ("l3-8b", 1100, {(8, 8, 2): 7166, (2, 8, 8): 6840}),
    ("13b", 513, {(8, 1): 4681, (6, 3): 4524, (3, 6): 4359}),
    ("13b", 777, {(8, 5): 6656, (7, 6): 6258}),
    ("13b", 1024, {(8, 8): 8246, (6, 6, 4): 8163, (4, 6, 6): 8041}),
    ("13b", 2000, {(8, 8, 8, 8): 18256, (6, 6, 6, 8, 6): 17121, (8, 6, 6, 6, 6): 16659}),
    ("13b", 3000, {(8, 8, 8, 8, 8, 7): 29746, (6, 6, 6, 6, 6, 6, 6, 5): 30210, (4, 6, 6, 6, 6, 6, 5, 8): 28048, (8, 6, 6, 6, 6, 8, 7): 28444}),
    ("d4608", 1300, {(8, 8, 5): 10677, (7, 7, 7): 10252}),
    ("d4608", 2500, {(8, 8, 8, 8, 8): 22786, (7, 7, 7, 7, 7, 5): 21357, (5, 7, 7, 7, 7, 7): 21068, (3, 8, 7, 7, 7, 8): 22127}),
]


def compile_plan(folder):
    (folder / "shim.cpp").write_text(SHIM)
    subprocess.run(["g++", "-O1", "-std=c++17", "-shared", "-fPIC", "-I", CSRC, "-o", str(folder / "shim.so"), str(folder / "shim.cpp")],
                   check=True)
    lib = ctypes.CDLL(str(folder / "shim.so"))
    lib.panel_us.restype = lib.rounds.restype = ctypes.c_double
    return lib


@pytest.fixture(scope="module")
def plan(tmp_path_factory):
    return compile_plan(tmp_path_factory.mktemp("plan"))


def _model(m, n_cu=256, max_tiles=8, max_seq=4200):
    """The plan's view of a workspace of up to 1 GB for such panels: regions of split partials, and the larger room for the others."""
    d, H, Hkv, hd, F = m
    hq, grp = H * hd, H // Hkv
    row = d * 4 + 2 * hq * 4 + 4 + 6 * max(d, hq) + 6 * F + 8 * d * 4
    region = -(-max_seq // 128) * 16 * grp * (hd + 2) * 4
    regions = min(512, ((1 << 30) - 64 * max_tiles * row) // region)
    room = max(8 * 64 * max_tiles * d, regions * region // 4)
    return (ctypes.c_int * 9)(d, hq, Hkv * hd, F, n_cu, hd, max_tiles, regions, room // 1024)


def cut(plan, m, n, n_cu=256, max_tiles=8, max_seq=4200):
    """Row tiles of the panels of an n-row prompt, as the prompt path asks for them."""
    v, out, pos = _model(m, n_cu, max_tiles, max_seq), [], 0
    while pos < n:
        tiles = (ctypes.c_int * 64)()
        k = plan.cut(v, n - pos, pos, tiles)
        assert 1 <= k <= 64 and all(1 <= t <= max_tiles for t in tiles[:k]), (n, pos, tiles[:k])
        out += tiles[:k]
        pos += 64 * sum(tiles[:k])
    assert pos - 64 < n
    return out


def full_panels_and_a_rest(n, max_tiles=8):
    tiles = -(-n // 64)
    return [max_tiles] * (tiles // max_tiles) + [tiles % max_tiles] * (tiles % max_tiles > 0)


def _us(plan, m, n_cu, max_tiles, n, tiles):
    v, pos, us = _model(m, n_cu, max_tiles), 0, 0.0
    for t in tiles:
        us += plan.panel_us(v, min(64 * t, n - pos), pos)
        pos += 64 * t
    return us


@pytest.mark.parametrize("model", MODELS)
@pytest.mark.parametrize("n_cu,max_tiles", [(256, 8), (256, 1), (256, 3), (256, 7), (64, 8), (4, 2)])
def test_cuts_cover_the_prompt(plan, model, n_cu, max_tiles):
    m = MODELS[model]
    for n in (1, 5, 63, 64, 65, 127, 129, 511, 512, 513, 576, 600, 777, 900, 1024, 1100, 2000, 2048, 2049, 4001, 4096, 4097, 5000, 9001):
        tiles = cut(plan, m, n, n_cu, max_tiles)
        plain = full_panels_and_a_rest(n, max_tiles)
        assert sum(tiles) == sum(plain)
        us, plain_us = (_us(plan, m, n_cu, max_tiles, n, c) for c in (tiles, plain))
        assert us <= plain_us * (1 + 1e-12) and (tiles == plain or us <= 0.975 * plain_us or n > 4096), (n, tiles)


@pytest.mark.parametrize("model,n,times", MEASURED)
def test_the_chosen_cut_is_a_quick_one(plan, model, n, times):
    tiles = tuple(cut(plan, MODELS[model], n))
    assert tiles in times and times[tiles] <= 1.035 * min(times.values()), tiles
    assert times[tiles] <= times[tuple(full_panels_and_a_rest(n))]


def test_tiles_and_groups(plan):
    # one workgroup per compute unit: four share groups of 64 workgroups; 80 are quicker in three rounds of one share
    assert [plan.groups(n, my, 256) for n, my in ((8, 8), (10, 8), (16, 8), (32, 8), (1, 1), (8, 4))] == [4, 8, 2, 1, 8, 8]
    # gate/up of 512 rows: 7B three tiles, Llama-3-8B two, 13B two; one of a short prompt
    assert [plan.wide(t, 8, 256) for t in (1376, 1792, 1728)] == [3, 2, 2] and plan.wide(1376, 1, 256) == 1
    # 36 columns of 7 row tiles: 252 workgroups, but 35 on an XCD's 32 compute units; two tiles per wave are the quicker two rounds
    assert [plan.rounds(c, my, 256) for c, my in ((36, 6), (36, 7), (32, 8), (40, 8), (1, 1), (264, 1))] == [1, 2, 1, 2, 1, 2]
    assert plan.wide(864, 6, 256) == 3 and plan.wide(864, 7, 256) == 2
