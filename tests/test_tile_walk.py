"""The tile walk of the persistent kernels (csrc/tile_walk.h), compiled for the host and enumerated: whatever the sizes and the
sharing of experts, the workgroups of a launch take every tile exactly once, whole or in all of its column parts."""
import ctypes
import os
import shutil
import subprocess

import numpy as np
import pytest

from paper_2604_26039_amd import build as lib_build

SOURCE = r"""
#include <cstdint>
#include "tile_walk.h"
struct Map {
    int n_tiles, group_m_req, group_m, group_n, blocks_n;
    unsigned long long block_magic, gm_magic, n_magic, bn_magic;
};
extern "C" int first_of_run(int m_tiles, int c) { return ramp::first_of_run(m_tiles, c); }
extern "C" int share_runs() { return ramp::kShareRuns; }
// taken[m_tiles][n_tiles]: quarters of the tile that have been taken; info: xm_log, and per workgroup the quarters taken by the one
// with the most and the least.  -1: a tile or a position out of range.
extern "C" int walk(int n_tiles, int group_m_req, int m_cap, int m_tiles, int same, int max_parts, int32_t *taken, int32_t *info)
{
    Map a = {n_tiles, group_m_req};
    ramp::tile_map(a);
    const int per_round = 8 * a.group_m;
    const long ids = (long)(m_cap + per_round - 1) / per_round * per_round * n_tiles;
    const int grid = ids < 256 ? (int)ids : 256;
    info[1] = 0, info[2] = 1 << 30;
    for (int id = 0; id < grid; ++id) {
        const ramp::TileWalk w = ramp::tile_walk(a, id & 7, id >> 3, grid >> 3, m_tiles, same, max_parts);
        int own = 0;
        info[0] = w.xm_log;
        for (int pos = ramp::walk_first(w); pos < w.whole; pos = ramp::walk_next(w, pos)) {
            int n = -1, m = -1;
            if (ramp::walk_slot(w, pos) >= w.total) return -1;
            ramp::tile_of_slot(a, w, ramp::walk_slot(w, pos), n, m);
            if (n < 0 || n >= n_tiles || m < 0 || m >= m_tiles) return -1;
            const int parts = pos < 0 ? 4 >> w.cut : 4;
            if (pos < 0 && (w.cut < 1 || 1 << w.cut > max_parts)) return -1;
            taken[m * n_tiles + n] += parts;
            if (pos < 0) taken[m * n_tiles + n] += 16 << w.part;   // each part once
            own += parts;
        }
        if (own > info[1]) info[1] = own;
        if (own < info[2]) info[2] = own;
    }
    return 0;
}
"""


@pytest.fixture(scope="module")
def walk(tmp_path_factory):
    gxx = shutil.which("g++")
    assert gxx, "needs a host compiler"
    d = tmp_path_factory.mktemp("walk")
    (d / "walk.cpp").write_text(SOURCE)
    subprocess.run([gxx, "-O2", "-Wall", "-Werror", "-std=c++17", "-shared", "-fPIC", "-I", lib_build.CSRC, "-o", str(d / "walk.so"),
                    str(d / "walk.cpp")], check=True)
    lib = ctypes.CDLL(str(d / "walk.so"))

    def run(n_tiles, group_m_req, m_tiles, same=0, max_parts=4, m_cap=None):
        taken = np.zeros((max(m_tiles, 1), n_tiles), np.int32)
        info = np.zeros(3, np.int32)
        rc = lib.walk(n_tiles, group_m_req, max(m_cap or m_tiles, 1), m_tiles, same, max_parts, taken.ctypes.data_as(ctypes.c_void_p),
                      info.ctypes.data_as(ctypes.c_void_p))
        assert rc == 0, (n_tiles, group_m_req, m_tiles, same, max_parts)
        return taken[:m_tiles], info
    run.lib = lib
    return run


M_TILES = [0, 1, 2, 3, 7, 8, 9, 13, 16, 17, 24, 31, 32, 33, 36, 40, 63, 64, 65, 72, 100, 128, 257, 300]


@pytest.mark.parametrize("n_tiles", [1, 2, 3, 4, 5, 6, 7, 8, 9, 11, 16, 17, 28, 32, 56, 112])
def test_every_tile_is_taken_once(walk, n_tiles):
    for group_m_req in (0, 2, 4, 8):
        for m_tiles in M_TILES:
            for same in (0, 12, 28):
                for max_parts in (1, 2, 4):
                    for m_cap in (m_tiles, m_tiles + 5 * n_tiles):
                        taken, info = walk(n_tiles, group_m_req, m_tiles, same, max_parts, m_cap)
                        whole = taken == 4
                        cut = (taken == 4 + 16 * 3) | (taken == 4 + 16 * 15)      # both of two parts, all of four
                        assert (whole | cut).all(), (n_tiles, group_m_req, m_tiles, same, max_parts, m_cap)
                        assert max_parts > 1 or whole.all()


@pytest.mark.parametrize("n_tiles,m_tiles,parts,longest,shortest", [
    (112, 13, 4, 24, 20),       # 1456 tiles over 8 x 32 workgroups: five or six each, no XCD has twice another's
    (8, 36, 4, 5, 4),           # one turn and four tiles an XCD: those in four parts
    (8, 36, 1, 8, 4),           # (not cut)
    (16, 13, 4, 4, 0), (16, 13, 1, 4, 0),       # 26 of 32: nothing to cut
    (8, 64, 1, 8, 8), (3, 1, 4, 1, 0)])
def test_shares(walk, n_tiles, m_tiles, parts, longest, shortest):
    _, info = walk(n_tiles, 0, m_tiles, 0, parts)
    assert (info[1], info[2]) == (longest, shortest)


def test_split_of_a_round(walk):
    """4 M-tiles x 8 N-tiles (xm = 2) where an XCD's block is one M-tile, 4 x 8 (xm = 4) where it is two; never for a GROUP_M shape or less
    than a round."""
    assert [walk(32, 0, 40, same)[1][0] for same in (0, 11, 12, 18, 19, 28)] == [3, 3, 2, 2, 1, 1]
    assert [walk(16, 0, 40, same)[1][0] for same in (0, 11, 12, 28)] == [3, 3, 2, 2]
    assert walk(32, 4, 40, 28)[1][0] == 3 and walk(32, 0, 7, 28)[1][0] == 3 and walk(8, 0, 40, 28)[1][0] == 3
    assert walk(33, 0, 40, 28)[1][0] == 3


def same_of(walk, tiles_per_expert):
    """What the kernels count on the tile table of these experts; every entry that they read exists."""
    table = np.repeat(np.arange(len(tiles_per_expert)), tiles_per_expert)
    same = 0
    for c in range(walk.lib.share_runs()):
        first = walk.lib.first_of_run(len(table), c)
        assert 0 <= first and first + 8 <= len(table)
        run = table[first:first + 8]
        same += int((run[1:] == run[:-1]).sum())
    return same, len(table)


def test_split_does_not_depend_on_the_order_of_the_experts(walk):
    """Rare experts in front of heavy ones, behind them and among them; the first eight M-tiles alone told these apart.  (Few heavy experts
    among many rare ones: which of them the runs meet is chance.)"""
    rng = np.random.default_rng(1)
    for tiles, split in (([1] * 8 + [8] * 8, True), ([1] * 12 + [9] * 3, True), ([1] * 40 + [8], False), ([1] * 100 + [5] * 8, False)):
        for order in [tiles, tiles[::-1]] + ([rng.permutation(tiles) for _ in range(20)] if split else []):
            same, m_tiles = same_of(walk, order)
            for n_tiles in (16, 112):
                assert (walk(n_tiles, 0, m_tiles, same)[1][0] != 3) == split, (n_tiles, tiles, same)


def test_split_by_tiles_per_expert(walk):
    """Two M-tiles an expert and more: split; four and more: by four, wherever the runs begin.  One: not split."""
    for lead in range(9):                                     # shifts the phase of the runs
        for n in (9, 16, 33, 64, 200):
            of = lambda t: walk(112, 0, *same_of(walk, [1 + lead % t] + [t] * n)[::-1])[1][0]
            assert of(1) == 3 and of(2) == 2 and of(4) == of(5) == of(9) == 1, (lead, n)


def test_table_reads_stay_inside(walk):
    for m_tiles in list(range(8, 400)) + [4096, 1 << 20]:
        assert [walk.lib.first_of_run(m_tiles, c) for c in (0, walk.lib.share_runs() - 1)] == [0, m_tiles - 8]
