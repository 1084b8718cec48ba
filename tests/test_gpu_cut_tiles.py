"""Persistent tiles cut in column parts where the whole turns of an XCD's 32 workgroups leave few: every element against a tile
that is never cut (the same fp32 sums in the same order, so the same bits), sampled rows against the oracle."""
import numpy as np
import pytest
import torch

import test_gpu_fp8
import test_gpu_moe
from paper_2604_26039_amd import ramp, synth

pytestmark = pytest.mark.gpu


# M-tiles of 128 rows x 3 N-tiles over 8 XCDs of 32 workgroups: less than a tile to an XCD; 4, 12 and 16 or 17 of 32; one turn and
# 1, 8, 16 and 17 tiles more; two turns and a few (past three turns nothing is cut).  One expert, and three that share M-tiles' turns.
@pytest.mark.parametrize("m_tiles", [1, 11, 32, 43, 45, 88, 107, 128, 132, 175, 260])
@pytest.mark.parametrize("E,H,I", [(1, 768, 384), (3, 640, 384)])
def test_every_element(m_tiles, E, H, I):
    against_a_tile_that_is_not_cut(m_tiles, E, H, I)


# Rounds that are split between the XCDs, with and without cut tiles behind them: 32 N-tiles of the up-projection (a block of one M-tile;
# split by four) and 16 of the up- or the down-projection (a block of two), 128-row and 256-row tiles; one expert, and three
@pytest.mark.parametrize("m_tiles,E,H,I", [(16, 1, 512, 4096), (18, 1, 512, 4096), (18, 3, 512, 4096), (34, 1, 512, 2048), (36, 3, 512, 2048),
                                           (17, 1, 4096, 384), (34, 1, 4096, 384), (37, 3, 4096, 384), (64, 1, 4096, 384)])
def test_every_element_of_split_rounds(m_tiles, E, H, I):
    against_a_tile_that_is_not_cut(m_tiles, E, H, I)


def against_a_tile_that_is_not_cut(m_tiles, E, H, I):
    s = synth.Shape("cut", H, I, E, 1)
    T = 128 * m_tiles - 37
    rng = np.random.default_rng(m_tiles)
    ids = rng.integers(0, E, (T, 1)).astype(np.int32)
    w = rng.uniform(0.25, 1.0, (T, 1)).astype(np.float32)
    rows = sorted(rng.choice(T, min(T, 12), replace=False).tolist())
    at = torch.tensor(rows, device="cuda:0")
    for fp8 in (False, True):
        mod = test_gpu_fp8 if fp8 else test_gpu_moe
        L = (mod.Fp8Layer if fp8 else mod.Layer)(s, T, seed=H, x_std=1.5)
        cfgs = ramp.fp8_configs(L.rs) if fp8 else ramp.configs(L.rs)
        plain = next(c for c in cfgs if not c.mode & 0x20700 and c.bm == (32 if fp8 else 128) and c.bn == 128)
        want = L.run(plain, ids, w).clone()
        mod.assert_close(want[at], L.oracle_rows(ids, w, rows=rows), f"{plain}")
        persistent = [c for c in cfgs if c.mode & ramp.PERSISTENT]
        assert {128, 256} <= {c.bm for c in persistent}
        for c in persistent:
            print(f"case E={E} T={T} {c}", flush=True)
            assert torch.equal(L.run(c, ids, w).view(torch.int16), want.view(torch.int16)), f"{c}"
