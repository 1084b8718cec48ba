"""The 256-wide persistent tiles on hidden sizes of 256 * n + 128, where the down-projection's last tile is half empty: bf16
against the oracle, FP8 bit for bit against the streaming and staged tiles' oracle."""
import numpy as np
import pytest
import torch

import test_gpu_fp8
import test_gpu_moe
from paper_2604_26039_amd import ramp, synth
from test_gpu_fp8_pingpong import routing_of_counts

pytestmark = pytest.mark.gpu
HALF = 0x20000


# one and a half tile, and more N-tiles than an XCD takes at a time; the last expert's last rows (nothing lies behind them in the
# packed weights); rows around the row blocks; fp32 and (last case) bf16 pair rows
@pytest.mark.parametrize("H,I,k,counts", [(384, 384, 1, [1, 16, 17, 0, 129, 257, 300]), (1152, 896, 2, [255, 256, 40, 288, 289, 3]),
                                          (4480, 512, 2, [700, 5, 800, 530, 1800])])
def test_against_the_oracle(H, I, k, counts):
    s = synth.Shape("half", H, I, len(counts), k)
    ids, w = routing_of_counts(counts, k, s.E, seed=H)
    T = ids.shape[0]
    rows = sorted(np.random.default_rng(1).choice(T, min(T, 40), replace=False).tolist())
    at = torch.tensor(rows, device="cuda:0")
    L = test_gpu_moe.Layer(s, T, seed=I, x_std=1.5)
    cfgs = [c for c in ramp.configs(L.rs) if c.mode & HALF]
    assert [c.bm for c in cfgs] == [128, 256, 288]
    ref = L.oracle_rows(ids, w, rows=rows)
    plain = next(c for c in ramp.configs(L.rs) if c.bm == 128 and c.bn == 128 and not c.mode & 0x700)
    want = L.run(plain, ids, w).float()
    for c in cfgs:
        print(f"case H={H} I={I} k={k} T={T} {c}", flush=True)
        out = L.run(c, ids, w)
        test_gpu_moe.assert_close(out[at], ref, f"{c}")
        assert (out.float() - want).norm() <= 5e-3 * want.norm()          # every row, against a tile that divides H
    F = test_gpu_fp8.Fp8Layer(s, T, seed=I, x_std=1.5)
    cfgs = [c for c in ramp.fp8_configs(F.rs) if c.mode & HALF]
    assert [c.bm for c in cfgs] == [128, 256]
    ref = F.oracle_rows(ids, w, rows=rows)
    plain = next(c for c in ramp.fp8_configs(F.rs) if c.bm == 32 and not c.mode & 0x500)
    want = F.run(plain, ids, w)
    test_gpu_fp8.assert_close(want[at], ref, f"{plain}")
    for c in cfgs:
        print(f"case fp8 H={H} I={I} k={k} T={T} {c}", flush=True)
        assert torch.equal(F.run(c, ids, w).view(torch.int16), want.view(torch.int16)), f"{c}"


def test_many_tiles_per_workgroup_run_twice():
    """Three turns and more of 128-row tiles (fewer of the others) over two N-tiles, the second half empty: the loads of the next tile
    follow a whole tile and half a one in turn.  Every element, twice: FP8 bit for bit, bf16 against a tile that divides H."""
    s = synth.Shape("half", 384, 384, 24, 1)
    T = 60_000
    ids, w = synth.routing(T, s, 0.7, seed=3)
    for fp8 in (False, True):
        mod = test_gpu_fp8 if fp8 else test_gpu_moe
        L = (mod.Fp8Layer if fp8 else mod.Layer)(s, T, seed=9, x_std=1.5)
        cfgs = (ramp.fp8_configs if fp8 else ramp.configs)(L.rs)
        plain = next(c for c in cfgs if c.bm == (32 if fp8 else 128) and c.bn == 128 and not c.mode & (0x700 | HALF))
        want = L.run(plain, ids, w).clone()
        rows = [0, 1, T // 2, T - 1]
        mod.assert_close(want[torch.tensor(rows, device="cuda:0")], L.oracle_rows(ids, w, rows=rows), f"{plain}")
        for c in [c for c in cfgs if c.mode & HALF]:
            print(f"case fp8={fp8} {c}", flush=True)
            outs = [L.run(c, ids, w).clone() for _ in range(2)]
            assert torch.equal(outs[0].view(torch.int16), outs[1].view(torch.int16)), f"{c}"
            if fp8:
                assert torch.equal(outs[0].view(torch.int16), want.view(torch.int16)), f"{c}"
            else:
                assert (outs[0].float() - want.float()).norm() <= 5e-3 * want.float().norm(), f"{c}"
