"""The weight-streaming FP8 kernels, which quantise their token operand in registers, against the FP8 oracle and the FP8 tiles."""
import numpy as np
import pytest
import torch

from paper_2604_26039_amd import ramp, synth
from test_gpu_fp8 import Fp8Layer, assert_close

pytestmark = pytest.mark.gpu


def stream_configs(rs):
    cfgs = [c for c in ramp.fp8_configs(ramp.Shape(1, 1, rs.E, rs.H, rs.I)) if c.mode & 0x100]
    assert len(cfgs) == 7
    return cfgs


# slices per wavefront: fewer than wavefronts (K/128 = 1, 3), uneven shares (5, 9, 17); k that divides 16 or does not; pairs at
# the limit of the two-launch form (64) and past it; rows around the 16-row block
@pytest.mark.parametrize("H,I,E,k,T", [(256, 128, 6, 4, 16), (384, 640, 5, 3, 21), (1152, 256, 4, 2, 33), (2176, 384, 40, 8, 8),
                                       (256, 1152, 3, 1, 49), (256, 128, 64, 16, 5)])
def test_shares_and_row_edges(H, I, E, k, T):
    s = synth.Shape("fp8s", H, I, E, k)
    L = Fp8Layer(s, T, seed=H + I, x_std=1.5)
    ids, w = synth.routing(T, s, 0.5, seed=T)
    ids = ids.copy()
    ids[1::6, 0] = -1                                     # some pairs dropped
    ref = L.oracle_rows(ids, w)
    for cfg in stream_configs(L.rs):
        print(f"case H={H} I={I} E={E} k={k} T={T} {cfg}", flush=True)
        got = L.run(cfg, ids, w)
        assert_close(got, ref, f"H={H} I={I} {cfg}")
        assert torch.equal(L.run(cfg, ids, w).view(torch.int16), got.view(torch.int16))


def test_scales_over_the_whole_range_infinities_and_nan():
    """One expert row per kind of value: codes of the register quantiser are those of the quantising pass, non-finite groups
    included (NaN has no magnitude and becomes +-448), so that streaming and staged tiles see the same operands."""
    s = synth.Shape("fp8s", 512, 256, 4, 1)
    T = 24
    L = Fp8Layer(s, T, seed=4)
    L.X[0] = 0
    for i in range(1, 9):
        L.X[i] *= 2.0 ** (-15 * i)                        # down to scales below the smallest E8M0 byte
    L.X[9, 5] = float("nan")
    L.X[10, 200:204] = float("nan")
    L.X[11, 300] = float("inf")
    L.X[12, 511] = float("-inf")
    L.X[13, 128:256] = float("nan")
    ids = (np.arange(T, dtype=np.int32) % s.E).reshape(T, 1)
    w = np.ones((T, 1), np.float32)
    base = next(c for c in ramp.fp8_configs(L.rs) if not c.mode & 0x500)
    want = L.run(base, ids, w).double().cpu().numpy()
    assert np.isfinite(want).all()
    for cfg in stream_configs(L.rs):
        got = L.run(cfg, ids, w).double().cpu().numpy()
        # same codes, fp32 sums in another order: what is left is the bf16 rounding of activation and output, or, per 128
        # features, the neighbouring scale (half a step of the coarser one, 2^-4, of one element against the row)
        err = np.linalg.norm(got - want, axis=1)
        assert (err <= 2.0 ** -6 * np.linalg.norm(want, axis=1)).all(), (cfg, err)


def test_bf16_pair_rows():
    s = synth.Shape("fp8s", 2048, 256, 8, 8)              # T*k*H >= 8 Mi elements
    T = 520
    L = Fp8Layer(s, T, seed=6)
    ids, w = synth.routing(T, s, 1.0, seed=2)
    rows = list(range(0, T, 40))
    ref = L.oracle_rows(ids, w, rows=rows)
    for cfg in stream_configs(L.rs):
        assert_close(L.run(cfg, ids, w)[torch.tensor(rows, device=L.X.device)], ref, f"{cfg}")
