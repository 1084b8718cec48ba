"""The persistent FP8 kernels against the FP8 oracle and, bit for bit, against a non-persistent FP8 tile: both add the
exact products of the same codes in fp32, one 128-wide k-block after the other, so every bit has to agree."""
import numpy as np
import pytest
import torch

from paper_2604_26039_amd import ramp, synth
from test_gpu_fp8 import DEV, Fp8Layer, assert_close

pytestmark = pytest.mark.gpu


def routing_of_counts(counts, k, E, seed):
    """One pair per token and choice j, expert e getting counts[e] pairs; tokens in random order."""
    rng = np.random.default_rng(seed)
    flat = np.repeat(np.arange(len(counts)), counts)
    flat = np.concatenate([flat, np.full(-len(flat) % k, E + 1)])        # pad to whole tokens with dropped pairs
    ids = rng.permutation(flat).reshape(-1, k).astype(np.int32)
    return ids, rng.random(ids.shape).astype(np.float32)


# rows per expert around the 16-row blocks, the 128-row halves and the 256-row tile; slices per tile: the smallest the
# kernels take (3), one and two more than a 16-slice chunk of scales, several chunks
@pytest.mark.parametrize("H,I,k", [(768, 384, 1), (512, 2176, 2), (4352, 512, 2)])
def test_tile_edges(H, I, k):
    counts = [1, 16, 17, 0, 127, 128, 129, 255, 256, 257, 400, 513]
    s = synth.Shape("pp", H, I, len(counts), k)
    ids, w = routing_of_counts(counts, k, s.E, seed=H)
    T = ids.shape[0]
    L = Fp8Layer(s, T, seed=I, x_std=1.5)
    cfgs = ramp.fp8_configs(L.rs)
    persistent = [c for c in cfgs if c.mode & ramp.PERSISTENT]
    assert {c.bm for c in persistent} == {128, 256}
    base = next(c for c in cfgs if c.bm == 128 and not c.mode & ramp.PERSISTENT)
    want = L.run(base, ids, w).clone()
    rows = sorted(np.random.default_rng(1).choice(T, 12, replace=False).tolist())
    assert_close(want[torch.tensor(rows, device=DEV)], L.oracle_rows(ids, w, rows=rows), f"H={H} I={I} {base}")
    for cfg in persistent:
        print(f"case H={H} I={I} k={k} T={T} {cfg}", flush=True)
        got = L.run(cfg, ids, w)
        assert torch.equal(got.view(torch.int16), want.view(torch.int16)), f"H={H} I={I} {cfg}"


def test_infinities_and_nan_in_the_quantised_activation():
    """Rows of every magnitude up to the largest bf16: products past it, infinities that cancel to NaN, and NaN and infinities in
    the hidden state.  The quantiser of the up-projection's epilogue has to agree with the quantising pass."""
    s = synth.Shape("pp", 512, 384, 3, 1)
    T = 3 * 140
    L = Fp8Layer(s, T, seed=8)
    scale = torch.exp2(torch.linspace(-60, 125, T // 3, device=DEV)).repeat_interleave(3)[:, None]
    L.X[:] = (L.X.float() * scale).bfloat16()
    L.X[3, 5] = float("nan")
    L.X[4, 128:256] = float("nan")
    L.X[5, 300] = float("inf")
    L.X[6, 511] = float("-inf")
    for W, f in ((L.Wg, 32.0), (L.Wu, 32.0), (L.Wd, 2.0 ** -12)):
        W *= f                                                       # activations overflow, outputs do not
    ramp.fp8_pack_weights(L.rs, L.Wg, L.Wu, L.Wd, L.packed)
    g, u = (L.X[9::3].cpu().float() @ W[0].cpu().float() for W in (L.Wg, L.Wu))   # expert 0's tokens, without the quantisation
    act = (torch.nn.functional.silu(g) * u).bfloat16()
    assert torch.isnan(act[-8:]).any() and torch.isinf(act).any() and torch.isfinite(act[:40]).all()
    ids = (np.arange(T, dtype=np.int32) % s.E).reshape(T, 1)
    w = np.ones((T, 1), np.float32)
    cfgs = ramp.fp8_configs(L.rs)
    want = L.run(next(c for c in cfgs if c.bm == 64), ids, w).clone()
    assert torch.isfinite(want.float()).all()
    for cfg in [c for c in cfgs if c.mode & ramp.PERSISTENT]:
        print(f"case {cfg}", flush=True)
        got = L.run(cfg, ids, w)
        assert torch.equal(got.view(torch.int16), want.view(torch.int16)), f"{cfg}"


@pytest.mark.parametrize("T,beta", [(1, 1.0), (300, 1.0), (2050, 0.3)])
def test_many_tiles_per_workgroup_and_bf16_pair_rows(T, beta):
    """One token; tiles fewer than workgroups; several tiles per workgroup with bf16 pair rows (T*k*H >= 8 Mi)."""
    s = synth.Shape("pp", 2048, 768, 24, 6)
    L = Fp8Layer(s, T, seed=T)
    ids, w = synth.routing(T, s, beta, seed=3)
    cfgs = ramp.fp8_configs(L.rs)
    want = L.run(next(c for c in cfgs if c.bm == 64), ids, w).clone()
    for cfg in [c for c in cfgs if c.mode & ramp.PERSISTENT]:
        print(f"case T={T} {cfg}", flush=True)
        for _ in range(2):
            got = L.run(cfg, ids, w)
            assert torch.equal(got.view(torch.int16), want.view(torch.int16)), f"T={T} {cfg}"
