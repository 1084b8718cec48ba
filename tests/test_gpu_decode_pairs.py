"""The two-launch decode form for every number of pairs per token it takes (1 .. 16), bf16 and FP8, against the oracles."""
import numpy as np
import pytest
import torch

import test_gpu_fp8
import test_gpu_moe
from paper_2604_26039_amd import ramp, synth

pytestmark = pytest.mark.gpu
DECODE = 0x2000


# wavefronts per pair 8, 4, 2, 1 with and without idle ones; one token and the most that 64 pairs allow; fewer k-steps than wavefronts
@pytest.mark.parametrize("k", [2, 3, 5, 6, 7, 9, 12, 15, 16])
@pytest.mark.parametrize("fp8", [False, True])
def test_every_number_of_pairs(k, fp8):
    s = synth.Shape("pairs", 384, 640, 24, k)
    T = 64 // k
    mod = test_gpu_fp8 if fp8 else test_gpu_moe
    L = mod.Fp8Layer(s, T, seed=k, x_std=1.5) if fp8 else mod.Layer(s, T, seed=k, x_std=1.5)
    for t in sorted({1, T}):
        rs = ramp.Shape(t, k, s.E, s.H, s.I)
        ids, w = synth.routing(T, s, 1.0, seed=k + t)
        ids = ids.copy()
        ids[-1, k // 2] = -1                              # a dropped pair
        if fp8:
            cfgs = [c for c in ramp.fp8_configs(rs) if c.mode & DECODE]
            if t != T:                                    # (its helper always runs the whole batch)
                continue
            ref = L.oracle_rows(ids, w)
            outs = [L.run(c, ids, w) for c in cfgs]
        else:
            cfgs = [c for c in ramp.configs(rs) if c.mode & DECODE]
            ids, w = ids[:t].copy(), w[:t].copy()
            ref = L.oracle_rows(ids, w, T=t)
            outs = [L.run(c, ids, w, T=t) for c in cfgs]
        assert len(cfgs) == (2 if fp8 else 7)
        for c, out in zip(cfgs, outs):
            print(f"case k={k} T={t} fp8={fp8} {c}", flush=True)
            mod.assert_close(out, ref, f"k={k} T={t} {c}")


def test_tokens_of_more_pairs_take_the_general_form():
    s = synth.Shape("pairs", 256, 256, 32, 17)
    L = test_gpu_moe.Layer(s, 3, seed=1, x_std=1.5)
    ids, w = synth.routing(3, s, 1.0, seed=1)
    ref = L.oracle_rows(ids, w)
    plain = {(c.bm, c.bn, c.bk, c.waves): c for c in ramp.configs(L.rs) if c.mode & 0x100 and not c.mode & DECODE}
    for c in ramp.configs(L.rs):
        if c.mode & DECODE:
            out = L.run(c, ids, w)
            test_gpu_moe.assert_close(out, ref, f"{c}")
            twin = plain.get((c.bm, c.bn, c.bk, c.waves))
            if twin is not None and twin.mode == c.mode & ~DECODE:
                assert torch.equal(L.run(twin, ids, w).view(torch.int16), out.view(torch.int16))
