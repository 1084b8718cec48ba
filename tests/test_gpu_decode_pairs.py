"""The two-launch decode form, bf16 and FP8: which calls take it (1 .. 16 pairs a token), and every number of pairs against the oracles."""
import numpy as np
import pytest
import torch

import test_gpu_fp8
import test_gpu_moe
from paper_2604_26039_amd import ramp, synth

pytestmark = pytest.mark.gpu
DEV = "cuda:0"
DECODE = 0x2000


def decode_configs(rs, fp8):
    cfgs = [c for c in (ramp.fp8_configs if fp8 else ramp.configs)(rs) if c.mode & 0x100 and c.mode & DECODE]
    assert len(cfgs) == (2 if fp8 else 7)
    return cfgs


# wavefronts per pair 8, 4, 2, 1 with and without idle ones; one token, the most that the form takes where k does not divide 16 (ten of
# H = 384), and the most that 64 pairs allow; fewer k-steps than wavefronts
@pytest.mark.parametrize("k", [2, 3, 5, 6, 7, 9, 12, 15, 16])
@pytest.mark.parametrize("fp8", [False, True])
def test_every_number_of_pairs(k, fp8):
    s = synth.Shape("pairs", 384, 640, 24, k)
    mod = test_gpu_fp8 if fp8 else test_gpu_moe
    for t in sorted({1, min(10, 64 // k), 64 // k}):
        L = (mod.Fp8Layer if fp8 else mod.Layer)(s, t, seed=k, x_std=1.5)
        ids, w = synth.routing(t, s, 1.0, seed=k + t)
        ids = ids.copy()
        ids[-1, k // 2] = -1                              # a dropped pair, of the only token where there is one
        ref = L.oracle_rows(ids, w)
        for c in decode_configs(L.rs, fp8):
            print(f"case k={k} T={t} fp8={fp8} {c}", flush=True)
            mod.assert_close(L.run(c, ids, w), ref, f"k={k} T={t} {c}")


# Both sides of T * H = 4096 where k does not divide 16, with T and with H; no such limit where it does; 17 pairs a token
@pytest.mark.parametrize("k,T,H,two", [(6, 3, 1152, True), (6, 4, 1152, False), (3, 10, 384, True), (3, 11, 384, False),
                                       (15, 1, 4096, True), (15, 1, 4224, False), (8, 8, 1152, True), (1, 64, 384, True),
                                       (17, 3, 256, False)])
@pytest.mark.parametrize("fp8", [False, True])
def test_which_calls_take_two_launches(k, T, H, two, fp8):
    """The general form leaves a row per pair in the workspace, its last section; the two-launch form does not touch it.  In the
    general form a configuration gives the bits of its twin without the mode bit."""
    s = synth.Shape("pairs", H, 128, 32, k)
    L = (test_gpu_fp8.Fp8Layer if fp8 else test_gpu_moe.Layer)(s, T, seed=1, x_std=1.5)
    ids, w = synth.routing(T, s, 1.0, seed=1)
    d_ids, d_w = torch.from_numpy(ids).to(DEV), torch.from_numpy(w).to(DEV)
    call, size, every = ((ramp.fused_moe_fp8, ramp.fused_moe_fp8_workspace_bytes, ramp.fp8_configs) if fp8 else
                         (ramp.fused_moe, ramp.fused_moe_workspace_bytes, ramp.configs))
    plain = {c.key(): c for c in every(L.rs)}
    ref, twins = L.oracle_rows(ids, w), 0
    for c in decode_configs(L.rs, fp8):
        print(f"case k={k} T={T} H={H} fp8={fp8} {c}", flush=True)
        ws = torch.full((size(L.rs, c),), 0xFF, dtype=torch.uint8, device=DEV)
        out = torch.empty((T, H), dtype=torch.bfloat16, device=DEV)
        call(L.rs, c, L.X, d_ids, d_w, L.packed, out, ws)
        untouched = bool((ws[-T * k * H * 4:] == 0xFF).all())
        assert untouched == two, f"{c}"
        (test_gpu_fp8 if fp8 else test_gpu_moe).assert_close(out, ref, f"{c}")
        twin = plain.get(c.key()[:5] + (c.mode & ~DECODE,))
        if twin is not None and not two:
            twins += 1
            assert torch.equal(L.run(twin, ids, w).view(torch.int16), out.view(torch.int16)), f"{c}"
    assert two or twins == (0 if fp8 else 6)
