"""Align inside a launch that does something else too: with the quantised hidden state of the FP8 layer, and once for all
candidates of the device-selected layer.  Sizes around a workgroup's 1024 pairs and the 2048 tokens where the align becomes
launches of its own again."""
import numpy as np
import pytest
import torch

from oracle import oracle
from paper_2604_26039_amd import ramp, synth, tuner
from test_gpu_fp8 import DEV, Fp8Layer, assert_close

pytestmark = pytest.mark.gpu
S = synth.Shape("am", 384, 384, 20, 2)


@pytest.mark.parametrize("T", [1, 33, 512, 513, 2048, 2049])
def test_fp8_layer(T):
    L = Fp8Layer(S, T, seed=T)
    ids, w = synth.routing(T, S, 0.5, seed=2)
    ids[T // 2, 1] = S.E + 3                                            # a dropped pair
    rows = sorted({0, T // 2, T - 1, *np.random.default_rng(T).integers(0, T, 6).tolist()})
    want = L.oracle_rows(ids, w, rows=rows)
    for cfg in [c for c in ramp.fp8_configs(L.rs) if not c.mode & 0x100]:
        print(f"case T={T} {cfg}", flush=True)
        assert_close(L.run(cfg, ids, w)[torch.tensor(rows, device=DEV)], want, f"T={T} {cfg}")


@pytest.mark.parametrize("T", [2048, 2049])
def test_selected_layer(T):
    X, Wg, Wu, Wd = synth.layer_tensors(S, T, seed=T, device=DEV, x_std=1.0)
    rs = ramp.Shape(T, S.k, S.E, S.H, S.I)
    packed = torch.empty(ramp.pack_bytes(rs), dtype=torch.uint8, device=DEV)
    ramp.pack_weights(rs, Wg, Wu, Wd, packed)
    ids, w = synth.routing(T, S, 0.5, seed=5)
    d_ids = torch.from_numpy(np.ascontiguousarray(ids, np.int32)).to(DEV)
    d_w = torch.from_numpy(np.ascontiguousarray(w, np.float32)).to(DEV)
    cfgs = tuner.Family.of(S, T).cfgs
    # a tile with per-slot weights, one without, and the smallest and the largest token block
    cands = [next(c for c in cfgs if c.mode & ramp.PERSISTENT), next(c for c in cfgs if not c.mode & 0x700),
             min(cfgs, key=lambda c: c.bm), max(cfgs, key=lambda c: c.bm)]
    nbytes = ramp.fused_moe_selected_workspace_bytes(rs, cands)
    for pos, cfg in enumerate(cands):
        print(f"case T={T} {cfg}", flush=True)
        ref, out = (torch.zeros((T, S.H), dtype=torch.bfloat16, device=DEV) for _ in range(2))
        ws = torch.full((ramp.fused_moe_workspace_bytes(rs, cfg),), 0xFF, dtype=torch.uint8, device=DEV)
        ramp.fused_moe(rs, cfg, X, d_ids, d_w, packed, ref, ws)
        ws = torch.full((nbytes,), 0xFF, dtype=torch.uint8, device=DEV)
        ramp.fused_moe_selected(rs, cands, torch.tensor([pos], dtype=torch.int32, device=DEV), X, d_ids, d_w, packed, out, ws)
        torch.cuda.synchronize()
        assert torch.equal(out.view(torch.int16), ref.view(torch.int16)), f"candidate {pos} {cfg}"


def check_tables(raw, base, ids, T, s, bm, what):
    """Sorted pairs, tile table, counts and meta at the front of a workspace against the oracle, surplus tiles (-1) included."""
    names = ("sorted", "tile_expert", "tile_rows", "counts", "meta")
    sorted_, table, counts, meta = oracle.align(ids.reshape(-1), T, s.k, s.E, bm)
    rows = np.zeros_like(table)
    at = base
    for name, want in zip(names, (sorted_, table, rows, counts, meta)):
        got = raw[at:at + want.nbytes].view(np.int32)
        if name != "tile_rows":
            assert np.array_equal(got, want), f"{what}: {name}"
        at += (want.nbytes + 255) // 256 * 256


@pytest.mark.parametrize("T", [3, 20, 700, 2049])
@pytest.mark.parametrize("fill", [0, 1])
def test_tables_written_beside_other_work(T, fill):
    """Every tile of the capacity has its entry: the kernels tell a surplus tile by its -1, so the workspace starts from ids of experts that
    exist (an entry left out would be taken for a tile), with the align of the device-selected layer, of the two-launch form, of the FP8
    layer and the quantiser in one launch and in two, and of a layer by itself."""
    value = torch.tensor([fill], dtype=torch.int32, device=DEV)
    ids, w = synth.routing(T, S, 0.5, seed=7)
    ids = ids.copy()
    ids[::5, 1] = -1
    d_ids, d_w = torch.from_numpy(ids).to(DEV), torch.from_numpy(w).to(DEV)
    X, Wg, Wu, Wd = synth.layer_tensors(S, T, seed=T, device=DEV, x_std=1.0)
    rs = ramp.Shape(T, S.k, S.E, S.H, S.I)
    packed = torch.empty(ramp.pack_bytes(rs), dtype=torch.uint8, device=DEV)
    ramp.pack_weights(rs, Wg, Wu, Wd, packed)
    packed8 = torch.empty(ramp.fp8_pack_bytes(rs), dtype=torch.uint8, device=DEV)
    ramp.fp8_pack_weights(rs, Wg, Wu, Wd, packed8)

    def workspace(nbytes):
        return value.repeat(nbytes // 4 + 1).view(torch.uint8)[:nbytes]

    cfgs = ramp.configs(rs)
    of = lambda want: next(c for c in cfgs if want(c))
    cands = [of(lambda c: c.mode & ramp.PERSISTENT), of(lambda c: not c.mode & (0x700 | ramp.PERSISTENT)),
             of(lambda c: c.mode & 0x100 and c.bm == 4), of(lambda c: c.mode & 0x100 and c.bm == 16),
             of(lambda c: c.mode & 0x100 and c.mode & 0x2000)]
    out = torch.empty((T, S.H), dtype=torch.bfloat16, device=DEV)
    size = ramp.fused_moe_selected_workspace_bytes(rs, cands)
    base = (T * S.k * S.H * 4 + 255) // 256 * 256
    for pos, cfg in enumerate(cands):
        print(f"case T={T} {cfg}", flush=True)
        ws = workspace(ramp.fused_moe_workspace_bytes(rs, cfg))
        ramp.fused_moe(rs, cfg, X, d_ids, d_w, packed, out, ws)
        ref = out.clone()
        check_tables(ws.cpu().numpy(), 0, ids, T, S, cfg.bm, f"layer {cfg}")
        ws = workspace(size)
        ramp.fused_moe_selected(rs, cands, torch.tensor([pos], dtype=torch.int32, device=DEV), X, d_ids, d_w, packed, out, ws)
        check_tables(ws.cpu().numpy(), base, ids, T, S, cfg.bm, f"selected {cfg}")
        assert torch.equal(out.view(torch.int16), ref.view(torch.int16)), f"{cfg}"
    outs = []
    for cfg in ramp.fp8_configs(rs):
        print(f"case T={T} {cfg}", flush=True)
        ws = workspace(ramp.fused_moe_fp8_workspace_bytes(rs, cfg))
        ramp.fused_moe_fp8(rs, cfg, X, d_ids, d_w, packed8, out, ws)
        check_tables(ws.cpu().numpy(), 0, ids, T, S, cfg.bm, f"fp8 {cfg}")
        outs.append(out.float().clone())
        assert (outs[-1] - outs[0]).norm() <= 5e-3 * outs[0].norm(), f"{cfg}"
