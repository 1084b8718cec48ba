"""GPU parity: ramp_fused_moe against the oracle's per-token definition (fp64, no intermediate
rounding), through the C ABI.

Tolerance (fp32-accumulated bf16 path, one bf16 rounding of the activation and one of the
output): max|d| <= 1e-2 * max|ref| and ||d||_2 / ||ref||_2 <= 5e-3.
Small cases compare every element for every configuration of the family; the benchmark-size
cases compare sampled token rows (rows are independent) in the launch configuration the
benchmark uses."""
import numpy as np
import pytest
import torch

from oracle import oracle
from paper_2604_26039_amd import ramp, synth

pytestmark = pytest.mark.gpu
DEV = "cuda:0"
MAX_TOL, L2_TOL = 1e-2, 5e-3


class Layer:
    """Device tensors of one synthetic layer plus its packed weights."""

    def __init__(self, shape: synth.Shape, T: int, seed: int, x_std=None):
        self.s, self.T = shape, T
        self.X, self.Wg, self.Wu, self.Wd = synth.layer_tensors(shape, T, seed, device=DEV, x_std=x_std)
        self.rs = ramp.Shape(T, shape.k, shape.E, shape.H, shape.I)
        self.packed = torch.empty(ramp.pack_bytes(self.rs), dtype=torch.uint8, device=DEV)
        ramp.pack_weights(self.rs, self.Wg, self.Wu, self.Wd, self.packed)
        torch.cuda.synchronize()

    def run(self, cfg, ids, w, T=None, poison=True):
        T = self.T if T is None else T
        rs = ramp.Shape(T, self.s.k, self.s.E, self.s.H, self.s.I)
        d_ids = torch.from_numpy(np.ascontiguousarray(ids, np.int32)).to(DEV)
        d_w = torch.from_numpy(np.ascontiguousarray(w, np.float32)).to(DEV)
        nbytes = ramp.fused_moe_workspace_bytes(rs, cfg)
        ws = torch.empty(nbytes + 1024, dtype=torch.uint8, device=DEV)
        if poison:
            ws.fill_(0xFF)  # NaN patterns: anything read before it is written shows up
        out = torch.full((T + 1, self.s.H), 777.0, dtype=torch.bfloat16, device=DEV)
        ramp.fused_moe(rs, cfg, self.X[:T], d_ids, d_w, self.packed, out, ws)
        torch.cuda.synchronize()
        assert (ws[nbytes:] == 0xFF).all() if poison else True, "write past the workspace"
        assert (out[T] == 777.0).all(), "write past the output"
        self.last_ws, self.last_rs = ws, rs
        return out[:T]

    def oracle_rows(self, ids, w, rows=None, T=None):
        T = self.T if T is None else T
        rows_l = list(range(T)) if rows is None else list(rows)
        used = sorted({int(e) for t in rows_l for e in ids[t] if 0 <= e < self.s.E})
        pick = lambda W: {e: synth.bits(W[e]) for e in used}
        return oracle.moe(synth.bits(self.X[:T]), ids, w, pick(self.Wg), pick(self.Wu), pick(self.Wd), E=self.s.E,
                          rows=None if rows is None else np.asarray(rows_l, np.int32))


def assert_close(got_bf16: torch.Tensor, ref: np.ndarray, what=""):
    got = got_bf16.float().cpu().numpy().astype(np.float64)
    assert np.isfinite(got).all(), f"{what}: non-finite output"
    d = got - ref
    scale = np.abs(ref).max()
    assert scale > 0
    max_err = np.abs(d).max() / scale
    l2 = np.linalg.norm(d) / np.linalg.norm(ref)
    assert max_err <= MAX_TOL and l2 <= L2_TOL, f"{what}: max {max_err:.3e} (tol {MAX_TOL}), L2 {l2:.3e} (tol {L2_TOL})"
    return max_err, l2


@pytest.fixture(scope="module")
def tiny():
    return Layer(synth.SHAPES["tiny"], 16, seed=1, x_std=2.0)


@pytest.mark.parametrize("beta", [1.0, 0.2])
def test_tiny_every_config(tiny, beta):
    ids, w = synth.routing(16, tiny.s, beta, seed=11)
    ref = tiny.oracle_rows(ids, w)
    cfgs = ramp.configs(tiny.rs)
    assert {4, 16} <= {c.bm for c in cfgs}
    for cfg in cfgs:
        assert_close(tiny.run(cfg, ids, w), ref, f"tiny beta={beta} {cfg}")


def test_tiny_default_scale_inputs():
    L = Layer(synth.SHAPES["tiny"], 16, seed=2)  # X ~ N(0, 1/sqrt(H)): SiLU nearly linear, tiny magnitudes
    ids, w = synth.routing(16, L.s, 0.2, seed=2)
    ref = L.oracle_rows(ids, w)
    for cfg in ramp.configs(L.rs):
        if cfg.bm in (4, 16):
            assert_close(L.run(cfg, ids, w), ref, f"{cfg}")


def test_workspace_holds_the_oracle_align(tiny):
    ids, w = synth.routing(16, tiny.s, 0.2, seed=5)
    for cfg in ramp.configs(tiny.rs):
        if cfg.bm not in (4, 16):
            continue
        tiny.run(cfg, ids, w)
        off = ramp.fused_moe_workspace_layout(tiny.last_rs, cfg)
        s, te, counts, meta = oracle.align(ids.reshape(-1), 16, tiny.s.k, tiny.s.E, cfg.bm)
        raw = tiny.last_ws.cpu().numpy()
        for o, ref in zip(off, (s, te, counts, meta)):
            got = raw[o:o + ref.nbytes].view(np.int32)
            assert np.array_equal(got, ref)


@pytest.fixture(scope="module")
def olmoe_small():
    return Layer(synth.SHAPES["olmoe"], 96, seed=3, x_std=1.0)


@pytest.mark.parametrize("T,beta", [(96, 0.2), (33, 1.0), (1, 1.0)])
def test_olmoe_small_every_config(olmoe_small, T, beta):
    L = olmoe_small
    ids, w = synth.routing(T, L.s, beta, seed=T)
    ref = L.oracle_rows(ids, w, T=T)
    outs = {}
    for cfg in ramp.configs(ramp.Shape(T, L.s.k, L.s.E, L.s.H, L.s.I)):
        out = L.run(cfg, ids, w, T=T)
        assert_close(out, ref, f"olmoe T={T} beta={beta} {cfg}")
        outs[cfg.key()] = out.float().cpu().numpy()
    # all configurations agree up to fp32 summation order and the two bf16 roundings
    vals = list(outs.values())
    for v in vals[1:]:
        assert np.linalg.norm(v - vals[0]) / np.linalg.norm(vals[0]) <= L2_TOL


@pytest.mark.parametrize("H,I,E,k,T,beta", [(128, 128, 4, 2, 700, 1.0), (256, 128, 6, 3, 1500, 0.5), (128, 384, 3, 1, 2500, 1.0)])
def test_smallest_dimensions_many_tiles(H, I, E, k, T, beta):
    """Shortest legal reduction lengths (a tile is as long as the load pipeline is deep) with enough pairs
    that the large-tile kernels walk several tiles per workgroup, full and ragged ones, on every configuration."""
    shape = synth.Shape("edge", H, I, E, k)
    L = Layer(shape, T, seed=H + I, x_std=1.5)
    ids, w = synth.routing(T, shape, beta, seed=T)
    ref = L.oracle_rows(ids, w)
    cfgs = ramp.configs(L.rs)
    assert any(c.mode & ramp.PERSISTENT for c in cfgs) and any(c.mode & 0x100 for c in cfgs)
    for cfg in cfgs:
        assert_close(L.run(cfg, ids, w), ref, f"H={H} I={I} {cfg}")


def test_expert_row_counts_around_the_tile_and_tail_block_sizes():
    """Experts whose pair counts sit on both sides of every row-block boundary that the large tiles know: 256 rows
    (a full tile of the 256-row configurations; the start of the 16-row tail blocks that the 272- and 288-row tiles
    share between their wavefront rows), 272 and 288 (those tiles full), one row more or less, two tiles, an empty
    expert, fewer rows than a block.  top-1 routing makes the counts exact; every element against the oracle on every
    ping-pong configuration."""
    counts = [256, 257, 260, 271, 272, 273, 287, 288, 289, 304, 529, 0, 15, 255, 544, 561, 577]
    shape = synth.Shape("edge", 256, 128, len(counts), 1)
    T = sum(counts)
    L = Layer(shape, T, seed=11, x_std=1.5)
    rng = np.random.default_rng(3)
    ids = np.repeat(np.arange(len(counts), dtype=np.int32), counts)
    rng.shuffle(ids)
    ids = ids.reshape(T, 1)
    w = rng.uniform(0.25, 1.0, size=(T, 1)).astype(np.float32)
    ref = L.oracle_rows(ids, w)
    cfgs = [c for c in ramp.configs(L.rs) if c.mode & ramp.PERSISTENT]
    assert {256, 272, 288} <= {c.bm for c in cfgs}
    for cfg in cfgs:
        assert_close(L.run(cfg, ids, w), ref, f"{cfg}")


def test_persistent_workgroups_walk_several_tiles_every_row():
    """More than 800 M-tiles of one N-tile each, so every one of the 256 persistent workgroups walks three or four
    tiles in both projections: the load stream crosses tile boundaries, the token and weight rings wrap, and the
    tail-block tiles keep the destination pairs and router weights of two tiles in LDS at a time.  Every element against
    the oracle on every ping-pong configuration; 24 experts with uneven counts give full tiles, tiles that end inside
    the tail blocks and ragged ones."""
    shape = synth.Shape("edge", 256, 128, 24, 1)
    T = 236_000
    L = Layer(shape, T, seed=29, x_std=1.5)
    ids, w = synth.routing(T, shape, 0.7, seed=31)
    rng = np.random.default_rng(5)
    w = rng.uniform(0.25, 1.0, size=w.shape).astype(np.float32)
    ref = L.oracle_rows(ids, w)
    cfgs = [c for c in ramp.configs(L.rs) if c.mode & ramp.PERSISTENT]
    assert {256, 272, 288} <= {c.bm for c in cfgs}
    for cfg in cfgs:
        print(f"case {cfg}", flush=True)
        assert ramp.align_capacity(T, 1, 24, cfg.bm) // cfg.bm > 3 * 256
        assert_close(L.run(cfg, ids, w), ref, f"{cfg}")


RANDOM_CASES = [  # H, I, E, k, T, beta: unusual tile counts (N-tiles 1, 3, 5, 6, 7, 10), few and many experts
    (384, 128, 5, 2, 900, 1.0), (256, 640, 7, 3, 400, 0.5), (768, 384, 12, 4, 260, 0.3), (128, 896, 3, 2, 1300, 1.0),
    (640, 256, 40, 6, 150, 0.2), (1280, 128, 9, 1, 2100, 1.0), (512, 768, 130, 5, 333, 0.1), (256, 256, 2, 2, 3000, 1.0),
]


@pytest.mark.parametrize("H,I,E,k,T,beta", RANDOM_CASES)
def test_irregular_shapes_every_third_config(H, I, E, k, T, beta):
    shape = synth.Shape("irregular", H, I, E, k)
    L = Layer(shape, T, seed=H * 7 + I, x_std=1.0)
    ids, w = synth.routing(T, shape, beta, seed=E * 100 + k)
    ref = L.oracle_rows(ids, w)
    cfgs = ramp.configs(L.rs)
    picked = cfgs[(H // 128) % 3::3] + [c for c in cfgs if c.mode & ramp.PERSISTENT]
    assert picked
    for cfg in picked:
        assert_close(L.run(cfg, ids, w), ref, f"H={H} I={I} E={E} k={k} T={T} {cfg}")


@pytest.mark.parametrize("seed", [1, 2, 3])
def test_randomized_shapes_sampled_rows(seed):
    """Seeded random shapes (H, I multiples of 128; 1 to 257 experts; top-1 to top-8), batch sizes from one token to
    a few thousand, four skews, some ids out of range; ten random configurations plus the ping-pong ones per case,
    sampled token rows against the oracle."""
    rng = np.random.default_rng(seed)
    for case in range(25):
        H, I = 128 * int(rng.integers(1, 9)), 128 * int(rng.integers(1, 9))
        E = int(rng.choice([1, 2, 3, 5, 8, 17, 33, 64, 100, 257]))
        k = int(rng.integers(1, min(E, 8) + 1))
        T = int(rng.choice([1, 2, 3, 15, 17, 63, 130, 255, 513, 1025, 2047, 3001]))
        beta = float(rng.choice([1.0, 0.5, 0.2, 0.08]))
        shape = synth.Shape("random", H, I, E, k)
        L = Layer(shape, T, seed=1000 * seed + case, x_std=float(rng.choice([0.5, 1.0, 2.0])))
        ids, w = synth.routing(T, shape, beta, seed=case)
        if rng.random() < 0.3:
            ids = ids.copy()
            ids.reshape(-1)[rng.integers(0, ids.size, max(1, ids.size // 10))] = rng.choice([-1, E, E + 5])
        rows = np.unique(rng.integers(0, T, min(T, 24)))
        if not any(0 <= e < E for t in rows for e in ids[t]):
            continue  # every sampled pair dropped: nothing to compare
        ref = L.oracle_rows(ids, w, rows=rows)
        if np.abs(ref).max() == 0:
            continue
        cfgs = ramp.configs(L.rs)
        picked = [cfgs[i] for i in rng.choice(len(cfgs), min(len(cfgs), 10), replace=False)]
        picked += [c for c in cfgs if c.mode & ramp.PERSISTENT][:3]
        sel = torch.from_numpy(rows).to(DEV)
        for cfg in picked:
            assert_close(L.run(cfg, ids, w)[sel], ref, f"seed={seed} case={case} H={H} I={I} E={E} k={k} T={T} beta={beta} {cfg}")


def test_fused_layer_replays_from_a_hip_graph(olmoe_small):
    """ramp_fused_moe only enqueues kernels on the caller's stream (no allocation, no memset node, no host
    synchronisation), so it can be captured once and replayed: every replay, with new inputs written into the
    captured buffers and eager work in between, is bit-identical to the eager call on the same inputs."""
    L = olmoe_small
    T = 96
    rs = ramp.Shape(T, L.s.k, L.s.E, L.s.H, L.s.I)
    cfgs = ramp.configs(rs)
    picked = [cfgs[0]] + [c for c in cfgs if c.mode & ramp.PERSISTENT][:1] + [c for c in cfgs if c.mode & 0x100][:1]
    for cfg in picked:
        d_ids = torch.zeros((T, L.s.k), dtype=torch.int32, device=DEV)
        d_w = torch.zeros((T, L.s.k), dtype=torch.float32, device=DEV)
        X = L.X[:T].clone()
        out = torch.zeros((T, L.s.H), dtype=torch.bfloat16, device=DEV)
        ws = torch.empty(ramp.fused_moe_workspace_bytes(rs, cfg), dtype=torch.uint8, device=DEV)
        side = torch.cuda.Stream()
        graph = torch.cuda.CUDAGraph()
        side.wait_stream(torch.cuda.current_stream())
        with torch.cuda.stream(side):
            ramp.fused_moe(rs, cfg, X, d_ids, d_w, L.packed, out, ws)       # warm-up outside the capture
            side.synchronize()
            with torch.cuda.graph(graph, stream=side):
                ramp.fused_moe(rs, cfg, X, d_ids, d_w, L.packed, out, ws, stream=side)
        torch.cuda.current_stream().wait_stream(side)
        for rep, beta in enumerate((0.2, 1.0, 0.5)):
            ids, w = synth.routing(T, L.s, beta, seed=40 + rep)
            d_ids.copy_(torch.from_numpy(np.ascontiguousarray(ids, np.int32)))
            d_w.copy_(torch.from_numpy(np.ascontiguousarray(w, np.float32)))
            X.copy_(L.X[:T] * (1.0 + 0.25 * rep))
            ws.fill_(0xFF)
            out.fill_(777.0)
            torch.cuda.synchronize()
            graph.replay()
            torch.cuda.synchronize()
            got = out.clone()
            eager = torch.zeros_like(out)
            ws2 = torch.full_like(ws, 0xFF)
            ramp.fused_moe(rs, cfg, X, d_ids, d_w, L.packed, eager, ws2)    # the program's own eager work between replays
            torch.cuda.synchronize()
            assert torch.equal(got.view(torch.int16), eager.view(torch.int16)), f"replay {rep} {cfg}"


def test_run_to_run_bit_identical(olmoe_small):
    L = olmoe_small
    ids, w = synth.routing(96, L.s, 0.2, seed=9)
    for cfg in ramp.configs(L.rs)[::5]:
        a = L.run(cfg, ids, w).view(torch.int16).cpu().numpy()
        b = L.run(cfg, ids, w, poison=False).view(torch.int16).cpu().numpy()
        assert np.array_equal(a, b), f"{cfg}"


def test_dropped_ids_zero_weights_and_empty_batch(olmoe_small):
    L = olmoe_small
    cfg = ramp.configs(L.rs)[3]
    ids, w = synth.routing(40, L.s, 0.5, seed=4)
    ids2 = ids.copy()
    ids2[::3, 2] = L.s.E + 5
    ids2[1::4, 0] = -1
    assert_close(L.run(cfg, ids2, w, T=40), L.oracle_rows(ids2, w, T=40), "dropped ids")
    z = L.run(cfg, ids, np.zeros_like(w), T=40)
    assert (z.float() == 0).all()
    all_dropped = np.full_like(ids, L.s.E)
    assert (L.run(cfg, all_dropped, w, T=40).float() == 0).all()
    L.run(cfg, ids[:0], w[:0], T=0)  # T = 0 is a no-op


def test_identical_experts_make_routing_irrelevant():
    s = synth.Shape("same", 256, 512, 16, 2)
    L = Layer(s, 48, seed=6, x_std=2.0)
    L.Wg[:] = L.Wg[0].clone(); L.Wu[:] = L.Wu[0].clone(); L.Wd[:] = L.Wd[0].clone()
    ramp.pack_weights(L.rs, L.Wg, L.Wu, L.Wd, L.packed)
    Xd = L.X.double().cpu()
    dense = (torch.nn.functional.silu(Xd @ L.Wg[0].double().cpu()) * (Xd @ L.Wu[0].double().cpu())) @ L.Wd[0].double().cpu()
    for beta in (1.0, 0.2):
        ids, w = synth.routing(48, s, beta, seed=7)
        scale = w.astype(np.float64).sum(1, keepdims=True)
        for cfg in ramp.configs(L.rs)[::4]:
            assert_close(L.run(cfg, ids, w), scale * dense.numpy(), f"identical experts {cfg}")


def test_rejects_bad_arguments(tiny):
    ids, w = synth.routing(16, tiny.s, 1.0, seed=1)
    cfg = ramp.configs(tiny.rs)[0]
    d_ids = torch.from_numpy(ids).to(DEV)
    d_w = torch.from_numpy(w).to(DEV)
    out = torch.empty((16, tiny.s.H), dtype=torch.bfloat16, device=DEV)
    small = torch.empty(256, dtype=torch.uint8, device=DEV)
    with pytest.raises(ramp.RampError) as ei:
        ramp.fused_moe(tiny.rs, cfg, tiny.X, d_ids, d_w, tiny.packed, out, small)
    assert ei.value.status == ramp.ENOSPC
    with pytest.raises(ramp.RampError) as ei:
        ramp.fused_moe(tiny.rs, ramp.Config(24, 64, 128, 2, 2, 0), tiny.X, d_ids, d_w, tiny.packed, out, small)
    assert ei.value.status == ramp.EUNSUPPORTED
    odd = ramp.Shape(16, 2, 16, 250, 512)
    with pytest.raises(ramp.RampError) as ei:
        ramp.fused_moe(odd, cfg, tiny.X, d_ids, d_w, tiny.packed, out, small)
    assert ei.value.status == ramp.EUNSUPPORTED


# ----------------------------------------------------------------------------- benchmark sizes, sampled rows

FULL = [
    # (shape, T, beta, n_sample_rows, configs to run: indices into the family by (bm, bn))
    ("olmoe", 4096, 1.0, 48), ("olmoe", 4096, 0.1, 48), ("olmoe", 1024, 0.2, 32),
    ("qwen3", 8192, 1.0, 32), ("qwen3", 512, 0.08, 32),
]


def sample_rows(ids, E, n, seed):
    """Seeded rows plus every... the first token of the most and the least loaded expert."""
    T = ids.shape[0]
    rng = np.random.default_rng(seed)
    rows = set(rng.choice(T, size=min(n, T), replace=False).tolist())
    counts = np.bincount(ids.reshape(-1), minlength=E)
    hot = int(counts.argmax())
    cold = int(np.where(counts > 0, counts, counts.max() + 1).argmin())
    for e in (hot, cold):
        toks = np.nonzero((ids == e).any(axis=1))[0]
        rows.update(toks[:2].tolist())
        rows.add(int(toks[-1]))
    return sorted(rows)


def pick_configs(rs, bms=(16, 64, 256)):
    out = {}
    for c in ramp.configs(rs):
        if c.bm in bms and c.bm not in out:
            out[c.bm] = c
    big = [c for c in ramp.configs(rs) if c.bm == 256]
    return list(out.values()) + big[-1:]


@pytest.mark.parametrize("name,T,beta,n", FULL)
def test_full_size_sampled_rows(name, T, beta, n):
    s = synth.SHAPES[name]
    L = Layer(s, T, seed=T % 97, x_std=1.0)
    ids, w = synth.routing(T, s, beta, seed=T + 1)
    rows = sample_rows(ids, s.E, n, seed=5)
    ref = L.oracle_rows(ids, w, rows=rows)
    for cfg in pick_configs(L.rs):
        out = L.run(cfg, ids, w, poison=False)
        assert_close(out[torch.tensor(rows, device=DEV)], ref, f"{name} T={T} beta={beta} {cfg}")
        # property that holds at any size: tokens routed nowhere new stay finite, output is deterministic
        assert torch.isfinite(out.float()).all()


@pytest.mark.parametrize("name,T,beta,n", [("mixtral", 1024, "zipf1.2", 6), ("dsv3", 2048, 0.1, 6)])
def test_large_layers_sampled_rows(name, T, beta, n):
    s = synth.SHAPES[name]
    L = Layer(s, T, seed=3, x_std=1.0)
    ids, w = synth.routing(T, s, beta, seed=T + 2)
    rng = np.random.default_rng(0)
    rows = sorted(rng.choice(T, size=n, replace=False).tolist())
    ref = L.oracle_rows(ids, w, rows=rows)
    for cfg in pick_configs(L.rs, bms=(32, 256)):
        out = L.run(cfg, ids, w, poison=False)
        assert_close(out[torch.tensor(rows, device=DEV)], ref, f"{name} T={T} beta={beta} {cfg}")


# ----------------------------------------------------------------------------- the largest benchmark points

_LAYERS = {}


def big_layer(name, T_max=8192):
    """One resident layer per shape for the large cases (the DeepSeek-V3-shaped one is 45 GB with its packed copy);
    switching shape frees the previous one."""
    if name not in _LAYERS:
        _LAYERS.clear()
        torch.cuda.empty_cache()
        _LAYERS[name] = Layer(synth.SHAPES[name], T_max, seed=3, x_std=1.0)
    return _LAYERS[name]


def large_tile_configs(rs):
    """Every persistent ping-pong configuration valid for the shape (what the large batches dispatch), plus the
    first LDS-ring configuration of each large token block and one mid-size block."""
    cfgs = ramp.configs(rs)
    picked = [c for c in cfgs if c.mode & ramp.PERSISTENT]
    assert any(c.key()[:5] == (256, 256, 32, 8, 3) for c in picked) and any(c.key()[:5] == (256, 256, 32, 8, 4) for c in picked)
    seen = set()
    for c in cfgs:
        if not (c.mode & 0x500) and c.bm in (64, 128, 256) and c.bm not in seen:
            seen.add(c.bm)
            picked.append(c)
    return picked


LARGEST = [("mixtral", 8192, 1.0, 8), ("mixtral", 8192, "zipf1.2", 8), ("dsv3", 8192, 1.0, 6), ("dsv3", 8192, 0.1, 6),
           ("dsv3", 512, 1.0, 6), ("qwen3", 2048, 0.08, 24), ("qwen3", 8192, 0.3, 24), ("olmoe", 4096, 0.5, 24)]


@pytest.mark.parametrize("name,T,beta,n", LARGEST)
def test_largest_points_sampled_rows_on_the_dispatched_kernels(name, T, beta, n):
    """Sampled token rows (seeded, plus tokens of the most and the least loaded expert) against the oracle at the
    largest benchmark points, on every ping-pong configuration: persistent workgroups walk many tiles each, the
    per-pair rows are bf16 and leave through the staged epilogue."""
    L = big_layer(name)
    s = L.s
    ids, w = synth.routing(T, s, beta, seed=T + 5)
    rows = sample_rows(ids, s.E, n, seed=7)
    ref = L.oracle_rows(ids, w, rows=rows, T=T)
    sel = torch.tensor(rows, device=DEV)
    rs = ramp.Shape(T, s.k, s.E, s.H, s.I)
    for cfg in large_tile_configs(rs):
        print(f"case {name} T={T} beta={beta} {cfg}", flush=True)
        out = L.run(cfg, ids, w, T=T, poison=False)
        assert_close(out[sel], ref, f"{name} T={T} beta={beta} {cfg}")
        assert torch.isfinite(out.float()).all()


@pytest.mark.parametrize("name,T,beta", [("olmoe", 4096, 1.0), ("olmoe", 4096, 0.1), ("mixtral", 8192, "zipf1.2"), ("dsv3", 8192, 1.0)])
def test_largest_points_run_twice_bit_identical(name, T, beta):
    """No atomics anywhere, so two runs of one configuration give the same bits; at these sizes every persistent
    workgroup walks several tiles (cross-tile load stream), which is what this check is for.  The second run starts
    from a workspace full of NaN patterns."""
    L = big_layer(name)
    s = L.s
    ids, w = synth.routing(T, s, beta, seed=T + 9)
    rs = ramp.Shape(T, s.k, s.E, s.H, s.I)
    for cfg in [c for c in ramp.configs(rs) if c.mode & ramp.PERSISTENT]:
        print(f"case {name} T={T} beta={beta} {cfg}", flush=True)
        a = L.run(cfg, ids, w, T=T, poison=False).clone()
        b = L.run(cfg, ids, w, T=T, poison=True)
        assert torch.equal(a.view(torch.int16), b.view(torch.int16)), f"{name} T={T} beta={beta} {cfg}"
