"""Calls whose align takes two launches, the second of which also quantises the hidden state: the sizes where that form begins
(2049 tokens; 16385 pairs and more), ids that are dropped, every row's codes used."""
import numpy as np
import pytest
import torch

from paper_2604_26039_amd import ramp, synth
from test_gpu_fp8 import DEV, Fp8Layer, assert_close

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("T,k,E,H", [(2049, 1, 3, 256), (1639, 10, 1024, 128), (1821, 9, 40, 384), (4099, 4, 8, 128)])
def test_align_and_quantiser_in_one_launch(T, k, E, H):
    s = synth.Shape("aq", H, 128, E, k)
    rng = np.random.default_rng(T)
    ids = np.argsort(rng.random((T, E)), axis=1)[:, :k].astype(np.int32)
    ids[rng.random((T, k)) < 0.1] = E + 1                                # dropped
    w = rng.random((T, k)).astype(np.float32)
    L = Fp8Layer(s, T, seed=k, x_std=1.5)
    rows = [0, 1023, 1024, T - 2, T - 1] + rng.choice(T, 8, replace=False).tolist()
    want = L.oracle_rows(ids, w, rows=rows)
    for cfg in [c for c in ramp.fp8_configs(L.rs) if not c.mode & 0x100][:3]:    # (a streaming tile aligns by itself)
        print(f"case T={T} k={k} E={E} H={H} {cfg}", flush=True)
        got = L.run(cfg, ids, w)
        assert_close(got[torch.tensor(rows, device=DEV)], want, f"T={T} k={k} {cfg}")
