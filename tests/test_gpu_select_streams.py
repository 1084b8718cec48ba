"""Weight-streaming candidates of a device-selected layer share one launch per projection: every candidate selected in turn gives
the bits of its eager call, whatever else is in the list."""
import numpy as np
import pytest
import torch

from paper_2604_26039_amd import ramp, synth
from test_gpu_moe import DEV, Layer

pytestmark = pytest.mark.gpu


# one and several tiles of a block's workgroups; an odd number of tiles for the blocks that hold two; dropped pairs; bf16 pair rows (last)
@pytest.mark.parametrize("H,I,E,k,T", [(256, 128, 6, 3, 23), (384, 640, 24, 6, 41), (1152, 256, 3, 2, 300), (4096, 128, 6, 4, 600)])
def test_every_streaming_candidate(H, I, E, k, T):
    s = synth.Shape("streams", H, I, E, k)
    L = Layer(s, T, seed=H, x_std=1.5)
    ids, w = synth.routing(T, s, 0.8, seed=T)
    ids = ids.copy()
    ids[::7, 0] = -1
    d_ids, d_w = torch.from_numpy(ids).to(DEV), torch.from_numpy(w).to(DEV)
    streams = [c for c in ramp.configs(L.rs) if c.mode & 0x100]
    other = next(c for c in ramp.configs(L.rs) if not c.mode & 0x700)
    assert len(streams) >= 20
    for i in range(0, len(streams), 14):
        cands = streams[i:i + 14] + [other]
        ws = torch.empty(ramp.fused_moe_selected_workspace_bytes(L.rs, cands), dtype=torch.uint8, device=DEV)
        for pick in list(range(len(cands))) + [-1, len(cands)]:
            ws.fill_(0xFF)
            out = torch.full((T, H), 7.0, dtype=torch.bfloat16, device=DEV)
            sel = torch.tensor([pick], dtype=torch.int32, device=DEV)
            ramp.fused_moe_selected(L.rs, cands, sel, L.X, d_ids, d_w, L.packed, out, ws)
            torch.cuda.synchronize()
            if not 0 <= pick < len(cands):
                assert (out == 7.0).all()
                continue
            want = L.run(cands[pick], ids, w)
            assert torch.equal(out.view(torch.int16), want.view(torch.int16)), f"{cands[pick]}"
