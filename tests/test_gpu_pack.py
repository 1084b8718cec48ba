"""GPU parity of the weight packing: the bf16 image against its definition, E4M3 codes and scales of every bf16 value."""
import numpy as np
import pytest
import torch

from oracle import fp8 as ofp8
from paper_2604_26039_amd import ramp, synth

pytestmark = pytest.mark.gpu
DEV = "cuda:0"


def row_feature(rb, r):
    """Feature held by row r of packed row block rb (interleave inside groups of four row blocks)."""
    return (rb // 4) * 64 + (r >> 2) * 16 + (rb % 4) * 4 + (r & 3)


def packed_matrix(W: np.ndarray) -> np.ndarray:
    """[K, F] -> [F/16][K/32][512]: lane l of a fragment holds row l%16 and k = 8*(l/16) .. +7."""
    K, F = W.shape
    rb, ks, lane, j = np.ogrid[:F // 16, :K // 32, :64, :8]
    return W[ks * 32 + (lane // 16) * 8 + j, row_feature(rb, lane % 16)].reshape(-1)


@pytest.mark.parametrize("E,H,I,shift", [(1, 128, 128, 0), (3, 256, 384, 0), (2, 640, 128, 1), (5, 384, 1152, 3)])
def test_bf16_pack_is_the_documented_image(E, H, I, shift):
    """shift: elements by which the sources miss a 16-byte boundary."""
    gen = torch.Generator(device=DEV).manual_seed(H + I)
    def weight(K, F):
        flat = torch.randint(-32768, 32767, (E * K * F + shift,), generator=gen, device=DEV, dtype=torch.int16)
        return flat[shift:].view(torch.bfloat16).view(E, K, F)
    Wg, Wu, Wd = weight(H, I), weight(H, I), weight(I, H)
    rs = ramp.Shape(1, 1, E, H, I)
    n = ramp.pack_bytes(rs)
    packed = torch.full((n + 256,), 0xA5, dtype=torch.uint8, device=DEV)
    ramp.pack_weights(rs, Wg, Wu, Wd, packed)
    got = packed.cpu().numpy()
    g, u, d = (synth.bits(w) for w in (Wg, Wu, Wd))
    want = np.concatenate([np.concatenate([packed_matrix(g[e]), packed_matrix(u[e])]) for e in range(E)]
                          + [packed_matrix(d[e]) for e in range(E)])
    assert np.array_equal(got[:want.nbytes].view(np.uint16), want)
    assert (got[n:] == 0xA5).all(), "write past the packed buffer"


def test_fp8_pack_codes_every_bf16_value_up_to_the_largest_code():
    """Blocks of scale 1 (largest value 448) that hold every bf16 bit pattern of magnitude <= 448, both signs: normal and
    subnormal codes, ties, values that round to zero."""
    H, I = 256, 384
    mag = np.arange(0x43E0 + 1, dtype=np.uint16)                  # 0x43E0 = 448
    pats = np.concatenate([mag, mag | 0x8000])
    blocks = np.full((6, 128 * 128), 0x43E0, np.uint16)
    per = 128 * 128 - 1                                           # one place of each block keeps the 448
    for b in range(3):
        part = pats[b * per:(b + 1) * per]
        blocks[b, 1:1 + part.size] = part
    assert 3 * per >= pats.size
    W = blocks.reshape(2, 3, 128, 128).transpose(0, 2, 1, 3).reshape(H, I)   # [K, F]
    Wg = torch.from_numpy(W.view(np.int16).copy()).view(torch.bfloat16).to(DEV)[None].contiguous()
    Wd = Wg.transpose(1, 2).contiguous()
    rs = ramp.Shape(1, 1, 1, H, I)
    packed = torch.zeros(ramp.fp8_pack_bytes(rs), dtype=torch.uint8, device=DEV)
    ramp.fp8_pack_weights(rs, Wg, Wg, Wd, packed)
    raw = packed.cpu().numpy()
    (w1_e, up_off, w2_base, w2_e, sc_base, _), strides = ramp.fp8_pack_layout(rs)
    Wf = synth.bits_to_f64(W)
    for off, M, scale_off, stride in ((0, Wf, 0, strides[0]), (up_off, Wf, (I // 128) * strides[0], strides[0]),
                                      (w2_base, Wf.T, 2 * (I // 128) * strides[0], strides[1])):
        K, F = M.shape
        want_c, want_s = ofp8.quantize_blocks(M)
        sc = raw[sc_base + scale_off: sc_base + scale_off + (F // 128) * stride].reshape(F // 128, stride)
        assert (want_s == 127).all() and np.array_equal(sc[:, :K // 128], want_s.T)
        rb, ks, h, lane, j = np.ogrid[:F // 16, :K // 128, :2, :64, :16]
        want = want_c[ks * 128 + (lane // 16) * 32 + h * 16 + j, row_feature(rb, lane % 16)]
        assert np.array_equal(raw[off: off + K * F].reshape(want.shape), want)


@pytest.mark.parametrize("fp8", [False, True])
def test_more_blocks_than_workgroups(fp8):
    """A layer of more than 2^20 blocks of 128 x 128 weights: workgroups take a second one.  Experts repeat three different ones, so
    the image has to repeat theirs."""
    H = I = 2048
    E = (1 << 20) // (3 * (H // 128) * (I // 128)) + 9
    assert 3 * E * (H // 128) * (I // 128) > 1 << 20
    gen = torch.Generator(device=DEV).manual_seed(1)
    base = (torch.randn((3, H, I), generator=gen, device=DEV) * torch.tensor([1.0, 0.1, 3.0], device=DEV)[:, None, None]).bfloat16()
    W = base.repeat(E // 3 + 1, 1, 1)[:E]
    pack, size = (ramp.fp8_pack_weights, ramp.fp8_pack_bytes) if fp8 else (ramp.pack_weights, ramp.pack_bytes)
    small, large = ramp.Shape(1, 1, 3, H, I), ramp.Shape(1, 1, E, H, I)
    want = torch.zeros(size(small), dtype=torch.uint8, device=DEV)
    pack(small, base, base, base, want)
    got = torch.zeros(size(large), dtype=torch.uint8, device=DEV)
    pack(large, W, W, W, got)
    one = 2 * H * I * (1 if fp8 else 2)                            # gate and up of an expert; half as much of down
    sections = [(0, 0, one), (3 * one, E * one, one // 2)]         # offset in the small and the large image, bytes of an expert
    if fp8:
        (_, _, _, _, sc3, sce), _ = ramp.fp8_pack_layout(small)
        (_, _, _, _, scE, _), _ = ramp.fp8_pack_layout(large)
        sections.append((sc3, scE, sce))
    for o3, oE, n in sections:
        w = want[o3:o3 + 3 * n].view(3, n)
        g = got[oE:oE + E * n].view(E, n)
        for e in range(E):
            assert torch.equal(g[e], w[e % 3]), (e, n)
