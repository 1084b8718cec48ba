// Weight-streaming form of the FP8 expert projections for small token blocks, and its two-launch form for calls of at most 64
// pairs.  Bound by HBM (a weight byte is used by at most 32 tokens), and below a few experts by launches and latency.
//
// As in moe_stream.h a wavefront owns FBW 16-row weight blocks and a 1/WK share of the reduction, and loads its 2 KB weight
// fragments straight into MFMA operand registers, one batch of U slices of 128 ahead; the WK partial sums meet in LDS once.
// The token operand is read as bf16 and quantised in registers (a lane holds 32 of the 128 values of a row's scale block, so
// the block maximum is two lane exchanges): the launches that quantise the hidden state and the activation, and their round
// trips through memory, are gone, for about 60 instructions per 16 rows and slice that hide under the weight loads.
//
// Measured (layer, best configuration of each family, against the best LDS-staged or persistent FP8 tile): OLMoE-shaped T = 1
// 36 -> 17 us (two launches instead of six; 20 us with the weights out of the memory-side cache), Qwen3-shaped T = 8 77 -> 56 us,
// Mixtral-shaped T = 1 221 -> 71 us and T = 32 293 -> 264 us (5.3 TB/s of weights), DeepSeek-V3-shaped T = 64 1652 -> 1573 us
// (6.5 TB/s).  Between 24 and 32 rows per expert the tiles with shared operands become the better ones (Mixtral-shaped: 16 rows
// 287 us against 307, 24 rows 303 against 306, 32 rows 452 against 315).
#pragma once

#include "align_tiny.h"
#include "fp8_format.h"
#include "moe_gemm.h"

namespace ramp {

struct Fp8StreamArgs {
    const uint8_t *wq;         // packed codes of this stage
    size_t expert_stride;      // bytes between experts
    uint32_t up_offset;        // stage 1: byte offset of the up rows inside an expert
    const uint8_t *wscale;     // first scale array of this stage (gate, or down)
    size_t wscale_expert_stride;
    uint32_t wscale_up_offset; // stage 1: gate -> up scale array
    int w_stride;              // scale row stride of the weights
};

// One wavefront's share: acc += weights (FBW fragments per slice) x tokens (NB blocks of 16 rows) over slices [ks0, ks1).
//   row[nb]: element offset of this lane's 32 values of slice 0 in `act`; live[nb]: this lane's row exists (others are zeros)
//   woff[i]: byte offset of weight block i, lane included; sw0/sw1: scale rows of the first and second half of the blocks
template <int FBW, int NB, int U>
__device__ __forceinline__ void fp8_stream_slices(floatx4 (&acc)[FBW][NB], const uint16_t *act, const uint32_t (&row)[NB],
                                                  const bool (&live)[NB], const uint8_t *w, const uint32_t (&woff)[FBW],
                                                  const uint8_t *sw0, const uint8_t *sw1, int ks0, int ks1)
{
    struct Batch {
        uint4 x[U][NB][4];
        intx4 w[U][FBW][2];
        uint32_t s[U][2];
    };
    auto load_batch = [&](Batch &b, int k) __attribute__((always_inline)) {
#pragma unroll
        for (int u = 0; u < U; ++u) {
            const int ks = min(k + u, ks1 - 1);  // past the end: the last slice again, its product is skipped
#pragma unroll
            for (int i = 0; i < FBW; ++i)
#pragma unroll
                for (int h = 0; h < 2; ++h)
                    b.w[u][i][h] = *reinterpret_cast<const intx4 *>(w + woff[i] + (size_t)ks * 2048 + h * 1024);
#pragma unroll
            for (int nb = 0; nb < NB; ++nb) {
#pragma unroll
                for (int p = 0; p < 4; ++p) b.x[u][nb][p] = make_uint4(0, 0, 0, 0);
                if (live[nb]) {
                    const uint4 *src = reinterpret_cast<const uint4 *>(act + row[nb] + (size_t)ks * 128);
#pragma unroll
                    for (int p = 0; p < 4; ++p) b.x[u][nb][p] = src[p];
                }
            }
            // wave-uniform, written by an earlier launch: scalar loads of the word that holds the byte
            const int word = ks & ~3;
            b.s[u][0] = *(const __attribute__((address_space(4))) uint32_t *)(sw0 + word) >> ((ks & 3) * 8);
            b.s[u][1] = *(const __attribute__((address_space(4))) uint32_t *)(sw1 + word) >> ((ks & 3) * 8);
        }
    };
    auto multiply = [&](const Batch &b, int k) __attribute__((always_inline)) {
#pragma unroll
        for (int u = 0; u < U; ++u) {
            if (k + u < ks1) {
#pragma unroll
                for (int nb = 0; nb < NB; ++nb) {
                    uint32_t raw[16], codes[8];
#pragma unroll
                    for (int p = 0; p < 4; ++p) {
                        raw[4 * p] = b.x[u][nb][p].x;
                        raw[4 * p + 1] = b.x[u][nb][p].y;
                        raw[4 * p + 2] = b.x[u][nb][p].z;
                        raw[4 * p + 3] = b.x[u][nb][p].w;
                    }
                    const uint32_t sx = quantise_group<16, 16, 64>(raw, codes);
                    const intx8 xf = {(int)codes[0], (int)codes[1], (int)codes[2], (int)codes[3],
                                      (int)codes[4], (int)codes[5], (int)codes[6], (int)codes[7]};
#pragma unroll
                    for (int i = 0; i < FBW; ++i) {
                        const intx4 lo = b.w[u][i][0], hi = b.w[u][i][1];
                        const intx8 wf = {lo[0], lo[1], lo[2], lo[3], hi[0], hi[1], hi[2], hi[3]};
                        acc[i][nb] = __builtin_amdgcn_mfma_scale_f32_16x16x128_f8f6f4(wf, xf, acc[i][nb], 0, 0, 0,
                                                                                      (int)b.s[u][2 * i >= FBW && FBW > 1], 0, (int)sx);
                    }
                }
            }
        }
    };
    if (ks0 >= ks1) return;
    Batch b0, b1;
    load_batch(b0, ks0);
    for (int k = ks0; k < ks1; k += 2 * U) {
        if (k + U < ks1) load_batch(b1, k + U);
        multiply(b0, k);
        if (k + 2 * U < ks1) load_batch(b0, k + 2 * U);
        if (k + U < ks1) multiply(b1, k + U);
    }
}

template <int BM, int FBW, int WF, int WK, int U>
struct Fp8StreamTraits {
    static constexpr int NB = (BM + 15) / 16;
    static constexpr int BN = WF * FBW * 16;                         // weight rows per workgroup tile
    static constexpr int RED_FLOATS = (WK - 1) * WF * FBW * NB * 256;  // partial sums parked in LDS
    static_assert(FBW % 2 == 0 && FBW <= 8, "gate and up row blocks come in pairs; a wavefront's features share a scale block");
    static_assert(RED_FLOATS * 4 <= 64 * 1024, "reduction buffer too large");
};

// Work of one workgroup on M-tile x feature tile.  pair_of[nb]: the pair of this lane's row, a.P for none; act_row[nb]: its row
// of the token operand; out_row(nb): its row of the activation (stage 1).
template <int STAGE, int BM, int FBW, int WF, int WK, int U, class OutRow>
__device__ __forceinline__ void fp8_stream_tile(const GemmArgs &a, const Fp8StreamArgs &f, float *red, int e, int n_tile, int wave,
                                                int lane, const int (&pair_of)[Fp8StreamTraits<BM, FBW, WF, WK, U>::NB],
                                                const uint32_t (&act_row)[Fp8StreamTraits<BM, FBW, WF, WK, U>::NB], OutRow out_row)
{
    using ST = Fp8StreamTraits<BM, FBW, WF, WK, U>;
    constexpr int NB = ST::NB;
    constexpr int FPW = (STAGE == 1) ? FBW / 2 : FBW;  // feature blocks per wavefront in the output
    const int wf = wave % WF, wk = wave / WF;
    const int q = lane >> 4;
    const int KT = a.K >> 7;
    const int rb0 = (n_tile * WF + wf) * FPW;
    const uint8_t *wexp = f.wq + (size_t)e * f.expert_stride;
    const uint8_t *sw = f.wscale + (size_t)e * f.wscale_expert_stride + (size_t)(rb0 >> 3) * f.w_stride;
    const int per = (KT + WK - 1) / WK;
    const int ks0 = wk * per, ks1 = min(KT, ks0 + per);
    uint32_t woff[FBW], row[NB];
    bool live[NB];
#pragma unroll
    for (int i = 0; i < FBW; ++i)
        woff[i] = (uint32_t)((rb0 + i % FPW) * KT) * 2048u + (i >= FPW ? f.up_offset : 0u) + (uint32_t)lane * 16u;
#pragma unroll
    for (int nb = 0; nb < NB; ++nb) {
        live[nb] = pair_of[nb] < a.P;
        row[nb] = act_row[nb] * (uint32_t)a.K + (uint32_t)(q * 32);
    }
    floatx4 acc[FBW][NB];
#pragma unroll
    for (int i = 0; i < FBW; ++i)
#pragma unroll
        for (int j = 0; j < NB; ++j) acc[i][j] = floatx4{0.f, 0.f, 0.f, 0.f};
    fp8_stream_slices<FBW, NB, U>(acc, a.act, row, live, wexp, woff, sw, STAGE == 1 ? sw + f.wscale_up_offset : sw, ks0, ks1);

    if (WK > 1) {
        if (wk > 0) {
#pragma unroll
            for (int i = 0; i < FBW; ++i)
#pragma unroll
                for (int nb = 0; nb < NB; ++nb)
                    *reinterpret_cast<floatx4 *>(&red[((((wk - 1) * WF + wf) * FBW + i) * NB + nb) * 256 + lane * 4]) = acc[i][nb];
        }
        __syncthreads();
        if (wk > 0) return;
#pragma unroll
        for (int s = 0; s < WK - 1; ++s)
#pragma unroll
            for (int i = 0; i < FBW; ++i)
#pragma unroll
                for (int nb = 0; nb < NB; ++nb)
                    acc[i][nb] += *reinterpret_cast<const floatx4 *>(&red[(((s * WF + wf) * FBW + i) * NB + nb) * 256 + lane * 4]);
    }
#pragma unroll
    for (int nb = 0; nb < NB; ++nb) {
        const int pair = pair_of[nb];
        if (pair >= a.P) continue;
        if (STAGE == 1)
            store_token_row<1, FPW>(a, &acc[0][nb], &acc[FBW / 2][nb], NB, out_row(nb), rb0, q, 1.0f);
        else
            store_token_row<2, FPW>(a, &acc[0][nb], &acc[0][nb], NB, (size_t)pair * a.F, rb0, q, a.topk_w[pair]);
    }
}

template <int STAGE, int BM, int FBW, int WF, int WK, int U>
__global__ __launch_bounds__(WF *WK * 64) void moe_fp8_stream_kernel(GemmArgs a, Fp8StreamArgs f)
{
    using ST = Fp8StreamTraits<BM, FBW, WF, WK, U>;
    constexpr int NB = ST::NB;
    __shared__ __attribute__((aligned(16))) float red[ST::RED_FLOATS > 0 ? ST::RED_FLOATS : 4];
    const int n_tile = blockIdx.x % a.n_tiles, m_tile = blockIdx.x / a.n_tiles;
    const int lane = threadIdx.x & 63, r16 = lane & 15;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    int pair_of[NB];
    uint32_t act_row[NB];
    // rows and expert on their way together; -1: past the real tiles (as in moe_stream_kernel)
#pragma unroll
    for (int nb = 0; nb < NB; ++nb) {
        const int tr = nb * 16 + r16;
        pair_of[nb] = a.sorted[m_tile * BM + (tr < BM ? tr : BM - 1)];
    }
    const int e = load_uniform_i32(a.tile_expert + m_tile);
    if (e < 0) return;
#pragma unroll
    for (int nb = 0; nb < NB; ++nb) {
        const int tr = nb * 16 + r16;
        const int slot = m_tile * BM + (tr < BM ? tr : BM - 1);
        const int pair = pair_of[nb];
        pair_of[nb] = tr < BM ? pair : a.P;
        act_row[nb] = (STAGE == 1) ? (uint32_t)(((unsigned long long)(uint32_t)pair * a.topk_magic) >> 40) : (uint32_t)slot;
    }
    fp8_stream_tile<STAGE, BM, FBW, WF, WK, U>(a, f, red, e, n_tile, wave, lane, pair_of, act_row,
                                               [&](int nb) { return (size_t)(m_tile * BM + nb * 16 + r16); });
}

// Two-launch form, first launch: every workgroup aligns the at most 64 pairs itself (moe_decode_up_kernel); the activation has
// one row per pair.
template <int BM, int FBW, int WF, int WK, int U>
__global__ __launch_bounds__(WF *WK * 64) void moe_fp8_decode_up_kernel(GemmArgs a, Fp8StreamArgs f, DecodeArgs d)
{
    using ST = Fp8StreamTraits<BM, FBW, WF, WK, U>;
    constexpr int NB = ST::NB;
    __shared__ __attribute__((aligned(16))) float red[ST::RED_FLOATS > 0 ? ST::RED_FLOATS : 4];
    __shared__ int n_lds[kAlignMaxE];
    __shared__ int toff[kAlignMaxE + 1];
    __shared__ int tile_pair[BM];
    __shared__ int tile_expert, tile_count;  // expert of this workgroup's M-tile, number of M-tiles of the call
    // workgroup 0 only writes the align result: in front of a tile of its own that would be the last tile to end
    const int tile = (int)blockIdx.x - 1;
    const int n_tile = tile % a.n_tiles;
    const int m_tile = tile < 0 ? a.m_tiles_cap : tile / a.n_tiles;
    const int lane = threadIdx.x & 63, r16 = lane & 15;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    for (int x = threadIdx.x; x < BM; x += blockDim.x) tile_pair[x] = a.P;
    __syncthreads();
    if (wave == 0) {
        int e, rank;
        tiny_align_wavefront(d.ids, a.P, d.E, BM, lane, n_lds, toff, e, rank);
        if (e >= 0) {
            const int slot = toff[e] + rank;
            if (slot / BM == m_tile) {
                tile_pair[slot - m_tile * BM] = lane;
                if (slot % BM == 0) tile_expert = e;  // the tile's first row: every tile has a pair there, one lane
            }
        }
        if (lane == 0) tile_count = toff[d.E] / BM;
        if (blockIdx.x == 0)
            tiny_align_emit(a.P, d.E, BM, d.cap, lane, n_lds, toff, e, rank, d.ids, d.sorted, d.tile_expert, d.tile_rows, d.counts,
                            d.meta);
    }
    __syncthreads();
    if (m_tile >= tile_count) return;
    const int e = __builtin_amdgcn_readfirstlane(tile_expert);
    int pair_of[NB];
    uint32_t act_row[NB];
#pragma unroll
    for (int nb = 0; nb < NB; ++nb) {
        const int tr = nb * 16 + r16;
        const int pair = tile_pair[tr < BM ? tr : BM - 1];
        pair_of[nb] = tr < BM ? pair : a.P;
        act_row[nb] = (uint32_t)(((unsigned long long)(uint32_t)pair * a.topk_magic) >> 40);
    }
    fp8_stream_tile<1, BM, FBW, WF, WK, U>(a, f, red, e, n_tile, wave, lane, pair_of, act_row,
                                           [&](int nb) { return (size_t)pair_of[nb]; });
}

// Second launch: down-projection, router weights and top-k sum of one token's 16 * FBW output features per workgroup, all of
// its k pairs (moe_decode_down_kernel).  grid = (H / (16*FBW)) * T workgroups of 16 wavefronts, WK as there.
template <int FBW, int U>
__global__ __launch_bounds__(1024) void moe_fp8_decode_down_kernel(DecodeDownArgs d, Fp8StreamArgs f)
{
    __shared__ float red[16][FBW * 16];
    __shared__ PairWeights weight;
    const int n_ft = d.H / (16 * FBW);
    const int t = blockIdx.x / n_ft, ft = blockIdx.x % n_ft;
    const PairWeight own_weight = load_pair_weight(d, t);
    const int lane = threadIdx.x & 63;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int WK = decode_pair_waves(d.k);
    const int j = wave / WK, wk = wave % WK;
    const int r16 = lane & 15, q = lane >> 4;
    const int pair = t * d.k + j;
    const int e = j < d.k ? __builtin_amdgcn_readfirstlane(d.ids[pair]) : -1;
    // To LDS here and not behind the slices: their batches leave no register for it under the 128 of sixteen wavefronts (it went
    // to scratch), and the wait for the id above, the younger load, has covered it.  Layer, T = 1: Mixtral-shaped 75.6 -> 73.6 us,
    // Qwen3-shaped 14.9 -> 14.7, OLMoE-shaped 17.1 as before; T = 8, OLMoE-shaped: 57.0 -> 56.7.
    store_pair_weight(weight, d, own_weight);
    const int KT = d.I >> 7;
    const int per = (KT + WK - 1) / WK;
    const int ks0 = wk * per, ks1 = min(KT, ks0 + per);
    floatx4 acc[FBW][1];
#pragma unroll
    for (int i = 0; i < FBW; ++i) acc[i][0] = floatx4{0.f, 0.f, 0.f, 0.f};
    if (e >= 0 && e < d.E) {
        const uint32_t row[1] = {(uint32_t)pair * (uint32_t)d.I + (uint32_t)(q * 32)};
        const bool live[1] = {r16 == 0};  // the token operand has one real column
        uint32_t woff[FBW];
#pragma unroll
        for (int i = 0; i < FBW; ++i) woff[i] = (uint32_t)((ft * FBW + i) * KT) * 2048u + (uint32_t)lane * 16u;
        const uint8_t *sw = f.wscale + (size_t)e * f.wscale_expert_stride + (size_t)((ft * FBW) >> 3) * f.w_stride;
        fp8_stream_slices<FBW, 1, U>(acc, d.act, row, live, f.wq + (size_t)e * f.expert_stride, woff, sw, sw, ks0, ks1);
    }
    if (r16 == 0) {
#pragma unroll
        for (int i = 0; i < FBW; ++i)
#pragma unroll
            for (int c = 0; c < 4; ++c) red[wave][i * 16 + q * 4 + c] = acc[i][0][c];
    }
    __syncthreads();
    if ((int)threadIdx.x < FBW * 16) {
        const int i = threadIdx.x / 16, r = threadIdx.x % 16;
        const float y = sum_of_pairs(WK, weight, [&](int w) { return red[w][threadIdx.x]; });
        d.out[(size_t)t * d.H + packed_row_feature(ft * FBW + i, r)] = f32_to_bf16_bits(y);
    }
}

template <int BM, int FBW, int WF, int WK, int U>
void launch_fp8_stream(int stage, const GemmArgs &a, const Fp8StreamArgs &f, hipStream_t stream)
{
    const dim3 grid((unsigned)a.n_tiles * (unsigned)a.m_tiles_cap), block(WF * WK * 64);
    if (grid.x == 0) return;
    if (stage == 1)
        hipLaunchKernelGGL((moe_fp8_stream_kernel<1, BM, FBW, WF, WK, U>), grid, block, 0, stream, a, f);
    else
        hipLaunchKernelGGL((moe_fp8_stream_kernel<2, BM, FBW, WF, WK, U>), grid, block, 0, stream, a, f);
}

template <int BM, int FBW, int WF, int WK, int U>
void launch_fp8_decode_up(const GemmArgs &a, const Fp8StreamArgs &f, const DecodeArgs &d, hipStream_t stream)
{
    if (a.n_tiles <= 0 || a.m_tiles_cap <= 0) return;
    const dim3 grid((unsigned)a.n_tiles * (unsigned)a.m_tiles_cap + 1), block(WF * WK * 64);
    hipLaunchKernelGGL((moe_fp8_decode_up_kernel<BM, FBW, WF, WK, U>), grid, block, 0, stream, a, f, d);
}

inline void launch_fp8_decode_down(const DecodeDownArgs &d, const Fp8StreamArgs &f, hipStream_t stream)
{
    if (d.T <= 0) return;
    // as launch_decode_down: 16 output features per workgroup fill the chip sooner, 32 halve the workgroups
    if ((size_t)d.H / 32 * d.T >= 2 * (size_t)kNumCU)
        hipLaunchKernelGGL((moe_fp8_decode_down_kernel<2, 1>), dim3((unsigned)(d.H / 32) * (unsigned)d.T), dim3(1024), 0, stream, d, f);
    else
        hipLaunchKernelGGL((moe_fp8_decode_down_kernel<1, 2>), dim3((unsigned)(d.H / 16) * (unsigned)d.T), dim3(1024), 0, stream, d, f);
}

}  // namespace ramp
