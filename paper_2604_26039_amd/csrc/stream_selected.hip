// One launch per projection for several weight-streaming candidates of a device-selected layer (ramp_fused_moe_selected).
//
// Every candidate's launches are enqueued and all but one return at once, but a launch that returns at once still takes its turn in
// the stream: 1.9 us in a captured graph, 2.9 with the grids of these kernels (3456 blocks of 512 threads).  So tiles that fit the same
// registers are cases of one kernel, which reads the selected position and runs that tile's code, with that candidate's bits.
//
// Two such kernels.  The first has blocks of 8 wavefronts, one workgroup of eight or two of four, and four wavefronts per SIMD (128
// registers): the tiles that need 90 to 122 have as many in their own kernels (16 on a unit; the one of four wavefronts and 88 registers
// has 20), and the two of 138 gain by it.  The second has blocks of four wavefronts and three per SIMD, as its tiles have on their own: in 128
// registers they lost more than the launches take (OLMoE-shaped T = 64, 13 experts, selected tile 16 rows x 4 weight blocks 63.0 -> 82.1 us;
// Mixtral-shaped T = 40 16 rows of four wavefronts without a shared reduction 534 -> 680).  Tiles that would spill, or lose in either (bm = 64,
// 32 rows x 4 weight blocks, 32 rows of four wavefronts), keep launches of their own.
// Selected layer in a graph, every candidate of fifteen calls selected in turn, against launches of their own: the four fastest
// configurations as candidates 0.96 of the time, eight 0.91, four of the streaming ones 0.95, two 0.98, none above 1.01 (Qwen3-shaped T = 32,
// 39 experts, four candidates 95 -> 84 us; H = 1152, I = 896 T = 16 75 -> 67; Mixtral-shaped T = 40, eight candidates 517 -> 484).
#include "config_list.h"
#include "moe_stream.h"

namespace ramp {
namespace {

#define X(BM, FBW, WF, WK, U) kShape_##BM##_##FBW##_##WF##_##WK##_##U,
enum : int { RAMP_STREAM_SELECTED_GROUP0(X) kEnd0, RAMP_STREAM_SELECTED_GROUP1(X) kEnd1 };
#undef X

constexpr int most(int a, int b) { return a > b ? a : b; }
// partial sums of the workgroups of one block
#define Y(BM, FBW, WF, WK, U) )
#define X(BM, FBW, WF, WK, U) most(stream_selected_waves(0) / (WF * WK) * StreamTraits<BM, FBW, WF, WK, U>::RED_FLOATS,
constexpr int kRedFloats0 = RAMP_STREAM_SELECTED_GROUP0(X) 0 RAMP_STREAM_SELECTED_GROUP0(Y);
#undef X
#define X(BM, FBW, WF, WK, U) most(stream_selected_waves(1) / (WF * WK) * StreamTraits<BM, FBW, WF, WK, U>::RED_FLOATS,
constexpr int kRedFloats1 = RAMP_STREAM_SELECTED_GROUP1(X) 0 RAMP_STREAM_SELECTED_GROUP1(Y);
#undef X
#undef Y

// Body of both kernels for the tile of one case.
template <int WAVES, int STAGE, int BM, int FBW, int WF, int WK, int U>
__device__ __forceinline__ void selected_tile(const GemmArgs &a, const StreamChoice &c, float *red, int wave, int lane)
{
    constexpr int PER_BLOCK = WAVES / (WF * WK);
    static_assert(WAVES % (WF * WK) == 0, "whole workgroups to a block");
    const int part = PER_BLOCK > 1 ? wave / (WF * WK) : 0;  // workgroup of the block
    const int id = (int)blockIdx.x * PER_BLOCK + part;
    const int m_tile = id / a.n_tiles, n_tile = id - m_tile * a.n_tiles;
    if (m_tile >= c.m_tiles_cap) {  // (the grid is the largest candidate's)
        if (PER_BLOCK > 1 && WK > 1) __syncthreads();
        return;
    }
    stream_tile<(PER_BLOCK > 1), STAGE, BM, FBW, WF, WK, U>(a, red + part * StreamTraits<BM, FBW, WF, WK, U>::RED_FLOATS, n_tile, m_tile,
                                                            wave - part * (WF * WK), lane);
}
template <int STAGE>
__device__ __forceinline__ bool selected_args(GemmArgs &a, StreamChoice &c, char *base, int features, int n_cand,
                                              const StreamChoices &choices)
{
    const int idx = *a.pred;
    if (idx < 0 || idx >= n_cand) return false;
    c = choices.c[idx];
    if (c.shape < 0) return false;
    a.sorted = reinterpret_cast<const int32_t *>(base + c.sorted);
    a.tile_expert = reinterpret_cast<const int32_t *>(base + c.tile_expert);
    a.n_tiles = features / c.bn;
    uint16_t *act = reinterpret_cast<uint16_t *>(base + c.a_buf);
    if (STAGE == 1) a.a_out = act;
    else a.act = act;
    return true;
}

template <int STAGE>
__global__ __launch_bounds__(512, 4) void moe_stream_selected0_kernel(GemmArgs a, char *base, int features, int n_cand,
                                                                      StreamChoices choices)
{
    __shared__ __attribute__((aligned(16))) float red[kRedFloats0];
    StreamChoice c;
    if (!selected_args<STAGE>(a, c, base, features, n_cand, choices)) return;
    const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    switch (c.shape) {
#define X(BM, FBW, WF, WK, U)                                                                                            \
    case kShape_##BM##_##FBW##_##WF##_##WK##_##U:                                                                        \
        selected_tile<stream_selected_waves(0), STAGE, BM, FBW, WF, WK, U>(a, c, red, wave, lane);                       \
        break;
        RAMP_STREAM_SELECTED_GROUP0(X)
    }
}
template <int STAGE>
__global__ __launch_bounds__(256) void moe_stream_selected1_kernel(GemmArgs a, char *base, int features, int n_cand,
                                                                   StreamChoices choices)
{
    __shared__ __attribute__((aligned(16))) float red[kRedFloats1];
    StreamChoice c;
    if (!selected_args<STAGE>(a, c, base, features, n_cand, choices)) return;
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    switch (c.shape) {
#undef X
#define X(BM, FBW, WF, WK, U)                                                                                            \
    case kShape_##BM##_##FBW##_##WF##_##WK##_##U:                                                                        \
        selected_tile<stream_selected_waves(1), STAGE, BM, FBW, WF, WK, U>(a, c, red, wave, lane);                       \
        break;
        RAMP_STREAM_SELECTED_GROUP1(X)
#undef X
    }
}

}  // namespace

int stream_selected_shape(const ramp_config &cfg)
{
    if (!(cfg.mode & kModeStream)) return -1;
#define X(BM, FBW, WF, WK, U)                                                                                            \
    if (cfg.bm == BM && cfg.bn == StreamTraits<BM, FBW, WF, WK, U>::BN && cfg.bk == U * 32 && cfg.waves == WF * WK &&     \
        (cfg.mode & 0xff) == WK)                                                                                         \
        return kShape_##BM##_##FBW##_##WF##_##WK##_##U;
    RAMP_STREAM_SELECTED_GROUP0(X)
    RAMP_STREAM_SELECTED_GROUP1(X)
#undef X
    return -1;
}

int stream_selected_group(int shape) { return shape < 0 ? -1 : shape < kEnd0 ? 0 : 1; }

int launch_stream_selected(int group, int stage, const GemmArgs &args, char *base, int features, int n_cand,
                           const StreamChoices &choices, unsigned blocks, hipStream_t stream)
{
    if (blocks == 0) return RAMP_OK;
    using Kernel = void (*)(GemmArgs, char *, int, int, StreamChoices);
    static const Kernel kernels[kStreamGroups][2] = {{&moe_stream_selected0_kernel<1>, &moe_stream_selected0_kernel<2>},
                                                     {&moe_stream_selected1_kernel<1>, &moe_stream_selected1_kernel<2>}};
    // a launch sees the candidates of its group alone
    StreamChoices own = choices;
    for (int c = 0; c < n_cand; ++c)
        if (stream_selected_group(own.c[c].shape) != group) own.c[c].shape = -1;
    hipLaunchKernelGGL(kernels[group][stage - 1], dim3(blocks), dim3(stream_selected_waves(group) * kWave), 0, stream, args, base,
                       features, n_cand, own);
    return check_launch("moe_stream_selected_kernel");
}

}  // namespace ramp
