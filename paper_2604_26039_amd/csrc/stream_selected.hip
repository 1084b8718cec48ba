// One launch per projection for all weight-streaming candidates of a device-selected layer (ramp_fused_moe_selected).
//
// Every candidate's launches are enqueued and all but one return at once, but a launch that returns at once still takes its turn in
// the stream: 1.9 us in a captured graph, 2.9 with the grids of these kernels (3456 blocks of 512 threads).  So the tiles that fit
// the same registers are cases of one kernel, which reads the selected position and runs that tile's code, with that
// candidate's bits.  A block is 8 wavefronts: one workgroup of eight, or two of four.  Four wavefronts per SIMD (128 registers)
// hold two blocks on a unit, as the tiles' own kernels have of eight wavefronts (one of the tiles, 16 rows x 4 weight blocks, keeps
// four values in scratch there); those that would spill much (bm = 64, 32 rows x 4 weight blocks) keep launches of their own.
// Replay of select + layer with four candidates, weights of three layers in turn: Qwen3-shaped T = 32 (39 experts) 102.6 -> 96.0 us
// and 104.0 -> 94.2 with two of the tiles selected, 105.6 as before with the one that spills; T = 16 181 -> 171; OLMoE-shaped
// T = 20 163 -> 149; H = 1152, I = 896 T = 40 66.5 -> 55; DeepSeek-V3-shaped T = 12 1199 -> 1160.
#include "config_list.h"
#include "moe_stream.h"

namespace ramp {
namespace {

#define X(BM, FBW, WF, WK, U) kShape_##BM##_##FBW##_##WF##_##WK##_##U,
enum : int { RAMP_STREAM_SELECTED_GROUP(X) kNumShapes };
#undef X

constexpr int most(int a, int b) { return a > b ? a : b; }
// partial sums of the workgroups of one block
#define X(BM, FBW, WF, WK, U) most(stream_selected_per_block(WF * WK) * StreamTraits<BM, FBW, WF, WK, U>::RED_FLOATS,
#define Y(BM, FBW, WF, WK, U) )
constexpr int kRedFloats = RAMP_STREAM_SELECTED_GROUP(X) 0 RAMP_STREAM_SELECTED_GROUP(Y);
#undef X
#undef Y

template <int STAGE>
__global__ __launch_bounds__(512, 4) void moe_stream_selected_kernel(GemmArgs a, char *base, int features, int n_cand,
                                                                     StreamChoices choices)
{
    __shared__ __attribute__((aligned(16))) float red[kRedFloats];
    const int idx = *a.pred;
    if (idx < 0 || idx >= n_cand) return;
    const StreamChoice c = choices.c[idx];
    if (c.shape < 0) return;
    a.sorted = reinterpret_cast<const int32_t *>(base + c.sorted);
    a.tile_expert = reinterpret_cast<const int32_t *>(base + c.tile_expert);
    a.n_tiles = features / c.bn;
    uint16_t *act = reinterpret_cast<uint16_t *>(base + c.a_buf);
    if (STAGE == 1) a.a_out = act;
    else a.act = act;
    const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    auto run = [&](auto tile, int waves, int red_floats) __attribute__((always_inline)) {
        const int part = wave / waves;  // workgroup of the block
        const int id = (int)blockIdx.x * (8 / waves) + part;
        const int m_tile = id / a.n_tiles, n_tile = id - m_tile * a.n_tiles;
        if (m_tile >= c.m_tiles_cap) return;  // (the grid is the largest candidate's)
        tile(red + part * red_floats, n_tile, m_tile, wave - part * waves);
    };
    switch (c.shape) {
#define X(BM, FBW, WF, WK, U)                                                                                            \
    case kShape_##BM##_##FBW##_##WF##_##WK##_##U:                                                                        \
        run([&](float *r, int n_tile, int m_tile, int w) __attribute__((always_inline)) {                                \
            stream_tile<STAGE, BM, FBW, WF, WK, U>(a, r, n_tile, m_tile, w, lane);                                       \
        }, WF * WK, StreamTraits<BM, FBW, WF, WK, U>::RED_FLOATS);                                                       \
        break;
        RAMP_STREAM_SELECTED_GROUP(X)
#undef X
    }
}

}  // namespace

int stream_selected_shape(const ramp_config &cfg)
{
    if (!(cfg.mode & kModeStream)) return -1;
#define X(BM, FBW, WF, WK, U)                                                                                            \
    static_assert(WF * WK == 8 || WF * WK == 4, "a block holds one or two workgroups");                                  \
    if (cfg.bm == BM && cfg.bn == StreamTraits<BM, FBW, WF, WK, U>::BN && cfg.bk == U * 32 && cfg.waves == WF * WK &&     \
        (cfg.mode & 0xff) == WK)                                                                                         \
        return kShape_##BM##_##FBW##_##WF##_##WK##_##U;
    RAMP_STREAM_SELECTED_GROUP(X)
#undef X
    return -1;
}

int launch_stream_selected(int stage, const GemmArgs &args, char *base, int features, int n_cand, const StreamChoices &choices,
                           unsigned blocks, hipStream_t stream)
{
    if (blocks == 0) return RAMP_OK;
    if (stage == 1)
        hipLaunchKernelGGL(moe_stream_selected_kernel<1>, dim3(blocks), dim3(512), 0, stream, args, base, features, n_cand, choices);
    else
        hipLaunchKernelGGL(moe_stream_selected_kernel<2>, dim3(blocks), dim3(512), 0, stream, args, base, features, n_cand, choices);
    return check_launch("moe_stream_selected_kernel");
}

}  // namespace ramp
