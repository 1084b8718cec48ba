// Persistent ping-pong form of the FP8 expert projections for large batches: 256 (or 128) token rows x 256 weight rows
// per tile, k-slices of 128, 8 wavefronts (2 token rows x 4 weight columns of the tile), v_mfma_scale_f32_16x16x128_f8f6f4.
//
// Schedule.  As in the bf16 ping-pong kernel two groups of four wavefronts (one of each per SIMD) are a phase apart: while
// one multiplies from registers (C), the other reads its operands from LDS and issues loads (M).  A slice of 128 k-values is
// twice the operand bytes of a bf16 slice of 32 k-values x 2, and a wavefront cannot hold the fragments of its 128 x 64
// part of the tile (8 token blocks x 8 + 4 weight blocks x 8 registers next to 128 accumulators), so a slice is
// multiplied in NH = bm / 128 steps of four token blocks: the first step reads the four weight fragments, which stay in
// registers, and the first half of the token rows, the second step the other half.  A step is 16 MFMAs of 32 clocks, as long
// as the 32 MFMAs of 16 clocks of a bf16 slice, and moves the same bytes, so the FP8 tile does twice the work per step.
// At the end of a tile the groups meet and run their epilogues side by side, then fall a phase apart again: one wavefront per
// SIMD leaves the vector unit idle most of an epilogue, and with the groups a phase apart the two came one after the other
// (5 + 6 of the 35 us of a Qwen3-shaped up-projection tile).  Kernel trace, up and down: Qwen3-shaped T = 3500 112.0 -> 107.3 and
// 84.0 -> 76.3 us, Mixtral-shaped T = 8192 1552 -> 1520 and 774 -> 759 us, OLMoE-shaped T = 1024 of 16 experts (128-row tile)
// 52.2 -> 51.1 and 42.0 -> 35.6 us.
//
// Rings.  Token rows go through LDS in halves (16 KB) that are free one step after they were read, weights in whole slices
// (32 KB) that are free after the first step of their slice: 5 halves + 2 weight slices (tile of 256, up-projection) keep
// every load four to six phases ahead of its use.  The number of loads between a load and the step that needs it is the
// same everywhere: the stream crosses into the next tile of the workgroup without a break, and past its last tile it goes on
// with loads that all lanes aim at one cache line, so the vmcnt waits are constants.
//
// Scales.  16 k-blocks of scale bytes per token row, and of the tile's weight rows, come into LDS with the weight slice that
// starts their 16-slice chunk (wavefronts 0-3: tokens, 4: weights; in the down-projection 5 and 6 bring the destination pair
// and router weight of every slot along with chunk 0).
//
// Re-quantisation.  The 128 features of an up-projection tile are one scale block, so its epilogue also quantises: row
// maxima meet in LDS across the four wavefronts of a token row (one barrier), codes and scale bytes are stored in the
// order the down-projection loads them, and the activation never exists in bf16 in memory.
// The epilogue is bound by its vector instructions (some 1900 a wavefront, two wavefronts a SIMD: 5.5 us of the 53 of a Mixtral-shaped
// tile), so the maxima are taken on the magnitude bits, two values an instruction, and v_cvt_scalef32_pk_fp8_bf16 scales and
// converts finite rows; rows with an infinity or NaN take the general conversion.  Up-projection, kernel trace: Mixtral-shaped
// T = 8192 1565 -> 1535 us, OLMoE-shaped T = 1024 of 16 experts (128-row tile) 54.6 -> 53.2, Qwen3-shaped T = 3500 120.7 -> 119.5.
//
// Measured: Mixtral-shaped layer, T = 8192 (5.8 TFLOP), 256-row tile, kernel trace: up-projection 1520 to 1580 us = 2.44 to 2.53 PFLOP/s
// and down-projection 770 to 800 us = 2.40 to 2.50 PFLOP/s, against 3073 + 320 (quantising pass) + 1302 us of the 128 x 256 tile with one
// barrier per slice.  The matrix pipes are busy 68 % of the up-projection's clocks and 78 % of the down-projection's, at 1.5 to 1.8 GHz:
// the chip holds these kernels at its power limit, so bytes that don't cross the fabric come back as clock.  What the loop waits
// for is its M phase, LDS reads at 128 bytes a clock and the issue of a 1 KB load every 16 clocks.
#pragma once

#include <type_traits>

#include "fp8_format.h"
#include "moe_gemm.h"

namespace ramp {

struct Fp8PingPongArgs {
    const uint8_t *act_q;      // token operand: codes row-major [T, H] (stage 1), fragments [slots/16][I/128][2 KB] (stage 2)
    const uint8_t *act_scale;  // [rows][act_stride] E8M0 bytes, rows padded to 16 k-blocks
    int act_stride;
    const uint8_t *wq;         // packed codes of this stage
    size_t expert_stride;      // bytes between experts
    uint32_t up_offset;        // stage 1: byte offset of the up rows inside an expert
    const uint8_t *wscale;     // first scale array of this stage (gate, or down)
    size_t wscale_expert_stride;
    uint32_t wscale_up_offset; // stage 1: gate -> up scale array
    int w_stride;              // scale row stride of the weights
    uint8_t *aq_out;           // stage 1: activation codes in stage 2's order
    uint8_t *as_out;           // stage 1: activation scale bytes [slots][as_stride]
    int as_stride;
};

template <int STAGE, int NH>
struct Fp8PingPongTraits {
    static constexpr int BM = 128 * NH, BN = 256;
    static constexpr int NB = 4 * NH;                            // token blocks per wavefront
    static constexpr int NW = (NH == 2) ? 2 : 3;                 // weight slices in LDS
    static constexpr int NXH = (NH == 1) ? 3 : (STAGE == 1 ? 5 : 4);  // token halves in LDS
    static constexpr int W_BYTES = 32 * 1024, XH_BYTES = 16 * 1024;
    static constexpr int SCALE_BYTES = BM * 16 + 256;            // one 16-slice chunk: token rows, then weight rows
    static constexpr int SLOT_BYTES = (STAGE == 2) ? BM * 8 : 0; // pair and router weight of every slot
    static constexpr int OFF_W = NXH * XH_BYTES, OFF_S = OFF_W + NW * W_BYTES, OFF_SLOT = OFF_S + 2 * SCALE_BYTES;
    static constexpr int STG_ROWS = 8 * NH;                      // output rows a wavefront stages at a time (128 bytes each)
    static constexpr int OFF_E = OFF_SLOT + 2 * SLOT_BYTES;      // epilogue: row maxima (stage 1), staged output rows (stage 2)
    static constexpr int LDS_BYTES = OFF_E + (STAGE == 1 ? BM * 16 : 8 * STG_ROWS * 128);
    static_assert(LDS_BYTES <= kLdsBytesPerCU, "tile does not fit in LDS");
    static constexpr int MIN_SLICES = 3;
    // loads of a wavefront that may stay in flight at the end of an M phase: those issued after what the next step reads
    static constexpr int WAIT = (NH == 1) ? 6 : (NXH == 5 ? 10 : 8);
};

template <int STAGE, int NH>
__global__ __launch_bounds__(512, 1) void moe_fp8_pingpong_kernel(GemmArgs a, Fp8PingPongArgs f)
{
    using PT = Fp8PingPongTraits<STAGE, NH>;
    constexpr int BM = PT::BM, NB = PT::NB, NW = PT::NW, NXH = PT::NXH;
    constexpr int FEAT = (STAGE == 1) ? 128 : 256;   // output features per tile
    constexpr int FB = (STAGE == 1) ? 2 : 4;         // 16-feature blocks of a wavefront (gate and up each in stage 1)

    __shared__ __attribute__((aligned(1024))) char lds[PT::LDS_BYTES];
    char *const lds_x = lds;
    char *const lds_w = lds + PT::OFF_W;
    char *const lds_s = lds + PT::OFF_S;
    char *const lds_slot = lds + PT::OFF_SLOT;
    char *const lds_e = lds + PT::OFF_E;

    const int lane = threadIdx.x & 63;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int wm = wave >> 2, wn = wave & 3;  // wm is also the phase group
    const int r16 = lane & 15, q = lane >> 4;
    const int KT = a.K >> 7;
    const int m_tiles = load_uniform_i32(a.meta + 1);

    // As in the bf16 kernel, but only a down-projection tile of 128 rows is cut, in halves: the 128 features of an up-projection tile
    // are quantised together, and the tile of 256 rows has no register to spare for it.
    constexpr bool CUTS = STAGE == 2 && NH == 1;
    const TileWalk walk = tile_walk(a, m_tiles, a.tile_expert, CUTS ? 2 : 1);
    auto tile_at = [&](int pos, int &n_tile, int &m_tile) __attribute__((always_inline)) -> bool {
        if (pos >= walk.whole) return false;
        tile_of_slot(a, walk, walk_slot(walk, pos), n_tile, m_tile);
        n_tile = __builtin_amdgcn_readfirstlane(n_tile);
        m_tile = __builtin_amdgcn_readfirstlane(m_tile);
        return true;
    };
    auto column_works = [&](int pos, int column) __attribute__((always_inline)) -> bool {
        return !CUTS || pos >= 0 || column / 2 == walk.part;
    };
    auto phase_barrier = [&]() __attribute__((always_inline)) {
        __builtin_amdgcn_sched_barrier(0);
        __builtin_amdgcn_s_barrier();
        __builtin_amdgcn_sched_barrier(0);
    };

    // ---- load stream.  Per tile: weights = expert codes + offset of this wavefront's first row block, tokens = one
    // offset per load of a half (two loads of 1 KB per wavefront and half), scales = one row per lane.
    struct TileSrc {
        const uint8_t *w;        // codes of row block wave/2 of the tile, half-fragment wave%2, slice 0
        const uint8_t *ws;       // weight scale row of the tile (gate, or down)
        uint32_t w_lane;         // lane * 16, or 0 past the last tile
        uint32_t w_second, s_second;  // from the first eight row blocks, and their scale row, to the other eight
    };
    auto weights_of = [&](int pos, int n_tile, int e) __attribute__((always_inline)) {
        TileSrc s;
        s.w = f.wq + (size_t)e * f.expert_stride + (size_t)(n_tile * (FEAT / 16) + (wave >> 1)) * (size_t)(KT * 2048) +
              (size_t)((wave & 1) * 1024);
        s.ws = f.wscale + (size_t)e * f.wscale_expert_stride + (size_t)(n_tile * (FEAT / 128)) * (size_t)f.w_stride;
        s.w_lane = (uint32_t)lane * 16u;
        // stage 1: the up rows; stage 2: the tile's other 128 features, or the same ones again where a last tile has none
        // or, of a cut tile, where a workgroup has 128 of them
        bool second = STAGE == 1 || n_tile * FEAT + 128 < a.F;
        if (CUTS && pos < 0) {
            if (walk.part && second) {
                s.w += (size_t)KT * (8 * 2048);
                s.ws += f.w_stride;
            }
            second = false;
        }
        s.w_second = STAGE == 1 ? f.up_offset : second ? (uint32_t)KT * (8u * 2048u) : 0u;
        s.s_second = STAGE == 1 ? f.wscale_up_offset : second ? (uint32_t)f.w_stride : 0u;
        return s;
    };
    // row block wave/2 + 4*s: stage 1 holds 8 gate row blocks, then the 8 up row blocks of the same features
    auto issue_w = [&](const TileSrc &src, int slice, int buf) __attribute__((always_inline)) {
        const uint8_t *base = src.w + (uint32_t)slice * 2048u;
        const uint32_t rb4 = (uint32_t)KT * (4u * 2048u);
#pragma unroll
        for (int s = 0; s < 4; ++s) {
            const uint32_t off = (uint32_t)(s & 1) * rb4 + (s >= 2 ? src.w_second : 0u);
            load_to_lds_16B(base + off + src.w_lane, lds_w + buf * PT::W_BYTES + (wave + 8 * s) * 1024);
        }
    };
    // rows of token loads: stage 1 takes 8 rows x 128 bytes per load, stage 2 one half-fragment of 16 slots
    auto load_row = [&](int h, int t) { return h * 128 + (wave + 8 * t) * 8 + (lane >> 3); };
    // pair index (stage 1: as loaded from the sorted list) -> byte offset of this lane's piece of slice 0
    auto token_offset = [&](int h, int t, uint32_t pair, int m_tile, int rows) __attribute__((always_inline)) -> uint32_t {
        if (STAGE == 1) {
            const int row = load_row(h, t);
            if (h * 128 + (wave + 8 * t) * 8 >= rows) return 0u;  // nothing but padding: one cache line for all lanes
            const uint32_t p = pair < (uint32_t)a.P ? pair : 0u;
            const uint32_t tok = (uint32_t)(((unsigned long long)p * a.topk_magic) >> 40);
            const uint32_t c = (uint32_t)((lane & 7) ^ ((row >> 1) & 7));  // piece 2*(c % 4) + c/4 of the row
            return tok * (uint32_t)a.K + ((c & 3u) * 2u + (c >> 2)) * 16u;
        }
        const int blk = h * 8 + ((wave + 8 * t) >> 1);
        const uint32_t l = (uint32_t)lane * 16u;
        if (blk * 16 >= rows) return l;
        return (uint32_t)(m_tile * (BM / 16) + blk) * (uint32_t)(KT * 2048) + (uint32_t)((wave & 1) * 1024) + l;
    };
    constexpr uint32_t XSTEP = (STAGE == 1) ? 128u : 2048u;
    uint32_t xoff[NH][2];
    auto issue_x = [&](int h, int slice, int buf) __attribute__((always_inline)) {
        const uint8_t *base = f.act_q + (uint32_t)slice * XSTEP;
#pragma unroll
        for (int t = 0; t < 2; ++t) load_to_lds_16B(base + xoff[h][t], lds_x + buf * PT::XH_BYTES + (wave + 8 * t) * 1024);
    };
    // scales of slices 16*chunk .. +15 of a tile; srow: byte offset of this lane's token scale row (wavefronts below BM/64)
    auto scale_row = [&](uint32_t pair, int m_tile) __attribute__((always_inline)) -> uint32_t {
        const int slot = m_tile * BM + (wave & (BM / 64 - 1)) * 64 + lane;
        if (STAGE == 2) return (uint32_t)slot * (uint32_t)f.act_stride;
        const uint32_t p = pair < (uint32_t)a.P ? pair : 0u;
        return (uint32_t)(((unsigned long long)p * a.topk_magic) >> 40) * (uint32_t)f.act_stride;
    };
    auto issue_s = [&](const TileSrc &src, uint32_t srow, int m_tile, int chunk, int buf, int slot_buf) __attribute__((always_inline)) {
        char *dst = lds_s + buf * PT::SCALE_BYTES;
        int role = wave;
        asm volatile("" : "+s"(role));  // opaque: the compiler would otherwise make a copy of the slice loop per role
        if (role < BM / 64) {
            load_to_lds_16B(f.act_scale + srow + (uint32_t)chunk * 16u, dst + wave * 1024);
        } else if (role == 4) {
            // lanes 0-3: the chunk's words of the (gate) scale row, 4-7: of the up row (stage 1) or of the second block of
            // 128 features (stage 2); words past the end of a row repeat its last one
            int word = chunk * 4 + (lane & 3);
            const int last = (KT - 1) >> 2;
            word = word < last ? word : last;
            const uint8_t *p = src.ws + ((lane & 4) ? src.s_second : 0u) + (uint32_t)word * 4u;
            __builtin_amdgcn_global_load_lds((const __attribute__((address_space(1))) void *)p,
                                             (__attribute__((address_space(3))) void *)(dst + BM * 16), 4, 0, 0);
        } else if (STAGE == 2 && chunk == 0 && (role == 5 || role == 6)) {
            if (lane < BM / 4) {
                const void *p = role == 5 ? (const void *)(a.sorted + (size_t)m_tile * BM + lane * 4)
                                          : (const void *)(a.slot_w + (size_t)m_tile * BM + lane * 4);
                load_to_lds_16B(p, lds_slot + slot_buf * PT::SLOT_BYTES + (role - 5) * BM * 4);
            }
        }
    };

    // ---- operands and accumulators
    floatx4 acc[4][NB];
    auto zero_acc = [&]() __attribute__((always_inline)) {
#pragma unroll
        for (int i = 0; i < 4; ++i)
#pragma unroll
            for (int j = 0; j < NB; ++j) acc[i][j] = floatx4{0.f, 0.f, 0.f, 0.f};
    };
    intx8 wf[4], xf[4];
    uint32_t sx[NB], sw[2];
    auto join = [](const intx4 &lo, const intx4 &hi) __attribute__((always_inline)) {
        return intx8{lo[0], lo[1], lo[2], lo[3], hi[0], hi[1], hi[2], hi[3]};
    };
    auto read_w = [&](int buf) __attribute__((always_inline)) {
        const char *p = lds_w + buf * PT::W_BYTES + lane * 16;
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            const int rb = (STAGE == 1) ? (i < 2 ? wn * 2 + i : 8 + wn * 2 + i - 2) : wn * 4 + i;
            wf[i] = join(*reinterpret_cast<const intx4 *>(p + rb * 2048), *reinterpret_cast<const intx4 *>(p + rb * 2048 + 1024));
        }
    };
    // token block nb of this wavefront inside a half is block 2*nb + wm (blocks are dealt to the two wavefront rows)
    const int xlane = (STAGE == 1) ? (r16 >> 3) * 1024 + (r16 & 7) * 128 + ((q ^ ((r16 >> 1) & 7)) * 16) : lane * 16;
    auto read_x = [&](int buf) __attribute__((always_inline)) {
        const char *p = lds_x + buf * PT::XH_BYTES + wm * 2048;
        const int lo = xlane, hi = (STAGE == 1) ? (xlane ^ 64) : xlane + 1024;
#pragma unroll
        for (int nb = 0; nb < 4; ++nb)
            xf[nb] = join(*reinterpret_cast<const intx4 *>(p + nb * 4096 + lo), *reinterpret_cast<const intx4 *>(p + nb * 4096 + hi));
    };
    // scale words of slices 4*(kt/4) .. +3
    auto read_s = [&](int buf, int kt) __attribute__((always_inline)) {
        const char *p = lds_s + buf * PT::SCALE_BYTES + ((kt >> 2) & 3) * 4;
#pragma unroll
        for (int nb = 0; nb < NB; ++nb) {
            const int row = (nb >> 2) * 128 + ((nb & 3) * 2 + wm) * 16 + r16;
            sx[nb] = *reinterpret_cast<const uint32_t *>(p + row * 16);
        }
        if (STAGE == 1) {
            sw[0] = *reinterpret_cast<const uint32_t *>(p + BM * 16);
            sw[1] = *reinterpret_cast<const uint32_t *>(p + BM * 16 + 16);
        } else {
            sw[0] = *reinterpret_cast<const uint32_t *>(p + BM * 16 + (wn >> 1) * 16);
        }
    };
    auto multiply = [&](int h, int sh) __attribute__((always_inline)) {
        const int s0 = (int)(sw[0] >> sh), s1 = (STAGE == 1) ? (int)(sw[1] >> sh) : s0;
#pragma unroll
        for (int nb = 0; nb < 4; ++nb) {
            const int sb = (int)(sx[h * 4 + nb] >> sh);
#pragma unroll
            for (int i = 0; i < 4; ++i)
                acc[i][h * 4 + nb] = __builtin_amdgcn_mfma_scale_f32_16x16x128_f8f6f4(wf[i], xf[nb], acc[i][h * 4 + nb], 0, 0, 0,
                                                                                      i < 2 ? s0 : s1, 0, sb);
        }
        // (no instruction) keeps the products in this phase: the compiler otherwise sinks them past the barrier, behind the
        // branches of the next M phase, where nothing runs beside them
#pragma unroll
        for (int nb = 0; nb < 4; ++nb)
#pragma unroll
            for (int i = 0; i < 4; ++i) asm volatile("" : "+v"(acc[i][h * 4 + nb]));
    };
    // token blocks with a real row (they come first) among those of this wavefront in a half
    auto blocks_of_half = [&](int rows, int h) __attribute__((always_inline)) {
        const int v = ((rows + 15) / 16 - h * 8 - wm + 1) / 2;
        return v < 0 ? 0 : (v > 4 ? 4 : v);
    };

    int n_tile, m_tile;
    auto opaque = [](int v) __attribute__((always_inline)) -> int {
        asm volatile("" : "+s"(v));
        return v;
    };
    int pos = opaque(walk_first(walk));
    if (!tile_at(pos, n_tile, m_tile)) return;
    int rows = load_uniform_i32(a.tile_rows + m_tile);
    TileSrc src = weights_of(pos, n_tile, load_uniform_i32(a.tile_expert + m_tile));
    int src_m = m_tile;       // tile the weight and scale loads are in
    uint32_t srow = 0;
    {
        if (STAGE == 1) {
#pragma unroll
            for (int h = 0; h < NH; ++h)
#pragma unroll
                for (int t = 0; t < 2; ++t) xoff[h][t] = (uint32_t)a.sorted[m_tile * BM + load_row(h, t)];
            srow = (uint32_t)a.sorted[m_tile * BM + (wave & (BM / 64 - 1)) * 64 + lane];
        }
#pragma unroll
        for (int h = 0; h < NH; ++h)
#pragma unroll
            for (int t = 0; t < 2; ++t) xoff[h][t] = token_offset(h, t, xoff[h][t], m_tile, rows);
        srow = scale_row(srow, m_tile);
    }
    zero_acc();

    // prologue: what the steps before step 0 would have issued, in their order
    int s_issue = 0, s_cur = 1;      // scale ring: next chunk to load / chunk being read (toggled at its first slice)
    int slot_cur = 0;                // slot table half of the current tile
    issue_s(src, srow, m_tile, 0, 0, 0);
    s_issue = 1;
    issue_w(src, 0, 0);
    issue_x(0, 0, 0);
    if (NH == 2) {
        issue_x(NH - 1, 0, 1);
        issue_w(src, 1, 1);
        issue_x(0, 1, 2);
        if (NXH == 5) issue_x(NH - 1, 1, 3);
    } else {
        issue_w(src, 1, 1);
        issue_x(0, 1, 1);
    }
    wait_vmcnt<PT::WAIT>();
    phase_barrier();

    int wb = 0, wb_issue = (NH == 2) ? 0 : 2;  // weight ring: buffer being read / being loaded
    int xb = 0, xb_issue = NXH - 1;            // token ring
    // slices the stream loads next (of this tile until they wrap to 0, then of the next): weights, token halves
    int wsl = 2, xsl[NH];
    xsl[0] = 2;
    if (NH == 2) xsl[NH - 1] = (NXH == 5) ? 2 : 1;
    while (true) {
        // the following tile of this workgroup, whose first slices are loaded while this one finishes
        int n_next = n_tile, m_next = m_tile;
        const int pos_next = opaque(walk_next(walk, pos));
        const bool has_next = tile_at(pos_next, n_next, m_next);
        if (!has_next) {
            n_next = n_tile;
            m_next = m_tile;
        }
        const int rows_next = has_next ? load_uniform_i32(a.tile_rows + m_next) : 0;
        TileSrc src_next = weights_of(pos_next, n_next, load_uniform_i32(a.tile_expert + m_next));
        if (!has_next) src_next.w_lane = 0;
        uint32_t xoff_n[NH][2] = {}, srow_n = 0;
        if (STAGE == 1) {
#pragma unroll
            for (int h = 0; h < NH; ++h)
#pragma unroll
                for (int t = 0; t < 2; ++t) xoff_n[h][t] = (uint32_t)a.sorted[m_next * BM + load_row(h, t)];
            srow_n = (uint32_t)a.sorted[m_next * BM + (wave & (BM / 64 - 1)) * 64 + lane];
        }
        const int no_chunk = has_next ? -1 : 0;  // past the last tile no scales are loaded
        int nbh[NH];
#pragma unroll
        for (int h = 0; h < NH; ++h) nbh[h] = blocks_of_half(rows, h);
#pragma unroll
        for (int nb = 0; nb < NB; ++nb) sx[nb] = 0;  // (read again at slice 0: nothing is carried from tile to tile)
        sw[0] = sw[1] = 0;

        // The load stream of a step: a token half and, once per slice, the weights two slices ahead go into the buffers that
        // became free.  cross_*() come first: where the stream enters the next tile it takes over that tile's
        // offsets, and where a weight slice begins a chunk of scales, it issues their loads.
        auto cross_x = [&](int h) __attribute__((always_inline)) {
            if (xsl[h] == 0) {
#pragma unroll
                for (int t = 0; t < 2; ++t) {
                    uint32_t p = xoff_n[h][t];
                    // keeps the arithmetic, and the wait for the index loads, here instead of in front of the slice loop
                    if (STAGE == 1) asm volatile("" : "+v"(p));
                    xoff[h][t] = token_offset(h, t, p, m_next, rows_next);
                }
            }
        };
        auto cross_w = [&]() __attribute__((always_inline)) {
            if (wsl == 0) {
                src = src_next;
                src_m = m_next;
                uint32_t p = srow_n;
                if (STAGE == 1) asm volatile("" : "+v"(p));
                srow = scale_row(p, m_next);
            }
            if ((wsl & 15) == 0 && wsl != no_chunk) {
                issue_s(src, srow, src_m, wsl >> 4, s_issue, slot_cur ^ 1);
                s_issue ^= 1;
            }
        };
        auto step = [&](int kt, auto h_c, auto live_c) __attribute__((always_inline)) {
            constexpr int h = decltype(h_c)::value;
            constexpr bool LIVE = decltype(live_c)::value;          // the half holds real rows
            constexpr bool W_STEP = (NH == 1) || h == 1;            // weight slices are issued in the last step of a slice
            constexpr int XH = (NXH == 4) ? 1 - h : h;              // half that is issued
            // ---- M phase
            cross_x(XH);
            if (W_STEP) cross_w();
            if (h == 0) {
                if ((kt & 15) == 0) s_cur ^= 1;
                if ((kt & 3) == 0) read_s(s_cur, kt);
                read_w(wb);
                wb = (wb + 1 == NW) ? 0 : wb + 1;
            }
            if (LIVE) read_x(xb);
            xb = (xb + 1 == NXH) ? 0 : xb + 1;
            if (W_STEP) {
                issue_w(src, wsl, wb_issue);
                wsl = (wsl + 1 == KT) ? 0 : wsl + 1;
                wb_issue = (wb_issue + 1 == NW) ? 0 : wb_issue + 1;
            }
            issue_x(XH, xsl[XH], xb_issue);
            xsl[XH] = (xsl[XH] + 1 == KT) ? 0 : xsl[XH] + 1;
            xb_issue = (xb_issue + 1 == NXH) ? 0 : xb_issue + 1;
            wait_vmcnt<PT::WAIT>();
            __builtin_amdgcn_s_waitcnt(0xc07f);  // lgkmcnt(0): operands in registers, buffers no longer read
            phase_barrier();
            // ---- C phase
            if (LIVE) multiply(h, (kt & 3) * 8);
            phase_barrier();
        };
        if (wm == 1) phase_barrier();  // stagger
        using H0 = std::integral_constant<int, 0>;
        using True = std::integral_constant<bool, true>;
        using False = std::integral_constant<bool, false>;
        if (NH == 1) {
            for (int kt = 0; kt < KT; ++kt) step(kt, H0{}, True{});
        } else if (rows > 128) {
            for (int kt = 0; kt < KT; ++kt) {
                step(kt, H0{}, True{});
                step(kt, std::integral_constant<int, NH - 1>{}, True{});
            }
        } else {  // nothing but padding in the second half: its steps only keep the loads and the phases going
            for (int kt = 0; kt < KT; ++kt) {
                step(kt, H0{}, True{});
                step(kt, std::integral_constant<int, NH - 1>{}, False{});
            }
        }

        if (wm == 0) phase_barrier();  // in step again
        // ---- epilogue: lane holds features 4*q + {0..3} of every 16-row block of token r16.  The lane index is made opaque:
        // addresses derived from it would otherwise be computed in front of the slice loop and spilled across it.
        int el = lane;
        asm volatile("" : "+v"(el));
        const int er = el & 15, eq = el >> 4;
        if (STAGE == 1) {
            // [BM][4] largest magnitude bits of a wavefront's 32 features; of rows with an infinity or NaN, marked by the top bit,
            // those without the NaNs
            uint32_t *row_top = reinterpret_cast<uint32_t *>(lds_e);
            auto across = [](uint32_t v) __attribute__((always_inline)) {
                v = max(v, (uint32_t)__shfl_xor((int)v, 16));
                return max(v, (uint32_t)__shfl_xor((int)v, 32));
            };
#pragma unroll
            for (int nb = 0; nb < NB; ++nb) {
                if ((nb & 3) < nbh[nb >> 2]) {
                    float v[8];
#pragma unroll
                    for (int i = 0; i < 2; ++i)
#pragma unroll
                        for (int c = 0; c < 4; ++c) v[i * 4 + c] = silu_f32(acc[i][nb][c]) * acc[2 + i][nb][c];
                    intx4 two;
                    ushortx2 m = {0, 0};
#pragma unroll
                    for (int c = 0; c < 4; ++c) {
                        two[c] = (int)f32x2_to_bf16x2(v[2 * c], v[2 * c + 1]);
                        m = max_bf16_bits(m, (uint32_t)two[c]);
                    }
                    acc[0][nb] = __builtin_bit_cast(floatx4, two);  // the 8 features wait in the accumulators' place
                    uint32_t top = across(m[0] > m[1] ? m[0] : m[1]);
                    if (__builtin_expect(top >= 0x7f80u, 0)) {
                        top = 0;
#pragma unroll
                        for (int c = 0; c < 4; ++c) {
                            const uint32_t lo = (uint32_t)two[c] & 0x7fffu, hi = ((uint32_t)two[c] >> 16) & 0x7fffu;
                            top = max(top, max(lo > 0x7f80u ? 0u : lo, hi > 0x7f80u ? 0u : hi));
                        }
                        top = across(top) | 0x80000000u;
                    }
                    const int row = (nb >> 2) * 128 + ((nb & 3) * 2 + wm) * 16 + er;
                    if (eq == 0) row_top[row * 4 + wn] = top;
                }
            }
            __builtin_amdgcn_s_waitcnt(0xc07f);
            phase_barrier();
            // the wavefront's 32 features of the block: k = 32*(wn/2 * 2 + eq/2) + 16*(eq%2) + 8*(wn%2) + 0..7 of the scale block
            const uint32_t k8 = (uint32_t)((wn >> 1) * 64 + eq * 16 + (wn & 1) * 8);
            uint8_t *dst = f.aq_out + (size_t)n_tile * 2048 + ((k8 >> 4) & 1u) * 1024u + ((k8 >> 5) * 16u + (uint32_t)er) * 16u + (k8 & 15u);
#pragma unroll
            for (int nb = 0; nb < NB; ++nb) {
                if ((nb & 3) < nbh[nb >> 2]) {
                    const int blk = (nb >> 2) * 8 + (nb & 3) * 2 + wm;
                    const uint4 t4 = *reinterpret_cast<const uint4 *>(row_top + (blk * 16 + er) * 4);
                    const uint32_t clear = 0x7fffffffu;
                    const uint32_t top = max(max(t4.x & clear, t4.y & clear), max(t4.z & clear, t4.w & clear));
                    const uint32_t b = e8m0_of_amax(bf16_bits_to_f32(top));
                    const intx4 two = __builtin_bit_cast(intx4, acc[0][nb]);
                    uint32_t codes[2];
                    if (__builtin_expect((int)(t4.x | t4.y | t4.z | t4.w) < 0, 0)) {
                        const float inv = inv_scale_of(b);
                        float v[8];
#pragma unroll
                        for (int c = 0; c < 4; ++c) {
                            v[2 * c] = bf16_bits_to_f32((uint32_t)two[c] & 0xffffu) * inv;
                            v[2 * c + 1] = bf16_bits_to_f32((uint32_t)two[c] >> 16) * inv;
                        }
                        codes[0] = e4m3x4_of_f32(v);
                        codes[1] = e4m3x4_of_f32(v + 4);
                    } else {
                        // (as in quantise_group: a finite row needs no saturation)
                        const float scale = __builtin_bit_cast(float, b << 23);
#pragma unroll
                        for (int c = 0; c < 2; ++c) {
                            const uint32_t lo = (uint32_t)two[2 * c], hi = (uint32_t)two[2 * c + 1];  // (values: __builtin_bit_cast takes a vector's element for its first)
                            shortx2 r = {0, 0};
                            r = __builtin_amdgcn_cvt_scalef32_pk_fp8_bf16(r, __builtin_bit_cast(bf16x2, lo), scale, false);
                            r = __builtin_amdgcn_cvt_scalef32_pk_fp8_bf16(r, __builtin_bit_cast(bf16x2, hi), scale, true);
                            codes[c] = __builtin_bit_cast(uint32_t, r);
                        }
                    }
                    const size_t frag = (size_t)(m_tile * (BM / 16) + blk) * (size_t)(a.F >> 7);
                    *reinterpret_cast<uint2 *>(dst + frag * 2048) = make_uint2(codes[0], codes[1]);
                    if (wn == 0 && eq == 0) f.as_out[(size_t)(m_tile * BM + blk * 16 + er) * (size_t)f.as_stride + n_tile] = (uint8_t)b;
                }
            }
        } else if (n_tile * FEAT + wn * 64 < a.F && column_works(pos, wn)) {  // (not the empty half of a last tile, nor what others have of a cut one)
            const int *pairs = reinterpret_cast<const int *>(lds_slot + slot_cur * PT::SLOT_BYTES);
            const float *wgts = reinterpret_cast<const float *>(pairs + BM);
            const int f0 = n_tile * FEAT + wn * 64;
            constexpr int SR = PT::STG_ROWS;
            char *stg = lds_e + wave * (SR * 128);
#pragma unroll
            for (int nb = 0; nb < NB; ++nb) {
                if ((nb & 3) >= nbh[nb >> 2]) continue;
                const int row0 = (nb >> 2) * 128 + ((nb & 3) * 2 + wm) * 16;
                const float wgt = wgts[row0 + er];
                if (a.y_bf16) {
                    // through a staging area of the wavefront, so that a store covers whole 128-byte lines
#pragma unroll
                    for (int p0 = 0; p0 < 16; p0 += SR) {
                        if (SR == 16 || (er & 8) == p0) {
#pragma unroll
                            for (int half = 0; half < 2; ++half) {
                                float w8[8];
#pragma unroll
                                for (int c = 0; c < 4; ++c) {
                                    w8[c] = wgt * acc[2 * half][nb][c];
                                    w8[4 + c] = wgt * acc[2 * half + 1][nb][c];
                                }
                                store_bf16x8(reinterpret_cast<uint16_t *>(stg + (er & (SR - 1)) * 128 + (((2 * eq + half) ^ ((er >> 1) & 7)) * 16)), w8);
                            }
                        }
#pragma unroll
                        for (int p = 0; p < SR; p += 8) {
                            const int r = p0 + p + (el >> 3);
                            const int pair = pairs[row0 + r];
                            const uint4 v = *reinterpret_cast<const uint4 *>(stg + (r & (SR - 1)) * 128 + (((el & 7) ^ ((r >> 1) & 7)) * 16));
                            if (pair < a.P)
                                *reinterpret_cast<uint4 *>(reinterpret_cast<uint16_t *>(a.y_out) + (size_t)pair * a.F + f0 + (el & 7) * 8) = v;
                        }
                    }
                } else {
                    store_pair_rows_f32<SR / 2>(a, stg, &acc[0][nb], NB, pairs[row0 + er], wgt, f0, el);
                }
            }
        }
        if (!has_next) break;
        pos = pos_next;
        n_tile = n_next;
        m_tile = m_next;
        rows = rows_next;
        slot_cur ^= 1;
        zero_acc();
    }
    wait_vmcnt<0>();               // no load may still write LDS when the workgroup ends
}

template <int NH>
void launch_fp8_pingpong(int stage, const GemmArgs &a, const Fp8PingPongArgs &f, hipStream_t stream)
{
    if (a.n_tiles <= 0 || a.m_tiles_cap <= 0) return;
    GemmArgs g = a;
    const unsigned tiles = xcd_grid(g);
    const dim3 grid(tiles < (unsigned)kNumCU ? tiles : (unsigned)kNumCU), block(512);
    if (stage == 1)
        hipLaunchKernelGGL((moe_fp8_pingpong_kernel<1, NH>), grid, block, 0, stream, g, f);
    else
        hipLaunchKernelGGL((moe_fp8_pingpong_kernel<2, NH>), grid, block, 0, stream, g, f);
}

}  // namespace ramp
