// Internal declarations shared by the library's translation units (not installed).
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>
#include <stdio.h>

#include "ramp.h"
#include "tile_walk.h"

namespace ramp {

// Thread-local message for ramp_last_error().
void set_error(const char *fmt, ...);

inline int check_launch(const char *what)
{
    hipError_t err = hipGetLastError();
    if (err != hipSuccess) {
        set_error("%s: %s", what, hipGetErrorString(err));
        return RAMP_EHIP;
    }
    return RAMP_OK;
}

constexpr int kNumCU = 256;           // MI355X compute units
constexpr int kLdsBytesPerCU = 160 * 1024;
constexpr int kWave = 64;

inline size_t align_up(size_t v, size_t a) { return (v + a - 1) / a * a; }

// ---- align ----
constexpr int kAlignThreads = 1024;   // one workgroup = 16 wavefronts
constexpr int kAlignChunk = 1024;     // pairs per workgroup in the multi-workgroup path
constexpr int kAlignSingleMaxP = 2048; // up to this many pairs no workspace is needed
// up to this many pairs and tokens every workgroup of one launch counts all pairs itself; past it, two launches share the counting
constexpr int kAlignOneLaunchMaxP = 16384;
constexpr int kAlignOneLaunchMaxT = 2048;
inline bool align_is_one_launch(int T, int k) { return T <= kAlignOneLaunchMaxT && (long long)T * k <= kAlignOneLaunchMaxP; }
constexpr int kAlignMaxE = 1024;

// Optional second output of the scatter: slot_w[s] = topk_w[sorted[s]] for the slots that hold a pair (the others are
// left as they are), so that a kernel can read the router weight of a slot without first waiting for its pair index.
struct AlignSlotWeights {
    const float *topk_w;
    float *slot_w;
};

int launch_align(const int32_t *ids, int T, int k, int E, int bm, int32_t *sorted, int32_t *tile_expert,
                 int32_t *tile_rows, int32_t *counts, int32_t *meta, void *ws, size_t ws_bytes, hipStream_t stream,
                 const int32_t *pred = nullptr, int pred_value = 0, AlignSlotWeights slot_weights = {nullptr, nullptr});

// Align for the device-selected layer: bm, capacity and workspace sections (byte offsets) of every candidate; bm = 0 for one
// that aligns in its own kernels.
constexpr int kMaxCandidates = 16;
struct AlignChoice {
    int32_t bm, cap, with_slot_w;
    size_t sorted, tile_expert, tile_rows, counts, meta, slot_w;
};
struct AlignChoices {
    AlignChoice c[kMaxCandidates];
};
int launch_align_selected(const int32_t *ids, int P, int E, const float *topk_w, char *base, const int32_t *sel, int n_cand,
                          const AlignChoices &choices, hipStream_t stream);

// bf16 rows to quantise to E4M3 codes and a scale byte per 128 values (fp8_format.h)
struct QuantRows {
    const uint16_t *src;
    int rows, K;
    uint8_t *codes, *sb;
    int stride;  // scale bytes per row
};
// Align of at least one pair and, by other workgroups of its only or its second launch, the quantised hidden state.  (A call of at
// most 64 pairs too takes the form of one launch.)
int launch_align_quant(const int32_t *ids, int T, int k, int E, int bm, int32_t *sorted, int32_t *tile_expert, int32_t *tile_rows,
                       int32_t *counts, int32_t *meta, void *ws, size_t ws_bytes, AlignSlotWeights slot_weights, const QuantRows &q,
                       hipStream_t stream);

// ---- packed weights ----
// 16 bytes of bf16 values at the alignment of one value: the caller's weights and rows to quantise may start anywhere
typedef uint32_t UnalignedWords4 __attribute__((ext_vector_type(4), aligned(2)));
// One fragment = 16 weight rows x 32 k-values = 512 bf16 = 1 KB, stored in the lane order
// of the A operand of v_mfma_f32_16x16x32_bf16: element (row r, k = 8*q + j) at (q*16 + r)*8 + j.
constexpr int kFragElems = 512;
// Which output feature sits in row r of packed row block rb.  Inside every group of 4 row blocks
// (64 features) the rows are interleaved so that, after the MFMA, lane group q of a wavefront holds
// 4 consecutive features per row block it owns, consecutive row blocks continuing the run: a lane
// that owns all 4 row blocks of a group stores 16 consecutive features (32 B of bf16) per token
// instead of 4 separate 8-byte pieces.  Pure relabelling: the packing kernel and the epilogues agree.
constexpr int kPermBlocks = 4;
__host__ __device__ inline int packed_row_feature(int rb, int r)
{
    return (rb / kPermBlocks) * (16 * kPermBlocks) + (r >> 2) * (4 * kPermBlocks) + (rb % kPermBlocks) * 4 + (r & 3);
}
// Element offset of (slot, feature) in the intermediate activation A = SiLU(G)*U.  A is private to the
// library, so the up-projection writes it in the order the down-projection consumes it: blocks of 16
// slots x 32 features stored as the 64-lane register image of one MFMA token operand (lane =
// 16*(feature/8 % 4) + slot % 16, 8 features per lane), k-steps of a slot block contiguous.  A k-step of
// 16 slots is then one contiguous 1 KB line, like a weight fragment.  kst = I / 32.
__host__ __device__ inline uint32_t act_elem(uint32_t slot, uint32_t feature, uint32_t kst)
{
    return ((slot >> 4) * kst + (feature >> 5)) * (uint32_t)kFragElems + ((((feature >> 3) & 3u) << 4) + (slot & 15u)) * 8u +
           (feature & 7u);
}
struct PackedLayout {
    size_t w1_expert_elems;  // gate then up: 2 * I * H
    size_t up_offset_elems;  // I * H
    size_t w2_expert_elems;  // H * I
    size_t w2_base_elems;    // E * 2 * I * H
    size_t total_bytes;
};
PackedLayout packed_layout(const ramp_shape &s);

// ---- projections ----
struct GemmArgs {
    const uint16_t *act;        // stage 1: X [T,H]; stage 2: A [cap,I]
    const uint16_t *wpacked;    // base of this stage's packed weights
    size_t expert_stride;       // elements between experts
    size_t up_offset;           // stage 1: offset of the up rows inside an expert
    const int32_t *sorted;      // [cap]
    const int32_t *tile_expert; // [cap/bm]
    const int32_t *tile_rows;   // [cap/bm] real rows per tile
    unsigned long long topk_magic;  // ceil(2^40 / k): pair / k == (pair * topk_magic) >> 40 for pair < 2^30
    const int32_t *meta;        // [4]
    const float *topk_w;        // stage 2: [P]
    const float *slot_w;        // stage 2, ping-pong kernels: router weight of every sorted slot that holds a pair [cap]
    uint16_t *a_out;            // stage 1: A [cap,I]
    float *y_out;               // stage 2: Y [P,H] (fp32, or bf16 in the same buffer when y_bf16 != 0)
    int y_bf16;                 // large batches keep the per-pair rows in bf16 to halve their HBM traffic
    int K;                      // reduction length (H or I)
    int F;                      // output features (I or H)
    int P;                      // pairs = T*k (the sentinel)
    int topk;                   // k
    int n_tiles;                // feature tiles of this stage
    int m_tiles_cap;            // launched M-tiles (upper bound)
    int group_m_req;            // GROUP_M of the configuration (mode bits 12-15): M-tiles per XCD block, 0 = automatic
    int group_m, group_n;       // M-tiles x N-tiles per XCD block of the workgroup->tile map (set by the launcher)
    int blocks_n;               // n_tiles / group_n
    // their divisors as multipliers (div_magic, set by the launcher): group_m * group_n, group_m, n_tiles, blocks_n
    unsigned long long block_magic, gm_magic, n_magic, bn_magic;
    int a_row_major;            // stage 1: A is written row-major [slot, I] instead of fragment-major (FP8 path)
    const int32_t *pred;        // device-side predicate: the launch does nothing unless *pred == pred_value (NULL: always runs)
    int pred_value;
};
// True when a predicated launch is not the one selected on the device.
__device__ __forceinline__ bool launch_deselected(const int32_t *pred, int pred_value)
{
    return pred != nullptr && *pred != pred_value;
}

// ramp_config.mode: bits 0-7 = WM-1 (token split of the wavefront grid), then the kernel family
constexpr int kModeStream = 0x100;    // weight-streaming kernel (moe_stream.h); bits 0-7 = WK instead
constexpr int kModePipe = 0x200;      // LDS-staged kernel with the register-pipelined main loop (moe_gemm.h)
constexpr int kModePingPong = 0x400;  // persistent ping-pong kernel (moe_pingpong.h)
// GROUP_M (Sec. 4.1, Eq. 4), XCD-aware: bits 12-15 = v > 0 makes every XCD take blocks of 2^v M-tiles x (32 >> v)
// N-tiles, so that the M-tiles of a block share the weight slices of its few N-tiles in that XCD's L2; 0 = a block
// spans all N-tiles (the token rows of its M-tiles stay in L2 instead).
constexpr int kModeDecode = 0x2000;   // with kModeStream: calls of at most 64 pairs run the two-launch form (moe_decode.h)
constexpr int kModeFp8 = 0x10000;     // W8A8 FP8 family (fp8.hip), listed by ramp_fp8_get_config
// in place of kModePingPong: a 256-wide persistent tile for H = 256 * n + 128.  The down-projection's last N-tile holds 128
// features; its other half re-reads the weights of the first (loads that hit, products that are not stored).  H = 1152, I = 896, E = 48, k = 6, against
// the best tile of 128 features (bf16 256 x 128, FP8 32 x 128): bf16 T = 1024 111 -> 103 us, 4096 230 -> 199, 8192 381 -> 330;
// FP8 T = 256 72 -> 60 us, 1024 140 -> 83, 8192 711 -> 259.  Below some 64 rows per expert the narrow tiles stay the better ones.
constexpr int kModeHalfTile = 0x20000;
constexpr bool mode_persistent(int mode) { return (mode & (kModePingPong | kModeHalfTile)) != 0; }
constexpr int kModeGroupShift = 12;
constexpr int kModeGroupMask = 0xF << kModeGroupShift;
inline int group_m_of_mode(int mode) { const int v = (mode & kModeGroupMask) >> kModeGroupShift; return v ? (1 << v) : 0; }

// The stream candidates of a device-selected call that share launches (stream_selected.hip): what differs between their arguments (byte
// offsets), and the number of a candidate's tile, -1 for one with launches of its own.
struct StreamChoice {
    int32_t shape, bn, m_tiles_cap;
    size_t sorted, tile_expert, a_buf;
};
struct StreamChoices {
    StreamChoice c[kMaxCandidates];
};
constexpr int kStreamGroups = 2;  // tiles of one group can share a launch
int stream_selected_shape(const ramp_config &cfg);  // -1: a tile of no group
int stream_selected_group(int shape);               // -1 of -1
// Wavefronts of a block of the group's kernel; a tile of fewer shares it with others
constexpr int stream_selected_waves(int group) { return group == 0 ? 8 : 4; }
// args: those of the candidates, without what `choices` holds; features: 2 * I, or H; blocks: the most that a candidate of the group needs
int launch_stream_selected(int group, int stage, const GemmArgs &args, char *base, int features, int n_cand,
                           const StreamChoices &choices, unsigned blocks, hipStream_t stream);

struct DecodeArgs;
struct DecodeDownArgs;
struct KernelInfo {
    ramp_config cfg;
    int wm, wn;                 // wavefront grid inside the workgroup (tokens x features)
    int lds_bytes;
    int acc_regs;               // fp32 accumulators per lane (stage 1, the larger one)
    void (*launch)(int stage, const GemmArgs &, hipStream_t);
    // decode-sized calls (kModeDecode): align + up-projection in one launch; NULL for every other configuration
    void (*launch_decode_up)(const GemmArgs &, const DecodeArgs &, hipStream_t);
    const void *kernel_fn[2];   // the two projection kernels (stage 1, stage 2), for occupancy queries
    int block_threads;
    const char *family;         // kernel template name and the template arguments of the stage-1 instantiation:
    int targs[8];               // the key into the compiler's per-kernel resource table (kernel_resources.inc)
    int n_targs;
};

// What the compiler reported for one kernel instantiation when the library was built (registers, LDS,
// wavefronts per SIMD that fit); generated by the build into kernel_resources.inc.
struct KernelResources {
    const char *family;
    int n_targs;
    int targs[8];
    int vgprs, agprs, lds_bytes, waves_per_simd;
};
const KernelResources *find_resources(const char *family, const int *targs, int n_targs);
int num_kernels();
const KernelInfo &kernel_info(int i);
const KernelInfo *find_kernel(const ramp_config &cfg);
bool config_valid_for_shape(const KernelInfo &ki, const ramp_shape &s);
// bn divides the features of both projections, or leaves half a tile of the down-projection's for a configuration made for that
inline bool bn_tiles_shape(const ramp_config &c, const ramp_shape &s)
{
    return (2 * s.I) % c.bn == 0 && s.H % c.bn == ((c.mode & kModeHalfTile) ? c.bn / 2 : 0);
}
bool config_in_pool(const KernelInfo &ki, const ramp_shape &s);
int occupancy_estimate(const ramp_config &cfg, const char *family, const int *targs, int n_targs);
int runtime_occupancy(const void *const kernel_fn[2], int block_threads, int *wg_per_cu);

// sel != NULL: the launch leaves `out` untouched unless 0 <= *sel < n_cand (device-selected layer) and bit *sel of
// skip_mask is clear (a candidate whose own launches write `out`).
// Two-launch form for decode-sized calls (moe_decode.h, instantiated in stream_group2.hip)
struct DecodeArgs {
    const int32_t *ids;      // [T*k]
    int E, bm, cap;          // bm is the kernels' template argument; without it here their argument loads are placed so that both
                             // decode forms run 0.5 to 0.9 % slower (FP8, OLMoE-shaped T = 8: 57.0 -> 57.4 us)
    int32_t *sorted, *tile_expert, *tile_rows, *counts, *meta;  // align result, written by workgroup 0
};
struct DecodeDownArgs {
    const uint16_t *act;       // A [P, I] bf16, row-major, one row per pair
    const uint16_t *wpacked;   // packed down-projection weights
    size_t expert_stride;      // elements between experts
    const int32_t *ids;        // [T, k]
    const float *topk_w;       // [T, k]
    uint16_t *out;             // [T, H] bf16
    int T, k, E, H, I;
    const int32_t *pred;
    int pred_value;
};

// Router weights of one token's pairs for the final sum of the decode down-projections.  Thread j < k loads pair j's when the
// kernel starts and stores them in LDS in front of its last barrier: read by the sum itself, id and weight of one pair after the
// other, they were 2 * k dependent loads behind it.
struct PairWeights {
    float w[16];
    int live[16];  // the pair's expert exists
};
struct PairWeight {
    int id;
    float w;
};
__device__ __forceinline__ PairWeight load_pair_weight(const DecodeDownArgs &d, int t)
{
    PairWeight p = {-1, 0.f};
    if ((int)threadIdx.x < d.k) p = PairWeight{d.ids[t * d.k + threadIdx.x], d.topk_w[t * d.k + threadIdx.x]};
    return p;
}
__device__ __forceinline__ void store_pair_weight(PairWeights &all, const DecodeDownArgs &d, PairWeight p)
{
    if (threadIdx.x >= 16) return;  // past the token's k pairs the id is -1
    all.w[threadIdx.x] = p.w;
    all.live[threadIdx.x] = p.id >= 0 && p.id < d.E;
}
// Sum over the 16 wavefronts' partial sums: the WK (a power of two) of one pair in order, weighted, then over the pairs in order.
// (wavefronts past the k-th pair's leave partial sums that no live pair owns)
template <class Partial>
__device__ __forceinline__ float sum_of_pairs(int WK, const PairWeights &p, Partial partial)
{
    float part[16];
#pragma unroll
    for (int w = 0; w < 16; ++w) part[w] = partial(w);
    const int shift = 31 - __clz(WK);
    float y = 0.f, s = 0.f;
#pragma unroll
    for (int w = 0; w < 16; ++w) {
        s = (w & (WK - 1)) ? s + part[w] : part[w];
        if ((w & (WK - 1)) == WK - 1 && p.live[w >> shift]) y += p.w[w >> shift] * s;
    }
    return y;
}
constexpr int kDecodeMaxPairs = 64;
// The two-launch form takes calls of at most 64 pairs whose tokens have at most 16: one wavefront or more of its down-projection
// to a pair.  Where k does not divide 16 some of the 16 wavefronts are idle, and every pair reads its expert's weights for itself where the
// general form reads them once per expert: it is the faster one while the down-projection's H / 16 * T workgroups fit on the units at
// once, and loses past that (both builds, all decode configurations, twelve layers of H = 1024 ... 7168 and k = 3 ... 15, with 16 to 64
// experts and with every token at all k of them): T * H <= 4096 0.57 to 0.99 of the general form's time (H = 1152, I = 896, k = 6, one
// token bf16 18.9 -> 14.1 us, FP8 17.6 -> 13.8), above it up to 1.7 of it (k = 6, T = 10 27.6 -> 39.1; H = 4096, E = 16, k = 5,
// T = 12 1.5 of it).
inline bool decode_in_two_launches(const ramp_shape &s)
{
    return s.k <= 16 && (long long)s.T * s.k <= kDecodeMaxPairs && (16 % s.k == 0 || (long long)s.T * s.H <= 16 * kNumCU);
}
// Wavefronts that share the reduction of one pair: the largest power of two that k pairs leave of 16.
__device__ __forceinline__ int decode_pair_waves(int k)
{
    return k > 8 ? 1 : k > 4 ? 2 : k > 2 ? 4 : k > 1 ? 8 : 16;
}
void launch_decode_down_any(const DecodeDownArgs &d, hipStream_t stream);

// shape limits shared by the fused entry points (fused.hip)
bool moe_shape_ok(const ramp_shape &s);
bool moe_pair_rows_bf16(const ramp_shape &s);      // per-pair rows kept in bf16 (large batches) instead of fp32
unsigned long long moe_topk_magic(int k);

int launch_combine(const float *Y, int y_bf16, const int32_t *ids, int T, int k, int E, int H, uint16_t *out,
                   hipStream_t stream, const int32_t *sel = nullptr, int n_cand = 0, unsigned skip_mask = 0);

}  // namespace ramp
