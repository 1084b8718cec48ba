// Which tiles a workgroup of a persistent kernel takes, and in which order.  Plain integer code without anything of the device
// in it, so that it is enumerated on the host too.
//
// Workgroup -> tile map of a launch (tile_map): every XCD takes blocks of group_m M-tiles x group_n N-tiles, the 8 XCDs 8 * group_m
// M-tiles per round.  The workgroups of the persistent kernels walk it: workgroup c of an XCD takes slots c, c + 32, ...  With the
// static map a workgroup gets the same position of every block and an XCD every eighth M-tile; where the experts have a full
// M-tile followed by a ragged one (two tiles per expert: block positions and XCDs alternate full, ragged) half of the
// workgroups, or half of the XCDs, then only ever get ragged tiles, finish early and run ahead of the siblings they
// share weights with.  So the position inside the block moves on by one per block, and the XCD -> M-tile assignment
// inside a round of 8 * group_m M-tiles by three per round: an XCD then steps through the M-tiles by 11 or 3 instead
// of 8, which does not stay in phase with 2, 3, 4, 8 or 9 tiles per expert (a shift of one, steps of 9, does with 3
// and 9: measured 7 % slower on such a layer).  The tiles an XCD works on at a time stay the same, who gets which
// changes.  Same-box A/B of the layer: DeepSeek-V3 T = 2048 at 52 active experts (two tiles each) 2010 -> 1766 us,
// Mixtral T = 8192 4980 -> 4880 us, T = 1024 1035 -> 1013 us, the other large points within +-1 %.
//
// The walk knows the real number of M-tiles (align's, on the device) and shares out three ways:
// - What whole rounds of 8 * group_m M-tiles leave is dealt to all XCDs evenly, M-tile by M-tile.  With the rounds of the map alone
//   13 M-tiles over rounds of 8 gave five XCDs twice the tiles of the other three (Mixtral-shaped, T = 1024 Zipf: up-projection
//   625 -> 568 us with the next point; T = 512 Zipf 485 -> 394).
// - Where M-tiles share an expert a round is split so that an XCD's 32 workgroups take up to 4 M-tiles x 8 N-tiles at a time, not
//   1 x 32 or 2 x 16: fewer bytes cross the fabric (FETCH_SIZE of the FP8 up-projection at Mixtral's T = 8192 8.3 -> 5.3 GB), and
//   the power that saves is clock for kernels held by it: 1691 -> 1575 us, bf16 2903 -> 2780.  With one M-tile per expert nothing is
//   shared and the default split is the better one (2016 against 2079 to 2108 us in the DeepSeek-V3-shaped down-projection at T = 8192).
//   Blocks of two M-tiles gain less than blocks of one, 128-row tiles more than 256-row ones; one loses: 128-row tiles and a reduction as
//   long as Mixtral's down-projection (K = 14336, T = 8192, default against split 1857 -> 1979 us), whose layer is the slower one all the same
//   with that launch alone left unsplit (5527 -> 5578, 4024 -> 4054 us at T = 6000: the up-projection beside it runs at a lower clock then).
//   The line lies at the share of M-tiles that have the expert of the one before: half of them, and for the split by four three quarters
//   (layers of 4 and 2 M-tiles an expert).  Default against split, us: none 273 -> 278, 598 -> 618, a third 1049 -> 1062 and 574 -> 547,
//   half 528 -> 530 and 273 -> 269, three quarters 3273 -> 3086 and 1727 -> 1645.
// - Of fewer than three turns of an XCD's workgroups, the tiles that fill no whole turn are cut in two or four column parts where
//   that many workgroups would idle, and come first: 36 M-tiles x 8 N-tiles on 256 units are one turn and 32 tiles (Qwen3-shaped,
//   T = 509: down-projection 41 -> 38 us; Mixtral-shaped, T = 200 207 -> 181; H = 1152, T = 777, up 50 -> 46).  A part takes as
//   many slices as a tile, with fewer weights, so behind three whole turns it gains under 1 %, and out of step with the tiles that
//   share its weights it can cost as much.
#pragma once

#ifdef __HIP__
#define RAMP_WALK __device__ __forceinline__
#define RAMP_WALK_UNIFORM(x) __builtin_amdgcn_readfirstlane(x)
#else
#define RAMP_WALK inline
#define RAMP_WALK_UNIFORM(x) (x)
#endif

namespace ramp {

// x / d as (x * ceil(2^40 / d)) >> 40: exact for x * d < 2^40, x < 2^24.  Of wave-uniform values it stays in scalar registers.
constexpr unsigned long long div_magic(int d) { return ((1ull << 40) + (unsigned)d - 1) / (unsigned)d; }
RAMP_WALK int div_by(int x, unsigned long long magic) { return (int)(((unsigned long long)(unsigned)x * magic) >> 40); }

// Block shape of the XCD-aware workgroup -> tile map of one launch: every XCD takes blocks of group_m M-tiles x
// group_n N-tiles, the 8 XCDs 8 * group_m M-tiles per hand-out round.  group_m_req > 0: the GROUP_M mode of the
// configuration (group_n = the largest divisor of n_tiles up to 32 / group_m).  Default: a block spans all N-tiles, so
// the token rows of its few M-tiles (group_m * bm * K * 2 bytes) stay in the 4 MB L2 across the walk over N while the
// 8 XCDs work on neighbouring M-tiles, i.e. mostly the same expert, and share its weights through the memory-side cache.
inline void xcd_block_shape(int n_tiles, int group_m_req, int *group_m, int *group_n)
{
    if (group_m_req > 0) {
        int gn = 32 / group_m_req;
        if (gn < 1) gn = 1;
        if (gn > n_tiles) gn = n_tiles;
        while (n_tiles % gn) --gn;
        *group_m = group_m_req;
        *group_n = gn;
    } else {
        int gm = 32 / n_tiles;
        if (gm < 1) gm = 1;
        if (gm > 8) gm = 8;
        *group_m = gm;
        *group_n = n_tiles;
    }
}

// Map: what holds n_tiles, group_m_req and the fields that this fills in from them (GemmArgs).
template <class Map>
inline void tile_map(Map &a)
{
    xcd_block_shape(a.n_tiles, a.group_m_req, &a.group_m, &a.group_n);
    a.blocks_n = a.n_tiles / a.group_n;
    a.block_magic = div_magic(a.group_m * a.group_n);
    a.gm_magic = div_magic(a.group_m);
    a.n_magic = div_magic(a.n_tiles);
    a.bn_magic = div_magic(a.blocks_n);
}

struct TileWalk {
    int xcd;
    int full, total;   // slots of this XCD in the whole rounds, and in all
    int m_full, tail0; // M-tiles of the whole rounds; first tile of this XCD's share of the rest
    int xm_log;        // log2 of xm: the round is split between xm x 8/xm XCDs
    int wg, wgs;       // this workgroup of its XCD, and how many there are
    int whole, cut;    // slots that the workgroups take one each, in whole turns; the others are cut in 1 << cut parts
    int part;          // this workgroup's part of a cut tile
};
// The sharing of experts is told from four runs of eight M-tiles, spread over the table: the first eight alone say nothing of a layer whose
// first experts are rare and others heavy (eight experts of one M-tile in front of eight of eight, H = 4096, I = 14336, T = 8192: layer of
// 128-row FP8 tiles 3310 -> 2969 us, 256-row 2514 -> 2485, bf16 6589 -> 5929 and 4981 -> 4830; in the opposite order as before).  Runs, not single pairs at
// a stride, which would be in step with two or four tiles an expert; scalar loads: with a wavefront's vector loads over 256 pairs the
// kernels spilled.  same counts those of their 28 pairs of neighbours that have one expert.
constexpr int kShareRuns = 4;
RAMP_WALK int first_of_run(int m_tiles, int c) { return (m_tiles - 8) * c / (kShareRuns - 1); }
RAMP_WALK bool walk_looks_at_experts(int group_m, int group_m_req, int m_tiles)
{
    return m_tiles >= 8 * group_m && group_m_req == 0 && group_m <= 2;
}
template <class Map>
RAMP_WALK TileWalk tile_walk(const Map &a, int xcd, int wg, int wgs, int m_tiles, int same, int max_parts)
{
    TileWalk w;
    const int per_round = 8 * a.group_m;
    const int rounds = div_by(m_tiles >> 3, a.gm_magic), rest = (m_tiles - rounds * per_round) * a.n_tiles;
    w.xcd = xcd;
    w.m_full = rounds * per_round;
    w.full = rounds * a.group_m * a.n_tiles;
    w.tail0 = (xcd * rest) >> 3;
    w.total = w.full + (((xcd + 1) * rest) >> 3) - w.tail0;
    w.xm_log = 3;
    if (walk_looks_at_experts(a.group_m, a.group_m_req, m_tiles)) {
        // (12: what the runs see of two tiles an expert at the worst; four tiles an expert show 20 to 24, three 16 to 20)
        if (a.group_m == 1 && same >= 19 && a.n_tiles % 4 == 0) w.xm_log = 1;
        else if (same >= 12 && a.n_tiles % 2 == 0) w.xm_log = 2;
    }
    w.wg = wg;
    w.wgs = wgs;
    const int left = RAMP_WALK_UNIFORM(w.total % w.wgs);
    w.cut = 0;
    if (left > 0 && w.total < 3 * w.wgs)
        while ((2 << w.cut) <= max_parts && (left * 2 << w.cut) <= w.wgs) ++w.cut;
    w.whole = w.cut > 0 ? w.total - left : w.total;
    w.part = w.wg & ((1 << w.cut) - 1);
    return w;
}
// What a workgroup takes: position -1 is its part of a cut tile, which comes first, s >= 0 the tile of slot s; a position of
// w.whole or more is past its last tile.
RAMP_WALK int walk_first(const TileWalk &w) { return w.cut > 0 && w.wg < (w.total - w.whole) << w.cut ? -1 : w.wg; }
RAMP_WALK int walk_next(const TileWalk &w, int pos) { return pos < 0 ? w.wg : pos + w.wgs; }
RAMP_WALK int walk_slot(const TileWalk &w, int pos) { return pos < 0 ? w.whole + (w.wg >> w.cut) : pos; }
// Tile of slot s < total.
template <class Map>
RAMP_WALK void tile_of_slot(const Map &a, const TileWalk &w, int s, int &n_tile, int &m_tile)
{
    if (s >= w.full) {
        const int f = w.tail0 + s - w.full;
        const int m = div_by(f, a.n_magic);
        m_tile = w.m_full + m;
        n_tile = f - m * a.n_tiles;
        return;
    }
    // an XCD's block: gm M-tiles x gn N-tiles
    const int xn_log = 3 - w.xm_log, gm = a.group_m << xn_log, gn = a.group_n >> xn_log;
    const int per_block = a.group_m * a.group_n;
    const int sb = div_by(s, a.block_magic);
    const int turn = s - sb * per_block + sb;
    const int v = turn - div_by(turn, a.block_magic) * per_block;
    const int dn = div_by(v >> xn_log, a.gm_magic), dm = v - dn * gm;
    const int mb = div_by(sb, a.bn_magic), nbi = sb - mb * a.blocks_n;
    const int x = (w.xcd + 3 * mb) & 7;
    const int xn = x >> w.xm_log, xm = x & ((1 << w.xm_log) - 1);
    n_tile = ((nbi << xn_log) + xn) * gn + dn;
    m_tile = ((mb << w.xm_log) + xm) * gm + dm;
}

}  // namespace ramp
