// Launch planning of the tiled GEMM (host) and the block -> tile map shared by
// the kernels and the host (host and device): which tile shape and K split a
// launch uses, its grid and split arguments, and which output tile and K range
// each block computes.  Kept apart from the kernels so that a host-only build
// (the CPU test of this map) can use the very same functions.
#pragma once

#include <algorithm>
#include <cmath>

#include "kernels.h"

namespace pb {

namespace {

#ifndef PB_GEMM_SPLIT_TARGET
#define PB_GEMM_SPLIT_TARGET 256  // blocks a split launch aims for
#endif
#ifndef PB_GEMM_MIN_KT
#define PB_GEMM_MIN_KT 8  // fewest K tiles a split-K block gets
#endif
#ifndef PB_GEMM_RAGGED
#define PB_GEMM_RAGGED 1  // split only the tail tiles of a ragged last round
#endif

constexpr int BK = 64;      // K tile
constexpr int GROUP_M = 8;  // tile-rows per group of the tile walk

struct SplitArgs {
    int splits;     // number of K splits (1 = none)
    int kt_split;   // K tiles per split (the LoRA tiles go to the last split)
    float* ws;      // [splits][M][N] fp32 partials when splits > 1
    // ragged-round split (full_tiles > 0): tiles [0, full_tiles) run whole
    // through the epilogue, only the tail tiles [full_tiles, full_tiles +
    // tail_tiles) are split `splits` ways, their partials packed as
    // [split][tail tile][BM][BN]; full_tiles and tail_tiles * splits are
    // multiples of 8
    int full_tiles, tail_tiles;
};

// Which output tile and K range a block works on: the hardware deals
// consecutive blocks round-robin to the 8 XCDs, so the block id is remapped to
// give each XCD a contiguous run; runs are split-major, and tiles are walked in
// groups of GROUP_M tile-rows so that blocks sharing an XCD's L2 share rows of
// X and of W.  Split s takes base K tiles [s kt, (s+1) kt), the last split
// also the LoRA K tiles of its output group (if that group is active).
struct TileJob {
    int m0, n0, split, nk1, t_begin, nk;
    bool partial;    // writes an fp32 partial tile (split along K) instead of the epilogue
    float* pbase;    // ... at pbase + (m - om) * ldp + (n - on)
    int ldp, om, on;
    const void* X2;  // LoRA activations of the tile's output group
};

// Output tile index -> its corner: tiles are walked in groups of GROUP_M
// tile-rows (blocks that share an XCD's L2 share rows of X and of W).
template <int BM, int BN>
__host__ __device__ __forceinline__ void tile_corner(const GemmParams& p, int tile, int& m0, int& n0) {
    const int tiles_m = (p.M + BM - 1) / BM;
    const int tiles_n = (p.N + BN - 1) / BN;
    const int per_group = GROUP_M * tiles_n;
    const int first_m = (tile / per_group) * GROUP_M;
    const int gsize = tiles_m - first_m < GROUP_M ? tiles_m - first_m : GROUP_M;
    m0 = (first_m + (tile % per_group) % gsize) * BM;
    n0 = ((tile % per_group) / gsize) * BN;
}

// (host-callable: block bid of a grid of nblk blocks)
template <int BM, int BN>
__host__ __device__ __forceinline__ TileJob tile_job(const GemmParams& p, const SplitArgs& sa, int bid, int nblk) {
    const int tiles_m = (p.M + BM - 1) / BM;
    const int tiles_n = (p.N + BN - 1) / BN;
    const int tiles = tiles_m * tiles_n;
    int tile, split;
    bool partial;
    if (sa.full_tiles > 0) {
        // the whole tiles first, then the split tail tiles, each part dealt
        // XCD-contiguously on its own so that the tail round spreads over all
        // eight XCDs
        if (bid < sa.full_tiles) {
            tile = (sa.full_tiles & 7) ? bid : (bid & 7) * (sa.full_tiles >> 3) + (bid >> 3);
            split = 0;
            partial = false;
        } else {
            const int r = bid - sa.full_tiles, nt = nblk - sa.full_tiles;
            const int rr = (nt & 7) ? r : (r & 7) * (nt >> 3) + (r >> 3);
            tile = sa.full_tiles + rr % sa.tail_tiles;
            split = rr / sa.tail_tiles;
            partial = true;
        }
    } else {
        if ((nblk & 7) == 0) bid = (bid & 7) * (nblk >> 3) + (bid >> 3);
        tile = bid % tiles;
        split = bid / tiles;
        partial = sa.splits > 1;
    }
    TileJob j;
    tile_corner<BM, BN>(p, tile, j.m0, j.n0);
    j.split = split;
    j.partial = partial;
    if (sa.full_tiles > 0) {
        j.pbase = sa.ws + ((int64_t)split * sa.tail_tiles + (tile - sa.full_tiles)) * (BM * BN);
        j.ldp = BN;
        j.om = j.m0;
        j.on = j.n0;
    } else {
        j.pbase = sa.ws + (int64_t)split * p.M * p.N;
        j.ldp = p.N;
        j.om = j.on = 0;
    }
    j.nk1 = p.K1 / BK;
    int nk2 = 0;
    j.X2 = p.X2;
    if (p.K2 > 0) {
        const int g = j.n0 / p.group;
        if ((p.k2_mask >> g) & 1u) {
            nk2 = p.K2 / BK;
            j.X2 = (const char*)p.X2 + (int64_t)g * p.x2_group_stride * 2;
        }
    }
    if (!partial) {
        j.t_begin = 0;
        j.nk = j.nk1 + nk2;
    } else {
        j.t_begin = split * sa.kt_split;
        const int t_end = (split == sa.splits - 1) ? j.nk1 + nk2
                          : (j.nk1 < j.t_begin + sa.kt_split ? j.nk1 : j.t_begin + sa.kt_split);
        j.nk = t_end - j.t_begin;
    }
    return j;
}

// K split into `splits` ranges: splits 0..S-2 take kt_split base tiles each,
// the last one the rest (and the LoRA tiles); S = ceil(nk1 / kt_split) leaves
// no split empty.
SplitArgs make_split(const GemmParams& p, const GemmWorkspace& wsp, int splits) {
    const int nk1 = p.K1 / BK;
    SplitArgs sa;
    sa.kt_split = (nk1 + splits - 1) / splits;
    sa.splits = (nk1 + sa.kt_split - 1) / sa.kt_split;
    sa.ws = (float*)wsp.ws;
    sa.full_tiles = sa.tail_tiles = 0;
    return sa;
}

// Grid and split arguments of a tile launch (host side): a uniform K split
// into `splits` ranges, or with ragged_tail > 0 the whole tiles first and the
// last `ragged_tail` tiles split (falling back to whole tiles only when the
// split does not come out as planned).
struct TileGeometry {
    SplitArgs sa;
    int grid;
};

template <int BM, int BN>
TileGeometry tile_geometry(const GemmParams& p, const GemmWorkspace& wsp, int splits, int ragged_tail) {
    const int tiles = ((p.M + BM - 1) / BM) * ((p.N + BN - 1) / BN);
    TileGeometry g;
    g.sa = make_split(p, wsp, splits);
    if (ragged_tail > 0) {
        if (g.sa.splits >= 2 && (tiles - ragged_tail) % 8 == 0 && (ragged_tail * g.sa.splits) % 8 == 0) {
            g.sa.full_tiles = tiles - ragged_tail;
            g.sa.tail_tiles = ragged_tail;
            g.grid = g.sa.full_tiles + ragged_tail * g.sa.splits;
            return g;
        }
        g.sa = make_split(p, wsp, 1);
    }
    g.grid = tiles * g.sa.splits;
    return g;
}

// Tile shape and K split of a launch, from a cost model: a block's time is
// its MFMA work at the rate of one CU with that tile (256 x 256 4.5 TFLOP/s, 128 x
// 128 2.6: measured with a plain ring in both; the 256 x 256 kernel now reaches
// 5.4, but another rate would move K ranges and with them the bits of results), blocks run in rounds of 256 (one per CU), and
// a split adds its fp32 partials (written, then read by the reduce) at
// ~4 TB/s.  Splits keep >= PB_GEMM_MIN_KT K tiles each and fit the workspace.
struct TilePlan {
    int tile;    // 256, 128 or 64
    int splits;
    int ragged_tail;  // > 0: whole tiles, then this many tail tiles split `splits` ways
};

TilePlan plan_tiles(const GemmParams& p, const GemmWorkspace& wsp) {
    const int nk1 = p.K1 / BK;
    const double out_bytes = (double)p.M * p.N * 4;
    // the LayerNorm that follows o or fc2 rides on a uniform split's reduce;
    // otherwise it is a pass of its own over the fp32 rows (read) and dt rows (write)
    const double ln_pass = p.ln_out ? (double)p.M * p.N * 6 / 4e12 : 0.0;
    TilePlan best{64, 1, 0};
    double best_t = 1e30;
    auto consider = [&](int t, double rate) {
        if (p.N % t) return;
        const long tiles = (long)((p.M + t - 1) / t) * (p.N / t);
        const double t_tile = 2.0 * t * t * p.K1 / rate;
        for (int s = 1; s <= 8; ++s) {
            if (s > 1 && (nk1 / s < PB_GEMM_MIN_KT || !wsp.ws || out_bytes * s > (double)wsp.bytes)) break;
            const long rounds = (tiles * s + 255) / 256;
            const double tt = rounds * (t_tile / s) + (s > 1 ? 2.0 * out_bytes * s / 4e12 : ln_pass);
            if (tt < best_t * 0.98) {  // prefer the simpler plan on near ties
                best_t = tt;
                best = {t, s, 0};
            }
        }
        // ragged last round: whole rounds unsplit, the tail tiles split to fill one round
        const long tail = tiles % 256, full = tiles - tail;
        if (PB_GEMM_RAGGED && full > 0 && tail > 0 && wsp.ws) {
            const int s = (int)std::min<long>(8, 256 / tail);
            const double pbytes = (double)tail * t * t * 4 * s;
            if (s >= 2 && nk1 / s >= PB_GEMM_MIN_KT && full % 8 == 0 && (tail * s) % 8 == 0 &&
                pbytes <= (double)wsp.bytes) {
                const double tt = (full / 256) * t_tile + t_tile / s + 2.0 * pbytes / 4e12 + ln_pass;
                if (tt < best_t * 0.98) {
                    best_t = tt;
                    best = {t, s, (int)tail};
                }
            }
        }
    };
    consider(256, 4.5e12);
    consider(128, 2.6e12);
    if (best_t >= 1e30) {  // N not a multiple of 128: 64 x 64 tiles, split when few
        const long tiles = (long)((p.M + 63) / 64) * (p.N / 64);
        int s = 1;
        if (tiles < 256 && wsp.ws) {
            s = std::min<long>((PB_GEMM_SPLIT_TARGET + tiles - 1) / tiles, std::max(1, nk1 / PB_GEMM_MIN_KT));
            while (s > 1 && out_bytes * s > (double)wsp.bytes) --s;
        }
        best = {64, std::max(1, s), 0};
    }
    return best;
}

// Launches between the GEMV and the large tiles: the streaming kernel (wide
// LDS rows, `bm` tokens x `bn` features per block) up to STREAM_MAX_ROWS rows,
// and tile shapes beside the square ones of plan_tiles.
constexpr int STREAM_MAX_ROWS = 512;

enum WideKind { WIDE_NONE = 0, WIDE_STREAM, WIDE_RING, WIDE_PINGPONG };

struct WidePlan {
    int kind;    // WideKind; WIDE_NONE: plan_tiles' choice stands
    int bm, bn;  // stream: 32 x 64, 32 x 32, 64 x 64, 128 x 64; ring: 192 x 128, 256 x 256; ping-pong: 128 or 192 x 256
    int bk;      // stream: K elements per ring stage (128 or 256)
    int splits;  // K ranges launched
    int kt;      // stream: K tiles (of 64) per range of plan_tiles' split (the sum's order), or all of them
};

// Block bid of a stream launch -> its tile corner, K split and stages of that
// split (split s takes stages [s kst, (s + 1) kst), the last one the rest).
// Token tiles of one feature block are neighbours within an XCD's run (they
// share its weight rows).
struct StreamJob {
    int m0, n0, split, t0, n;
};

template <int BM, int BN, int BKE>
__host__ __device__ __forceinline__ StreamJob stream_job(const GemmParams& p, int kst, int bid, int nblk) {
    const int nbm = (p.M + BM - 1) / BM, tiles = p.N / BN * nbm;
    if (nbm > 1 && (nblk & 7) == 0) bid = (bid & 7) * (nblk >> 3) + (bid >> 3);
    StreamJob j;
    j.split = bid / tiles;
    j.m0 = bid % tiles % nbm * BM;
    j.n0 = bid % tiles / nbm * BN;
    const int nk = p.K1 / BKE;
    j.t0 = j.split * kst;
    j.n = nk - j.t0 < kst ? nk - j.t0 : kst;
    return j;
}

// What a K split or its absence costs beside the product: partials written and
// read (mostly from the last-level cache: ~8 TB/s) and a reduce launch of its
// own (`launch`, as fitted in recorded graphs) unless the LayerNorm that follows is
// that reduce; without a split that LayerNorm is a pass.
inline double split_cost(const GemmParams& p, int splits, double launch) {
    const double out = (double)p.M * p.N * 4;
    if (splits > 1) return 2.0 * out * splits / 8e12 + (p.ln_out ? 0.0 : launch);
    return p.ln_out ? out * 1.5 / 4e12 + 3e-6 : 0.0;
}

// Eight K ranges a multiple of 4 KB apart read the same HBM channels (N 4096 in
// 128 x 128 tiles, one round of 256 blocks: K 16384 in eight ranges 49 us for 50
// rows and 53 for 100, in six 38 and 42; K 12288, 3 KB apart, in eight 28 and 30).
inline bool same_channels(const GemmParams& p, int splits) { return splits == 8 && p.K1 / 8 * 2 % 4096 == 0; }

// Times of a tile and of a stream launch, fitted together to 5600 launches (the
// projections of d_model 768 .. 9216, 9 .. 2000 rows, cold weights; mean error 8%).
//
// Tiles: rounds of 256 blocks (one per CU) at a time per 64-wide K tile, cold
// weights in 128-byte row pieces at 6.8 TB/s, 0.29 of the shorter left over; and
// the launch, the ring's first tiles and the epilogue.
inline double tile_time(const GemmParams& p, int bm, int bn, int splits) {
    const long blocks = (long)((p.M + bm - 1) / bm) * ((p.N + bn - 1) / bn) * splits, rounds = (blocks + 255) / 256;
    double per_kt;
    if (bn == 256) per_kt = bm == 256 ? 1.43e-6 : bm == 192 ? 1.18e-6 : 0.88e-6;
    else if (bm == 192) per_kt = 0.76e-6;
    else if (bm == 128) per_kt = 0.32e-6 + 0.26e-6 * (double)std::min<long>(blocks, 256) / 256;
    else per_kt = 0.30e-6;
    double work = (double)rounds * (double)((p.K1 / BK + splits - 1) / splits) * per_kt;
    if (rounds == 1 && same_channels(p, splits)) work *= 1.43;
    const double hbm = (double)p.N * p.K1 * 2 / 6.8e12;
    return (bn == 256 ? 7.7e-6 : 7.0e-6) + std::max(work, hbm) + 0.29 * std::min(work, hbm) + split_cost(p, splits, 1e-6);
}

// Streams: a CU copies 70 GB/s into LDS whatever the block shape (blocks on one
// CU share it), the chip streams cold weights at 7.1 TB/s (32-row blocks less
// when their rounds leave CUs idle), 0.46 of the shorter left over, and 2.4 us per
// further round of blocks that fill a CU's LDS (all but the 32-row ones).
inline double stream_time(const GemmParams& p, int bm, int bn, int splits) {
    const long blocks = (long)((p.M + bm - 1) / bm) * (p.N / bn) * splits, rounds = (blocks + 255) / 256;
    const double copy = rounds * ((double)p.K1 / splits) * (bm + bn) * 2 / 70e9;
    double hbm = (double)p.N * p.K1 * 2 / 7.1e12;
    if (bm == 32) hbm /= std::pow((double)blocks / (256.0 * rounds), 0.2);
    if (same_channels(p, splits)) hbm *= bm == 32 ? 1.43 : 1.67;
    const double t = std::max(copy, hbm) + 0.46 * std::min(copy, hbm) + (bm > 32 ? (rounds - 1) * 2.4e-6 : 0.0);
    return 4.1e-6 + (bn == 32 ? 1.05 * t : t) + split_cost(p, splits, 2.4e-6);  // bn 32: two waves, fewer copies in flight
}

// K elements per ring stage of 32-row blocks: unsplit with at most a block per
// CU, 512-byte rows (144 KB of ring) measured 6-8% faster than 256-byte rows.
inline int wide_row_stage(const GemmParams& p, int bn, int splits) {
    return bn == 64 && splits == 1 && p.K1 % 256 == 0 && p.N / 64 <= 256 ? 256 : 128;
}

// Split launches planned on the square 256 x 256 tile keep its plain two-stage
// ring, before any other shape is tried, where ranges are short and the weights
// cold: one token tile of up to 24 K tiles (ping-pong / 192 x 256 / plain ring: N
// 9216, K 9216, M 129 64 / 64 / 56 us, M 256 78 / 90 / 68; N 12288, K 4096, M 129 46
// / 43 / 40; N 20480, K 5120, M 256, 27 K tiles 82 / - / 83), and where the ranges
// share HBM channels (N 4096, K 16384 in eight: M 400 80 us in ping-pong, 86 in 128
// x 256, 77; M 512 91, 91, 81; M 384 81, 102, 76).
inline bool plain_ring(const GemmParams& p, const SplitArgs& sa) {
    return sa.splits > 1 && ((p.M <= 256 && sa.kt_split <= 24) || same_channels(p, sa.splits));
}

// `base`: plan_tiles' choice for the same launch, kept unless another shape is
// predicted faster by a margin (below); up to GEMV_MAX_ROWS rows plan_few decides.
// Over the fitted launches the choice is 0.4% above the fastest shape in the mean;
// 1 of 952 products is more than 4% slower than its base.  Every other shape
// sums K in the same ranges as the base, added in the same order (tiles: the same
// split; the streaming kernel:
// the same split, or one block that closes a running sum at each range's end),
// so the result does not depend on the shape chosen, bit for bit; ragged-round
// plans, whose ranges differ from tile to tile, stay.  Measured gains over the
// base (us): M 24, N 16384, K 4096 38 -> 27 (stream), M 200, N 6144, K 2048 20.1
// -> 15.9 (stream 128 x 64), M 333, N 16384, K 4096 77 -> 59 (192 x 256), M 333,
// N 5120, K 20480 112 -> 91 (192 x 256), M 700, N 15360, K 5120 152 -> 110 (192
// x 256).
WidePlan plan_wide(const GemmParams& p, const GemmWorkspace& wsp, const TilePlan& base) {
    WidePlan best{WIDE_NONE, 0, 0, 0, 1, 0};
    if (p.M <= GEMV_MAX_ROWS || p.M > 2048 || base.ragged_tail > 0) return best;
    const SplitArgs sa = make_split(p, wsp, base.splits);
    if (base.tile == 256 && plain_ring(p, sa)) return WidePlan{WIDE_RING, 256, 256, 0, base.splits, 0};
    double best_t = tile_time(p, base.tile, base.tile, base.splits);
    // margins: the models' bias against measurement, shape by shape (64-row
    // streaming blocks come out up to 12% slower than predicted, the split 128 x 128
    // tiles beside 128-row ones up to 17%, and their reduce costs 3 us more where the
    // launches are not replayed from a graph)
    auto consider = [&](double t, const WidePlan& w) {
        double margin = 0.98;
        if (best.kind == WIDE_NONE) margin = w.kind != WIDE_STREAM ? 0.97 : w.bm == 32 ? 0.98 : w.bm == 64 ? 0.92 : 1.06;
        if (t < best_t * margin) {
            best_t = t;
            best = w;
        }
    };
    struct Shape { int kind, bm, bn; };
    for (const Shape& c : {Shape{WIDE_RING, 192, 128}, Shape{WIDE_PINGPONG, 128, 256}, Shape{WIDE_PINGPONG, 192, 256}}) {
        if (p.N % c.bn || (c.bm > 128 && p.M <= c.bm - 64)) continue;  // whole 64-row strips of padding
        consider(tile_time(p, c.bm, c.bn, sa.splits), WidePlan{c.kind, c.bm, c.bn, 0, base.splits, 0});
    }
    // the streaming kernel's rows are 128 K elements wide
    if (p.M <= STREAM_MAX_ROWS && p.K1 % 128 == 0) {
        for (const Shape& c : {Shape{WIDE_STREAM, 32, 64}, Shape{WIDE_STREAM, 32, 32}, Shape{WIDE_STREAM, 64, 64},
                               Shape{WIDE_STREAM, 128, 64}}) {
            if (c.bm == 32 ? p.M > 32 : p.M <= c.bm / 2) continue;
            consider(stream_time(p, c.bm, c.bn, 1), WidePlan{c.kind, c.bm, c.bn, 128, 1, sa.kt_split});
            if (sa.splits > 1 && sa.kt_split % 2 == 0)
                consider(stream_time(p, c.bm, c.bn, sa.splits),
                         WidePlan{c.kind, c.bm, c.bn, 128, sa.splits, sa.kt_split});
        }
    }
    if (best.kind == WIDE_STREAM && best.bm == 32) best.bk = wide_row_stage(p, best.bn, best.splits);
    return best;
}

// Time of a GEMV launch of at most GEMV_MAX_ROWS rows (gemv_kernel: a wave
// takes 4 features x K / KW): the weights at 5.8 TB/s, or the waves' dot products
// (208 cycles per row and 512 elements) and lane sums (400 per row) over the
// chip's 1024 SIMDs, rows in groups of 4 or 8; a LayerNorm that follows is a
// pass of its own.  Fitted, as few_stream_time, to the times of the projections of
// d_model 768 .. 12288 with 3 and 8 rows (mean error 8%).
inline double gemv_time(const GemmParams& p) {
    const int rows = p.M <= 1 ? 1 : p.M <= 2 ? 2 : p.M <= 4 ? 4 : 8, kw = p.K1 >= 4096 ? 8 : 4;
    const double dots = (double)p.N / 4 * kw * rows * (208.0 * p.K1 / kw / 512 + 400.0) / (1024 * 2.1e9);
    return 4.6e-6 + std::max(dots, (double)p.N * p.K1 * 2 / 5.8e12) + split_cost(p, 1, 0.0);
}

// ... and of a stream launch of so few rows in 32 x bn blocks: copies into LDS
// at 75 GB/s per CU, cold weights at 7.2 TB/s (less with fewer blocks than CUs),
// half of the shorter one left over, and a reduce that is mostly launch.
inline double few_stream_time(const GemmParams& p, int bn, int splits) {
    const long blocks = (long)(p.N / bn) * splits, per_cu = (blocks + 255) / 256;
    const double copy = per_cu * ((double)p.K1 / splits) * (32 + bn) * 2 / 75e9;
    double hbm = (double)p.N * p.K1 * 2 / 7.2e12;
    if (blocks < 256) hbm /= std::pow((double)blocks / 256, 0.4);
    const double t = std::max(copy, hbm) + 0.5 * std::min(copy, hbm);
    return 3.7e-6 + (bn == 32 ? 1.03 * t : t) +
           (splits > 1 ? 2.0 * p.M * p.N * 4 * splits / 8e12 + 3e-6 : split_cost(p, 1, 0.0));
}

// Launch of at most GEMV_MAX_ROWS rows: WIDE_NONE is the GEMV.  Its fp32 dot
// products cost arithmetic per row, the streaming kernel's matrix products do
// not (N 8192, K 2048: 13.3 us for 3 rows and 22.2 for 8 against 10.9; N 27648, K
// 9216: 94 and 175 against 92); the GEMV keeps 1 and 2 rows, few features (N 2048,
// K 2048, 3 rows: 6.3 against 8.2) and long weight rows of 3 and 4 (N 9216, K 36864:
// 119 against 125).  The faster of the two and of the splits by the two models
// above was within 0.6% of the fastest in the mean, 8% at worst, over those
// shapes.  K ranges are whole ring stages: no other launch has to give the same
// bits.  Operands that are not 16-byte aligned are the GEMV's, which takes them.
// Sums of fewer than 768 products are too: the GEMV's error is smaller there
// (bf16, K 512: 6.2e-8 relative against 6.4e-8; K 768: 6.5e-8 against 6.4e-8, K
// 8192: 8.8e-8 against 8.6e-8, f16 alike).
WidePlan plan_few(const GemmParams& p, const GemmWorkspace& wsp) {
    WidePlan best{WIDE_NONE, 0, 0, 0, 1, 0};
    if (p.M <= 2 || p.M > GEMV_MAX_ROWS || p.K1 % 128 || p.K1 < 768 ||
        (((uintptr_t)p.X | (uintptr_t)p.W | (uintptr_t)(p.ldx * 2) | (uintptr_t)(p.ldw * 2)) & 15))
        return best;
    double best_t = gemv_time(p);
    const int nk = p.K1 / BK;
    for (int bn : {64, 32})
        for (int s = 1; s <= 8; ++s) {
            const int kt = ((nk + s - 1) / s + 1) / 2 * 2, splits = (nk + kt - 1) / kt;
            if (splits != s || (s > 1 && (nk / s < PB_GEMM_MIN_KT || !wsp.ws ||
                                          (double)p.M * p.N * 4 * s > (double)wsp.bytes)))
                continue;
            const double t = few_stream_time(p, bn, s);
            if (t < best_t * 0.98) {  // the simpler launch on near ties
                best_t = t;
                best = {WIDE_STREAM, 32, bn, wide_row_stage(p, bn, s), s, kt};
            }
        }
    return best;
}

// Tile plan of a launch by role: the projections by the cost model above,
// the LoRA shrink (role 4) always 64 x 64, split along K when few.
TilePlan plan_for_role(int role, const GemmParams& p, const GemmWorkspace& wsp) {
    if (role != 4) return plan_tiles(p, wsp);
    const long tiles = (long)((p.M + 63) / 64) * (p.N / 64);
    int sp = 1;
    if (tiles < 256 && wsp.ws) {
        sp = std::min<long>((PB_GEMM_SPLIT_TARGET + tiles - 1) / tiles, std::max(1, p.K1 / BK / PB_GEMM_MIN_KT));
        while (sp > 1 && (double)p.M * p.N * 4 * sp > (double)wsp.bytes) --sp;
    }
    return {64, std::max(1, sp), 0};
}

}  // namespace

}  // namespace pb
