// MFMA GEMM for the decoder's projections on gfx950.
//
// Y[M, N] = X[M, K] W[N, K]^T with fp32 accumulation in v_mfma_f32_16x16x32_{f16,bf16}.
// The MFMA's A operand is the weight tile (rows = output features n) and its B
// operand the activation tile (columns = tokens m), so each lane ends up with
// four consecutive output features of one token: the epilogue writes 8-byte
// (dt) or 16-byte (fp32 residual) vectors.
//
// Block tile BM x BN, K tile 64: 256 x 256 (two wave groups in ping-pong over
// a 2-stage ring, 128 KiB of LDS: gemm_pingpong_kernel; a plain ring for short
// cold K ranges: plain_ring) or 128 x 128 (3-stage
// ring: with few tiles the weights arrive cold from HBM and a deeper ring
// hides more of that latency) with 8 waves (2 x 4, two waves per SIMD), chosen
// by how many tiles the shape gives, and 64 x 64 with 4 waves for N not a
// multiple of 128.  Tiles go straight from global memory
// into the S-stage LDS ring (LDS-DMA, no staging registers), so S-1 tiles are
// in flight while one is multiplied; one barrier per K tile.  The operand
// reads from LDS, not the MFMA rate, bound the smaller tiles: a wave's
// WM x WN sub-tile reads (WM + WN) rows per K tile.
// LDS rows are 128 bytes (64 elements) with the 16-byte chunks XOR-swizzled by
// the row index so that the MFMA operand reads of 16 consecutive rows are free
// of bank conflicts (the DMA writes the swizzle by choosing which chunk each
// lane fetches).
//
// Block order: the hardware deals consecutive blocks round-robin to the 8
// XCDs; the block id is remapped so that each XCD gets a contiguous run of
// tiles, walked in groups of 8 tile-rows, so blocks that share an XCD's L2
// share rows of X and of W.
//
// Small grids are split along K (deterministically: every split writes its
// fp32 partial tile to a workspace and a reduce kernel sums the splits in a
// fixed order before the epilogue).  The tile shape and split of a launch,
// its grid and the block -> tile map live in gemm_plan.h (host and device).
//
// The LoRA expand (Section 2.1: the adapter adds s (u A) B on top of the fixed
// W) is folded into the same accumulation as extra K tiles: [X | Z][W | Bcat]^T
// where Z holds s * (u A_slot) in the row's slot columns and zeros elsewhere,
// so sequences with different adapters (or none) share one launch.
#include <algorithm>
#include <type_traits>

#include "common.h"
#include "gemm_plan.h"
#include "kernels.h"

namespace pb {

namespace {

#ifndef PB_GEMM_S128
#define PB_GEMM_S128 3  // LDS ring depth of the 128 x 128 tiles
#endif
#ifndef PB_GEMM_S64
#define PB_GEMM_S64 4  // ... of the 64 x 64 tiles
#endif
#ifndef PB_GEMM_GEMV
#define PB_GEMM_GEMV 1  // dot-product kernel for few token rows (plan_few)
#endif
#ifndef PB_GEMV_KW8
#define PB_GEMV_KW8 1  // GEMV rows of K >= 4096 split over eight waves
#endif
#ifndef PB_GEMV_NT
#define PB_GEMV_NT 1  // weights streamed by the GEMV with non-temporal loads
#endif
#ifndef PB_GEMV_RPB
#define PB_GEMV_RPB 4  // output features per GEMV block
#endif

constexpr int ROW_BYTES = BK * 2;

// Physical 16-byte chunk of logical chunk ch in LDS row `row`.  chunk ^ (row & 7)
// measured conflict-free on gfx950 for the operand reads (16 rows, one chunk
// per lane group) with the bank-conflict counter.
__device__ __forceinline__ int swz(int row, int ch) { return ch ^ (row & 7); }

// Epilogue of four consecutive output features n..n+3 of token m.
template <typename T, int EPI>
__device__ __forceinline__ void epilogue4(const GemmParams& p, int m, int n, f32x4 v) {
    if (EPI == EPI_SHRINK) {
        const int slot = p.row_slot[m];
        const int c = n % p.kw;  // slot_width is a multiple of 4
        const bool keep = slot >= 0 && (c / p.slot_width) == slot;
        const float f = keep ? p.slot_scale[slot] : 0.f;
        *(u32x2*)((T*)p.C + (int64_t)m * p.ldc + n) =
            pack4<T>(keep ? v[0] * f : 0.f, keep ? v[1] * f : 0.f, keep ? v[2] * f : 0.f,
                     keep ? v[3] * f : 0.f);
        return;
    }
    const u32x2 braw = *(const u32x2*)((const T*)p.bias + n);
    T bb[4];
    __builtin_memcpy(bb, &braw, 8);
    float y[4];
#pragma unroll
    for (int r = 0; r < 4; ++r) y[r] = v[r] + (float)bb[r];
    if (EPI == EPI_QKV) {
        float sc[4];
#pragma unroll
        for (int r = 0; r < 4; ++r) sc[r] = n + r < p.qcols ? p.qscale : 1.f;
        const u32x2 out = pack4<T>(y[0] * sc[0], y[1] * sc[1], y[2] * sc[2], y[3] * sc[3]);
        *(u32x2*)((T*)p.C + (int64_t)m * p.ldc + n) = out;
        if (p.kv && n >= p.qcols) {  // qcols is a multiple of 4: the group is all key or all value
            const int64_t row = (int64_t)(m / p.kv_T) * p.kv_seq + (int64_t)(*p.kv_pos + m % p.kv_T) * 2 * p.qcols;
            *(u32x2*)((T*)p.kv + row + (n - p.qcols)) = out;
        }
    } else if (EPI == EPI_RELU) {
        *(u32x2*)((T*)p.C + (int64_t)m * p.ldc + n) =
            pack4<T>(fmaxf(y[0], 0.f), fmaxf(y[1], 0.f), fmaxf(y[2], 0.f), fmaxf(y[3], 0.f));
    } else {  // EPI_RESID
        f32x4* rp = (f32x4*)(p.R + (int64_t)m * p.ldr + n);
        f32x4 rv = *rp;
        rv[0] += y[0];
        rv[1] += y[1];
        rv[2] += y[2];
        rv[3] += y[3];
        *rp = rv;
    }
}

// Epilogue of a wave's accumulators: acc[i][j] holds output features
// nb + 16 i + 4 lg + r (r = 0..3) of token mb + 16 j + lr.
template <typename T, int EPI, int MF, int NF>
__device__ __forceinline__ void store_tile(const GemmParams& p, const TileJob& jb, int mb, int nb, int lr, int lg,
                                           const f32x4 (&acc)[NF][MF]) {
#pragma unroll
    for (int j = 0; j < MF; ++j) {
        const int m = mb + j * 16 + lr;
        if (m >= p.M) continue;
#pragma unroll
        for (int i = 0; i < NF; ++i) {
            const int n = nb + i * 16 + 4 * lg;
            if (n >= p.N) continue;
            if (jb.partial)
                *(f32x4*)(jb.pbase + (int64_t)(m - jb.om) * jb.ldp + (n - jb.on)) = acc[i][j];
            else
                epilogue4<T, EPI>(p, m, n, acc[i][j]);
        }
    }
}

// (at least two waves per SIMD as the register budget: with more registers the
// compiler moves accumulators between register files around every MFMA)
template <typename T, int EPI, int BM, int BN, int WGM, int WGN, int ROLE, int S>
__global__ __launch_bounds__(64 * WGM * WGN) __attribute__((amdgpu_waves_per_eu(2)))
void gemm_kernel(GemmParams p, SplitArgs sa) {
    typedef typename Mfma<T>::vec8 vec8;
    constexpr int NW = WGM * WGN;               // waves per block
    constexpr int WM = BM / WGM, WN = BN / WGN;  // wave tile
    constexpr int MF = WM / 16, NF = WN / 16;   // 16x16 fragments per wave
    constexpr int NL = (BM + BN) / (8 * NW);    // LDS-DMA instructions per wave per K tile
    constexpr int NLX = BM / (8 * NW);          // ... of which carry X rows
    constexpr int STAGE = (BM + BN) * ROW_BYTES;
    static_assert(BM % (8 * NW) == 0 && BN % (8 * NW) == 0, "DMA slots split into X and W");
    static_assert(S >= 2 && (S - 2) * NL < 64, "pipeline depth");
    extern __shared__ __attribute__((aligned(16))) uint8_t smem[];

    const int tid = threadIdx.x;
    const int lane = tid & 63, wave = tid >> 6;
    const int wm = wave % WGM, wn = wave / WGM;
    const TileJob jb = tile_job<BM, BN>(p, sa, (int)blockIdx.x, (int)gridDim.x);
    const int m0 = jb.m0, n0 = jb.n0, nk1 = jb.nk1, t_begin = jb.t_begin, nk = jb.nk;
    const T* X2 = (const T*)jb.X2;

    // DMA instruction j of this wave fills LDS rows 8g .. 8g+7, g = wave + NW j;
    // rows < BM hold X (tokens), the rest W (output features): slots j < NLX.
    // Lane i writes row 8g + i/8, physical chunk i%8, which holds logical K
    // chunk (i%8) ^ (row & 7) = (i%8) ^ (i/8) for every j.  Rows past the
    // matrix edge re-read its last row.
    const int lrow = lane >> 3;
    const int chk = swz(lrow, lane & 7) * 8;
    const int xr0 = m0 + 8 * wave + lrow, wr0 = n0 + 8 * wave + lrow - BM;
    const T* Xb = (const T*)p.X;
    const T* Wb = (const T*)p.W;
    const T* W2 = (const T*)p.W2;
    const uint32_t lds0 = (uint32_t)(uintptr_t)smem;
    // each slot's row is the same in every K tile: its byte offset (row and
    // chunk) is taken once and a tile moves the operand's scalar base by its
    // K offset, so the lanes' offsets cost no VALU work per tile (measured:
    // 46 -> 14 vector adds per K tile, the large projections 1.3-1.9% faster
    // under the power limit); byte offsets fit in 32 bits (the launcher keeps
    // rows * leading dimension below 2^31 elements)
    uint32_t soff[NL];
#pragma unroll
    for (int j = 0; j < NL; ++j)
        soff[j] = j < NLX ? ((uint32_t)min(xr0 + 8 * NW * j, p.M - 1) * (uint32_t)p.ldx + chk) * 2
                          : ((uint32_t)min(wr0 + 8 * NW * j, p.N - 1) * (uint32_t)p.ldw + chk) * 2;
    auto issue = [&](int t, int stage) {
        const uint32_t sbase = lds0 + stage * STAGE;
        if (t < nk1) {
            const int64_t kb = (int64_t)t * BK * 2;
            const char* xk = (const char*)Xb + kb;
            const char* wk = (const char*)Wb + kb;
#pragma unroll
            for (int j = 0; j < NL; ++j)
                dma16s(j < NLX ? xk : wk, soff[j],
                       sbase + (uint32_t)__builtin_amdgcn_readfirstlane((wave + NW * j) * 1024));
        } else {  // LoRA K tiles: [Z | B] rows of the same slots
            const int64_t kb = (int64_t)(t - nk1) * BK * 2;
            const char* xk = (const char*)X2 + kb;
            const char* wk = (const char*)W2 + kb;
#pragma unroll
            for (int j = 0; j < NL; ++j) {
                const uint32_t off = j < NLX ? ((uint32_t)min(xr0 + 8 * NW * j, p.M - 1) * (uint32_t)p.ldx2 + chk) * 2
                                             : ((uint32_t)min(wr0 + 8 * NW * j, p.N - 1) * (uint32_t)p.ldw2 + chk) * 2;
                dma16s(j < NLX ? xk : wk, off,
                       sbase + (uint32_t)__builtin_amdgcn_readfirstlane((wave + NW * j) * 1024));
            }
        }
    };

    f32x4 acc[NF][MF];
#pragma unroll
    for (int i = 0; i < NF; ++i)
#pragma unroll
        for (int j = 0; j < MF; ++j) acc[i][j] = f32x4{0.f, 0.f, 0.f, 0.f};

    const int lr = lane & 15, lg = lane >> 4;
    auto compute = [&](int stage) {
        const uint8_t* s = smem + stage * STAGE;
#pragma unroll
        for (int kk = 0; kk < 2; ++kk) {
            const int ch = kk * 4 + lg;
            vec8 b[MF];
#pragma unroll
            for (int j = 0; j < MF; ++j) {
                const int row = wm * WM + j * 16 + lr;
                b[j] = as_vec8<T>(*(const u32x4*)(s + row * ROW_BYTES + (swz(row, ch) << 4)));
            }
#pragma unroll
            for (int i = 0; i < NF; ++i) {
                const int row = BM + wn * WN + i * 16 + lr;
                const vec8 a = as_vec8<T>(*(const u32x4*)(s + row * ROW_BYTES + (swz(row, ch) << 4)));
#pragma unroll
                for (int j = 0; j < MF; ++j) acc[i][j] = Mfma<T>::mma(a, b[j], acc[i][j]);
            }
        }
    };

    // S-stage ring: tiles t+1 .. t+S-1 are in flight while tile t is multiplied.
    // Steady state first (branch-free), then the tail that drains the ring.
#pragma unroll
    for (int q = 0; q < S - 1; ++q)
        if (q < nk) issue(t_begin + q, q);
    int t = 0;
    for (; t + S - 1 < nk; ++t) {
        wait_vmcnt<(S - 2) * NL>();  // tiles t+1 .. t+S-2 may still fly
        __syncthreads();             // tile t visible to all waves; stage of tile t-1 free
        issue(t_begin + t + S - 1, (t + S - 1) % S);
        compute(t % S);
    }
    for (; t < nk; ++t) {
        wait_vmcnt<0>();
        __syncthreads();
        compute(t % S);
    }

    store_tile<T, EPI, MF, NF>(p, jb, m0 + wm * WM, n0 + wn * WN, lr, lg, acc);
}

// ---- 256-feature tiles: two wave groups in ping-pong ----------------------------
// Tiles of 64 XF tokens (XF = 2, 3 or 4) x 256 features; eight waves (2 x 4),
// wave tile 32 XF tokens x 64 features, K tile 64, two LDS stages.  A K tile is
// four phases, one per quadrant (16 XF tokens x 32 features) of the wave tile, and a phase has two slots, each closed by a barrier: a
// memory slot (operand reads of the quadrant into registers, one or two copies)
// and a product slot (4 XF products at raised wave priority).  Waves 4-7 run one slot
// behind waves 0-3, and waves w and w + 4 share a SIMD, so one of the two is
// always in its product slot while the other reads LDS: the matrix unit is not
// left idle by operand reads, copy waits or the barrier, which held one third
// of the cycles of the plain ring (0.60 MFMA busy).
//
// A stage is four regions in order of need: Wa (32 of each wave's 64 features),
// X0 (half of its tokens), Wb, X1.  Quadrants go (Wa, X0), (Wb, X0),
// (Wb, X1), (Wa, X1); Wa of the next tile is read in the last phase, into the
// registers of this tile's Wb, so even tiles start with feature half 0 and odd
// ones with half 1 and each memory slot holds 4 or 2 XF reads.  A region is free
// once both groups have read it, one slot later, and is then refilled with
// tile t + 2: every copy has seven phases to land with two stages only, and
// every wait is for all but the youngest one and a half tiles of a wave's copies.  Past the last
// tile the copies re-read it (they land in regions nobody reads).
//
// Bound by the matrix units (0.74 - 0.78 busy in counter runs at the OPT-66B
// shapes, the plain ring 0.60) at the clock the power limit leaves (1.7 GHz,
// 1.95 there); OPT-66B fc1
// (M 4096, N 36864, K 9216, f16) 2235 -> 2000 us (1245 -> 1395 TFLOP/s, the
// vendor library 1406), M 2000, N 20480, K 5120 416 -> 361 us.  The K order of
// every output is that of the plain loop (bit-identical results).
template <typename T, int EPI, int XF, int ROLE>
__global__ __launch_bounds__(512) __attribute__((amdgpu_waves_per_eu(2)))
void gemm_pingpong_kernel(GemmParams p, SplitArgs sa) {
    typedef typename Mfma<T>::vec8 vec8;
    constexpr int BM = 64 * XF, BN = 256;
    constexpr int XH = 16 * XF;            // tokens of a wave's X half
    constexpr int XC = BM / 2 / 8;         // copies of an X region
    constexpr int XQ = (XC + 7) / 8;       // ... per wave (XF = 3: four waves repeat the last one)
    constexpr int LAG = (4 + 2 * XQ) * 3 / 2;  // copies younger than the one a slot needs
    constexpr int STAGE = (BM + BN) * ROW_BYTES;
    extern __shared__ __attribute__((aligned(16))) uint8_t smem[];
    const int lane = threadIdx.x & 63;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int wm = wave & 1, wn = wave >> 1;
    const TileJob jb = tile_job<BM, BN>(p, sa, (int)blockIdx.x, (int)gridDim.x);
    const int m0 = jb.m0, n0 = jb.n0, nk1 = jb.nk1, t_begin = jb.t_begin, nk = jb.nk;

    // copies: region X h is token rows (2 g + h) XH .. + XH - 1 (g = 0, 1),
    // region W h feature rows 64 g + 32 h .. + 31 (g = 0 .. 3), 8 rows per copy;
    // copy q of this wave is number wave + 8 q of its region.  Lane i writes
    // row i / 8, physical chunk i % 8.
    const int lrow = lane >> 3;
    const int chk = swz(lrow, lane & 7) * 8;
    const uint32_t lds0 = (uint32_t)(uintptr_t)smem;
    int xrow[2 * XQ], wrow[4];  // first row of copy q of region h: [XQ h + q], [2 h + q]
    uint32_t xoff[2 * XQ], woff[4];
#pragma unroll
    for (int i = 0; i < 2 * XQ; ++i) {
        const int h = i / XQ, c = min(wave + 8 * (i % XQ), XC - 1);
        xrow[i] = (2 * (c / (XC / 2)) + h) * XH + (c % (XC / 2)) * 8;
        xoff[i] = ((uint32_t)min(m0 + xrow[i] + lrow, p.M - 1) * (uint32_t)p.ldx + chk) * 2;
    }
#pragma unroll
    for (int i = 0; i < 4; ++i) {
        const int h = i >> 1, c = wave + 8 * (i & 1);
        wrow[i] = (c >> 2) * 64 + h * 32 + (c & 3) * 8;
        woff[i] = ((uint32_t)min(n0 + wrow[i] + lrow, p.N - 1) * (uint32_t)p.ldw + chk) * 2;
    }
    // the LoRA K tiles' offsets are taken where they are used (the empty asm
    // keeps the compiler from holding them in registers through the base tiles)
    auto copy_x = [&](int t, int stage, int h) {
        const uint32_t sb = lds0 + stage * STAGE;
        t += t_begin;
        if (t < nk1) {
            const char* b = (const char*)p.X + (int64_t)t * BK * 2;
#pragma unroll
            for (int i = XQ * h; i < XQ * h + XQ; ++i) dma16s(b, xoff[i], sb + xrow[i] * ROW_BYTES);
        } else {
            const char* b = (const char*)jb.X2 + (int64_t)(t - nk1) * BK * 2;
#pragma unroll
            for (int i = XQ * h; i < XQ * h + XQ; ++i) {
                int r = m0 + xrow[i] + lrow;
                asm volatile("" : "+v"(r));
                dma16s(b, ((uint32_t)min(r, p.M - 1) * (uint32_t)p.ldx2 + chk) * 2, sb + xrow[i] * ROW_BYTES);
            }
        }
    };
    auto copy_w = [&](int t, int stage, int h) {
        const uint32_t sb = lds0 + stage * STAGE + BM * ROW_BYTES;
        t += t_begin;
        if (t < nk1) {
            const char* b = (const char*)p.W + (int64_t)t * BK * 2;
#pragma unroll
            for (int i = 2 * h; i < 2 * h + 2; ++i) dma16s(b, woff[i], sb + wrow[i] * ROW_BYTES);
        } else {
            const char* b = (const char*)p.W2 + (int64_t)(t - nk1) * BK * 2;
#pragma unroll
            for (int i = 2 * h; i < 2 * h + 2; ++i) {
                int r = n0 + wrow[i] + lrow;
                asm volatile("" : "+v"(r));
                dma16s(b, ((uint32_t)min(r, p.N - 1) * (uint32_t)p.ldw2 + chk) * 2, sb + wrow[i] * ROW_BYTES);
            }
        }
    };

    f32x4 acc[4][2 * XF];
#pragma unroll
    for (int i = 0; i < 4; ++i)
#pragma unroll
        for (int j = 0; j < 2 * XF; ++j) acc[i][j] = f32x4{0.f, 0.f, 0.f, 0.f};
    const int lr = lane & 15, lg = lane >> 4;
    vec8 w0[2][2], w1[2][2], x[XF][2];  // [fragment][k half]
    const uint32_t lk[2] = {(uint32_t)(lr * ROW_BYTES + (swz(lr, lg) << 4)),
                            (uint32_t)(lr * ROW_BYTES + (swz(lr, 4 + lg) << 4))};
    auto read_w = [&](vec8 (&w)[2][2], int stage, int h) {
        const uint8_t* s = smem + stage * STAGE + (BM + wn * 64 + h * 32) * ROW_BYTES;
#pragma unroll
        for (int i = 0; i < 2; ++i)
#pragma unroll
            for (int kk = 0; kk < 2; ++kk) w[i][kk] = as_vec8<T>(*(const u32x4*)(s + i * 16 * ROW_BYTES + lk[kk]));
    };
    auto read_x = [&](int stage, int h) {
        const uint8_t* s = smem + stage * STAGE + (2 * wm + h) * XH * ROW_BYTES;
#pragma unroll
        for (int j = 0; j < XF; ++j)
#pragma unroll
            for (int kk = 0; kk < 2; ++kk) x[j][kk] = as_vec8<T>(*(const u32x4*)(s + j * 16 * ROW_BYTES + lk[kk]));
    };
    // nothing moves across the end of a slot
    auto barrier = [] { asm volatile("s_barrier" ::: "memory"); };
    auto end_memory = [&] {
        __builtin_amdgcn_sched_barrier(0);
        asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory");
        __builtin_amdgcn_sched_barrier(0);
    };
    auto products = [&](const vec8 (&w)[2][2], int fi, int fj) {
        __builtin_amdgcn_s_setprio(1);
#pragma unroll
        for (int kk = 0; kk < 2; ++kk)
#pragma unroll
            for (int i = 0; i < 2; ++i)
#pragma unroll
                for (int j = 0; j < XF; ++j)
                    acc[fi + i][fj + j] = Mfma<T>::mma(w[i][kk], x[j][kk], acc[fi + i][fj + j]);
        __builtin_amdgcn_s_setprio(0);
        __builtin_amdgcn_sched_barrier(0);
        barrier();
        __builtin_amdgcn_sched_barrier(0);
    };

    const int last = nk - 1;
    auto fill = [&](int t, int stage) {  // a whole stage, in order of need
        copy_w(t, stage, stage);
        copy_x(t, stage, 0);
        copy_w(t, stage, 1 - stage);
        copy_x(t, stage, 1);
    };
    fill(0, 0);
    fill(min(1, last), 1);
    wait_vmcnt<LAG>();
    barrier();
    read_w(w0, 0, 0);
    end_memory();               // both groups hold Wa of tile 0: its region may be refilled
    if (wave >= 4) barrier();  // one slot behind from here on
    auto tile = [&](int t, auto parity) {
        constexpr int P = decltype(parity)::value;  // t % 2: the stage, and the feature half of Wa
        auto& wa = P ? w1 : w0;
        auto& wb = P ? w0 : w1;
        const int tn = min(t + 2, last);
        read_x(P, 0);
        copy_w(tn, P, P);
        wait_vmcnt<LAG>();  // Wb landed
        end_memory();
        products(wa, 2 * P, 0);
        read_w(wb, P, 1 - P);
        copy_x(tn, P, 0);
        wait_vmcnt<LAG>();  // X1 landed
        end_memory();
        products(wb, 2 - 2 * P, 0);
        read_x(P, 1);
        copy_w(tn, P, 1 - P);
        wait_vmcnt<LAG>();  // Wa of t + 1 landed
        end_memory();
        products(wb, 2 - 2 * P, XF);
        read_w(wb, 1 - P, 1 - P);  // Wa of t + 1
        copy_x(tn, P, 1);
        wait_vmcnt<LAG>();  // X0 of t + 1 landed
        end_memory();
        products(wa, 2 * P, XF);
    };
    const std::integral_constant<int, 0> even;
    const std::integral_constant<int, 1> odd;
    int t = 0;
    for (; t + 1 < nk; t += 2) {
        tile(t, even);
        tile(t + 1, odd);
    }
    if (t < nk) tile(t, even);
    if (wave < 4) barrier();  // as many barriers in both groups

    store_tile<T, EPI, 2 * XF, 4>(p, jb, m0 + wm * 2 * XH, n0 + wn * 64, lr, lg, acc);
    wait_vmcnt<0>();  // the last copies have landed before the block's LDS is given back
}

// ---- few rows (batched decode, short prompts): wide-row weight streaming ------
// One block computes BM tokens (all of them up to 32 or 64) x BN output features
// over one K range; its waves split the features (and the tokens when WGM > 1).  A ring
// stage holds BKE (128 or 256) K elements of the BM token rows and BN weight
// rows, so a copy instruction fetches whole 256- or 512-byte row pieces; the
// 128-byte pieces of the tiles above reach 3.5 TB/s on such products, these
// 4.9 (N 16384, K 4096, 32 rows: 27.4 us against 37.3; N 2048, K 8192: 8.7
// and a reduce against 16.6).  HBM-bound for large N, by its fixed ~3 us for
// small ones.  An unsplit launch still adds the K ranges of plan_tiles' split
// one after another (the same result as its partials and reduce, bit for bit).
// Up to GEMV_MAX_ROWS rows, which the GEMV's dot products serve as well, a
// chain of MFMA sums ends after 128 elements and the running sum keeps the
// rounding errors of its additions (two-sum).  Chains as long as a K range lost
// more than the dot products' short ones (relative error of the sums, K 2048 ..
// 36864: 1.5e-7 .. 4.6e-7 with a workspace, up to 1.2e-6 without, the GEMV's
// 0.9e-7 .. 1.3e-7, these 0.8e-7 .. 1.0e-7).
// The base K ranges are independent of the LoRA segment (B = 0 stays
// bit-identical to the base), whose few columns are read
// straight into registers: the first 64, requested ahead of the ring, have
// landed by the time the base is done.
template <typename T, int EPI, int BM, int BN, int WGM, int WGN, int BKE, int S, int ROLE, bool FEW>
__global__ __launch_bounds__(64 * WGM * WGN) void stream_kernel(GemmParams p, SplitArgs sa, int kst) {
    typedef typename Mfma<T>::vec8 vec8;
    constexpr int NW = WGM * WGN;
    constexpr int WM = BM / WGM, WN = BN / WGN;
    constexpr int MF = WM / 16, NF = WN / 16;
    constexpr int RB = BKE * 2;                // bytes per LDS row
    constexpr int CPR = RB / 16;               // 16-byte chunks per row
    constexpr int RPI = 1024 / RB;             // rows per copy instruction
    constexpr int NL = (BM + BN) / RPI / NW;   // copy instructions per wave per stage
    constexpr int STAGE = (BM + BN) * RB;
    static_assert(BM % (RPI * NW) == 0 && BN % (RPI * NW) == 0, "copy slots split into X and W");
    static_assert(S >= 2 && (S - 2) * NL < 64, "pipeline depth");
    extern __shared__ __attribute__((aligned(16))) uint8_t smem[];

    const int lane = threadIdx.x & 63;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int wm = wave % WGM, wn = wave / WGM;
    const int lr = lane & 15, lg = lane >> 4;
    const StreamJob job = stream_job<BM, BN, BKE>(p, kst, (int)blockIdx.x, (int)gridDim.x);
    const int split = job.split, m0 = job.m0, n0 = job.n0, t0 = job.t0, n = job.n;

    // copy j of this wave fills rows RPI (wave + NW j) .. of a stage, tokens
    // first; the 16-byte chunks of a row are XOR-permuted by its low row bits
    // (all 16 rows of an operand read then hit distinct banks)
    uint32_t off[NL];
#pragma unroll
    for (int j = 0; j < NL; ++j) {
        const int row = (wave + NW * j) * RPI + lane / CPR;
        const int ch = (lane % CPR) ^ (row & 15);
        off[j] = (wave + NW * j) * RPI < BM
                     ? ((uint32_t)min(m0 + row, p.M - 1) * (uint32_t)p.ldx + ch * 8) * 2
                     : ((uint32_t)(n0 + row - BM) * (uint32_t)p.ldw + ch * 8) * 2;
    }
    const uint32_t lds0 = (uint32_t)(uintptr_t)smem;
    auto issue = [&](int t, int stage) {
        const int64_t kb = (int64_t)t * RB;
        const char* xk = (const char*)p.X + kb;
        const char* wk = (const char*)p.W + kb;
#pragma unroll
        for (int j = 0; j < NL; ++j) {
            const int I = wave + NW * j;
            dma16s(I * RPI < BM ? xk : wk, off[j], lds0 + stage * STAGE + I * 1024);
        }
    };

    // acc: the K range at hand; sum: the ranges closed so far (-0 + x is x)
    f32x4 acc[NF][MF], sum[NF][MF];
#pragma unroll
    for (int i = 0; i < NF; ++i)
#pragma unroll
        for (int j = 0; j < MF; ++j) {
            acc[i][j] = f32x4{0.f, 0.f, 0.f, 0.f};
            sum[i][j] = f32x4{-0.f, -0.f, -0.f, -0.f};
        }
    auto close_range = [&] {
#pragma unroll
        for (int i = 0; i < NF; ++i)
#pragma unroll
            for (int j = 0; j < MF; ++j)
#pragma unroll
                for (int r = 0; r < 4; ++r) {
                    sum[i][j][r] += acc[i][j][r];
                    acc[i][j][r] = 0.f;
                }
    };
    int left = sa.kt_split;  // K tiles of 64 until the range at hand ends
    auto compute = [&](int stage) {
        const uint8_t* s = smem + stage * STAGE;
#pragma unroll
        for (int kk = 0; kk < BKE / 32; ++kk) {
            if (kk % 2 == 0 && left-- == 0) {  // the tile after a range's last
                close_range();
                left = sa.kt_split - 1;
            }
            const int ch = kk * 4 + lg;
            vec8 b[MF];
#pragma unroll
            for (int j = 0; j < MF; ++j) {
                const int row = wm * WM + j * 16 + lr;
                b[j] = as_vec8<T>(*(const u32x4*)(s + row * RB + ((ch ^ (row & 15)) << 4)));
            }
#pragma unroll
            for (int i = 0; i < NF; ++i) {
                const int row = BM + wn * WN + i * 16 + lr;
                const vec8 a = as_vec8<T>(*(const u32x4*)(s + row * RB + ((ch ^ (row & 15)) << 4)));
#pragma unroll
                for (int j = 0; j < MF; ++j) acc[i][j] = Mfma<T>::mma(a, b[j], acc[i][j]);
            }
        }
    };

    // FEW: only the first 16 tokens exist; low holds the rounding errors of sum (a
    // kernel of its own: the same choice made in the loop cost more rows 1 us)
    f32x4 low[NF];
#pragma unroll
    for (int i = 0; i < NF; ++i) low[i] = f32x4{0.f, 0.f, 0.f, 0.f};
    auto compute_few = [&](int stage) {
        const uint8_t* s = smem + stage * STAGE;
#pragma unroll
        for (int h = 0; h < BKE / 128; ++h) {
            f32x4 c[NF];
#pragma unroll
            for (int i = 0; i < NF; ++i) c[i] = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
            for (int kk = 4 * h; kk < 4 * h + 4; ++kk) {
                const int ch = kk * 4 + lg;
                const vec8 b = as_vec8<T>(*(const u32x4*)(s + lr * RB + ((ch ^ lr) << 4)));
#pragma unroll
                for (int i = 0; i < NF; ++i) {
                    const int row = BM + wn * WN + i * 16 + lr;
                    c[i] = Mfma<T>::mma(as_vec8<T>(*(const u32x4*)(s + row * RB + ((ch ^ (row & 15)) << 4))), b, c[i]);
                }
            }
#pragma unroll
            for (int i = 0; i < NF; ++i)
#pragma unroll
                for (int r = 0; r < 4; ++r) {
                    const float x = sum[i][0][r], y = c[i][r], t = x + y, yy = t - x;
                    low[i][r] += (x - (t - yy)) + (y - yy);
                    sum[i][0][r] = t;
                }
        }
    };
    auto step = [&](int stage) {
        if constexpr (FEW) compute_few(stage);
        else compute(stage);
    };

    // LoRA segment of this block's output group (last split): operands of one
    // 32-wide step straight from global memory
    int nk2 = 0;
    const T* X2 = (const T*)p.X2;
    if (p.K2 > 0 && split == sa.splits - 1) {
        const int g = n0 / p.group;  // the group size is a multiple of BN
        if ((p.k2_mask >> g) & 1u) {
            nk2 = p.K2 / 32;
            X2 += (int64_t)g * p.x2_group_stride;
        }
    }
    struct Ops {
        u32x4 w[NF], x[MF];
    };
    auto load2 = [&](Ops& o, int t) {
#pragma unroll
        for (int i = 0; i < NF; ++i)
            o.w[i] = *(const u32x4*)((const T*)p.W2 + (int64_t)(n0 + wn * WN + i * 16 + lr) * p.ldw2 + t * 32 + 8 * lg);
#pragma unroll
        for (int j = 0; j < MF; ++j)
            o.x[j] = *(const u32x4*)(X2 + (int64_t)min(m0 + wm * WM + j * 16 + lr, p.M - 1) * p.ldx2 + t * 32 + 8 * lg);
    };
    auto mul2 = [&](const Ops& o) {
#pragma unroll
        for (int i = 0; i < NF; ++i)
#pragma unroll
            for (int j = 0; j < MF; ++j) acc[i][j] = Mfma<T>::mma(as_vec8<T>(o.w[i]), as_vec8<T>(o.x[j]), acc[i][j]);
    };
    Ops l0, l1;
    if (nk2 > 0) {  // K2 is a multiple of 64: at least two steps
        load2(l0, 0);
        load2(l1, 1);
    }

#pragma unroll
    for (int q = 0; q < S - 1; ++q)
        if (q < n) issue(t0 + q, q);
    int t = 0, st = 0;
    for (; t + S - 1 < n; ++t) {
        wait_vmcnt<(S - 2) * NL>();
        __syncthreads();  // stage st visible to all waves; the stage before it free
        issue(t0 + t + S - 1, st == 0 ? S - 1 : st - 1);
        step(st);
        st = st == S - 1 ? 0 : st + 1;
    }
    for (; t < n; ++t) {
        wait_vmcnt<0>();
        __syncthreads();
        step(st);
        st = st == S - 1 ? 0 : st + 1;
    }
    if (nk2 > 0) {
        mul2(l0);
        mul2(l1);
        for (int q = 2; q < nk2; q += 2) {
            load2(l0, q);
            load2(l1, q + 1);
            mul2(l0);
            mul2(l1);
        }
    }
    if constexpr (FEW) {
#pragma unroll
        for (int i = 0; i < NF; ++i)
#pragma unroll
            for (int r = 0; r < 4; ++r)  // acc: the LoRA columns; an overflowed sum has a NaN for its error
                sum[i][0][r] += fabsf(sum[i][0][r]) < INFINITY ? low[i][r] + acc[i][0][r] : acc[i][0][r];
    } else {
        close_range();
    }
    TileJob jb;
    jb.partial = sa.splits > 1;
    jb.pbase = sa.ws + (int64_t)split * p.M * p.N;
    jb.ldp = p.N;
    jb.om = jb.on = 0;
    store_tile<T, EPI, MF, NF>(p, jb, m0 + wm * WM, n0 + wn * WN, lr, lg, sum);
}

// Sum the split-K partials in split order, then apply the epilogue.
template <typename T, int EPI, int ROLE>
__global__ __launch_bounds__(256) void splitk_reduce_kernel(GemmParams p, SplitArgs sa) {
    const int64_t q = (int64_t)blockIdx.x * 256 + threadIdx.x;  // index of a group of 4 columns
    const int64_t per_row = p.N / 4;
    if (q >= (int64_t)p.M * per_row) return;
    const int m = (int)(q / per_row), n = (int)(q % per_row) * 4;
    const int64_t stride = (int64_t)p.M * p.N;
    const float* src = sa.ws + (int64_t)m * p.N + n;
    f32x4 v = *(const f32x4*)src;
    for (int s = 1; s < sa.splits; ++s) {
        const f32x4 w = *(const f32x4*)(src + s * stride);
        v[0] += w[0];
        v[1] += w[1];
        v[2] += w[2];
        v[3] += w[3];
    }
    epilogue4<T, EPI>(p, m, n, v);
}

// Reduce of a ragged-round split: only the tail tiles' partials, summed in
// split order, then the epilogue.  One thread per group of 4 columns.
template <typename T, int EPI, int ROLE, int BM, int BN>
__global__ __launch_bounds__(256) void tail_reduce_kernel(GemmParams p, SplitArgs sa) {
    constexpr int GPT = BM * BN / 4;  // column groups per tile
    const int64_t q = (int64_t)blockIdx.x * 256 + threadIdx.x;
    if (q >= (int64_t)sa.tail_tiles * GPT) return;
    const int tt = (int)(q / GPT);
    int m0, n0;
    tile_corner<BM, BN>(p, sa.full_tiles + tt, m0, n0);
    const int e = (int)(q % GPT);
    const int m = m0 + e / (BN / 4), n = n0 + (e % (BN / 4)) * 4;
    if (m >= p.M || n >= p.N) return;
    const int64_t stride = (int64_t)sa.tail_tiles * BM * BN;
    const float* src = sa.ws + (int64_t)tt * BM * BN + (int64_t)(m - m0) * BN + (n - n0);
    f32x4 v = *(const f32x4*)src;
    for (int s = 1; s < sa.splits; ++s) {
        const f32x4 w = *(const f32x4*)(src + s * stride);
        v[0] += w[0];
        v[1] += w[1];
        v[2] += w[2];
        v[3] += w[3];
    }
    epilogue4<T, EPI>(p, m, n, v);
}

// Row-wise split-K reduce of a residual projection fused with the LayerNorm
// that follows it: R[m] += (sum of partials in split order) + bias, then
// ln_out[m] = dt(LN(R[m]) * g + b) with fp32 statistics, and optionally the
// row's LoRA shrink.  One block per row; MAXC float4 chunks per thread (N <=
// 1024 MAXC); NS splits known at compile time (0: any count, summed in a loop)
// so that every partial of a chunk is in flight at once.
constexpr int RLN_MAXC = 16;  // largest chunk count: N <= 16384

template <typename T, int ROLE, int MAXC, int NS>
__global__ __launch_bounds__(256) void splitk_resid_ln_kernel(GemmParams p, SplitArgs sa) {
    __shared__ float red[4];
    const int m = blockIdx.x;
    const int nc = p.N / 4;
    const int64_t stride = (int64_t)p.M * p.N;
    float* xr = p.R + (int64_t)m * p.ldr;
    const float* wr = sa.ws + (int64_t)m * p.N;
    // every load of every chunk first (the stores to R below would otherwise
    // order the next chunk's loads behind them), then sums and stores; with
    // few chunks the loads are unconditional, a chunk past nc re-reading the
    // last one, so that no branch splits them into batches
    constexpr int NL = NS > 0 ? NS : 1;
    f32x4 v[MAXC], w[MAXC][NL];
    u32x2 braw[MAXC];
#pragma unroll
    for (int i = 0; i < MAXC; ++i) {
        int c = threadIdx.x + 256 * i;
        if (MAXC <= 4) c = min(c, nc - 1);
        else if (c >= nc) continue;
#pragma unroll
        for (int s = 0; s < NL; ++s) w[i][s] = *(const f32x4*)(wr + s * stride + 4 * c);
        braw[i] = *(const u32x2*)((const T*)p.bias + 4 * c);
        v[i] = *(const f32x4*)(xr + 4 * c);
    }
    float sum = 0.f;
#pragma unroll
    for (int i = 0; i < MAXC; ++i) {
        const int c = threadIdx.x + 256 * i;
        if (c < nc) {
            f32x4 a = w[i][0];
#pragma unroll
            for (int s = 1; s < NS; ++s)
                a = f32x4{a[0] + w[i][s][0], a[1] + w[i][s][1], a[2] + w[i][s][2], a[3] + w[i][s][3]};
            if (NS == 0)
                for (int s = 1; s < sa.splits; ++s) {
                    const f32x4 u = *(const f32x4*)(wr + s * stride + 4 * c);
                    a = f32x4{a[0] + u[0], a[1] + u[1], a[2] + u[2], a[3] + u[3]};
                }
            T bb[4];
            __builtin_memcpy(bb, &braw[i], 8);
            f32x4 x = v[i];
#pragma unroll
            for (int r = 0; r < 4; ++r) x[r] += a[r] + (float)bb[r];
            *(f32x4*)(xr + 4 * c) = x;
            v[i] = x;
            sum += (x[0] + x[1]) + (x[2] + x[3]);
        }
    }
    row_layernorm<T, MAXC, false>(v, sum, nc, (const T*)p.ln_g, (const T*)p.ln_b,
                                  (T*)p.ln_out + (int64_t)m * p.N, p.ln_eps, red);
    if (p.shrink.Acat) {
        __shared__ float red16[4][16];
        row_shrink<T, MAXC>(p.shrink, m, p.N, v, red16);
    }
}

template <typename T, int ROLE>
hipError_t launch_resid_ln(const GemmParams& all, const SplitArgs& sa, hipStream_t s) {
#define PB_RLN(MAXC, NS) \
    PB_LAUNCH((splitk_resid_ln_kernel<T, ROLE, MAXC, NS>), dim3(p.M), dim3(256), 0, s, p, sa)
    // few rows: the row's shrink on one block walks its rank groups one after
    // another (12 rows, d 4096, q,k,v rank 16: 19.7 us against 6.3 without it);
    // a launch of its own spreads them over blocks
    const bool apart = all.shrink.Acat && all.M <= ROW_SHRINK_APART;
    GemmParams p = all;
    if (apart) p.shrink.Acat = nullptr;
    // few rows (latency-bound): every partial in flight at once; many rows:
    // occupancy hides the latency and registers matter more
#define PB_RLN_NS(MAXC)                       \
    do {                                      \
        if (sa.splits == 2) PB_RLN(MAXC, 2);      \
        else if (sa.splits == 3) PB_RLN(MAXC, 3); \
        else if (sa.splits == 4) PB_RLN(MAXC, 4); \
        else if (sa.splits == 5) PB_RLN(MAXC, 5); \
        else if (sa.splits == 6) PB_RLN(MAXC, 6); \
        else if (sa.splits == 7) PB_RLN(MAXC, 7); \
        else if (sa.splits == 8) PB_RLN(MAXC, 8); \
        else PB_RLN(MAXC, 0);                     \
    } while (0)
    if (p.N <= 2048) PB_RLN_NS(2);
    else if (p.N <= 4096) PB_RLN_NS(4);
    else if (p.N <= 8192) PB_RLN(8, 0);
    else PB_RLN(RLN_MAXC, 0);
#undef PB_RLN_NS
#undef PB_RLN
    const hipError_t e = hipGetLastError();
    if (e != hipSuccess || !apart) return e;
    return launch_row_shrink(std::is_same<T, _Float16>::value ? 1 : 0, p.ln_out, all.shrink, p.M, p.N, s);
}

// After a split launch: the row-wise reduce (fused with the residual and the
// following LayerNorm where the caller asks for it).
template <typename T, int EPI, int ROLE>
hipError_t finish_split(const GemmParams& p, const SplitArgs& sa, hipStream_t s) {
    if (EPI == EPI_RESID && p.ln_out && p.N <= 256 * 4 * RLN_MAXC) {
        const hipError_t e = launch_resid_ln<T, ROLE>(p, sa, s);
        if (e == hipSuccess && p.ln_done) *p.ln_done = true;
        return e;
    }
    const int64_t groups = (int64_t)p.M * (p.N / 4);
    PB_LAUNCH((splitk_reduce_kernel<T, EPI, ROLE>), dim3((unsigned)((groups + 255) / 256)), dim3(256), 0,
                       s, p, sa);
    return hipGetLastError();
}

template <typename T, int EPI, int BM, int BN, int WGM, int WGN, int ROLE, int S, bool RING = BN != 256>
hipError_t launch_cfg(const GemmParams& p, const GemmWorkspace& wsp, int splits, int ragged_tail, hipStream_t s) {
    constexpr int LDS = S * (BM + BN) * ROW_BYTES;
    constexpr auto kernel = [] {
        if constexpr (RING) return &gemm_kernel<T, EPI, BM, BN, WGM, WGN, ROLE, S>;
        else return &gemm_pingpong_kernel<T, EPI, BM / 64, ROLE>;
    }();
    static bool attr_set = false;
    if (!attr_set) {
        hipError_t e =
            hipFuncSetAttribute((const void*)kernel, hipFuncAttributeMaxDynamicSharedMemorySize, LDS);
        if (e != hipSuccess) return e;
        attr_set = true;
    }
    const TileGeometry g = tile_geometry<BM, BN>(p, wsp, splits, ragged_tail);
    const SplitArgs& sa = g.sa;
    PB_LAUNCH(kernel, dim3(g.grid), dim3(64 * WGM * WGN), LDS, s, p, sa);
    const hipError_t e = hipGetLastError();
    if (e != hipSuccess || sa.splits == 1) return e;
    if constexpr (BM == BN) {
        if (sa.full_tiles > 0) {  // whole tiles, then the tail split
            const int64_t groups = (int64_t)sa.tail_tiles * (BM * BN / 4);
            PB_LAUNCH((tail_reduce_kernel<T, EPI, ROLE, BM, BN>), dim3((unsigned)((groups + 255) / 256)), dim3(256),
                      0, s, p, sa);
            return hipGetLastError();
        }
    }
    return finish_split<T, EPI, ROLE>(p, sa, s);
}

template <typename T, int EPI, int BM, int BN, int WGM, int WGN, int BKE, int S, int ROLE, bool FEW = false>
hipError_t launch_stream_cfg(const GemmParams& p, const GemmWorkspace& wsp, const WidePlan& w, hipStream_t s) {
    constexpr int LDS = S * (BM + BN) * BKE * 2;
    static bool attr_set = false;
    if (!attr_set) {
        hipError_t e = hipFuncSetAttribute((const void*)stream_kernel<T, EPI, BM, BN, WGM, WGN, BKE, S, ROLE, FEW>,
                                           hipFuncAttributeMaxDynamicSharedMemorySize, LDS);
        if (e != hipSuccess) return e;
        attr_set = true;
    }
    SplitArgs sa{};
    sa.splits = w.splits;
    sa.kt_split = w.kt;
    sa.ws = (float*)wsp.ws;
    const int kst = w.splits > 1 ? w.kt * BK / BKE : p.K1 / BKE;  // ring stages per launched range
    PB_LAUNCH((stream_kernel<T, EPI, BM, BN, WGM, WGN, BKE, S, ROLE, FEW>), dim3((unsigned)((p.M + BM - 1) / BM * (p.N / BN) * w.splits)),
              dim3(64 * WGM * WGN), LDS, s, p, sa, kst);
    const hipError_t e = hipGetLastError();
    if (e != hipSuccess || w.splits == 1) return e;
    return finish_split<T, EPI, ROLE>(p, sa, s);
}

template <typename T, int EPI, int ROLE>
hipError_t launch_wide(const GemmParams& p, const GemmWorkspace& wsp, const WidePlan& w, hipStream_t s) {
    if (w.kind == WIDE_RING) {
        if (w.bm == 256) return launch_cfg<T, EPI, 256, 256, 2, 4, ROLE, 2, true>(p, wsp, w.splits, 0, s);
        return launch_cfg<T, EPI, 192, 128, 2, 4, ROLE, 4>(p, wsp, w.splits, 0, s);
    }
    if (w.kind == WIDE_PINGPONG) {
        if (w.bm == 192) return launch_cfg<T, EPI, 192, 256, 2, 4, ROLE, 2>(p, wsp, w.splits, 0, s);
        return launch_cfg<T, EPI, 128, 256, 2, 4, ROLE, 2>(p, wsp, w.splits, 0, s);
    }
    if (w.bm == 128) return launch_stream_cfg<T, EPI, 128, 64, 4, 2, 128, 3, ROLE>(p, wsp, w, s);
    if (w.bm == 64) return launch_stream_cfg<T, EPI, 64, 64, 1, 4, 128, 4, ROLE>(p, wsp, w, s);
    if (p.M <= GEMV_MAX_ROWS) {
        if (w.bn == 32) return launch_stream_cfg<T, EPI, 32, 32, 1, 2, 128, 4, ROLE, true>(p, wsp, w, s);
        if (w.bk == 256) return launch_stream_cfg<T, EPI, 32, 64, 1, 4, 256, 3, ROLE, true>(p, wsp, w, s);
        return launch_stream_cfg<T, EPI, 32, 64, 1, 4, 128, 3, ROLE, true>(p, wsp, w, s);
    }
    if (w.bn == 32) return launch_stream_cfg<T, EPI, 32, 32, 1, 2, 128, 4, ROLE>(p, wsp, w, s);
    if (w.bk == 256) return launch_stream_cfg<T, EPI, 32, 64, 1, 4, 256, 3, ROLE>(p, wsp, w, s);
    return launch_stream_cfg<T, EPI, 32, 64, 1, 4, 128, 3, ROLE>(p, wsp, w, s);
}

template <typename T, int EPI>
hipError_t launch_gemv(const GemmParams& p, hipStream_t s);

// Few rows: the GEMV unless the streaming kernel is planned (never for the LoRA
// shrink, whose epilogue it does not know); more: tiles or the streaming kernel.
template <typename T, int EPI, int ROLE>
hipError_t launch_role(const GemmParams& p, const GemmWorkspace& wsp, hipStream_t s) {
    if (PB_GEMM_GEMV && p.M <= GEMV_MAX_ROWS) {
        if constexpr (ROLE != 4) {
            const WidePlan w = plan_few(p, wsp);
            if (w.kind != WIDE_NONE) return launch_wide<T, EPI, ROLE>(p, wsp, w, s);
        }
        return launch_gemv<T, EPI>(p, s);
    }
    const TilePlan tp = plan_for_role(ROLE, p, wsp);
    if constexpr (ROLE != 4) {
        const WidePlan w = plan_wide(p, wsp, tp);
        if (w.kind != WIDE_NONE) return launch_wide<T, EPI, ROLE>(p, wsp, w, s);
    }
    if constexpr (ROLE == 4) {
        return launch_cfg<T, EPI, 64, 64, 2, 2, 4, 4>(p, wsp, tp.splits, 0, s);
    } else {
        if (tp.tile == 256)
            return launch_cfg<T, EPI, 256, 256, 2, 4, ROLE, 2>(p, wsp, tp.splits, tp.ragged_tail, s);
        if (tp.tile == 128)
            return launch_cfg<T, EPI, 128, 128, 2, 4, ROLE, PB_GEMM_S128>(p, wsp, tp.splits, tp.ragged_tail, s);
        return launch_cfg<T, EPI, 64, 64, 2, 2, ROLE, PB_GEMM_S64>(p, wsp, tp.splits, tp.ragged_tail, s);
    }
}

template <typename T>
hipError_t launch_typed(int role, const GemmParams& p, const GemmWorkspace& wsp, hipStream_t s) {
    switch (role) {
        case 0: return launch_role<T, EPI_QKV, 0>(p, wsp, s);
        case 1: return launch_role<T, EPI_RESID, 1>(p, wsp, s);
        case 2: return launch_role<T, EPI_RELU, 2>(p, wsp, s);
        case 3: return launch_role<T, EPI_RESID, 3>(p, wsp, s);
        case 4: return launch_role<T, EPI_SHRINK, 4>(p, wsp, s);
        default: break;
    }
    return hipErrorInvalidValue;
}

// ---- few rows (decode steps): weight streaming without tiles ---------------
// A block owns four consecutive output features n0..n0+3; its four waves
// (eight for rows of 4096 or more) split K (and the LoRA K2 columns) into
// equal contiguous parts, so a matrix of N features is streamed by N / 4
// blocks and every CU has many waves' loads in flight (measured: four
// features per block beat eight or sixteen).  In a part, lane i takes elements 8i..8i+7 of each
// 512-element chunk (a feature's chunk is one contiguous 1 KiB read), two
// chunks per step, accumulating all MR token rows at once (MR <= GEMV_MAX_ROWS: the rows
// of X are re-read from cache by every wave).  Each wave sums its lanes, the
// parts are added in wave order through LDS, and the usual epilogue is
// applied to the four features of each token.
template <typename T, int MR, int RPB>
__device__ __forceinline__ void gemv_dot(const T* __restrict__ X, int64_t ldx, const T* __restrict__ W,
                                         int64_t ldw, int n0, int M, int kb, int ke, int lane,
                                         float (&acc)[RPB][MR]) {
    for (int c0 = kb + lane * 8; c0 < ke; c0 += 2 * 512) {
        u32x4 wr[2][RPB], xr[2][MR];
#pragma unroll
        for (int u = 0; u < 2; ++u) {
            const int c = min(c0 + u * 512, ke - 8);  // in bounds; the excess is not accumulated
#pragma unroll
            for (int r = 0; r < RPB; ++r) {
                const u32x4* src = (const u32x4*)(W + (int64_t)(n0 + r) * ldw + c);
#if PB_GEMV_NT
                wr[u][r] = __builtin_nontemporal_load(src);  // each weight is read once per step
#else
                wr[u][r] = *src;
#endif
            }
#pragma unroll
            for (int m = 0; m < MR; ++m) xr[u][m] = *(const u32x4*)(X + (int64_t)min(m, M - 1) * ldx + c);
        }
#pragma unroll
        for (int u = 0; u < 2; ++u) {
            if (c0 + u * 512 >= ke) break;
#pragma unroll
            for (int m = 0; m < MR; ++m) {
                T xe[8];
                __builtin_memcpy(xe, &xr[u][m], 16);
#pragma unroll
                for (int r = 0; r < RPB; ++r) {
                    T we[8];
                    __builtin_memcpy(we, &wr[u][r], 16);
#pragma unroll
                    for (int e = 0; e < 8; ++e) acc[r][m] += (float)we[e] * (float)xe[e];
                }
            }
        }
    }
}

// RPB output features per block (a multiple of 4: the epilogue writes four
// consecutive features of one token), K split over KW waves
template <typename T, int EPI, int MR, int RPB, int KW>
__global__ __launch_bounds__(64 * KW) void gemv_kernel(GemmParams p) {
    __shared__ float part[KW][RPB][MR];  // [wave][feature][token]
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const int n0 = blockIdx.x * RPB;
    float acc[RPB][MR];
#pragma unroll
    for (int r = 0; r < RPB; ++r)
#pragma unroll
        for (int m = 0; m < MR; ++m) acc[r][m] = 0.f;
    const int q1 = p.K1 / KW;  // K1, K2 are multiples of 64: the parts are multiples of 8
    gemv_dot<T, MR, RPB>((const T*)p.X, p.ldx, (const T*)p.W, p.ldw, n0, p.M, wave * q1, (wave + 1) * q1, lane,
                         acc);
    if (p.K2 > 0) {
        const int g = n0 / p.group;  // the group size is a multiple of RPB
        const int q2 = p.K2 / KW;
        if ((p.k2_mask >> g) & 1u)
            gemv_dot<T, MR, RPB>((const T*)p.X2 + (int64_t)g * p.x2_group_stride, p.ldx2, (const T*)p.W2, p.ldw2,
                                 n0, p.M, wave * q2, (wave + 1) * q2, lane, acc);
    }
#pragma unroll
    for (int r = 0; r < RPB; ++r)
#pragma unroll
        for (int m = 0; m < MR; ++m) acc[r][m] = wave_sum(acc[r][m]);
    if (lane == 0)
#pragma unroll
        for (int r = 0; r < RPB; ++r)
#pragma unroll
            for (int m = 0; m < MR; ++m) part[wave][r][m] = acc[r][m];
    __syncthreads();
    const int m = threadIdx.x % MR, f4 = threadIdx.x / MR;  // token, group of four features
    if (f4 < RPB / 4 && m < p.M) {
        f32x4 v;
#pragma unroll
        for (int r = 0; r < 4; ++r) {
            const int rr = 4 * f4 + r;
            float t = part[0][rr][m];
#pragma unroll
            for (int w = 1; w < KW; ++w) t += part[w][rr][m];
            v[r] = t;
        }
        epilogue4<T, EPI>(p, m, n0 + 4 * f4, v);
    }
}

template <typename T, int EPI>
hipError_t launch_gemv(const GemmParams& p, hipStream_t s) {
    constexpr int RPB = PB_GEMV_RPB;
    const dim3 grid(p.N / RPB);
#define PB_GEMV(MR, KW) PB_LAUNCH((gemv_kernel<T, EPI, MR, RPB, KW>), grid, dim3(64 * KW), 0, s, p)
#define PB_GEMV_M(KW)                \
    do {                             \
        if (p.M <= 1) PB_GEMV(1, KW);      \
        else if (p.M <= 2) PB_GEMV(2, KW); \
        else if (p.M <= 4) PB_GEMV(4, KW); \
        else PB_GEMV(8, KW);               \
    } while (0)
    // long rows: eight waves share the K range so each walks at most 1024
    // elements (measured: eight waves for short rows of few blocks is slower)
    if (PB_GEMV_KW8 && p.K1 >= 4096) PB_GEMV_M(8);
    else PB_GEMV_M(4);
#undef PB_GEMV_M
#undef PB_GEMV
    return hipGetLastError();
}

}  // namespace

hipError_t launch_gemm(int dtype, int role, int epi, const GemmParams& p, const GemmWorkspace& wsp,
                       hipStream_t s) {
    if (p.M <= 0 || p.N <= 0) return hipSuccess;
    if (p.N % 64 || p.K1 % BK || p.K2 % BK || p.K1 <= 0 || p.K2 < 0) return hipErrorInvalidValue;
    const int64_t lim = (int64_t)1 << 31;
    if ((int64_t)p.M * p.ldx >= lim || (int64_t)p.N * p.ldw >= lim ||
        (p.K2 > 0 && ((int64_t)p.M * p.ldx2 >= lim || (int64_t)p.N * p.ldw2 >= lim)))
        return hipErrorInvalidValue;
    const int expect[5] = {EPI_QKV, EPI_RESID, EPI_RELU, EPI_RESID, EPI_SHRINK};
    if (role < 0 || role > 4 || expect[role] != epi) return hipErrorInvalidValue;
    if (dtype == 1) return launch_typed<_Float16>(role, p, wsp, s);
    return launch_typed<__bf16>(role, p, wsp, s);
}

}  // namespace pb
