// LM head of several sequences on the matrix units: logits[b, v] = z[b] . E[v]
// with z held in fp32, E streamed once for up to 32 sequences.
//
// The dot-product head (misc.hip) is bound by its fp32 arithmetic from two
// sequences on (OPT-1.3B embedding, 206 MB: 36 us for one sequence, 217 for
// four) and takes at most four sequences per pass over E.  Here z enters the
// MFMA as three terms of dt whose sum carries every bit of its fp32 value, so
// nothing is rounded that the dot products kept:
//   bf16: z = h + l + m, 8 + 8 + 8 significant bits;
//   f16:  z = 2^e (h + 2^-11 l + 2^-22 m), |h| <= 1, 11 bits each (the power
//         of two keeps the terms inside f16's range whatever the row's scale;
//         elements below about 2^-25 of the row's largest lose bits, all of them
//         below 2^-46 of it).
// Products are exact in fp32 and accumulate in fp32, one accumulator per term,
// the first term's sums of 128 products added up with their rounding errors
// kept (two-sum): one long chain of fp32 additions would lose more than the
// dot products' short ones (relative error 4e-7 against 1.1e-7 at d 4096).
#include <algorithm>

#include "common.h"
#include "kernels.h"

namespace pb {

namespace {

constexpr float TERM_STEP = 2048.f;  // 2^11 between the f16 terms

template <typename T> struct TermScale;
template <> struct TermScale<__bf16> { static constexpr float step = 1.f; };
template <> struct TermScale<_Float16> { static constexpr float step = TERM_STEP; };

// zs[term][rows][d] and scale[rows] of z [B][d]; rows past B are zeros.  One
// block per row.
template <typename T>
__global__ __launch_bounds__(256) void split_terms_kernel(const float* __restrict__ z, int B, int rows, int d,
                                                         T* __restrict__ zs, float* __restrict__ scale) {
    __shared__ float red[4];
    const int r = blockIdx.x;
    const float* zr = z + (int64_t)min(r, B - 1) * d;
    float down = 1.f, up = 1.f;
    if (TermScale<T>::step != 1.f) {
        float mx = 0.f;
        for (int c = threadIdx.x; c < d; c += 256) mx = fmaxf(mx, fabsf(zr[c]));
        mx = wave_max(mx);
        if ((threadIdx.x & 63) == 0) red[threadIdx.x >> 6] = mx;
        __syncthreads();
        mx = fmaxf(fmaxf(red[0], red[1]), fmaxf(red[2], red[3]));
        int e = 0;
        if (mx > 0.f && mx < INFINITY) (void)frexpf(mx, &e);  // mx 2^-e in [0.5, 1)
        e = min(max(e, -120), 120);
        down = ldexpf(1.f, -e);
        up = ldexpf(1.f, e);
    }
    if (threadIdx.x == 0) scale[r] = up;
    const int64_t plane = (int64_t)rows * d;
    T* out = zs + (int64_t)r * d;
    for (int c = threadIdx.x; c < d; c += 256) {
        const float v = r < B ? zr[c] * down : 0.f;
        const T h = (T)v;
        // an infinite value is carried by its first term alone
        const float r1 = fabsf((float)h) < INFINITY ? (v - (float)h) * TermScale<T>::step : 0.f;
        const T l = (T)r1;
        const T m = (T)((r1 - (float)l) * TermScale<T>::step);
        out[c] = h;
        out[plane + c] = l;
        out[2 * plane + c] = m;
    }
}

__device__ __forceinline__ bool ranks_first(float v, int i, float bv, int bi) {
    return v > bv || (v == bv && i < bi);
}

// Block = 4 waves, 64 rows of E (16 per wave) x NG groups of 16 sequences; K
// stages of 128 elements arrive in an S-stage LDS ring in 256-byte row pieces
// (16-byte chunks XOR-permuted by the low row bits).  HBM-bound: the rows of
// E are the only cold data, the terms of z (3 x 16 NG rows) come from L2.
constexpr int LMM_ROWS = 64;

template <typename T, int NG, int S>
__global__ __launch_bounds__(256) void lm_head_mfma_kernel(const T* __restrict__ zs, const float* __restrict__ scale,
                                                          int nb, int b0, const T* __restrict__ E, int V, int d,
                                                          float* __restrict__ logits, float* __restrict__ pval,
                                                          int* __restrict__ pidx, int nblk) {
    typedef typename Mfma<T>::vec8 vec8;
    constexpr int NZ = 3 * NG;               // 16-column operand tiles of z
    constexpr int ZR = 16 * NZ;              // rows of z terms in a stage
    constexpr int RB = 256;                  // bytes per LDS row (128 elements)
    constexpr int STAGE = (ZR + LMM_ROWS) * RB;
    constexpr int NL = STAGE / 1024 / 4;     // copies per wave per stage
    static_assert(STAGE % 4096 == 0, "whole copies per wave");
    extern __shared__ __attribute__((aligned(16))) uint8_t smem[];
    const int lane = threadIdx.x & 63;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int lr = lane & 15, lg = lane >> 4;
    const int v0 = (int)blockIdx.x * LMM_ROWS;
    uint32_t off[NL];
#pragma unroll
    for (int j = 0; j < NL; ++j) {
        const int row = (wave + 4 * j) * 4 + (lane >> 4);
        const int ch = (lane & 15) ^ (row & 15);
        // z terms: plane row / (16 NG), row within it; [term][16 NG][d] is one array of ZR rows
        off[j] = row < ZR ? ((uint32_t)row * (uint32_t)d + ch * 8) * 2
                          : ((uint32_t)min(v0 + row - ZR, V - 1) * (uint32_t)d + ch * 8) * 2;
    }
    const uint32_t lds0 = (uint32_t)(uintptr_t)smem;
    auto issue = [&](int t, int stage) {
        const char* zk = (const char*)zs + (int64_t)t * RB;
        const char* ek = (const char*)E + (int64_t)t * RB;
#pragma unroll
        for (int j = 0; j < NL; ++j) {
            const int I = wave + 4 * j;
            dma16s(I * 4 < ZR ? zk : ek, off[j], lds0 + stage * STAGE + I * 1024);
        }
    };
    f32x4 acc[NZ];
#pragma unroll
    for (int j = 0; j < NZ; ++j) acc[j] = f32x4{0.f, 0.f, 0.f, 0.f};
    float sum[NG][4], low[NG][4];  // first term: running sums and their rounding errors
#pragma unroll
    for (int g = 0; g < NG; ++g)
#pragma unroll
        for (int r = 0; r < 4; ++r) sum[g][r] = low[g][r] = 0.f;
    auto compute = [&](int stage) {
        const uint8_t* s = smem + stage * STAGE;
#pragma unroll
        for (int g = 0; g < NG; ++g) acc[g] = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
        for (int kk = 0; kk < 4; ++kk) {
            const int ch = kk * 4 + lg;
            const int er = ZR + wave * 16 + lr;
            const vec8 a = as_vec8<T>(*(const u32x4*)(s + er * RB + ((ch ^ (er & 15)) << 4)));
#pragma unroll
            for (int j = 0; j < NZ; ++j) {
                const int row = j * 16 + lr;
                acc[j] = Mfma<T>::mma(a, as_vec8<T>(*(const u32x4*)(s + row * RB + ((ch ^ lr) << 4))), acc[j]);
            }
        }
#pragma unroll
        for (int g = 0; g < NG; ++g)
#pragma unroll
            for (int r = 0; r < 4; ++r) {
                const float y = acc[g][r], t = sum[g][r] + y, yy = t - sum[g][r];
                low[g][r] += (sum[g][r] - (t - yy)) + (y - yy);
                sum[g][r] = t;
            }
    };
    const int n = d / 128;
#pragma unroll
    for (int q = 0; q < S - 1; ++q)
        if (q < n) issue(q, q);
    int t = 0, st = 0;
    for (; t + S - 1 < n; ++t) {
        wait_vmcnt<(S - 2) * NL>();
        __syncthreads();
        issue(t + S - 1, st == 0 ? S - 1 : st - 1);
        compute(st);
        st = st == S - 1 ? 0 : st + 1;
    }
    for (; t < n; ++t) {
        wait_vmcnt<0>();
        __syncthreads();
        compute(st);
        st = st == S - 1 ? 0 : st + 1;
    }
    // lane (lr, lg): rows v0 + 16 wave + 4 lg + r of sequence 16 g + lr; per
    // block the (maximum, lowest index) of its rows for every sequence
    constexpr float inv = 1.f / TermScale<T>::step;
    __shared__ float sv[4][16 * NG];
    __shared__ int si[4][16 * NG];
    const int v = v0 + 16 * wave + 4 * lg;
#pragma unroll
    for (int g = 0; g < NG; ++g) {
        const int b = 16 * g + lr;
        const float up = scale[b];
        float best = -INFINITY;
        int bi = 0x7fffffff;
#pragma unroll
        for (int r = 0; r < 4; ++r) {
            const float rest = low[g][r] + inv * (acc[NG + g][r] + inv * acc[2 * NG + g][r]);
            // an overflowed sum stays as it is (its rounding error is a NaN)
            const float x = (fabsf(sum[g][r]) < INFINITY ? sum[g][r] + rest : sum[g][r]) * up;
            if (b < nb && v + r < V) {
                logits[(int64_t)(b0 + b) * V + v + r] = x;
                if (ranks_first(x, v + r, best, bi)) {
                    best = x;
                    bi = v + r;
                }
            }
        }
#pragma unroll
        for (int o = 16; o < 64; o <<= 1) {
            const float ov = __shfl_xor(best, o, 64);
            const int oi = __shfl_xor(bi, o, 64);
            if (ranks_first(ov, oi, best, bi)) {
                best = ov;
                bi = oi;
            }
        }
        if (lg == 0) {
            sv[wave][b] = best;
            si[wave][b] = bi;
        }
    }
    __syncthreads();
    const int b = threadIdx.x;
    if (b < nb) {
        float best = sv[0][b];
        int bi = si[0][b];
#pragma unroll
        for (int w = 1; w < 4; ++w)
            if (ranks_first(sv[w][b], si[w][b], best, bi)) {
                best = sv[w][b];
                bi = si[w][b];
            }
        pval[(int64_t)(b0 + b) * nblk + blockIdx.x] = best;
        pidx[(int64_t)(b0 + b) * nblk + blockIdx.x] = bi;
    }
}

template <typename T, int NG, int S>
hipError_t launch_group(const T* zs, const float* scale, int nb, int b0, const T* E, int V, int d, float* logits,
                        float* pval, int* pidx, int nblk, hipStream_t s) {
    constexpr int LDS = S * (48 * NG + LMM_ROWS) * 256;
    static bool attr_set = false;
    if (!attr_set) {
        const hipError_t e = hipFuncSetAttribute((const void*)lm_head_mfma_kernel<T, NG, S>,
                                                 hipFuncAttributeMaxDynamicSharedMemorySize, LDS);
        if (e != hipSuccess) return e;
        attr_set = true;
    }
    PB_LAUNCH((lm_head_mfma_kernel<T, NG, S>), dim3(nblk), dim3(256), LDS, s, zs, scale, nb, b0, E, V, d, logits,
              pval, pidx, nblk);
    return hipGetLastError();
}

template <typename T>
hipError_t launch_typed(const float* z, int B, const T* E, int V, int d, float* logits, float* pval, int* pidx,
                        void* scratch, hipStream_t s) {
    const int nblk = lm_head_mfma_blocks(V);
    T* zs = (T*)scratch;
    for (int b0 = 0; b0 < B; b0 += 32) {
        const int nb = std::min(32, B - b0), rows = nb > 16 ? 32 : 16;
        float* scale = (float*)(zs + (int64_t)3 * rows * d);
        PB_LAUNCH(split_terms_kernel<T>, dim3(rows), dim3(256), 0, s, z + (int64_t)b0 * d, nb, rows, d, zs, scale);
        hipError_t e = hipGetLastError();
        if (e != hipSuccess) return e;
        e = rows == 16 ? launch_group<T, 1, 2>(zs, scale, nb, b0, E, V, d, logits, pval, pidx, nblk, s)
                       : launch_group<T, 2, 3>(zs, scale, nb, b0, E, V, d, logits, pval, pidx, nblk, s);
        if (e != hipSuccess) return e;
    }
    return hipSuccess;
}

}  // namespace

// One pass of the dot-product head serves 4, 2 or 1 sequences (d <= 4096, <=
// 10240, above) and its time grows with them where the arithmetic bounds it
// (one chunk per thread: d <= 2048); a pass here costs about one and a half
// of its single-sequence passes for up to 16 sequences.  Measured (vocab
// 50272): d 2048, 2 sequences 55 us against 72; d 4096, 2: 105 against 68,
// 3: 107 against 137, 12: 107 against 389; d 9216, 2: 209 against 141, 3: 209
// against 279.  Narrow rows stay with the dot products, whose error is smaller
// there (f16, relative: d 128 7.4-7.9e-8 against 7.6-9.3e-8, d 256 7.7-8.7e-8
// against 7.7-9.0e-8; d 512 8.1-8.9e-8 against 7.7-8.6e-8, d 4096 1.0-1.1e-7 against
// 7.7-8.9e-8).
bool lm_head_use_mfma(int B, int V, int d) {
    if (d < 512 || d % 128 || (int64_t)V * d >= ((int64_t)1 << 31)) return false;
    return B >= 3 || (B == 2 && (d <= 2048 || d > 10240));
}

int lm_head_mfma_blocks(int V) { return (V + LMM_ROWS - 1) / LMM_ROWS; }

size_t lm_head_mfma_scratch(int d) { return (size_t)3 * 32 * d * 2 + 32 * 4; }

hipError_t launch_lm_head_mfma(int dtype, const float* z, int B, const void* E, int V, int d, float* logits,
                               float* pval, int* pidx, void* scratch, hipStream_t s) {
    if (B <= 0 || V <= 0) return hipSuccess;
    // copy offsets are 32-bit bytes into E
    if (d % 128 || (int64_t)V * d >= ((int64_t)1 << 31)) return hipErrorInvalidValue;
    return dtype == 1
               ? launch_typed<_Float16>(z, B, (const _Float16*)E, V, d, logits, pval, pidx, scratch, s)
               : launch_typed<__bf16>(z, B, (const __bf16*)E, V, d, logits, pval, pidx, scratch, s);
}

}  // namespace pb
