// Device code of the row kernels that also run beside a product in one launch (gemm_generic.hip): RMSNorm backward of any type,
// and the sums of the gain gradients' partial rows.  Work-groups of 256 threads.
#pragma once
#include "kernels.h"

namespace alch {

static constexpr int kNormBwdBlocks = 1024;
static constexpr int kNormMaxCols = 32;  // columns per thread: width <= 8192

__device__ __forceinline__ float wave_sum(float v) {
#pragma unroll
    for (int d = 32; d > 0; d >>= 1) v += __shfl_xor(v, d, 64);
    return v;
}

// RMSNorm backward with residual, the rows block, block + blocks, ...:
//   dX = resid + r*(g*dH) - X * r^3/width * sum(g*dH*X);   partial[block] = sum over the block's rows of dH*X*r
// A row is one chain of load, two sums, store: everything of a row is requested at once, and both sums meet in one exchange.
// kCols: columns per thread (all 32 of them for hidden 256 were 5 us of predicated code for 256 rows, one is 4).
template <typename T, int kCols>
__device__ __forceinline__ void rmsnorm_bwd_rows(const NormBwdRows& a, int block, int blocks, float* red /*[8]*/) {
    const T *dH = static_cast<const T*>(a.dH), *X = static_cast<const T*>(a.X), *g = static_cast<const T*>(a.g), *resid = static_cast<const T*>(a.resid);
    T *dX = static_cast<T*>(a.dX), *hn_out = static_cast<T*>(a.hn_out);
    const int width = a.width, wave = threadIdx.x >> 6;
    float dgp[kCols], gv[kCols];
#pragma unroll
    for (int i = 0; i < kCols; ++i) {
        dgp[i] = 0.f;
        const int c = threadIdx.x + 256 * i;
        gv[i] = c < width ? (float)g[c] : 0.f;
    }
    for (long long row = block; row < a.Trows; row += blocks) {
        float xv[kCols], dv[kCols], rv[kCols <= 4 ? kCols : 1];
        const bool keep = resid && !(a.resid_mask && a.resid_mask[row] == 0);
        float ss = 0.f, dot = 0.f;
#pragma unroll
        for (int i = 0; i < kCols; ++i) {
            const int c = threadIdx.x + 256 * i;
            xv[i] = c < width ? (float)X[row * width + c] : 0.f;
            dv[i] = c < width ? (float)dH[row * width + c] : 0.f;
            if constexpr (kCols <= 4) rv[i] = keep && c < width ? (float)resid[row * width + c] : 0.f;
        }
#pragma unroll
        for (int i = 0; i < kCols; ++i) {
            ss += xv[i] * xv[i];
            dot += gv[i] * dv[i] * xv[i];
        }
        ss = wave_sum(ss);
        dot = wave_sum(dot);
        __syncthreads();  // (the sums of the row before have been read)
        if ((threadIdx.x & 63) == 0) { red[wave] = ss; red[4 + wave] = dot; }
        __syncthreads();
        ss = red[0] + red[1] + red[2] + red[3];
        dot = red[4] + red[5] + red[6] + red[7];
        const float r = rsqrtf(ss / (float)width + a.eps);
        const float coef = r * r * r / (float)width * dot;
#pragma unroll
        for (int i = 0; i < kCols; ++i) {
            const int c = threadIdx.x + 256 * i;
            if (c < width) {
                float v = r * gv[i] * dv[i] - xv[i] * coef;
                if constexpr (kCols <= 4) v = keep ? v + rv[i] : v;
                else if (keep) v += (float)resid[row * width + c];
                dX[row * width + c] = (T)v;
                if (hn_out) hn_out[row * width + c] = (T)(xv[i] * r * gv[i]);  // the normalised row
                dgp[i] += dv[i] * xv[i] * r;
            }
        }
    }
    if (a.partial) {
#pragma unroll
        for (int i = 0; i < kCols; ++i) {
            const int c = threadIdx.x + 256 * i;
            if (c < width) a.partial[(long long)block * width + c] = dgp[i];
        }
    }
}

// dg[c] (+)= sum over the partial rows, 64 columns c0 .. by kWaves wavefronts: 16 groups of rows (rg, rg + 16, ...), their
// sums folded through LDS in order.  Several rows of every group are requested before the first is added: one after the other
// their latencies were the kernel's time.
template <typename T, int kWaves>
__device__ __forceinline__ void gain_sums(const GainSums& sums, int which, int c0, int width, int accumulate, float (*red)[64]) {
    const float* __restrict__ partial = sums.of[which].partial;
    T* __restrict__ dg = static_cast<T*>(sums.of[which].dg);
    const int nblk = sums.of[which].rows, lane = threadIdx.x & 63, wave = threadIdx.x >> 6, c = c0 + lane;
    constexpr int kGroups = 16 / kWaves, kBatch = 8 / (kGroups > 2 ? 2 : 1);
    float s[kGroups];
#pragma unroll
    for (int j = 0; j < kGroups; ++j) s[j] = 0.f;
    if (c < width)
        for (int b = 0; b < nblk; b += 16 * kBatch) {
            float v[kBatch][kGroups];
#pragma unroll
            for (int i = 0; i < kBatch; ++i)
#pragma unroll
                for (int j = 0; j < kGroups; ++j) {
                    const int row = b + 16 * i + wave + kWaves * j;
                    v[i][j] = row < nblk ? partial[(long long)row * width + c] : 0.f;
                }
#pragma unroll
            for (int i = 0; i < kBatch; ++i)
#pragma unroll
                for (int j = 0; j < kGroups; ++j) s[j] += v[i][j];
        }
#pragma unroll
    for (int j = 0; j < kGroups; ++j) red[wave + kWaves * j][lane] = s[j];
    __syncthreads();
    if (wave == 0 && c < width) {
        float t = 0.f;
#pragma unroll
        for (int i = 0; i < 16; ++i) t += red[i][lane];
        if (accumulate) t += (float)dg[c];
        dg[c] = (T)t;
    }
}

}  // namespace alch
