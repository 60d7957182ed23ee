// Low-rank adapter (LoRA) kernels: the rank-r products around a projection y = x W^T + s (x A^T) B^T
// (Section 3, assumption A1 and Section 6 of the paper: parameter-efficient fine-tuning, rank 8).
//
// With r = 8 every one of these products streams a [T, width] activation once and does 8 multiply-adds per element: HBM-bound where
// the matrix cores do them ("down" in bf16 here, "up" in bf16 and both in one pass in lora_pass.hip), near it on the vector ALU
// (fp32, other widths, more partial sums than the scratch of a shared pass holds):
//   down:  Y[T, r]  = alpha * X[T, K] * S         (S = A^T or B; "t1 = x A^T", "t2 = dy B")
//   up:    C[r, N]  = alpha * S[T, r]^T * X[T, N] (adapter gradients dA = t2^T x, dB^T = t1^T dy)
// Storage type T is float or bf16, arithmetic fp32, sums over tokens in a fixed order (deterministic).
#include <algorithm>

#include "kernels.h"

namespace alch {

typedef __attribute__((ext_vector_type(8))) __bf16 bf16x8_l;
typedef __attribute__((ext_vector_type(4))) float f32x4_l;

__device__ __forceinline__ void load8(const __bf16* p, float (&v)[8]) {
    const bf16x8_l t = *reinterpret_cast<const bf16x8_l*>(p);
#pragma unroll
    for (int e = 0; e < 8; ++e) v[e] = (float)t[e];
}
__device__ __forceinline__ void load8(const float* p, float (&v)[8]) {
    const f32x4_l a = *reinterpret_cast<const f32x4_l*>(p), b = *reinterpret_cast<const f32x4_l*>(p + 4);
#pragma unroll
    for (int e = 0; e < 4; ++e) { v[e] = a[e]; v[4 + e] = b[e]; }
}

// ---- down, vector-ALU version (any dtype): 16 rows per work-group (4 per wavefront), 8 output columns
// per blockIdx.y.  S(k, j) = S[j*lds + k] (an [r, K] matrix: A, or B transposed).  Columns j >= r of the
// slot_cols-wide output slot are written as zeros (the slot is later read as a zero-padded operand of a
// matrix-core product).
template <typename T>
__global__ __launch_bounds__(256) void k_lora_down(const T* __restrict__ X, long long ldx, int Trows, int K,
                                                   const T* __restrict__ S, long long lds, int r, float alpha,
                                                   T* __restrict__ Y, long long ldy) {
    __shared__ float red[4][64][33];
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const int j0 = blockIdx.y * 8;
    const long long t0 = (long long)blockIdx.x * 16 + wave * 4;
    if (j0 >= r) {
        if (lane < 32 && t0 + (lane >> 3) < Trows) Y[(t0 + (lane >> 3)) * ldy + j0 + (lane & 7)] = (T)0.f;
        return;
    }
    float acc[4][8];
#pragma unroll
    for (int i = 0; i < 4; ++i)
#pragma unroll
        for (int j = 0; j < 8; ++j) acc[i][j] = 0.f;
    for (int k0 = lane * 8; k0 < K; k0 += 512) {
        float x[4][8];
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            if (t0 + i < Trows) {
                load8(X + (t0 + i) * ldx + k0, x[i]);
            } else {
#pragma unroll
                for (int e = 0; e < 8; ++e) x[i][e] = 0.f;
            }
        }
#pragma unroll
        for (int q = 0; q < 8; ++q) {
            float s[8];
            load8(S + (long long)(j0 + q) * lds + k0, s);
#pragma unroll
            for (int i = 0; i < 4; ++i)
#pragma unroll
                for (int e = 0; e < 8; ++e) acc[i][q] = __builtin_fmaf(x[i][e], s[e], acc[i][q]);
        }
    }
#pragma unroll
    for (int i = 0; i < 4; ++i)
#pragma unroll
        for (int j = 0; j < 8; ++j) red[wave][lane][i * 8 + j] = acc[i][j];
    __syncthreads();
    if (lane < 32) {
        float s = 0.f;
        for (int l = 0; l < 64; ++l) s += red[wave][l][lane];
        const long long t = t0 + (lane >> 3);
        if (t < Trows) Y[t * ldy + j0 + (lane & 7)] = (T)(alpha * s);
    }
}

// ---- down on the matrix cores (bf16, K a multiple of 64): eight multiply-adds per streamed element are
// too many for the vector ALU to keep up with HBM, so the [32 rows x 16 k] x [16 k x 32 columns] MFMA does
// them.  A matrix-instruction operand wants one row per lane (a wave-wide load of that shape touches 64 cache
// lines for 1 KB); the rows are fetched as whole 128-byte lines straight into LDS instead (buffer_load ... lds,
// eight lanes per line) and the operands are read from there, which also lets several S share one pass over X.
//
// A problem = one streamed X [Trows, K] and up to four groups of eight columns of the output, each with its
// own [rows <= 8, K] matrix S and its own destination (problems that share X are merged by the host: the t1
// of q, k, v, or of gate and up, cost one pass).  A work-group owns kRows rows (32, fewer in a short batch); its kWaves
// wavefronts split K in chunks of 64 and fold their sums through LDS in a fixed order.  Every wavefront runs a private ring of
// stages [X kRows rows x 128 B | S 8 rows x 128 B per group]: no barrier inside the loop.  16-byte piece c of
// row r sits at position c ^ ((r >> 1) & 7) of the row, which makes the operand reads conflict-free.
typedef __attribute__((ext_vector_type(16))) float f32x16_l;
typedef __attribute__((ext_vector_type(4))) int i32x4_l;
struct LoraDownGroup {
    const __bf16* S; long long lds; int rows;  // rows = 0: no such group
    __bf16* Y;                                 // first of the group's eight output columns
};
static constexpr int kDownProblems = 6;
struct LoraDownProblem {
    const __bf16* X; long long ldx; int K, ngroups;
    LoraDownGroup g[kDownGroups];
};
struct LoraDownParams {
    LoraDownProblem pr[kDownProblems];
    __bf16* slot[3]; int slot_r[3]; int nslots;  // output slots: columns slot_r .. slot_cols-1 are zero-filled
    int Trows; long long ldy; float alpha; int slot_cols;
    const int* rows_dev;
};
template <int kG, int kRows, int kWaves> struct DownCfg {
    static constexpr int kStageBytes = kRows * 128 + kG * 1024;
    static constexpr int kStages = 144 * 1024 / kWaves / kStageBytes < 2 ? 2 : 144 * 1024 / kWaves / kStageBytes;  // 36 KB per wavefront of four
};
// (s_nop: a load into LDS takes one wait state after a scalar write of m0, which the compiler does not see to in assembly)
__device__ __forceinline__ void lora_dma16(i32x4_l r, uint32_t lds_addr, uint32_t voff) {
    asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tbuffer_load_dwordx4 %1, %2, 0 offen lds" ::"s"(lds_addr), "v"(voff), "s"(r)
                 : "memory", "m0");
}
__device__ __forceinline__ i32x4_l lora_rsrc(const void* p, long long bytes) {
    const uint32_t n = bytes <= 0 ? 0u : (bytes > 0x7fffffffLL ? 0x7fffffffu : (uint32_t)bytes);
    const uint64_t a = reinterpret_cast<uint64_t>(p);
    i32x4_l r;
    r[0] = __builtin_amdgcn_readfirstlane((int)(uint32_t)a);
    r[1] = __builtin_amdgcn_readfirstlane((int)((uint32_t)(a >> 32) & 0xffffu));
    r[2] = __builtin_amdgcn_readfirstlane((int)n);
    r[3] = 0x00020000;
    return r;
}
template <int kG, int kRows, int kWaves>
__global__ __launch_bounds__(kWaves * 64) void k_lora_down_mfma(LoraDownParams p) {
    constexpr int kStageBytes = DownCfg<kG, kRows, kWaves>::kStageBytes, kStages = DownCfg<kG, kRows, kWaves>::kStages;
    constexpr int kLoadsX = kRows / 8, kElems = kRows / 2;  // (accumulator elements whose row is one of kRows)
    constexpr uint32_t kS = kRows * 128;  // S behind X in a stage
    __shared__ __attribute__((aligned(1024))) char smem[kWaves * kStages * kStageBytes];
    float (*red)[64][kElems + 1] = reinterpret_cast<float (*)[64][kElems + 1]>(smem);  // the stages have been read by then
    static_assert(sizeof(float) * (kWaves - 1) * 64 * (kElems + 1) <= sizeof(smem), "");
    const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int c = lane & 31, kh = lane >> 5;
    const long long t0 = (long long)blockIdx.x * kRows;
    const int Trows = p.rows_dev ? min(__builtin_amdgcn_readfirstlane(*p.rows_dev), p.Trows) : p.Trows;
    if (t0 >= Trows) return;
    const int rows_valid = (int)(Trows - t0 < kRows ? Trows - t0 : kRows);
    if (blockIdx.y == 0) {  // the columns past the rank of every output slot
        const int pieces = p.slot_cols >> 3;
        const bf16x8_l z = {(__bf16)0.f, (__bf16)0.f, (__bf16)0.f, (__bf16)0.f, (__bf16)0.f, (__bf16)0.f, (__bf16)0.f, (__bf16)0.f};
        for (int sl = 0; sl < p.nslots; ++sl)
            for (int idx = threadIdx.x; idx < kRows * pieces; idx += kWaves * 64) {
                const int row = idx / pieces, piece = idx % pieces;
                if (row < rows_valid && piece * 8 >= p.slot_r[sl])
                    *reinterpret_cast<bf16x8_l*>(p.slot[sl] + (t0 + row) * p.ldy + piece * 8) = z;
            }
    }
    const LoraDownProblem& pb = p.pr[blockIdx.y];
    if (pb.ngroups == 0) return;
    const int nc = pb.K >> 6;
    const int c_lo = wave * nc / kWaves, n = (wave + 1) * nc / kWaves - c_lo;  // this wavefront's chunks of 64 k
    char* wbase = smem + wave * (kStages * kStageBytes);
    const uint32_t lds_w = (uint32_t)(uintptr_t)((__attribute__((address_space(3))) void*)wbase);
    // per-lane source offsets of the loads: lane -> (row 8j + lane/8, piece (lane & 7) ^ swizzle of the LDS row)
    const int row8 = lane >> 3, q = lane & 7;
    uint32_t voff_x[kLoadsX], voff_s[kG];
#pragma unroll
    for (int j = 0; j < kLoadsX; ++j) {
        const int row = 8 * j + row8;
        voff_x[j] = (uint32_t)(row * pb.ldx * 2 + ((q ^ ((row >> 1) & 7)) << 4));
    }
#pragma unroll
    for (int g = 0; g < kG; ++g) voff_s[g] = (uint32_t)(row8 * pb.g[g].lds * 2 + ((q ^ (((8 * g + row8) >> 1) & 7)) << 4));
    const __bf16* xb = pb.X + t0 * pb.ldx + (long long)c_lo * 64;
    const long long x_bytes = rows_valid > 0 ? ((long long)(rows_valid - 1) * pb.ldx + 64) * 2 : 0;
    auto issue = [&](int i) {
        const uint32_t st = lds_w + (uint32_t)(i % kStages) * kStageBytes;
        const bool live = i < n;
        const i32x4_l rx = lora_rsrc(xb + (long long)i * 64, live ? x_bytes : 0);
#pragma unroll
        for (int j = 0; j < kLoadsX; ++j) lora_dma16(rx, st + (uint32_t)j * 1024u, voff_x[j]);
#pragma unroll
        for (int g = 0; g < kG; ++g) {
            const LoraDownGroup& gr = pb.g[g];
            const i32x4_l rs = lora_rsrc(gr.S + (long long)(c_lo + i) * 64,
                                         live && gr.rows > 0 ? ((long long)(gr.rows - 1) * gr.lds + 64) * 2 : 0);
            lora_dma16(rs, st + kS + (uint32_t)g * 1024u, voff_s[g]);
        }
    };
    f32x16_l acc;
#pragma unroll
    for (int e = 0; e < 16; ++e) acc[e] = 0.f;
    // operand read offsets inside a stage: X row c, S row c (rows and columns past those of the stage read one that
    // exists; their results are never stored)
    const int cs = c < 8 * kG ? c : (c & 7), cx = c & (kRows - 1);
    uint32_t off_a[4], off_b[4];
#pragma unroll
    for (int u = 0; u < 4; ++u) {
        off_a[u] = (uint32_t)(cx * 128 + (((2 * u + kh) ^ ((cx >> 1) & 7)) << 4));
        off_b[u] = (uint32_t)(kS + cs * 128 + (((2 * u + kh) ^ ((cs >> 1) & 7)) << 4));
    }
#pragma unroll
    for (int s = 0; s < kStages - 1; ++s) issue(s);
    for (int i = 0; i < n; ++i) {
        issue(i + kStages - 1);
        asm volatile("s_waitcnt vmcnt(%0)" ::"n"((kStages - 1) * (kLoadsX + kG)) : "memory");
        const char* st = wbase + (i % kStages) * kStageBytes;
        bf16x8_l a[4], b[4];
#pragma unroll
        for (int u = 0; u < 4; ++u) {
            a[u] = *reinterpret_cast<const bf16x8_l*>(st + off_a[u]);
            b[u] = *reinterpret_cast<const bf16x8_l*>(st + off_b[u]);
        }
#pragma unroll
        for (int u = 0; u < 4; ++u) acc = __builtin_amdgcn_mfma_f32_32x32x16_bf16(a[u], b[u], acc, 0, 0, 0);
        // this stage has been read before the next loads overwrite it (the products have waited for it, but may move)
        asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
    }
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
    __syncthreads();
    if (wave > 0) {
#pragma unroll
        for (int e = 0; e < kElems; ++e) red[wave - 1][lane][e] = acc[e];
    }
    __syncthreads();
    if (wave == 0) {
        __bf16* yp = nullptr;
        int yrows = 0;
#pragma unroll
        for (int g = 0; g < kG; ++g)
            if ((c >> 3) == g && g < pb.ngroups) { yp = pb.g[g].Y; yrows = pb.g[g].rows; }
        // accumulator element e: row 8*(e>>2) + 4*kh + (e&3), column c
#pragma unroll
        for (int e = 0; e < kElems; ++e) {
            float v = acc[e];
#pragma unroll
            for (int w = 0; w < kWaves - 1; ++w) v += red[w][lane][e];
            const int row = 8 * (e >> 2) + 4 * kh + (e & 3);
            if (row < rows_valid && (c & 7) < yrows) yp[(t0 + row) * p.ldy + (c & 7)] = (__bf16)(p.alpha * v);
        }
    }
}

// ---- up, pass 1: partial[jc][split][j][n] = sum over the rows of the split of S[t, 8*jc + j] * X[t, n] ----
// work-group = 512 columns (8 per lane) x one row split; its four wavefronts interleave the rows and
// fold their sums through LDS in a fixed order.
typedef __attribute__((ext_vector_type(2))) __bf16 bf16x2_l;
typedef __attribute__((ext_vector_type(4))) unsigned int u32x4_l;

// One token (float storage) or one pair of tokens (bf16 storage) of the rank-8 outer-product sum
// acc[j][c] += S[t, j] * X[t, c].  For bf16 the two tokens of a pair are interleaved into (t, t+1)
// halfword pairs (one byte-permute per pair) and each 2-term sum is one packed dot-product instruction
// accumulating in fp32: half the vector instructions of convert + multiply-add per element.
__device__ __forceinline__ void up_step(const float* xr, const float* sr, long long, long long, bool, float (&acc)[8][8]) {
    float x[8], s[8];
    load8(xr, x);
    load8(sr, s);
#pragma unroll
    for (int j = 0; j < 8; ++j)
#pragma unroll
        for (int c = 0; c < 8; ++c) acc[j][c] = __builtin_fmaf(s[j], x[c], acc[j][c]);
}
__device__ __forceinline__ void up_step(const __bf16* xr, const __bf16* sr, long long ldx, long long lds, bool second,
                                        float (&acc)[8][8]) {
    const u32x4_l zero = {0u, 0u, 0u, 0u};
    const u32x4_l x0 = *reinterpret_cast<const u32x4_l*>(xr), s0 = *reinterpret_cast<const u32x4_l*>(sr);
    const u32x4_l x1 = second ? *reinterpret_cast<const u32x4_l*>(xr + ldx) : zero;
    const u32x4_l s1 = second ? *reinterpret_cast<const u32x4_l*>(sr + lds) : zero;
    unsigned xp[8], sp[8];
#pragma unroll
    for (int m = 0; m < 4; ++m) {
        xp[2 * m] = __builtin_amdgcn_perm(x1[m], x0[m], 0x05040100u);      // (x[t][2m],   x[t+1][2m])
        xp[2 * m + 1] = __builtin_amdgcn_perm(x1[m], x0[m], 0x07060302u);  // (x[t][2m+1], x[t+1][2m+1])
        sp[2 * m] = __builtin_amdgcn_perm(s1[m], s0[m], 0x05040100u);
        sp[2 * m + 1] = __builtin_amdgcn_perm(s1[m], s0[m], 0x07060302u);
    }
#pragma unroll
    for (int j = 0; j < 8; ++j)
#pragma unroll
        for (int c = 0; c < 8; ++c)
            acc[j][c] = __builtin_amdgcn_fdot2_f32_bf16(__builtin_bit_cast(bf16x2_l, sp[j]), __builtin_bit_cast(bf16x2_l, xp[c]),
                                                        acc[j][c], false);
}
template <typename T> struct UpStep { static constexpr int kTokens = 1; };
template <> struct UpStep<__bf16> { static constexpr int kTokens = 2; };

// blockIdx.z = (job - first) * (r / 8) + chunk of eight rank rows; work-groups beyond a job's column slabs or row splits exit
template <typename T>
__global__ __launch_bounds__(256) void k_lora_up_partial(LoraUpParams p, int first) {
    __shared__ float red[3][64][65];
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const int chunks = p.r >> 3;
    const LoraUpJob jb = p.job[first + blockIdx.z / chunks];
    const int jc = blockIdx.z % chunks;
    const int N = jb.N, nsplit = jb.nsplit, split = blockIdx.y;
    if ((int)blockIdx.x * 512 >= N || split >= nsplit) return;
    const T* __restrict__ S = static_cast<const T*>(jb.S);
    const T* __restrict__ X = static_cast<const T*>(jb.X);
    const long long lds = jb.lds, ldx = jb.ldx;
    const int Trows = p.Trows, rows_per_split = jb.rows_per_split;
    float* __restrict__ partial = p.scratch + jb.scratch_off;
    const int n0 = blockIdx.x * 512 + lane * 8;
    const long long r0 = (long long)split * rows_per_split;
    const long long r1 = r0 + rows_per_split < Trows ? r0 + rows_per_split : Trows;
    constexpr int kTok = UpStep<T>::kTokens;
    float acc[8][8];
#pragma unroll
    for (int j = 0; j < 8; ++j)
#pragma unroll
        for (int c = 0; c < 8; ++c) acc[j][c] = 0.f;
    if (n0 < N) {
#pragma unroll 2
        for (long long t = r0 + wave * kTok; t < r1; t += 4 * kTok)
            up_step(X + t * ldx + n0, S + t * lds + jc * 8, ldx, lds, t + 1 < r1, acc);
    }
    if (wave > 0) {
#pragma unroll
        for (int j = 0; j < 8; ++j)
#pragma unroll
            for (int c = 0; c < 8; ++c) red[wave - 1][lane][j * 8 + c] = acc[j][c];
    }
    __syncthreads();
    if (wave == 0 && n0 < N) {
        float* out = partial + ((long long)(jc * nsplit + split) * 8) * N + n0;
#pragma unroll
        for (int j = 0; j < 8; ++j) {
            f32x4_l lo, hi;
#pragma unroll
            for (int c = 0; c < 8; ++c) {
                const float v = ((acc[j][c] + red[0][lane][j * 8 + c]) + red[1][lane][j * 8 + c]) + red[2][lane][j * 8 + c];
                if (c < 4) lo[c] = v; else hi[c - 4] = v;
            }
            *reinterpret_cast<f32x4_l*>(out + (long long)j * N) = lo;
            *reinterpret_cast<f32x4_l*>(out + (long long)j * N + 4) = hi;
        }
    }
}

// ---- up, pass 2: C(j, n) (+)= alpha * sum over splits, written as C[j*ldc + n] or transposed C[n*ldc + j].
// Eight lanes share four neighbouring outputs: lane q adds splits q, q+8, ... and the eight sums are folded in a fixed order.
// The sums of all adapters of a layer are one launch (with one for every group of projections, of single outputs, a layer
// of 900 tokens spent 32 us in four of them).
static constexpr int kSumsPerGroup = 128;  // outputs of a work-group
template <typename T>
__global__ __launch_bounds__(256) void k_lora_up_finish(LoraUpParams p) {
    int at = 0;
    for (int i = 1; i < p.n_jobs; ++i)
        if ((int)blockIdx.x >= p.job[i].first_group) at = i;
    const LoraUpJob jb = p.job[at];
    const int N = jb.N, nsplit = jb.nsplit;
    const int live_splits = jb.rows_dev ? min((max(*jb.rows_dev, 0) + jb.rows_dev_split - 1) / jb.rows_dev_split, nsplit) : nsplit;
    const long long idx = (long long)((int)blockIdx.x - jb.first_group) * kSumsPerGroup + (threadIdx.x >> 3) * 4;
    const int q = threadIdx.x & 7;
    const bool live = idx < (long long)N * p.r;
    // consecutive outputs walk n: the partial sums are read in order (C itself is small; N is a multiple of 8)
    const int jj = !live ? 0 : (int)(idx / N);
    const int n = !live ? 0 : (int)(idx % N);
    const float* src = p.scratch + jb.scratch_off + ((long long)(jj >> 3) * nsplit * 8 + (jj & 7)) * N + n;
    f32x4_l s = {0.f, 0.f, 0.f, 0.f};
    if (live)
        for (int k = q; k < live_splits; k += 8) s += *reinterpret_cast<const f32x4_l*>(src + (long long)k * 8 * N);
#pragma unroll
    for (int d = 1; d < 8; d <<= 1)
#pragma unroll
        for (int e = 0; e < 4; ++e) s[e] += __shfl_xor(s[e], d, 64);
    if (live && q < 4) {  // lane e writes output e
        const float v = q == 0 ? s[0] : q == 1 ? s[1] : q == 2 ? s[2] : s[3];
        T* C = static_cast<T*>(jb.C);
        T* dst = jb.transposed ? C + (long long)(n + q) * jb.ldc + jj : C + (long long)jj * jb.ldc + n + q;
        float o = v * p.alpha;
        if (p.accumulate) o += (float)*dst;
        *dst = (T)o;
    }
}

// ---- operand preparation, all adapters of a layer in one launch: job z writes dst [rows_out, cols] with
// dst[i, c] = i < r ? (transpose ? src[c*r + i] : src[i*cols + c]) : 0   (src null: all zeros).
// Used for the zero-padded stacks of the A matrices (extra operand of the data-gradient products) and for
// B^T (so that both rank-r "down" products read an [r, K] matrix).
template <typename T>
__global__ __launch_bounds__(256) void k_lora_prep(LoraPrepParams p) {
    const LoraPrepJob jb = p.job[blockIdx.y];
    const T* src = static_cast<const T*>(jb.src);
    T* dst = static_cast<T*>(jb.dst);
    const long long first = (long long)blockIdx.x * 256 + threadIdx.x, step = (long long)gridDim.x * 256;
    // eight elements a thread (14 jobs of the 8B shape: 6.8 us one by one); dst lies in the workspace, aligned
    struct alignas(8 * sizeof(T)) Eight { T v[8]; };
    if (jb.cols % 8 == 0 && jb.r % 8 == 0 && reinterpret_cast<uintptr_t>(src) % sizeof(Eight) == 0) {
        const long long n8 = jb.transpose ? (long long)jb.cols * (jb.r / 8) : (long long)jb.rows_out * jb.cols / 8;
        for (long long i = first; i < n8; i += step) {
            Eight e;
#pragma unroll
            for (int k = 0; k < 8; ++k) e.v[k] = (T)0.f;
            if (jb.transpose) {  // rows_out = r: eight rows of column c
                const int c = (int)(i % jb.cols), row = (int)(i / jb.cols) * 8;
                if (src) e = *reinterpret_cast<const Eight*>(src + (long long)c * jb.r + row);
#pragma unroll
                for (int k = 0; k < 8; ++k) dst[(long long)(row + k) * jb.cols + c] = e.v[k];
            } else {
                if (src && i * 8 < (long long)jb.r * jb.cols) e = *reinterpret_cast<const Eight*>(src + i * 8);
                *reinterpret_cast<Eight*>(dst + i * 8) = e;
            }
        }
        return;
    }
    const long long n = (long long)jb.rows_out * jb.cols;
    for (long long idx = first; idx < n; idx += step) {
        const int i = (int)(idx / jb.cols), c = (int)(idx % jb.cols);
        T v = (T)0.f;
        if (src && i < jb.r) v = jb.transpose ? src[(long long)c * jb.r + i] : src[idx];
        dst[idx] = v;
    }
}

static int up_splits(int Trows, int N) {
    const int slabs = ceil_div(N, 512);
    int n = ceil_div(256, slabs);
    if (n < 4) n = 4;
    if (n > kLoraMaxSplits) n = kLoraMaxSplits;
    // At least 64 rows to a split: the partial sums of shorter ones are more to write and read than the activations (layer of
    // the 8B shape, us in all pieces of the gradients with splits of any length / 32 / 64 rows: 200 tokens 57 / 39 / 39, 900
    // tokens 82 / 74 / 68, 1700 tokens 106 / 104 / 99).
    if (n > ceil_div(Trows, 64)) n = Trows > 0 ? ceil_div(Trows, 64) : 1;
    return n;
}

size_t lora_up_scratch_bytes(int rank, int n_sum) {
    return (size_t)ceil_div(rank, 8) * kLoraMaxSplits * 8 * (size_t)n_sum * sizeof(float);
}

template <typename T>
static int lora_down_valu(const LoraDown& j, int Trows, float alpha, long long ldy, int slot_cols, hipStream_t stream) {
    const dim3 grid(ceil_div(Trows, 16), slot_cols / 8);
    k_lora_down<T><<<grid, 256, 0, stream>>>((const T*)j.X, j.ldx, Trows, j.K, (const T*)j.S, j.lds, j.r, alpha, (T*)j.Y, ldy);
    return ALCH_OK;
}

template <int kRows, int kWaves>
static void launch_down(const LoraDownParams& p, int groups, int Trows, int problems, hipStream_t stream) {
    const dim3 grid(ceil_div(Trows, kRows), std::max(problems, 1));
    if (groups <= 1) k_lora_down_mfma<1, kRows, kWaves><<<grid, kWaves * 64, 0, stream>>>(p);
    else if (groups == 2) k_lora_down_mfma<2, kRows, kWaves><<<grid, kWaves * 64, 0, stream>>>(p);
    else if (groups == 3) k_lora_down_mfma<3, kRows, kWaves><<<grid, kWaves * 64, 0, stream>>>(p);
    else k_lora_down_mfma<4, kRows, kWaves><<<grid, kWaves * 64, 0, stream>>>(p);
}

// Few rows leave compute units without a work-group, and a wavefront alone on its SIMD takes 0.37 us for a chunk (load,
// read, four dependent products, one after the other): work-groups of fewer rows and more wavefronts, as long as
// each finds a compute unit (the sums of a row are then folded from 8 or 16 parts of K instead of 4).  8B shape, us a launch of
// 32 rows by 4 / 16 rows by 8 / 8 rows by 16 wavefronts: 200 tokens, K 14336 21.5 / 13.6 / 10.2, K 4096 10.3 / 7.4 / 6.2; 900 tokens, two of K 14336 23.4 / 17.9 / 14.8; 2000
// tokens, one 29.2 / 22.4 / 17.3 and two (500 work-groups of 8 rows) 34.7 / 25.2 / 30.6; 5120 tokens 40.9 / 46.3 / 44.0.
int lora_down_parts(int Trows, int problems, int n_cu) {
    return ceil_div(Trows, 8) * problems <= n_cu ? 16 : ceil_div(Trows, 16) * problems <= n_cu ? 8 : 4;
}

int launch_lora_down(alch_dtype dt, const LoraDown* jobs, int n_jobs, int Trows, float alpha, long long ldy,
                     int slot_cols, hipStream_t stream, int as_problems, const int* rows_dev) {
    if (n_jobs < 1 || n_jobs > 3) return fail(ALCH_ERR_INVALID_ARG, "adapter product: 1..3 problems per launch");
    double flops = 0, bytes = 0;
    bool fast = dt == ALCH_BF16;
    for (int i = 0; i < n_jobs; ++i) {
        const LoraDown& j = jobs[i];
        if (j.K % 8 || j.ldx % 8 || j.r % 8 || (j.r > 0 && j.lds % 8))
            return fail(ALCH_ERR_UNSUPPORTED, "adapter product: widths, strides and rank must be multiples of 8");
        if (j.r > 0) { flops += 2.0 * Trows * j.K * j.r; bytes += (double)Trows * j.K * dtype_size(dt); }
        if (j.r > slot_cols) return fail(ALCH_ERR_INVALID_ARG, "adapter product: rank exceeds the output slot");
        fast = fast && j.K % 64 == 0 && aligned16(j.X) && aligned16(j.Y) && (j.r == 0 || aligned16(j.S)) && 32 * j.ldx < (1LL << 30);
    }
    if (slot_cols % 8 || ldy % 8) return fail(ALCH_ERR_UNSUPPORTED, "adapter product: slot width must be a multiple of 8");
    if (Trows <= 0) return ALCH_OK;
    // algorithmic bytes: each streamed activation once (nothing for slots that are only zero-filled)
    if (fast) {
        // problems: the eight-column groups of all jobs, those of equal X merged four at a time
        LoraDownParams p = {};
        int np = 0, most = 0;
        p.nslots = n_jobs;
        for (int i = 0; i < n_jobs; ++i) {
            const LoraDown& j = jobs[i];
            p.slot[i] = (__bf16*)j.Y;
            p.slot_r[i] = j.r;
            for (int g0 = 0; g0 < j.r; g0 += 8) {
                LoraDownProblem* pb = np > 0 ? &p.pr[np - 1] : nullptr;
                if (!pb || pb->X != (const __bf16*)j.X || pb->ldx != j.ldx || pb->K != j.K || pb->ngroups == kDownGroups) {
                    pb = &p.pr[np++];
                    pb->X = (const __bf16*)j.X; pb->ldx = j.ldx; pb->K = j.K; pb->ngroups = 0;
                }
                pb->g[pb->ngroups++] = LoraDownGroup{(const __bf16*)j.S + (long long)g0 * j.lds, j.lds, 8, (__bf16*)j.Y + g0};
                most = std::max(most, pb->ngroups);
            }
        }
        p.Trows = Trows; p.ldy = ldy; p.alpha = alpha; p.slot_cols = slot_cols;
        p.rows_dev = rows_dev;
        bytes = 0;
        if (rows_dev) flops = 0;  // (what is done only the device knows)
        for (int i = 0; i < np && !rows_dev; ++i) bytes += (double)Trows * p.pr[i].K * dtype_size(dt);
        TraceScope ts(kTraceLora, flops, bytes, stream);
        int n_cu = 0;
        ALCH_TRY(compute_units(&n_cu));
        const int parts = lora_down_parts(Trows, as_problems > 0 ? as_problems : np, n_cu);
        if (parts == 16) launch_down<8, 16>(p, most, Trows, np, stream);
        else if (parts == 8) launch_down<16, 8>(p, most, Trows, np, stream);
        else launch_down<32, 4>(p, most, Trows, np, stream);
    } else {
        if (rows_dev) return fail(ALCH_ERR_UNSUPPORTED, "adapter product: a row count on the device needs the matrix-core kernel");
        TraceScope ts(kTraceLora, flops, bytes, stream);
        for (int i = 0; i < n_jobs; ++i) {
            if (dt == ALCH_BF16) lora_down_valu<__bf16>(jobs[i], Trows, alpha, ldy, slot_cols, stream);
            else lora_down_valu<float>(jobs[i], Trows, alpha, ldy, slot_cols, stream);
        }
    }
    ALCH_HIP_TRY(hipGetLastError());
    return ALCH_OK;
}

void add_lora_up_job(LoraUpSums& sums, const LoraUp& j, int nsplit, const int* rows_dev, int rows_dev_split) {
    LoraUpParams& p = sums.p;
    const LoraUpJob* before = p.n_jobs > 0 ? &p.job[p.n_jobs - 1] : nullptr;
    const int first_group = before ? before->first_group + ceil_div((long long)before->N * p.r, (long long)kSumsPerGroup) : 0;
    p.job[p.n_jobs++] = LoraUpJob{j.S, j.lds, j.X, j.ldx, j.N, nsplit, nsplit > 0 ? ceil_div(p.Trows, nsplit) : 0, j.C, j.ldc,
                                  j.transposed, first_group, sums.floats, rows_dev, rows_dev_split};
    sums.floats += (long long)p.r * nsplit * j.N;
}

int launch_lora_up(alch_dtype dt, const LoraUp* jobs, int n_jobs, LoraUpSums& sums, hipStream_t stream) {
    LoraUpParams& p = sums.p;
    const int r = p.r, Trows = p.Trows;
    if (n_jobs < 1 || n_jobs > kLoraUpJobs) return fail(ALCH_ERR_INVALID_ARG, "adapter gradient: 1..%d problems per launch", kLoraUpJobs);
    if (r % 8 || r <= 0) return fail(ALCH_ERR_UNSUPPORTED, "adapter gradient: rank must be a positive multiple of 8");
    long long need = 0;
    for (int i = 0; i < n_jobs; ++i) {
        const LoraUp& j = jobs[i];
        if (j.N % 8 || j.ldx % 8 || j.lds % 8)
            return fail(ALCH_ERR_UNSUPPORTED, "adapter gradient: widths and strides must be multiples of 8");
        need += (long long)r * (Trows > 0 ? up_splits(Trows, j.N) : 0) * j.N;
    }
    if (p.n_jobs + n_jobs > kLoraUpSums || sums.floats + need > sums.capacity) ALCH_TRY(launch_lora_up_sums(dt, sums, stream));
    double flops = 0, bytes = 0;
    int max_slabs = 1, max_split = 0;
    const int first = p.n_jobs;
    for (int i = 0; i < n_jobs; ++i) {
        const LoraUp& j = jobs[i];
        const int nsplit = Trows > 0 ? up_splits(Trows, j.N) : 0;
        add_lora_up_job(sums, j, nsplit);
        flops += 2.0 * Trows * j.N * r;
        bytes += (double)Trows * j.N * dtype_size(dt);
        max_slabs = std::max(max_slabs, ceil_div(j.N, 512));
        max_split = std::max(max_split, nsplit);
    }
    TraceScope ts(kTraceLora, flops, bytes, stream);
    const dim3 grid(max_slabs, max_split, n_jobs * (r / 8));
    if (max_split > 0) {
        if (dt == ALCH_BF16) k_lora_up_partial<__bf16><<<grid, 256, 0, stream>>>(p, first);
        else k_lora_up_partial<float><<<grid, 256, 0, stream>>>(p, first);
    }
    ALCH_HIP_TRY(hipGetLastError());
    return ALCH_OK;
}

int launch_lora_up_sums(alch_dtype dt, LoraUpSums& sums, hipStream_t stream) {
    LoraUpParams& p = sums.p;
    if (p.n_jobs == 0) return ALCH_OK;
    const LoraUpJob& last = p.job[p.n_jobs - 1];
    const int groups = last.first_group + ceil_div((long long)last.N * p.r, (long long)kSumsPerGroup);
    {
        TraceScope ts(kTraceLora, 0.0, 0.0, stream);
        if (dt == ALCH_BF16) k_lora_up_finish<__bf16><<<groups, 256, 0, stream>>>(p);
        else k_lora_up_finish<float><<<groups, 256, 0, stream>>>(p);
    }
    p.n_jobs = 0;
    sums.floats = 0;
    ALCH_HIP_TRY(hipGetLastError());
    return ALCH_OK;
}

int launch_lora_prep(alch_dtype dt, const LoraPrepParams& p, int n_jobs, hipStream_t stream) {
    if (n_jobs <= 0) return ALCH_OK;
    long long most = 0;
    for (int i = 0; i < n_jobs; ++i) most = std::max(most, (long long)p.job[i].rows_out * p.job[i].cols);
    int gx = ceil_div(most, 256LL * 8);
    if (gx > 128) gx = 128;
    if (gx < 1) gx = 1;
    if (dt == ALCH_BF16) k_lora_prep<__bf16><<<dim3(gx, n_jobs), 256, 0, stream>>>(p);
    else k_lora_prep<float><<<dim3(gx, n_jobs), 256, 0, stream>>>(p);
    ALCH_HIP_TRY(hipGetLastError());
    return ALCH_OK;
}

}  // namespace alch
