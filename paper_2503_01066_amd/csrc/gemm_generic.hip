// GEMM in fp32 arithmetic for the fp32 storage type and for bf16 problems whose shapes or alignments the bf16
// matrix-core kernel does not take.  Same contract as that kernel (operand pairs, split outputs, accumulate).
//
// The multiply-adds run on the fp32 form of the matrix instruction (v_mfma_f32_32x32x2_f32: fp32 operands and
// accumulation, 157 TFLOP/s on this chip, twice the unpacked vector rate), in two kernels chosen by the number of
// output tiles:
//   k_gemm_f32_slices  one 32x32 tile per work-group of 4, 8 or 16 wavefronts that each take a slice of the
//                      contraction, operands straight from memory into registers, the slices' sums folded through LDS in
//                      a fixed order.  A problem of a few hundred rows has few tiles and a long serial contraction: what
//                      bounds it is the latency of that chain, so it is cut (256 x 256 x 2048: 445 -> 13 us).
//   k_gemm_f32_tiled   128x128 tiles staged through LDS, for problems with enough of them to fill the compute units
//                      (4096 x 4096 x 2048: 93 - 107 TFLOP/s; vector multiply-adds on 64x64 tiles: 50).
#include <algorithm>
#include <type_traits>

#include "kernels.h"
#include "row_sums.h"

namespace alch {

typedef __attribute__((ext_vector_type(16))) float f32x16;
typedef __attribute__((ext_vector_type(4))) float f32x4;
typedef __attribute__((ext_vector_type(4))) __bf16 bf16x4;

struct GenericGemmParams {
    int M, N, n_seg, n_out, accumulate, a_kmajor, b_kmajor, tiles_n;
    const void* A[kMaxGemmSegs];
    const void* B[kMaxGemmSegs];
    int K[kMaxGemmSegs];
    long long lda[kMaxGemmSegs], ldb[kMaxGemmSegs];
    int a_vec[kMaxGemmSegs], b_vec[kMaxGemmSegs];  // base and stride allow loads of four elements
    void* C[3];
    int m_begin[3];
    long long ldc[3];
    int c_vec[3];  // (as a_vec)
    int epilogue;
    const void* G;
    const void* U;
    long long ldgu;
    void* act_out;
};

template <typename T> __device__ __forceinline__ float ld(const T* p) { return (float)*p; }
template <typename T> __device__ __forceinline__ void st(T* p, float v) { *p = (T)v; }
__device__ __forceinline__ f32x4 ld4(const float* p) { return *reinterpret_cast<const f32x4*>(p); }
__device__ __forceinline__ f32x4 ld4(const __bf16* p) {
    const bf16x4 v = *reinterpret_cast<const bf16x4*>(p);
    return f32x4{(float)v[0], (float)v[1], (float)v[2], (float)v[3]};
}

__device__ __forceinline__ void st4(float* p, const f32x4& v) { *reinterpret_cast<f32x4*>(p) = v; }
__device__ __forceinline__ void st4(__bf16* p, const f32x4& v) {
    *reinterpret_cast<bf16x4*>(p) = bf16x4{(__bf16)v[0], (__bf16)v[1], (__bf16)v[2], (__bf16)v[3]};
}

// What the output of element (m, n) needs of memory: G and U, or its old value.
template <typename T>
__device__ __forceinline__ void element_operands(const GenericGemmParams& p, int m, int n, float (&x)[2]) {
    if (m >= p.M || n >= p.N) return;
    if (p.epilogue == kEpiSwigluBwd) {
        x[0] = ld(static_cast<const T*>(p.G) + (long long)m * p.ldgu + n);
        x[1] = ld(static_cast<const T*>(p.U) + (long long)m * p.ldgu + n);
    } else if (p.accumulate) {
        int oseg = 0;
        for (int s = 1; s < p.n_out; ++s)
            if (m >= p.m_begin[s]) oseg = s;
        x[0] = ld(static_cast<const T*>(p.C[oseg]) + (long long)(m - p.m_begin[oseg]) * p.ldc[oseg] + n);
    }
}
// One element of the product -> the output; x: its element_operands.
template <typename T>
__device__ __forceinline__ void store_element(const GenericGemmParams& p, int m, int n, float acc, const float (&x)[2]) {
    if (m >= p.M || n >= p.N) return;
    int oseg = 0;
    for (int s = 1; s < p.n_out; ++s)
        if (m >= p.m_begin[s]) oseg = s;
    T* C = static_cast<T*>(p.C[oseg]);
    const long long ldc = p.ldc[oseg];
    if (p.epilogue == kEpiSwigluBwd) {
        const float g = x[0], u = x[1];
        const float d = (float)(T)acc;
        const float sg = 1.f / (1.f + expf(-g));
        st(C + (long long)m * ldc + n, d * u * sg * (1.f + g * (1.f - sg)));
        st(C + (long long)m * ldc + p.N + n, d * g * sg);
        if (p.act_out) st(static_cast<T*>(p.act_out) + (long long)m * p.N + n, g * sg * u);
    } else {
        st(C + (long long)(m - p.m_begin[oseg]) * ldc + n, p.accumulate ? acc + x[0] : acc);
    }
}

// Elements (idx, k .. k+3) of an operand, zero from k_end on.  idx lies inside the operand.  whole: k + 4 <= k_end
// for every lane (uniform, so that the usual case has no per-element branches).
template <typename T>
__device__ __forceinline__ f32x4 operand4(const T* base, long long ld_, bool kmajor, bool vec, bool whole, int idx, int k, int k_end) {
    const T* q = kmajor ? base + (long long)idx * ld_ + k : base + (long long)k * ld_ + idx;
    const long long step = kmajor ? 1 : ld_;
    if (whole) {
        if (kmajor && vec) return ld4(q);
        return f32x4{ld(q), ld(q + step), ld(q + 2 * step), ld(q + 3 * step)};
    }
    f32x4 v = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int i = 0; i < 4; ++i)
        if (k + i < k_end) v[i] = ld(q + i * step);
    return v;
}

// kTile 32: v_mfma_f32_32x32x2_f32, kTile 16: v_mfma_f32_16x16x4_f32.  A lane gives one (row, k) element of A and one
// (k, column) element of B, k = lane / kTile.  Which k meet in an instruction is free as long as A and B agree: with
// kParts = 64 / kTile, part h of the wavefront holds k0 + 4h .. k0 + 4h + 3 of a chunk of 4 kParts, and instruction i
// multiplies k0 + i, k0 + 4 + i, ...
template <int kTile> struct F32Tile;
template <> struct F32Tile<32> {
    typedef f32x16 Acc;
    static __device__ __forceinline__ Acc mac(float a, float b, Acc c) { return __builtin_amdgcn_mfma_f32_32x32x2f32(a, b, c, 0, 0, 0); }
    static __device__ __forceinline__ int row(int e, int lane) { return 8 * (e >> 2) + 4 * (lane >> 5) + (e & 3); }
};
template <> struct F32Tile<16> {
    typedef f32x4 Acc;
    static __device__ __forceinline__ Acc mac(float a, float b, Acc c) { return __builtin_amdgcn_mfma_f32_16x16x4f32(a, b, c, 0, 0, 0); }
    static __device__ __forceinline__ int row(int e, int lane) { return 4 * (lane >> 4) + e; }
};

// kForm: 0..3 = (a_kmajor, b_kmajor << 1) with contractions of whole chunks, one at least (a pair of length zero may have no
// operands), and, for a k-major operand, rows that allow
// loads of four elements: no load then depends on a condition, so that all of a batch are requested before the first is
// waited for (the eight products of a layer backward of 256 tokens, hidden 256, ffn 1024: 77 us with the conditions, 63 us
// without); -1 = everything else.
// `wave` of the kWaves that form tile `tile`; `red` holds their sums.  Every wavefront of the work-group takes part in the
// one barrier; whether the tile is written may differ.
template <typename T, int kTile, int kWaves, int kForm>
__device__ __forceinline__ void slices_tile(const GenericGemmParams& p, int tile, int wave, float (*red)[kTile * kTile / 64][64], bool written) {
    constexpr int kElems = kTile * kTile / 64, kChunk = 256 / kTile;
    const int lane = threadIdx.x & 63, part = lane / kTile;
    const int m0 = tile / p.tiles_n * kTile, n0 = tile % p.tiles_n * kTile;
    const int m = min(m0 + lane % kTile, p.M - 1), n = min(n0 + lane % kTile, p.N - 1);
    constexpr bool kPlain = kForm >= 0;
    const bool ak = kPlain ? (kForm & 1) != 0 : p.a_kmajor != 0, bk = kPlain ? (kForm & 2) != 0 : p.b_kmajor != 0;
    constexpr int kBatch = 4;
    typename F32Tile<kTile>::Acc acc;
#pragma unroll
    for (int e = 0; e < kElems; ++e) acc[e] = 0.f;
    // kBatch chunks are requested together, and the next batch is on its way during the current one.  Behind the last one there is
    // none to request: with its last chunk asked for four times more, and waited for, a layer backward of 2 x 128 tokens,
    // hidden 256, took 81.8 us, now 72.4 (dH2 of it 15.3 -> 9.7, dAct 9.9 -> 8.7 with what its output needs ahead of the products);
    // 97 tokens 86.9 -> 74.3, 664 tokens 164 -> 142, same bits.  The first batch of the next operand pair ahead of the last
    // products of this one: 72.1, 664 tokens 158.
    auto load = [&](const T* A, const T* B, long long lda, long long ldb, bool av, bool bv, int c, int hi, int k_end, f32x4 (&a)[kBatch],
                    f32x4 (&b)[kBatch]) {
#pragma unroll
        for (int q = 0; q < kBatch; ++q) {
            // (past the slice, whose products are left out below: its last chunk again)
            const int k = (kPlain ? max(min(c + q, hi - 1), 0) : c + q) * kChunk + 4 * part;
            const bool whole = kPlain || (c + q + 1) * kChunk <= k_end;
            a[q] = operand4(A, lda, ak, av, whole, m, k, k_end);
            b[q] = operand4(B, ldb, bk, bv, whole, n, k, k_end);
        }
    };
    auto products = [&](int c, int hi, const f32x4 (&a)[kBatch], const f32x4 (&b)[kBatch]) {
#pragma unroll
        for (int q = 0; q < kBatch; ++q)
            if (!kPlain || c + q < hi) {
#pragma unroll
                for (int i = 0; i < 4; ++i) acc = F32Tile<kTile>::mac(a[q][i], b[q][i], acc);
            }
    };
    // The elements of the tile that this thread writes, and what the output needs of memory for them, which is on its way
    // during the products (asked for behind them, element by element, it was four latencies of the dAct product).
    constexpr int kMine = (kElems + kWaves - 1) / kWaves;
    float more[kMine][2];
    constexpr bool kAhead = kForm != 0;
    if (kAhead && written) {
#pragma unroll
        for (int i = 0; i < kMine; ++i) {
            const int q = (i * kWaves + wave) * 64 + lane;
            if (q < kElems * 64) element_operands<T>(p, m0 + F32Tile<kTile>::row(q >> 6, q & 63), n0 + (q & 63) % kTile, more[i]);
        }
    }
    for (int s = 0; s < p.n_seg; ++s) {
        const T* A = static_cast<const T*>(p.A[s]);
        const T* B = static_cast<const T*>(p.B[s]);
        const long long lda = p.lda[s], ldb = p.ldb[s];
        const bool av = kPlain || p.a_vec[s], bv = kPlain || p.b_vec[s];
        const int chunks = (p.K[s] + kChunk - 1) / kChunk;
        const int lo = wave * chunks / kWaves, hi = (wave + 1) * chunks / kWaves;
        const int k_end = min(p.K[s], hi * kChunk);
        f32x4 a0[kBatch], b0[kBatch];
        load(A, B, lda, ldb, av, bv, lo, hi, k_end, a0, b0);
        int c = lo;
        for (; c + kBatch < hi; c += kBatch) {
            f32x4 a1[kBatch], b1[kBatch];
            load(A, B, lda, ldb, av, bv, c + kBatch, hi, k_end, a1, b1);
            products(c, hi, a0, b0);
#pragma unroll
            for (int q = 0; q < kBatch; ++q) { a0[q] = a1[q]; b0[q] = b1[q]; }
        }
        products(c, hi, a0, b0);
    }
#pragma unroll
    for (int e = 0; e < kElems; ++e) red[wave][e][lane] = acc[e];
    __syncthreads();
    if (!written) return;
#pragma unroll
    for (int i = 0; i < kMine; ++i) {
        const int q = (i * kWaves + wave) * 64 + lane;
        if (q >= kElems * 64) break;
        const int e = q >> 6, l = q & 63;
        float v = red[0][e][l];
#pragma unroll
        for (int w = 1; w < kWaves; ++w) v += red[w][e][l];
        const int row = m0 + F32Tile<kTile>::row(e, l), col = n0 + l % kTile;
        if (!kAhead) element_operands<T>(p, row, col, more[i]);
        store_element<T>(p, row, col, v, more[i]);
    }
}

template <typename T, int kTile, int kWaves, int kForm>
__global__ __launch_bounds__(kWaves * 64) void k_gemm_f32_slices(GenericGemmParams p) {
    __shared__ float red[kWaves][kTile * kTile / 64][64];
    slices_tile<T, kTile, kWaves, kForm>(p, (int)blockIdx.x, __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), red, true);
}

// A data gradient (form 1) and, in the work-groups from n_data on, a weight gradient (form 0) that does not depend on it:
// either is a chain of latencies on part of the chip (layer of 2 x 128 tokens, hidden 256: dO 4.5 us and [dWg; dWu] 10, now
// 11.7 together; dH1 10.2 and dWo 3.9, now 12.3; layer backward of 256 tokens, all gradients, 105.5 -> 101.8 us; four shapes from 1
// to 2000 tokens, none slower).  Each takes its own tile size and wavefronts per tile (kWaves at most); a work-group holds as
// many tiles as fit.  Work-groups of 16 wavefronts are left out: one fills a compute
// unit's registers, so that the second product's wait for the first one's to end (dH2 15.5 and dWd 5.5 us, together 28).
struct SlicesJob { GenericGemmParams p; int tiles, tile, waves; };
template <int kTile, int kWaves, int kPer, int kForm>
__device__ __forceinline__ void slices_tiles(const SlicesJob& job, int block, float* red) {
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), sub = wave / kPer;
    constexpr int kEach = kTile * kTile / 64 * 64;
    const int t = block * (kWaves / kPer) + sub;
    slices_tile<float, kTile, kPer, kForm>(job.p, min(t, job.tiles - 1), wave % kPer,
                                           reinterpret_cast<float (*)[kTile * kTile / 64][64]>(red + sub * kPer * kEach), t < job.tiles);
}
template <int kWaves, int kForm>
__device__ __forceinline__ void slices_job(const SlicesJob& job, int block, float* red) {
    if (job.tile == 32) {
        if (job.waves == kWaves) slices_tiles<32, kWaves, kWaves, kForm>(job, block, red);
        else slices_tiles<32, kWaves, 4, kForm>(job, block, red);
    } else {
        if (job.waves == kWaves) slices_tiles<16, kWaves, kWaves, kForm>(job, block, red);
        else slices_tiles<16, kWaves, 4, kForm>(job, block, red);
    }
}
template <int kWaves>
__global__ __launch_bounds__(kWaves * 64) void k_gemm_f32_two(SlicesJob data, SlicesJob weight, int n_data) {
    __shared__ float red[kWaves * 16 * 64];
    if ((int)blockIdx.x < n_data) slices_job<kWaves, 1>(data, (int)blockIdx.x, red);
    else slices_job<kWaves, 0>(weight, (int)blockIdx.x - n_data, red);
}

// A weight gradient of four wavefronts a tile behind the rows of an RMSNorm backward, or the sums of the gain gradients, which
// take a few latencies each on their own (layer of 2 x 128 tokens, hidden 256: dWd 5.8 us and the norm 5.0, dWqkv 6.9 and the sums
// 3.9).  Same bits.
template <int kCols>
__global__ __launch_bounds__(256) void k_gemm_f32_norm(SlicesJob weight, NormBwdRows rows, int n_rows) {
    __shared__ float red[4 * 16 * 64];
    if ((int)blockIdx.x < n_rows) rmsnorm_bwd_rows<float, kCols>(rows, (int)blockIdx.x, n_rows, red);
    else slices_job<4, 0>(weight, (int)blockIdx.x - n_rows, red);
}
__global__ __launch_bounds__(256) void k_gemm_f32_gains(SlicesJob weight, GainSums sums, int width, int accumulate, int slabs) {
    __shared__ float red[4 * 16 * 64];
    const int n_sums = slabs * sums.n, block = (int)blockIdx.x;
    if (block < n_sums) gain_sums<float, 4>(sums, block / slabs, block % slabs * 64, width, accumulate, reinterpret_cast<float (*)[64]>(red));
    else slices_job<4, 0>(weight, block - n_sums, red);
}

template <typename T>
__global__ __launch_bounds__(256) void k_gemm_f32_tiled(GenericGemmParams p) {
    constexpr int TB = 128, TK = 32, kLd = TB + 4;
    __shared__ __attribute__((aligned(16))) float As[2][TK][kLd];
    __shared__ __attribute__((aligned(16))) float Bs[2][TK][kLd];
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6, half = lane >> 5;
    const int wm = (wave >> 1) * 64, wn = (wave & 1) * 64;
    const int m0 = (int)(blockIdx.x / p.tiles_n) * TB, n0 = (int)(blockIdx.x % p.tiles_n) * TB;
    f32x16 acc[2][2];
#pragma unroll
    for (int i = 0; i < 2; ++i)
#pragma unroll
        for (int j = 0; j < 2; ++j)
#pragma unroll
            for (int e = 0; e < 16; ++e) acc[i][j][e] = 0.f;
    // this thread's 16 elements of an operand tile: k-major: row tid/2, k (tid&1)*16 ..+15; else k tid/16 and 16 further,
    // columns (tid&15)*8 ..+7
    const int kr = threadIdx.x >> 1, kk = (threadIdx.x & 1) * 16, mk = threadIdx.x >> 4, mc = (threadIdx.x & 15) * 8;
    auto load = [&](const T* P, long long ld_, bool kmajor, bool vec, int r0, int r_end, int k0, int K, f32x4 (&v)[4]) {
        const bool inside = kmajor ? k0 + TK <= K : k0 + TK <= K && r0 + TB <= r_end;
        const int r = min(r0 + kr, r_end - 1);
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            const int k = k0 + mk + 16 * (i >> 1), c = r0 + mc + 4 * (i & 1);
            if (kmajor) v[i] = operand4(P, ld_, true, vec, inside, r, k0 + kk + 4 * i, K);
            else if (inside || k < K) v[i] = operand4(P, ld_, true, vec, inside, k, c, r_end);  // four columns of a row of k
            else v[i] = f32x4{0.f, 0.f, 0.f, 0.f};
        }
    };
    auto store = [&](float (&S)[TK][kLd], bool kmajor, const f32x4 (&v)[4]) {
        if (kmajor) {
#pragma unroll
            for (int i = 0; i < 16; ++i) S[kk + i][kr] = v[i >> 2][i & 3];
        } else {
#pragma unroll
            for (int i = 0; i < 4; ++i) *reinterpret_cast<f32x4*>(&S[mk + 16 * (i >> 1)][mc + 4 * (i & 1)]) = v[i];
        }
    };
    for (int s = 0; s < p.n_seg; ++s) {
        const T* A = static_cast<const T*>(p.A[s]);
        const T* B = static_cast<const T*>(p.B[s]);
        const int K = p.K[s], nk = (K + TK - 1) / TK;
        f32x4 a[4], b[4];
        load(A, p.lda[s], p.a_kmajor, p.a_vec[s], m0, p.M, 0, K, a);
        load(B, p.ldb[s], p.b_kmajor, p.b_vec[s], n0, p.N, 0, K, b);
        __syncthreads();  // (the previous pair's last stage has been read)
        for (int t = 0; t < nk; ++t) {
            store(As[t & 1], p.a_kmajor, a);
            store(Bs[t & 1], p.b_kmajor, b);
            __syncthreads();  // one barrier per stage: stage t+1 goes to the other half of the buffers
            if (t + 1 < nk) {
                load(A, p.lda[s], p.a_kmajor, p.a_vec[s], m0, p.M, (t + 1) * TK, K, a);
                load(B, p.ldb[s], p.b_kmajor, p.b_vec[s], n0, p.N, (t + 1) * TK, K, b);
            }
#pragma unroll
            for (int k = 0; k < TK; k += 2) {
                float fa[2], fb[2];
#pragma unroll
                for (int i = 0; i < 2; ++i) {
                    fa[i] = As[t & 1][k + half][wm + i * 32 + (lane & 31)];
                    fb[i] = Bs[t & 1][k + half][wn + i * 32 + (lane & 31)];
                }
#pragma unroll
                for (int i = 0; i < 2; ++i)
#pragma unroll
                    for (int j = 0; j < 2; ++j) acc[i][j] = __builtin_amdgcn_mfma_f32_32x32x2f32(fa[i], fb[j], acc[i][j], 0, 0, 0);
            }
        }
    }
    // A tile of one output leaves through LDS as 16-byte (bf16: 8-byte) pieces of whole rows, 64x64 per wavefront, columns
    // turned by 32 in every other group of four rows so that the two halves of a wavefront write to different banks.  Element
    // by element the stores were what short contractions took: 4096 x 1312, K 32 28 us, now 14;
    // 8192 x 8192, K 16 208 us, now 91, K 64 226 us, now 120; 4096 x 4096, K 2048 736 us, now 706.
    int oseg = 0;
    for (int s = 1; s < p.n_out; ++s)
        if (m0 >= p.m_begin[s]) oseg = s;
    if (p.epilogue == kEpiNone && p.N % 4 == 0 && p.c_vec[oseg] && (oseg + 1 >= p.n_out || m0 + TB <= p.m_begin[oseg + 1])) {
        __syncthreads();  // (the last stage has been read)
        float* st = (wave < 2 ? &As[0][0][0] : &Bs[0][0][0]) + (wave & 1) * 4096;
#pragma unroll
        for (int i = 0; i < 2; ++i)
#pragma unroll
            for (int j = 0; j < 2; ++j)
#pragma unroll
                for (int e = 0; e < 16; ++e) {
                    const int r = i * 32 + 8 * (e >> 2) + 4 * half + (e & 3);
                    st[r * 64 + ((j * 32 + (lane & 31)) ^ (half * 32))] = acc[i][j][e];
                }
        const long long ldc = p.ldc[oseg];
        const int rows = p.M - (m0 + wm + (lane >> 4));  // of this lane's: row 4 k is inside for 4 k < rows
        if (n0 + wn + 4 * (lane & 15) >= p.N) return;
        T* C = static_cast<T*>(p.C[oseg]) + (long long)(m0 - p.m_begin[oseg] + wm + (lane >> 4)) * ldc + n0 + wn + 4 * (lane & 15);
#pragma unroll
        for (int q = 0; q < 16; q += 8) {
            f32x4 old[8];
            if (p.accumulate)
#pragma unroll
                for (int k = 0; k < 8; ++k)
                    if (4 * (q + k) < rows) old[k] = ld4(C + (long long)(4 * (q + k)) * ldc);
#pragma unroll
            for (int k = 0; k < 8; ++k) {
                const int r = 4 * (q + k) + (lane >> 4);
                f32x4 v = *reinterpret_cast<const f32x4*>(st + r * 64 + ((4 * (lane & 15)) ^ ((((q + k) & 1)) * 32)));
                if (p.accumulate) v += old[k];
                if (4 * (q + k) < rows) st4(C + (long long)(4 * (q + k)) * ldc, v);
            }
        }
        return;
    }
#pragma unroll
    for (int i = 0; i < 2; ++i)
#pragma unroll
        for (int j = 0; j < 2; ++j)
#pragma unroll
            for (int e = 0; e < 16; ++e)
            {
                const int m = m0 + wm + i * 32 + 8 * (e >> 2) + 4 * half + (e & 3), n = n0 + wn + j * 32 + (lane & 31);
                float more[2];
                element_operands<T>(p, m, n, more);
                store_element<T>(p, m, n, acc[i][j][e], more);
            }
}

// From this many 128x128 tiles on the tiled kernel is the faster one (K 1024, three layouts, slices against tiled:
// 121 tiles 88 / 95 / 103 against 125 / 139 / 99 us, 182 tiles 129 / 141 / 150 against 125 / 138 / 99 us,
// 256 tiles 174 / 191 / 203 against 126 / 139 / 101 us; K 256: 156 tiles 36 / 36 / 37 against 34 / 37 / 30 us).
static constexpr int kTiledFrom = 160;
// Below this many 32x32 tiles the slices kernel takes 16x16 ones: four times as many work-groups share the reads
// (256 x 256 x 2048, 64 tiles of 32x32: 24 against 12.4 us; 192 tiles, K 256: equal; 512^3, 256 tiles: 10.6 against 13.7 us).
static constexpr int kWideFrom = 128;

// Wavefronts per tile: slices of at least 64 k.
static int slices_waves(int k_total) { return k_total >= 1024 ? 16 : k_total >= 512 ? 8 : 4; }
// Contractions of whole chunks and, for k-major operands, rows that allow loads of four elements (kForm >= 0).
static bool slices_plain(const GenericGemmParams& p, int tile) {
    bool plain = true;
    for (int s = 0; s < p.n_seg; ++s)
        plain = plain && p.K[s] > 0 && p.K[s] % (256 / tile) == 0 && (!p.a_kmajor || p.a_vec[s]) && (!p.b_kmajor || p.b_vec[s]);
    return plain;
}

template <typename T, int kTile, int kForm>
static void gemm_slices_form(GenericGemmParams& p, int k_total, hipStream_t stream) {
    p.tiles_n = ceil_div(p.N, kTile);
    const int grid = ceil_div(p.M, kTile) * p.tiles_n, waves = slices_waves(k_total);
    if (waves == 16) k_gemm_f32_slices<T, kTile, 16, kForm><<<grid, 1024, 0, stream>>>(p);
    else if (waves == 8) k_gemm_f32_slices<T, kTile, 8, kForm><<<grid, 512, 0, stream>>>(p);
    else k_gemm_f32_slices<T, kTile, 4, kForm><<<grid, 256, 0, stream>>>(p);
}
template <typename T, int kTile>
static void gemm_slices_t(GenericGemmParams& p, int k_total, hipStream_t stream) {
    if constexpr (std::is_same<T, float>::value) {
        if (slices_plain(p, kTile)) {
            if (p.a_kmajor && p.b_kmajor) return gemm_slices_form<T, kTile, 3>(p, k_total, stream);
            if (p.b_kmajor) return gemm_slices_form<T, kTile, 2>(p, k_total, stream);
            if (p.a_kmajor) return gemm_slices_form<T, kTile, 1>(p, k_total, stream);
            return gemm_slices_form<T, kTile, 0>(p, k_total, stream);
        }
    }
    gemm_slices_form<T, kTile, -1>(p, k_total, stream);
}

static int total_k(const GenericGemmParams& p) {
    int k = 0;
    for (int s = 0; s < p.n_seg; ++s) k += p.K[s];
    return k;
}
// Rows and columns of a tile: 128 (tiled kernel), 32 or 16 (slices).
static int generic_tile(const GenericGemmParams& p) {
    if ((long long)ceil_div(p.M, 128) * ceil_div(p.N, 128) >= kTiledFrom) return 128;
    return (long long)ceil_div(p.M, 32) * ceil_div(p.N, 32) >= kWideFrom ? 32 : 16;
}

template <typename T>
static void gemm_generic_t(GenericGemmParams& p, hipStream_t stream) {
    const int tile = generic_tile(p);
    if (tile == 128) {
        p.tiles_n = ceil_div(p.N, 128);
        k_gemm_f32_tiled<T><<<ceil_div(p.M, 128) * p.tiles_n, 256, 0, stream>>>(p);
    } else if (tile == 32) {
        gemm_slices_t<T, 32>(p, total_k(p), stream);
    } else {
        gemm_slices_t<T, 16>(p, total_k(p), stream);
    }
}

static GenericGemmParams generic_params(const GemmDesc& d) {
    GenericGemmParams p;
    p.M = d.M; p.N = d.N; p.n_seg = d.n_seg; p.n_out = d.n_out; p.accumulate = d.accumulate;
    p.a_kmajor = d.a_kmajor; p.b_kmajor = d.b_kmajor;
    const size_t E = dtype_size(d.dtype);
    auto vec_ok = [&](const void* q, long long ld_) { return reinterpret_cast<uintptr_t>(q) % (4 * E) == 0 && ld_ % 4 == 0; };
    for (int s = 0; s < kMaxGemmSegs; ++s) {
        const bool on = s < d.n_seg;
        p.A[s] = on ? d.seg[s].A : nullptr;
        p.B[s] = on ? d.seg[s].B : nullptr;
        p.K[s] = on ? d.seg[s].K : 0;
        p.lda[s] = on ? d.seg[s].lda : 0;
        p.ldb[s] = on ? d.seg[s].ldb : 0;
        p.a_vec[s] = on && vec_ok(d.seg[s].A, d.seg[s].lda);
        p.b_vec[s] = on && vec_ok(d.seg[s].B, d.seg[s].ldb);
    }
    for (int s = 0; s < kMaxGemmOuts; ++s) {
        const bool oo = s < d.n_out;
        p.C[s] = oo ? d.out[s].C : nullptr;
        p.m_begin[s] = oo ? d.out[s].m_begin : 0x7fffffff;
        p.ldc[s] = oo ? d.out[s].ldc : 0;
        p.c_vec[s] = oo && vec_ok(d.out[s].C, d.out[s].ldc);
    }
    p.epilogue = d.epilogue; p.G = d.G; p.U = d.U; p.ldgu = d.ldgu; p.act_out = d.act_out;
    return p;
}

int launch_gemm_generic(const GemmDesc& d, hipStream_t stream) {
    GenericGemmParams p = generic_params(d);
    if (d.dtype == ALCH_BF16) gemm_generic_t<__bf16>(p, stream);
    else gemm_generic_t<float>(p, stream);
    ALCH_HIP_TRY(hipGetLastError());
    return ALCH_OK;
}

static bool slices_job_of(const GemmDesc& d, SlicesJob& job) {
    job.p = generic_params(d);
    job.tile = generic_tile(job.p);
    if (job.tile == 128 || !slices_plain(job.p, job.tile)) return false;
    job.p.tiles_n = ceil_div(d.N, job.tile);
    job.tiles = ceil_div(d.M, job.tile) * job.p.tiles_n;
    job.waves = slices_waves(total_k(job.p));
    return true;
}
static bool slices_jobs(const GemmDesc& data, const GemmDesc& weight, SlicesJob& a, SlicesJob& b) {
    if (data.dtype != ALCH_F32 || weight.dtype != ALCH_F32 || data.m_dev || weight.k_dev || data.by_cols || weight.by_cols) return false;
    if (!data.a_kmajor || data.b_kmajor || weight.a_kmajor || weight.b_kmajor) return false;
    return slices_job_of(data, a) && slices_job_of(weight, b) && std::max(a.waves, b.waves) < 16;
}
static int launch_slices_jobs(const SlicesJob& a, const SlicesJob& b, hipStream_t stream) {
    const int waves = std::max(a.waves, b.waves), n_data = ceil_div(a.tiles, waves / a.waves);
    const int grid = n_data + ceil_div(b.tiles, waves / b.waves);
    if (waves == 8) k_gemm_f32_two<8><<<grid, 512, 0, stream>>>(a, b, n_data);
    else k_gemm_f32_two<4><<<grid, 256, 0, stream>>>(a, b, n_data);
    ALCH_HIP_TRY(hipGetLastError());
    return ALCH_OK;
}

static double job_flops(const GemmDesc& d, double& bytes) {
    double k_total = 0;
    for (int s = 0; s < d.n_seg; ++s) k_total += d.seg[s].K;
    bytes = ((double)d.M * k_total + (double)d.N * k_total + (double)d.M * d.N) * dtype_size(d.dtype);
    return 2.0 * d.M * d.N * k_total;
}
static bool job_beside_rows(const GemmDesc& weight, SlicesJob& job) {
    if (weight.M <= 0 || weight.N <= 0 || weight.dtype != ALCH_F32 || weight.k_dev || weight.m_dev || weight.by_cols) return false;
    return !weight.a_kmajor && !weight.b_kmajor && slices_job_of(weight, job) && job.waves == 4;
}
bool gemm_beside_rows(const GemmDesc& weight, int width) {
    SlicesJob job;
    return width <= 1024 && job_beside_rows(weight, job);
}
int launch_gemm_beside_norm(const GemmDesc& weight, NormBwdRows rows, void* dg, GainSums& sums, hipStream_t stream) {
    SlicesJob job;
    if (!job_beside_rows(weight, job) || rows.width > 1024 || rows.Trows <= 0) return fail(ALCH_ERR_UNSUPPORTED, "a product that does not run beside rows");
    const int n_rows = std::min(rows.Trows, kNormBwdBlocks);
    if (dg) {
        sums.of[sums.n].partial = rows.partial;
        sums.of[sums.n].dg = dg;
        sums.of[sums.n++].rows = n_rows;
    } else {
        rows.partial = nullptr;
    }
    double bytes;
    const double flops = job_flops(weight, bytes);
    TraceScope ts(kTraceGemmGeneric, flops, bytes, stream);
    if (rows.width <= 256) k_gemm_f32_norm<1><<<n_rows + job.tiles, 256, 0, stream>>>(job, rows, n_rows);
    else k_gemm_f32_norm<4><<<n_rows + job.tiles, 256, 0, stream>>>(job, rows, n_rows);
    ALCH_HIP_TRY(hipGetLastError());
    return ALCH_OK;
}
int launch_gemm_beside_gains(const GemmDesc& weight, const GainSums& sums, int width, int accumulate, hipStream_t stream) {
    SlicesJob job;
    if (!job_beside_rows(weight, job)) return fail(ALCH_ERR_UNSUPPORTED, "a product that does not run beside rows");
    double bytes;
    const double flops = job_flops(weight, bytes);
    TraceScope ts(kTraceGemmGeneric, flops, bytes, stream);
    const int slabs = ceil_div(width, 64);
    k_gemm_f32_gains<<<slabs * sums.n + job.tiles, 256, 0, stream>>>(job, sums, width, accumulate, slabs);
    ALCH_HIP_TRY(hipGetLastError());
    return ALCH_OK;
}

// The matrix-core kernel addresses an operand through one buffer descriptor and refuses operands of 2 GiB or more.
// The operands that grow with the batch are indexed by tokens: the rows of a k-major A (data gradients, forward)
// or the contraction index of a weight gradient.  A product refused for that reason alone is cut along that
// index into bands the kernel takes: row bands are independent products; contraction bands accumulate into the
// output one after the other (sum in fp32 inside a band, one rounding to the storage type per band).
// Returns true when the product was launched that way (rc holds the status).
static bool launch_gemm_in_bands(const GemmDesc& d, hipStream_t stream, int& rc) {
    if (d.dtype != ALCH_BF16 || d.m_dev || d.k_dev || d.n_out != 1 || d.out[0].m_begin != 0) return false;
    const long long kLimit = (1LL << 31) - 1;
    const bool rows = d.a_kmajor;                        // bands over M
    const bool contr = !d.a_kmajor && !d.b_kmajor;       // bands over K (single operand pair)
    if (!rows && !contr) return false;
    if (contr && d.n_seg != 1) return false;
    long long ld_max = 1;
    for (int s = 0; s < d.n_seg; ++s) ld_max = std::max(ld_max, contr ? std::max(d.seg[s].lda, d.seg[s].ldb) : d.seg[s].lda);
    if (d.epilogue == kEpiSwigluBwd) ld_max = std::max(ld_max, std::max(d.ldgu, d.out[0].ldc));
    const long long total = rows ? d.M : d.seg[0].K;
    long long band = kLimit / (ld_max * 2) / 256 * 256;
    if (band < 256 || band >= total) return false;       // nothing to gain, or not the reason of the refusal
    auto band_desc = [&](long long b0, long long n) {
        GemmDesc e = d;
        if (rows) {
            e.M = (int)n;
            for (int s = 0; s < d.n_seg; ++s) e.seg[s].A = static_cast<const char*>(d.seg[s].A) + b0 * d.seg[s].lda * 2;
            e.out[0].C = static_cast<char*>(d.out[0].C) + b0 * d.out[0].ldc * 2;
            if (d.epilogue == kEpiSwigluBwd) {
                e.G = static_cast<const char*>(d.G) + b0 * d.ldgu * 2;
                e.U = static_cast<const char*>(d.U) + b0 * d.ldgu * 2;
                if (d.act_out) e.act_out = static_cast<char*>(d.act_out) + b0 * (long long)d.N * 2;
            }
        } else {
            e.seg[0].K = (int)n;
            e.seg[0].A = static_cast<const char*>(d.seg[0].A) + b0 * d.seg[0].lda * 2;
            e.seg[0].B = static_cast<const char*>(d.seg[0].B) + b0 * d.seg[0].ldb * 2;
            e.accumulate = b0 == 0 ? d.accumulate : 1;
        }
        return e;
    };
    for (long long b0 = 0; b0 < total; b0 += band)
        if (!gemm_mfma_supported(band_desc(b0, std::min(band, total - b0)))) return false;
    rc = ALCH_OK;
    for (long long b0 = 0; b0 < total && rc == ALCH_OK; b0 += band) {
        const GemmDesc e = band_desc(b0, std::min(band, total - b0));
        double k_total = 0;
        for (int s = 0; s < e.n_seg; ++s) k_total += e.seg[s].K;
        TraceScope ts(kTraceGemmMfma, 2.0 * e.M * e.N * k_total, ((double)e.M * k_total + (double)e.N * k_total + (double)e.M * e.N) * 2, stream);
        rc = launch_gemm_mfma(e, stream);
    }
    return true;
}

int launch_gemm(const GemmDesc& d, hipStream_t stream) {
    if (d.M <= 0 || d.N <= 0) return ALCH_OK;
    double k_total = 0;
    for (int s = 0; s < d.n_seg; ++s) k_total += d.seg[s].K;
    // a size that lives on the device is not known here: such launches are traced with zero work and the
    // caller accounts for them from the row count it knows
    const bool dev_sized = d.m_dev || d.k_dev;
    const double flops = dev_sized ? 0.0 : 2.0 * d.M * d.N * k_total;
    const size_t E = dtype_size(d.dtype);
    const double bytes = dev_sized ? 0.0 : ((double)d.M * k_total + (double)d.N * k_total + (double)d.M * d.N) * E;
    if (dev_sized && !d.by_cols && !gemm_mfma_supported(d))
        return fail(ALCH_ERR_UNSUPPORTED, "device-resident sizes need the matrix-core kernel (bf16, aligned, K %% 64 == 0)");
    if (gemm_mfma_supported(d) && (!d.by_cols || gemm_cols_together(d))) {
        TraceScope ts(kTraceGemmMfma, flops, bytes, stream);
        return launch_gemm_mfma(d, stream);
    }
    if (d.by_cols) {  // one product per column range
        for (int o = 0; o < d.n_out; ++o) {
            GemmDesc r = d;
            r.by_cols = false;
            r.N = (o + 1 < d.n_out ? d.out[o + 1].m_begin : d.N) - d.out[o].m_begin;
            r.seg[0].B = d.out[o].B;
            r.n_out = 1;
            r.out[0] = GemmOut{d.out[o].C, 0, d.out[o].ldc};
            ALCH_TRY(launch_gemm(r, stream));
        }
        return ALCH_OK;
    }
    if (d.residual) {  // (C is the whole of its rows)
        ALCH_TRY(launch_masked_copy(d.dtype, d.residual, nullptr, d.out[0].C, d.M, d.N, stream));
        GemmDesc r = d;
        r.residual = nullptr;
        return launch_gemm(r, stream);
    }
    int rc = ALCH_OK;
    if (launch_gemm_in_bands(d, stream, rc)) return rc;
    TraceScope ts(kTraceGemmGeneric, flops, bytes, stream);
    return launch_gemm_generic(d, stream);
}

bool gemm_together(const GemmDesc& data, const GemmDesc& weight) {
    if (data.M <= 0 || data.N <= 0 || weight.M <= 0 || weight.N <= 0) return false;
    SlicesJob a, b;
    return data.dtype == ALCH_F32 ? slices_jobs(data, weight, a, b) : gemm_mfma_together(data, weight);
}

int launch_gemm_together(const GemmDesc& data, const GemmDesc& weight, hipStream_t stream) {
    double flops = 0, bytes = 0;
    for (const GemmDesc* d : {&data, &weight}) {
        if (d->m_dev || d->k_dev) continue;  // (as in launch_gemm)
        double k_total = 0;
        for (int s = 0; s < d->n_seg; ++s) k_total += d->seg[s].K;
        flops += 2.0 * d->M * d->N * k_total;
        bytes += ((double)d->M * k_total + (double)d->N * k_total + (double)d->M * d->N) * dtype_size(d->dtype);
    }
    TraceScope ts(data.dtype == ALCH_F32 ? kTraceGemmGeneric : kTraceGemmMfma, flops, bytes, stream);
    if (data.dtype != ALCH_F32) return launch_gemm_mfma_together(data, weight, stream);
    SlicesJob a, b;
    if (!slices_jobs(data, weight, a, b)) return fail(ALCH_ERR_UNSUPPORTED, "products that do not run together");
    return launch_slices_jobs(a, b, stream);
}

}  // namespace alch
