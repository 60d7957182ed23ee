// Cross-entropy on chunks of LM-head logits (Section 5 of the paper: the continual-pre-training
// loss is computed from the saved prefill output and the prompt's own tokens as labels).
// Logits are produced chunk by chunk by the GEMM and turned into their gradient in place, so the
// [tokens, vocab] matrix is never stored whole.
#include "kernels.h"

namespace alch {

template <typename T> __device__ __forceinline__ float ldf(const T* p) { return (float)*p; }
template <typename T> __device__ __forceinline__ void stf(T* p, float v) { *p = (T)v; }

__device__ __forceinline__ float wmax(float v) {
#pragma unroll
    for (int d = 32; d > 0; d >>= 1) v = fmaxf(v, __shfl_xor(v, d, 64));
    return v;
}
__device__ __forceinline__ float wsum2(float v) {
#pragma unroll
    for (int d = 32; d > 0; d >>= 1) v += __shfl_xor(v, d, 64);
    return v;
}

// A position counts when its label names a vocabulary entry (0 <= label < vocab) and its loss-mask byte, if a
// mask is given, is nonzero: one predicate for the count, the counted mask and the row kernels.
__device__ __forceinline__ bool label_counts(int label, int vocab) { return (unsigned)label < (unsigned)vocab; }

__global__ __launch_bounds__(256) void k_count_labels(const int* __restrict__ labels, const uint8_t* __restrict__ mask,
                                                      int T, int vocab, int* __restrict__ n_counted,
                                                      float* __restrict__ row_loss, uint8_t* __restrict__ counted) {
    // single block: deterministic count
    __shared__ int part[4];
    int c = 0;
    for (int t = threadIdx.x; t < T; t += 256) {
        const int one = (label_counts(labels[t], vocab) && (!mask || mask[t] != 0)) ? 1 : 0;
        c += one;
        if (counted) counted[t] = (uint8_t)one;
        row_loss[t] = 0.f;
    }
#pragma unroll
    for (int d = 32; d > 0; d >>= 1) c += __shfl_xor(c, d, 64);
    if ((threadIdx.x & 63) == 0) part[threadIdx.x >> 6] = c;
    __syncthreads();
    if (threadIdx.x == 0) n_counted[0] = part[0] + part[1] + part[2] + part[3];
}

template <typename T>
__global__ __launch_bounds__(256) void k_ce_chunk(T* __restrict__ logits, long long ld, int vocab,
                                                  const int* __restrict__ labels, const uint8_t* __restrict__ mask,
                                                  const int* __restrict__ n_counted, float* __restrict__ row_loss,
                                                  const int* __restrict__ rows_dev) {
    __shared__ float red[4];
    const int r = blockIdx.x;
    if (rows_dev && r >= *rows_dev) return;  // row count decided on the device (compacted rows)
    T* row = logits + (long long)r * ld;
    const int label = labels[r];
    const bool counted = label_counts(label, vocab) && (!mask || mask[r] != 0);
    if (!counted) {
        for (int v = threadIdx.x; v < vocab; v += 256) row[v] = (T)0.f;
        return;
    }
    float m = -INFINITY;
    for (int v = threadIdx.x; v < vocab; v += 256) m = fmaxf(m, ldf(row + v));
    m = wmax(m);
    if ((threadIdx.x & 63) == 0) red[threadIdx.x >> 6] = m;
    __syncthreads();
    m = fmaxf(fmaxf(red[0], red[1]), fmaxf(red[2], red[3]));
    __syncthreads();
    float s = 0.f;
    for (int v = threadIdx.x; v < vocab; v += 256) s += __expf(ldf(row + v) - m);
    s = wsum2(s);
    if ((threadIdx.x & 63) == 0) red[threadIdx.x >> 6] = s;
    __syncthreads();
    s = red[0] + red[1] + red[2] + red[3];
    const float logz = m + __logf(s);
    const float inv_n = 1.f / (float)n_counted[0];
    const float x_label = ldf(row + label);
    __syncthreads();  // everyone has read the label logit before it is overwritten
    for (int v = threadIdx.x; v < vocab; v += 256) {
        float p = __expf(ldf(row + v) - logz);
        if (v == label) p -= 1.f;
        stf(row + v, p * inv_n);
    }
    if (threadIdx.x == 0) row_loss[r] = logz - x_label;
}

// bf16 fast path: a 1024-thread work-group keeps a whole row in registers (kChunks chunks of 8 logits per thread, 16 of
// them for vocab <= 131072), so that the logits are read once and the gradient written once: the three passes (max, sum of
// exponentials, gradient) run on registers.  A row is half of a compute unit's registers: one work-group fits, and with a
// row to a work-group its loads, arithmetic and stores ran one after the other (6001 x 128256: 885 us, 3.5 TB/s).  The
// work-groups are therefore persistent, one per compute unit, and fetch the next row while they work on the present one:
// 9 of 16 chunks wait in LDS (144 KB), the others in registers: 615 us, 5.0 TB/s, what a large copy reaches.  A row that does
// not count is neither fetched nor worked on, only cleared (three quarters of these rows: 623 -> 396 us): the label and the mask byte
// of a row are read two rows ahead, so that they are there when its logits are to be requested.
typedef __attribute__((ext_vector_type(8))) __bf16 bf16x8_c;
typedef __attribute__((ext_vector_type(4))) unsigned int u32x4_c;
typedef __attribute__((ext_vector_type(4))) int i32x4_c;
static constexpr int kCeThreads = 1024, kCeChunks = 16;

__device__ __forceinline__ i32x4_c ce_row(const void* p, int vocab) {  // the bytes of a row: reads past it are zero, writes dropped
    const uint64_t a = reinterpret_cast<uint64_t>(p);
    i32x4_c r;
    r[0] = __builtin_amdgcn_readfirstlane((int)(uint32_t)a);
    r[1] = __builtin_amdgcn_readfirstlane((int)((uint32_t)(a >> 32) & 0xffffu));
    r[2] = __builtin_amdgcn_readfirstlane(vocab * 2);
    r[3] = 0x00020000;
    return r;
}

template <int kChunks>
__global__ __launch_bounds__(kCeThreads) void k_ce_chunk_bf16_row(__bf16* __restrict__ logits, long long ld, int rows, int vocab,
                                                                   const int* __restrict__ labels,
                                                                   const uint8_t* __restrict__ mask,
                                                                   const int* __restrict__ n_counted,
                                                                   float* __restrict__ row_loss,
                                                                   const int* __restrict__ rows_dev) {
    constexpr int kLds = kChunks * 9 / 16, kRegs = kChunks - kLds;
    __shared__ __attribute__((aligned(1024))) bf16x8_c ahead[kLds * kCeThreads];
    __shared__ float red[2 * kCeThreads / 64];
    const int tid = threadIdx.x, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int n_rows = rows_dev ? min(*rows_dev, rows) : rows;  // (compacted rows: decided on the device)
    if ((int)blockIdx.x >= n_rows) return;
    const int nchunks = vocab >> 3, step = (int)gridDim.x;
    const float inv_n = 1.f / (float)n_counted[0];
    const uint32_t lds0 = (uint32_t)(uintptr_t)(__attribute__((address_space(3))) void*)ahead + (uint32_t)wave * 1024u;
    bf16x8_c next[kRegs];
    // The loads of a row: a wavefront fetches what its own lanes will use.  kChunks loads, every one issued whether or not
    // the row reaches it.
    auto fetch = [&](int r, bool wanted) {
        const i32x4_c src = ce_row(logits + (long long)r * ld, wanted ? vocab : 0);
        uint32_t at = (uint32_t)tid * 16u;
        asm volatile("" : "+v"(at));  // (one register, not one per chunk kept across the loop)
#pragma unroll
        for (int k = 0; k < kLds; ++k)  // (s_nop: a load into LDS takes one wait state after a scalar write of m0)
            asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tbuffer_load_dwordx4 %1, %2, 0 offen lds" ::"s"(lds0 + k * kCeThreads * 16),
                         "v"(at + k * kCeThreads * 16), "s"(src)
                         : "memory", "m0");
#pragma unroll
        for (int k = 0; k < kRegs; ++k)
            next[k] = __builtin_bit_cast(bf16x8_c, __builtin_amdgcn_raw_buffer_load_b128(
                          __builtin_amdgcn_make_buffer_rsrc(logits + (long long)r * ld, 0, wanted ? vocab * 2 : 0, 0x00020000),
                          at + (kLds + k) * kCeThreads * 16, 0, 0));
    };
    auto label_of = [&](int r) { return labels[min(r, n_rows - 1)]; };
    auto mask_of = [&](int r) {  // (scalar at once: a vector register carried over would make the maskless case wait for its load)
        int mk = 1;
        if (mask) mk = __builtin_amdgcn_readfirstlane((int)mask[min(r, n_rows - 1)]);
        return mk;
    };
    auto counts = [&](int r, int label, int mk) {
        return r < n_rows && label_counts(label, vocab) && mk != 0;
    };
    int label = label_of(blockIdx.x), label1 = label_of(blockIdx.x + step), mask1 = mask_of(blockIdx.x + step);
    bool counted = counts(blockIdx.x, label, mask_of(blockIdx.x));
    fetch(blockIdx.x, counted);
    __builtin_amdgcn_s_waitcnt(0x0f70);  // vmcnt(0), known to the compiler: inside the loop it then counts the stores, too
    for (int r = blockIdx.x; r < n_rows; r += step) {
        // the row's loads have landed; the kChunks stores of the row before may still be on their way
        asm volatile("s_waitcnt vmcnt(%0)" ::"n"(kChunks) : "memory");
        const bool counted1 = counts(r + step, label1, mask1);
        const int label2 = label_of(r + 2 * step), mask2 = mask_of(r + 2 * step);
        if (!counted) {
            fetch(r + step, counted1);
            int at = tid;
            asm volatile("" : "+v"(at));
            const auto dst = __builtin_amdgcn_make_buffer_rsrc(logits + (long long)r * ld, 0, vocab * 2, 0x00020000);
#pragma unroll
            for (int k = 0; k < kChunks; ++k) __builtin_amdgcn_raw_buffer_store_b128(u32x4_c{0, 0, 0, 0}, dst, (at + k * kCeThreads) * 16, 0, 0);
            label = label1; label1 = label2; mask1 = mask2; counted = counted1;
            continue;
        }
        bf16x8_c x[kChunks];
#pragma unroll
        for (int k = 0; k < kLds; ++k) x[k] = ahead[k * kCeThreads + tid];
#pragma unroll
        for (int k = 0; k < kRegs; ++k) x[kLds + k] = next[k];
        asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
#pragma unroll
        for (int k = 0; k < kChunks; ++k) asm volatile("" : "+v"(x[k]));  // (in registers before the next row overwrites them)
        fetch(r + step, counted1);
        float m = -INFINITY;
#pragma unroll
        for (int k = 0; k < kChunks; ++k)
            if (tid + k * kCeThreads < nchunks) {
#pragma unroll
                for (int e = 0; e < 8; ++e) m = fmaxf(m, (float)x[k][e]);
            }
        m = wmax(m);
        if ((tid & 63) == 0) red[wave] = m;
        __syncthreads();
        m = red[0];
#pragma unroll
        for (int w = 1; w < kCeThreads / 64; ++w) m = fmaxf(m, red[w]);
        const float kL2e = 1.4426950408889634f;
        float s = 0.f;
        // (the empty asm keeps the row packed in registers between passes: without it the compiler carries the
        // converted fp32 copies across and runs out of registers)
#pragma unroll
        for (int k = 0; k < kChunks; ++k) {
            asm volatile("" : "+v"(x[k]));
            if (tid + k * kCeThreads < nchunks) {
#pragma unroll
                for (int e = 0; e < 8; ++e) s += __builtin_amdgcn_exp2f(((float)x[k][e] - m) * kL2e);
            }
        }
        s = wsum2(s);
        if ((tid & 63) == 0) red[kCeThreads / 64 + wave] = s;
        __syncthreads();
        s = 0.f;
#pragma unroll
        for (int w = 0; w < kCeThreads / 64; ++w) s += red[kCeThreads / 64 + w];
        const float logz = m + __logf(s);
        int at = tid;
        asm volatile("" : "+v"(at));
        const auto dst = __builtin_amdgcn_make_buffer_rsrc(logits + (long long)r * ld, 0, vocab * 2, 0x00020000);
#pragma unroll
        for (int k = 0; k < kChunks; ++k) {
            asm volatile("" : "+v"(x[k]));
            const int c = at + k * kCeThreads;
            bf16x8_c o;
#pragma unroll
            for (int e = 0; e < 8; ++e) o[e] = (__bf16)0.f;
            if (c < nchunks) {
#pragma unroll
                for (int e = 0; e < 8; ++e) o[e] = (__bf16)(__builtin_amdgcn_exp2f(((float)x[k][e] - logz) * kL2e) * inv_n);
                if (c == label >> 3) {  // one thread of the work-group
                    float xl = 0.f;
#pragma unroll
                    for (int e = 0; e < 8; ++e)
                        if (e == (label & 7)) {
                            xl = (float)x[k][e];
                            o[e] = (__bf16)((__builtin_amdgcn_exp2f((xl - logz) * kL2e) - 1.f) * inv_n);
                        }
                    row_loss[r] = logz - xl;
                }
            }
            __builtin_amdgcn_raw_buffer_store_b128(__builtin_bit_cast(u32x4_c, o), dst, c * 16, 0, 0);
        }
        label = label1; label1 = label2; mask1 = mask2; counted = counted1;
    }
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
}

__global__ __launch_bounds__(256) void k_finish_loss(const float* __restrict__ row_loss, const int* __restrict__ n_counted,
                                                     float* __restrict__ loss_out, int T) {
    __shared__ float red[4];
    float s = 0.f;
    for (int t = threadIdx.x; t < T; t += 256) s += row_loss[t];
    s = wsum2(s);
    if ((threadIdx.x & 63) == 0) red[threadIdx.x >> 6] = s;
    __syncthreads();
    if (threadIdx.x == 0) {
        const int n = n_counted[0];
        loss_out[0] = n > 0 ? (red[0] + red[1] + red[2] + red[3]) / (float)n : 0.f;
    }
}

int launch_count_labels(const int* labels, const uint8_t* loss_mask, int T, int vocab, int* n_counted, float* row_loss, uint8_t* counted,
                        hipStream_t stream) {
    k_count_labels<<<1, 256, 0, stream>>>(labels, loss_mask, T, vocab, n_counted, row_loss, counted);
    ALCH_HIP_TRY(hipGetLastError());
    return ALCH_OK;
}

int launch_ce_chunk(alch_dtype dt, void* logits, long long ld, int rows, int vocab, const int* labels,
                    const uint8_t* loss_mask, const int* n_counted, float* row_loss, hipStream_t stream,
                    const int* rows_dev) {
    if (rows <= 0) return ALCH_OK;
    if (dt == ALCH_BF16 && vocab % 8 == 0 && ld % 8 == 0 && vocab <= kCeThreads * kCeChunks * 8 && aligned16(logits))
    {
        int n_cu = 0;
        ALCH_TRY(compute_units(&n_cu));
        const int chunks = ceil_div(vocab, 8 * kCeThreads), slots = chunks <= 4 ? 2 * n_cu : n_cu, grid = rows < slots ? rows : slots;
        auto kernel = chunks <= 4 ? k_ce_chunk_bf16_row<4> : chunks <= 8 ? k_ce_chunk_bf16_row<8> : k_ce_chunk_bf16_row<kCeChunks>;
        kernel<<<grid, kCeThreads, 0, stream>>>((__bf16*)logits, ld, rows, vocab, labels, loss_mask, n_counted, row_loss, rows_dev);
    }
    else if (dt == ALCH_BF16)
        k_ce_chunk<__bf16><<<rows, 256, 0, stream>>>((__bf16*)logits, ld, vocab, labels, loss_mask, n_counted, row_loss, rows_dev);
    else
        k_ce_chunk<float><<<rows, 256, 0, stream>>>((float*)logits, ld, vocab, labels, loss_mask, n_counted, row_loss, rows_dev);
    ALCH_HIP_TRY(hipGetLastError());
    return ALCH_OK;
}

int launch_finish_loss(const float* row_loss, const int* n_counted, float* loss_out, int T, hipStream_t stream) {
    k_finish_loss<<<1, 256, 0, stream>>>(row_loss, n_counted, loss_out, T);
    ALCH_HIP_TRY(hipGetLastError());
    return ALCH_OK;
}

}  // namespace alch
