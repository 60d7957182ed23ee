// Causal grouped-query attention in fp32 arithmetic, float or bf16 storage, any even head_dim up to 256: the fp32
// storage type and the head sizes that the bf16 matrix-core kernels (attn_mfma_kernels.h) do not take.
//
// Backward from the saved record (Section 4.1 of the paper: Q, K, V of the prompt tokens are what
// the serving side keeps): p_ij = exp(q_i.k_j/sqrt(D) - LSE_i) for j <= i in the same sequence,
// dV_j = sum_i p_ij dO_i, ds_ij = p_ij (dO_i.v_j - delta_i), dQ_i = sum_j ds_ij k_j / sqrt(D),
// dK_j = sum_i ds_ij q_i / sqrt(D); K/V gradients are summed over the query heads of a group.
// A sequence with a prefix (responses on the saved KV cache of their prompt, Section 4.1) also sees
// every key of the prefix sequence; the keys of a prefix collect gradient from all sequences that
// name it.
//
// All contractions run on the fp32 matrix instruction 32x32x2 (fp32 operands and sums).  A work-group owns 32 queries of
// one (sequence, head) -- or 32 keys of one (sequence, kv head) -- and its four wavefronts take the 32-key (32-query)
// blocks in turn; their sums meet in LDS in wavefront order, so results are deterministic.  Scores come out of the
// matrix unit in the layout in which they are an operand of the second contraction: lane = the row the work-group owns,
// register e of half h = row r(e, h) = 8 (e / 4) + 4 h + e % 4 of the other side.  Operands are read straight from
// memory: the row-major ones 16 bytes per lane along the head, those of the second contraction as whole 128-byte lines.
// What bounds it at the sizes it serves is latency, so the blocks of one work-group are spread over its wavefronts.
// A wavefront per row with two lane reductions per (row, key) pair took, 2 sequences x 128 tokens, 4 heads of 64, fp32:
// dQ 78 us, dK/dV 63 us, plus 9 us for delta and the RoPE backward.  With loads that depend on the head size by a branch,
// wavefronts adding their sums in turn and a launch for each gradient it was 21 + 31 us, without these 19 us in all.
#include <initializer_list>
#include <type_traits>

#include "attn_rows.h"

namespace alch {

typedef __attribute__((ext_vector_type(16))) float f32x16;
typedef __attribute__((ext_vector_type(4))) float f32x4;
typedef __attribute__((ext_vector_type(4))) __bf16 bf16x4;

static constexpr int kWaves = 4, kBlk = 32;

template <typename T> __device__ __forceinline__ float ldf(const T* p) { return (float)*p; }
template <typename T> __device__ __forceinline__ void stf(T* p, float v) { *p = (T)v; }
__device__ __forceinline__ f32x4 ld4(const float* p) { return *reinterpret_cast<const f32x4*>(p); }
__device__ __forceinline__ f32x4 ld4(const __bf16* p) {
    const bf16x4 v = *reinterpret_cast<const bf16x4*>(p);
    return f32x4{(float)v[0], (float)v[1], (float)v[2], (float)v[3]};
}

template <typename T>
struct AttnPlainParams {
    const T *Q, *K, *V, *O, *dO;
    float* LSE;  // read by the backward, written by the forward
    float* delta;
    T *dQ, *dK, *dV, *Oout;
    const int *cu, *prefix, *positions;
    int n_seqs, seq_begin, blocks, short_upto, Hq, Hkv, D;  // the grid: (head, block of 32 rows) x sequences from seq_begin on
    long long ldo;          // row stride of dQ, dK, dV
    float scale, log2_base;
    int rope;               // dQ and dK are rotated by minus the RoPE angle
    int vec;                // rows allow loads of four elements
};

// Elements d .. d+3 of a head row, zero from D on.
template <typename T>
__device__ __forceinline__ f32x4 head4(const T* row, int d, int D, bool vec) {
    if (vec && d + 4 <= D) return ld4(row + d);
    f32x4 v = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int i = 0; i < 4; ++i)
        if (d + i < D) v[i] = ldf(row + d + i);
    return v;
}

// A B^T over the head: rows ra (this lane's row of A) and rb (of B), both [*, D].  kFull: D = NB * 32 and rows that
// allow loads of four elements, so that no load depends on a condition.  Every 16 terms (heads of up to 32: all)
// are added in two sums of their own: one sum of all D terms rounds more often than the sum over the lanes of a wavefront by
// which the scores were formed before.  Errors against 64 bits, 2 x 128 tokens, heads of 64: O 1.25e-7, dQ 3.5e-7 (one sum:
// 2.0e-7, 4.3e-7; the lanes' sum: 1.6e-7, 3.6e-7); 1024 tokens, heads of 128: O 1.8e-7 (3.3e-7, 3.3e-7).  Unrolled, the loop
// has every block's loads in flight and spills from heads of 128 on.
template <typename T, int NB, bool kFull>
__device__ __forceinline__ f32x16 rows_product(const T* ra, const T* rb, int D, bool vec, int half) {
    constexpr int kRun = NB == 1 ? 4 : 2;
    f32x16 total;
#pragma unroll
    for (int e = 0; e < 16; ++e) total[e] = 0.f;
#pragma unroll 1
    for (int nb = 0; nb < NB; ++nb) {
        f32x4 a[4], b[4];
        const bool whole = kFull || (vec && nb * 32 + 32 <= D);
#pragma unroll
        for (int c = 0; c < 4; ++c) {
            const int d = nb * 32 + 8 * c + 4 * half;
            a[c] = whole ? ld4(ra + d) : head4(ra, d, D, vec);
            b[c] = whole ? ld4(rb + d) : head4(rb, d, D, vec);
        }
#pragma unroll
        for (int c = 0; c < 4; c += kRun) {
            f32x16 acc[2];
#pragma unroll
            for (int e = 0; e < 16; ++e) acc[0][e] = acc[1][e] = 0.f;
#pragma unroll
            for (int i = 0; i < 4 * kRun; ++i)
                acc[i & 1] = __builtin_amdgcn_mfma_f32_32x32x2f32(a[c + (i >> 2)][i & 3], b[c + (i >> 2)][i & 3], acc[i & 1], 0, 0, 0);
            total += acc[0] + acc[1];
        }
    }
    return total;
}
__device__ __forceinline__ int row_of(int e, int half) { return 8 * (e >> 2) + 4 * half + (e & 3); }

// Sums of the wavefronts on their way to a row-major block of 32 rows; value e of block nb of a lane is element
// (row_of(e), nb*32 + lane&31), or its transpose.  Up to 128 columns every wavefront has a block of its own in LDS and the
// reader adds them in order; beyond that they are added in turn into one.
template <int NB> struct FoldBuf {
    static constexpr int kLd = NB * 32 + 1, kBlocks = NB <= 4 ? kWaves : 1, kPitch = kBlk * kLd;
    float at[kBlocks * kPitch];
    __device__ __forceinline__ float sum(int i) const {
        float v = at[i];
#pragma unroll
        for (int w = 1; w < kBlocks; ++w) v += at[w * kPitch + i];
        return v;
    }
};
template <int NB, bool kTransposed>
__device__ __forceinline__ void fold(FoldBuf<NB>& buf, const f32x16 (&x)[NB], int wave, int lane, float factor) {
    constexpr int ld = FoldBuf<NB>::kLd;
    constexpr bool kOwn = FoldBuf<NB>::kBlocks > 1;
    __syncthreads();  // (the buffer has been read)
    for (int w = 0; w < (kOwn ? 1 : kWaves); ++w) {
        if (kOwn || wave == w) {
            float* base = buf.at + (kOwn ? wave * FoldBuf<NB>::kPitch : 0);
#pragma unroll
            for (int nb = 0; nb < NB; ++nb)
#pragma unroll
                for (int e = 0; e < 16; ++e) {
                    const int r = row_of(e, lane >> 5), c = lane & 31;
                    float* q = kTransposed ? base + c * ld + nb * 32 + r : base + r * ld + nb * 32 + c;
                    const float v = x[nb][e] * factor;
                    *q = kOwn || w == 0 ? v : *q + v;
                }
        }
        __syncthreads();
    }
}

// Any sum of the work-group not finite (the wavefronts' flags of not_finite)
__device__ __forceinline__ bool any_not_finite(float flag) { return __syncthreads_or(!(flag == 0.f)) != 0; }
// A row formed anew, in place of the sums of the wavefronts
template <int NB, typename T, int E>
__device__ __forceinline__ void replace_row(FoldBuf<NB>& buf, int r, const HeadRow<T, E>& x, int D) {
#pragma unroll
    for (int e = 0; e < E; ++e) {
        const int d = (int)(threadIdx.x & 63) + 64 * e;
        if (d >= D) continue;
        for (int w = 0; w < FoldBuf<NB>::kBlocks; ++w) buf.at[w * FoldBuf<NB>::kPitch + r * FoldBuf<NB>::kLd + d] = w == 0 ? x.v[e] : 0.f;
    }
}

// LDS [32][ld] -> rows of the output, scaled and, with `rope`, rotated by minus the RoPE angle.
template <typename T, int NB>
__device__ __forceinline__ void store_rows(const FoldBuf<NB>& buf, T* out, long long ldo, int rows, int D, float scale,
                                           bool rope, float log2_base, const int* positions, int token0, int row0) {
    constexpr int ld = FoldBuf<NB>::kLd;
    if (rope) {
        const int hd = D >> 1;
        for (int q = threadIdx.x; q < rows * hd; q += kWaves * 64) {
            const int r = q / hd, k = q - r * hd;
            const int pos = positions ? positions[token0 + r] : row0 + r;
            float sn, cs;
            sincosf((float)pos * exp2f(-2.f * (float)k / (float)D * log2_base), &sn, &cs);
            const float a = buf.sum(r * ld + k) * scale, b = buf.sum(r * ld + k + hd) * scale;
            stf(out + (long long)r * ldo + k, a * cs + b * sn);
            stf(out + (long long)r * ldo + k + hd, b * cs - a * sn);
        }
        return;
    }
    for (int q = threadIdx.x; q < rows * D; q += kWaves * 64) {
        const int r = q / D, k = q - r * D;
        stf(out + (long long)r * ldo + k, buf.sum(r * ld + k) * scale);
    }
}

// The key blocks that the queries i0 .. i0+31 of a sequence see: those of its prefix, then its own up to the diagonal.
struct KeyBlocks {
    int own0, len, pre0, pre_len, n_pre, n;
    __device__ __forceinline__ KeyBlocks(const int* cu, const int* prefix, int seq, int i0) {
        own0 = cu[seq];
        len = cu[seq + 1] - own0;
        const int pre = prefix ? prefix[seq] : -1;
        pre0 = pre >= 0 ? cu[pre] : 0;
        pre_len = pre >= 0 ? cu[pre + 1] - pre0 : 0;
        n_pre = (pre_len + kBlk - 1) / kBlk;
        n = n_pre + min(i0 + kBlk - 1, len - 1) / kBlk + 1;
    }
    __device__ __forceinline__ SeenKeys seen_by(int i) const { return SeenKeys{pre0, pre_len, own0, pre_len + i + 1}; }
    // first key of block b, keys of its sequence, its first row in the batch
    __device__ __forceinline__ void at(int b, int& j0, int& keys, int& row0) const {
        const bool in_pre = b < n_pre;
        j0 = (in_pre ? b : b - n_pre) * kBlk;
        keys = in_pre ? pre_len : len;
        row0 = in_pre ? pre0 : own0;
    }
};

template <typename T, int NB, bool kFull>
__global__ __launch_bounds__(kWaves * 64) void k_attn_fwd_plain(AttnPlainParams<T> p) {
    __shared__ FoldBuf<NB> buf;
    __shared__ float ml[2][kWaves][kBlk];
    const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), half = lane >> 5;
    const int seq = p.seq_begin + blockIdx.y, h = (int)blockIdx.x % p.Hq, kv = h / (p.Hq / p.Hkv), D = kFull ? NB * 32 : p.D;
    const int i0 = (p.blocks - 1 - (int)blockIdx.x / p.Hq) * kBlk;  // the longest rows first
    const KeyBlocks kb(p.cu, p.prefix, seq, i0);
    if (i0 >= kb.len || kb.len <= p.short_upto) return;
    const long long ldq = (long long)p.Hq * D, ldk = (long long)p.Hkv * D;
    const int i = min(i0 + (lane & 31), kb.len - 1);  // this lane's query
    const T* q = p.Q + (kb.own0 + i) * ldq + (long long)h * D;
    f32x16 Ot[NB];  // transposed: rows d, columns queries
#pragma unroll
    for (int nb = 0; nb < NB; ++nb)
#pragma unroll
        for (int e = 0; e < 16; ++e) Ot[nb][e] = 0.f;
    float m = -INFINITY, l = 0.f;
    for (int b = wave; b < kb.n; b += kWaves) {
        int j0, keys, row0;
        kb.at(b, j0, keys, row0);
        const int lim = b < kb.n_pre ? keys - 1 : i;  // last visible key
        f32x16 S = rows_product<T, NB, kFull>(p.K + (row0 + min(j0 + (lane & 31), keys - 1)) * ldk + (long long)kv * D, q, D, p.vec, half);
        float mx = m;
#pragma unroll
        for (int e = 0; e < 16; ++e) {
            S[e] = j0 + row_of(e, half) <= lim ? S[e] * p.scale : -INFINITY;
            mx = fmaxf(mx, S[e]);
        }
        mx = fmaxf(mx, __shfl_xor(mx, 32, 64));
        const float alpha = expf(m - mx);  // every query sees at least one key of every block: mx is finite
        m = mx;
        float sum = 0.f;
#pragma unroll
        for (int e = 0; e < 16; ++e) {
            S[e] = expf(S[e] - mx);
            sum += S[e];
        }
        l = l * alpha + sum + __shfl_xor(sum, 32, 64);
#pragma unroll
        for (int nb = 0; nb < NB; ++nb)
#pragma unroll
            for (int e = 0; e < 16; ++e) Ot[nb][e] *= alpha;
        const T* v = p.V + row0 * ldk + (long long)kv * D;
#pragma unroll
        for (int e = 0; e < 16; ++e) {
            const T* vr = v + min(j0 + row_of(e, half), keys - 1) * ldk;
#pragma unroll
            for (int nb = 0; nb < NB; ++nb) {
                const int d = nb * 32 + (lane & 31);
                Ot[nb] = __builtin_amdgcn_mfma_f32_32x32x2f32(kFull || d < D ? ldf(vr + d) : 0.f, S[e], Ot[nb], 0, 0, 0);
            }
        }
    }
    if (half == 0) { ml[0][wave][lane] = m; ml[1][wave][lane] = l; }
    __syncthreads();
    float M = -INFINITY, L = 0.f;
#pragma unroll
    for (int w = 0; w < kWaves; ++w) M = fmaxf(M, ml[0][w][lane & 31]);
#pragma unroll
    for (int w = 0; w < kWaves; ++w) L += ml[1][w][lane & 31] * expf(ml[0][w][lane & 31] - M);
    const int rows = min(kBlk, kb.len - i0);
    float flag = 0.f;
#pragma unroll
    for (int nb = 0; nb < NB; ++nb) flag = not_finite(Ot[nb], flag);
    if (any_not_finite(flag)) {  // formed again from the visible keys alone (attn_rows.h)
        for (int r = wave; r < rows; r += kWaves) {
            HeadRow<T, (NB + 1) / 2> o;
            float lse;
            attn_fwd_row(p.Q + (kb.own0 + i0 + r) * ldq + (long long)h * D, p.K + (long long)kv * D, p.V + (long long)kv * D, ldk,
                         kb.seen_by(i0 + r), D, p.scale, o, lse);
            replace_row(buf, r, o, D);
        }
        __syncthreads();
    } else {
        fold<NB, true>(buf, Ot, wave, lane, expf(m - M) / L);
    }
    store_rows(buf, p.Oout + (kb.own0 + i0) * ldq + (long long)h * D, ldq, rows, D, 1.f, false, 0.f, nullptr, 0, 0);
    if (wave == 0 && half == 0 && lane < rows) p.LSE[(long long)(kb.own0 + i0 + lane) * p.Hq + h] = M + logf(L);
}

// delta_i = sum_d dO O of one row, half of the elements per lane, in four sums
template <typename T>
__device__ __forceinline__ float row_delta(const T* go, const T* o, int D, bool vec, int half) {
    f32x4 part = {0.f, 0.f, 0.f, 0.f};
    for (int d = 4 * half; d < D; d += 8) {
        const f32x4 a = head4(go, d, D, vec), b = head4(o, d, D, vec);
#pragma unroll
        for (int c = 0; c < 4; ++c) part[c] = __builtin_fmaf(a[c], b[c], part[c]);
    }
    const float del = (part[0] + part[1]) + (part[2] + part[3]);
    return del + __shfl_xor(del, 32, 64);
}

// dQ of block `block` (heads first, then 32-query blocks); kDelta: also writes delta
template <typename T, int NB, bool kFull, bool kDelta>
__device__ __forceinline__ void attn_bwd_dq_block(const AttnPlainParams<T>& p, FoldBuf<NB>& buf, int block) {
    const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), half = lane >> 5;
    const int seq = p.seq_begin + blockIdx.y, h = block % p.Hq, kv = h / (p.Hq / p.Hkv), D = kFull ? NB * 32 : p.D;
    const int i0 = (p.blocks - 1 - block / p.Hq) * kBlk;
    const KeyBlocks kb(p.cu, p.prefix, seq, i0);
    if (i0 >= kb.len || kb.len <= p.short_upto) return;
    const long long ldq = (long long)p.Hq * D, ldk = (long long)p.Hkv * D;
    const int i = min(i0 + (lane & 31), kb.len - 1);
    const long long qoff = (kb.own0 + i) * ldq + (long long)h * D, roff = (long long)(kb.own0 + i) * p.Hq + h;
    const T *q = p.Q + qoff, *go = p.dO + qoff, *o = p.O + qoff;
    const float del = row_delta(go, o, D, kFull || p.vec, half);
    if (kDelta && wave == 0 && half == 0 && i0 + lane < kb.len) p.delta[roff] = del;
    const float lse = p.LSE[roff];
    f32x16 dQ[NB];
#pragma unroll
    for (int nb = 0; nb < NB; ++nb)
#pragma unroll
        for (int e = 0; e < 16; ++e) dQ[nb][e] = 0.f;
    for (int b = wave; b < kb.n; b += kWaves) {
        int j0, keys, row0;
        kb.at(b, j0, keys, row0);
        const int lim = b < kb.n_pre ? keys - 1 : i;
        const long long koff = (row0 + min(j0 + (lane & 31), keys - 1)) * ldk + (long long)kv * D;
        f32x16 S = rows_product<T, NB, kFull>(p.K + koff, q, D, p.vec, half);
        const f32x16 dP = rows_product<T, NB, kFull>(p.V + koff, go, D, p.vec, half);
#pragma unroll
        for (int e = 0; e < 16; ++e)
            S[e] = j0 + row_of(e, half) <= lim ? expf(S[e] * p.scale - lse) * (dP[e] - del) : 0.f;
        const T* k = p.K + row0 * ldk + (long long)kv * D;
#pragma unroll
        for (int e = 0; e < 16; ++e) {
            const T* kr = k + min(j0 + row_of(e, half), keys - 1) * ldk;
#pragma unroll
            for (int nb = 0; nb < NB; ++nb) {
                const int d = nb * 32 + (lane & 31);
                dQ[nb] = __builtin_amdgcn_mfma_f32_32x32x2f32(S[e], kFull || d < D ? ldf(kr + d) : 0.f, dQ[nb], 0, 0, 0);
            }
        }
    }
    float flag = 0.f;
#pragma unroll
    for (int nb = 0; nb < NB; ++nb) flag = not_finite(dQ[nb], flag);
    if (any_not_finite(flag)) {
        for (int r = wave; r < min(kBlk, kb.len - i0); r += kWaves) {
            const long long at = (kb.own0 + i0 + r) * ldq + (long long)h * D;
            HeadRow<T, (NB + 1) / 2> x;
            float del_again;
            attn_dq_row(p.Q + at, p.dO + at, p.O + at, p.K + (long long)kv * D, p.V + (long long)kv * D, ldk, kb.seen_by(i0 + r), D,
                        p.scale, p.LSE[(long long)(kb.own0 + i0 + r) * p.Hq + h], x, del_again);
            replace_row(buf, r, x, D);
        }
        __syncthreads();
    } else {
        fold<NB, false>(buf, dQ, wave, lane, 1.f);
    }
    store_rows(buf, p.dQ + (kb.own0 + i0) * p.ldo + (long long)h * D, p.ldo, min(kBlk, kb.len - i0), D, p.scale,
               p.rope, p.log2_base, p.positions, kb.own0 + i0, i0);
}

// dK, dV of block `block` (kv heads first, then 32-key blocks); kDelta: forms delta of the queries it meets by itself
// instead of reading it
template <typename T, int NB, bool kFull, bool kDelta>
__device__ __forceinline__ void attn_bwd_dkv_block(const AttnPlainParams<T>& p, FoldBuf<NB>& buf, int block) {
    const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), half = lane >> 5;
    const int seq = p.seq_begin + blockIdx.y, kv = block % p.Hkv, G = p.Hq / p.Hkv, D = kFull ? NB * 32 : p.D;
    const int own0 = p.cu[seq], len = p.cu[seq + 1] - own0, j0 = block / p.Hkv * kBlk;
    if (j0 >= len || len <= p.short_upto) return;
    const long long ldq = (long long)p.Hq * D, ldk = (long long)p.Hkv * D;
    const int j = min(j0 + (lane & 31), len - 1);  // this lane's key
    const T *k = p.K + (own0 + j) * ldk + (long long)kv * D, *v = p.V + (own0 + j) * ldk + (long long)kv * D;
    f32x16 dK[NB], dV[NB];
#pragma unroll
    for (int nb = 0; nb < NB; ++nb)
#pragma unroll
        for (int e = 0; e < 16; ++e) dK[nb][e] = dV[nb][e] = 0.f;
    // query blocks: those of the key's own sequence from the diagonal on, then all of every sequence that names it as
    // prefix, each for every head of the group; block number `turn` goes to wavefront turn % kWaves
    int turn = 0;
    for (int c = seq; c < p.n_seqs; ++c) {
        if (c > seq && !(p.prefix && p.prefix[c] == seq)) continue;
        const int row0 = p.cu[c], n = p.cu[c + 1] - row0;
        for (int i0 = c == seq ? j0 : 0; i0 < n; i0 += kBlk)
            for (int h = kv * G; h < (kv + 1) * G; ++h, ++turn) {
                if (turn % kWaves != wave) continue;
                const long long qoff = (row0 + min(i0 + (lane & 31), n - 1)) * ldq + (long long)h * D;
                float lse = 0.f, del = 0.f;  // of this lane's query row
                if constexpr (kDelta) {
                    lse = p.LSE[(long long)(row0 + min(i0 + (lane & 31), n - 1)) * p.Hq + h];
                    del = row_delta(p.dO + qoff, p.O + qoff, D, kFull || p.vec, half);
                }
                f32x16 S = rows_product<T, NB, kFull>(p.Q + qoff, k, D, p.vec, half);
                f32x16 dP = rows_product<T, NB, kFull>(p.dO + qoff, v, D, p.vec, half);
#pragma unroll
                for (int e = 0; e < 16; ++e) {
                    const int i = i0 + row_of(e, half);
                    const long long roff = (long long)(row0 + min(i, n - 1)) * p.Hq + h;
                    const bool seen = i < n && (c > seq || i >= j0 + (lane & 31));
                    const float le = kDelta ? __shfl(lse, row_of(e, half), 64) : p.LSE[roff];
                    const float de = kDelta ? __shfl(del, row_of(e, half), 64) : p.delta[roff];
                    S[e] = seen ? expf(S[e] * p.scale - le) : 0.f;
                    dP[e] = S[e] * (dP[e] - de);
                }
                const T *qh = p.Q + row0 * ldq + (long long)h * D, *gh = p.dO + row0 * ldq + (long long)h * D;
                if constexpr (kFull) {
                    // the elements of four rows are on their way while those of the four before are multiplied (left to the
                    // compiler, each load of heads of 128 stood before its use: 870 us for 2000 tokens, 504 us so)
                    float gb[2][4][NB], qb[2][4][NB];
                    auto load = [&](int e0, float (&g)[4][NB], float (&q)[4][NB]) {
#pragma unroll
                        for (int e = 0; e < 4; ++e) {
                            const long long ro = min(i0 + row_of(e0 + e, half), n - 1) * ldq + (lane & 31);
#pragma unroll
                            for (int nb = 0; nb < NB; ++nb) {
                                g[e][nb] = ldf(gh + ro + nb * 32);
                                q[e][nb] = ldf(qh + ro + nb * 32);
                            }
                        }
                    };
                    load(0, gb[0], qb[0]);
#pragma unroll
                    for (int e0 = 0; e0 < 16; e0 += 4) {
                        if (e0 + 4 < 16) load(e0 + 4, gb[(e0 / 4 + 1) & 1], qb[(e0 / 4 + 1) & 1]);
                        __builtin_amdgcn_sched_barrier(0);
#pragma unroll
                        for (int e = 0; e < 4; ++e)
#pragma unroll
                            for (int nb = 0; nb < NB; ++nb) {
                                dV[nb] = __builtin_amdgcn_mfma_f32_32x32x2f32(S[e0 + e], gb[(e0 / 4) & 1][e][nb], dV[nb], 0, 0, 0);
                                dK[nb] = __builtin_amdgcn_mfma_f32_32x32x2f32(dP[e0 + e], qb[(e0 / 4) & 1][e][nb], dK[nb], 0, 0, 0);
                            }
                        __builtin_amdgcn_sched_barrier(0);
                    }
                    continue;
                }
#pragma unroll
                for (int e = 0; e < 16; ++e) {
                    const long long ro = min(i0 + row_of(e, half), n - 1) * ldq;
#pragma unroll
                    for (int nb = 0; nb < NB; ++nb) {
                        const int d = nb * 32 + (lane & 31);
                        dV[nb] = __builtin_amdgcn_mfma_f32_32x32x2f32(S[e], kFull || d < D ? ldf(gh + ro + d) : 0.f, dV[nb], 0, 0, 0);
                        dK[nb] = __builtin_amdgcn_mfma_f32_32x32x2f32(dP[e], kFull || d < D ? ldf(qh + ro + d) : 0.f, dK[nb], 0, 0, 0);
                    }
                }
            }
        if (!p.prefix) break;
    }
    const int rows = min(kBlk, len - j0);
    const long long out = (own0 + j0) * p.ldo + (long long)kv * D;
    float flag = 0.f;
#pragma unroll
    for (int nb = 0; nb < NB; ++nb) flag = not_finite(dV[nb], not_finite(dK[nb], flag));
    if (any_not_finite(flag)) {
        for (int r = wave; r < rows; r += kWaves) {
            HeadRow<T, (NB + 1) / 2> dk, dv;
            const long long at = (own0 + j0 + r) * ldk + (long long)kv * D;
            attn_dkv_row(p.K + at, p.V + at, p.Q, p.dO, p.O, p.LSE, nullptr, p.Hq, kv * G, (kv + 1) * G, p.cu, p.prefix, p.n_seqs, seq,
                         j0 + r, D,
                         p.scale, dk, dv);
            replace_row(buf, r, dk, D);
#pragma unroll
            for (int e = 0; e < (NB + 1) / 2; ++e)
                if (lane + 64 * e < D) stf(p.dV + out + (long long)r * p.ldo + lane + 64 * e, dv.v[e]);
        }
        __syncthreads();
        store_rows(buf, p.dK + out, p.ldo, rows, D, p.scale, p.rope, p.log2_base, p.positions, own0 + j0, j0);
        return;
    }
    fold<NB, false>(buf, dK, wave, lane, 1.f);
    store_rows(buf, p.dK + out, p.ldo, rows, D, p.scale, p.rope, p.log2_base, p.positions, own0 + j0, j0);
    fold<NB, false>(buf, dV, wave, lane, 1.f);
    store_rows(buf, p.dV + out, p.ldo, rows, D, 1.f, false, 0.f, nullptr, 0, 0);
}

template <typename T, int NB, bool kFull>
__global__ __launch_bounds__(kWaves * 64) void k_attn_bwd_dq_plain(AttnPlainParams<T> p) {
    __shared__ FoldBuf<NB> buf;
    attn_bwd_dq_block<T, NB, kFull, true>(p, buf, (int)blockIdx.x);
}
template <typename T, int NB, bool kFull>
__global__ __launch_bounds__(kWaves * 64) void k_attn_bwd_dkv_plain(AttnPlainParams<T> p) {
    __shared__ FoldBuf<NB> buf;
    attn_bwd_dkv_block<T, NB, kFull, false>(p, buf, (int)blockIdx.x);
}
// Both in one launch: key blocks first (they take longer), then query blocks.
template <typename T, int NB, bool kFull>
__global__ __launch_bounds__(kWaves * 64) void k_attn_bwd_plain(AttnPlainParams<T> p) {
    __shared__ FoldBuf<NB> buf;
    const int key_blocks = p.blocks * p.Hkv;
    if ((int)blockIdx.x < key_blocks) attn_bwd_dkv_block<T, NB, kFull, true>(p, buf, (int)blockIdx.x);
    else attn_bwd_dq_block<T, NB, kFull, false>(p, buf, (int)blockIdx.x - key_blocks);
}

// ---- a row at a time, for sequences of up to short_upto tokens: a wavefront takes one head of one sequence,
// or every gridDim.z-th row of it
template <typename T, int E>
__device__ __forceinline__ void store_row(const HeadRow<T, E>& x, float* tmp, T* out, int D, float scale, bool rope, float log2_base, int pos) {
    const int lane = threadIdx.x & 63;
    if (rope)
#pragma unroll
        for (int e = 0; e < E; ++e)
            if (lane + 64 * e < D) tmp[lane + 64 * e] = x.v[e];  // (of this wavefront alone)
#pragma unroll
    for (int e = 0; e < E; ++e) {
        const int d = lane + 64 * e, hd = D >> 1, k = d < hd ? d : d - hd;
        if (d >= D) continue;
        float v = x.v[e] * scale;
        if (rope) {
            float sn, cs;
            sincosf((float)pos * exp2f(-2.f * (float)k / (float)D * log2_base), &sn, &cs);
            const float other = tmp[d < hd ? d + hd : d - hd] * scale;
            v = d < hd ? v * cs + other * sn : v * cs - other * sn;
        }
        stf(out + d, v);
    }
}

template <typename T, int E>
__global__ __launch_bounds__(kWaves * 64) void k_attn_fwd_rows(AttnPlainParams<T> p) {
    const int seq = p.seq_begin + blockIdx.y, row0 = p.cu[seq], len = p.cu[seq + 1] - row0;
    const int h = (int)blockIdx.x * kWaves + __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), kv = h / (p.Hq / p.Hkv), lane = threadIdx.x & 63;
    if (len > p.short_upto || h >= p.Hq) return;
    const long long ldq = (long long)p.Hq * p.D, ldk = (long long)p.Hkv * p.D, kvo = (long long)kv * p.D;
    for (int i = blockIdx.z; i < len; i += gridDim.z) {
        HeadRow<T, E> o;
        float lse;
        const long long at = (row0 + i) * ldq + (long long)h * p.D;
        attn_fwd_row(p.Q + at, p.K + kvo, p.V + kvo, ldk, SeenKeys{0, 0, row0, i + 1}, p.D, p.scale, o, lse);
#pragma unroll
        for (int e = 0; e < E; ++e)
            if (lane + 64 * e < p.D) stf(p.Oout + at + lane + 64 * e, o.v[e]);
        if (lane == 0) p.LSE[(long long)(row0 + i) * p.Hq + h] = lse;
    }
}

template <typename T, int E>
__global__ __launch_bounds__(kWaves * 64) void k_attn_bwd_dq_rows(AttnPlainParams<T> p) {  // also writes delta
    __shared__ float tmp[kWaves][64 * E];
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), lane = threadIdx.x & 63, D = p.D;
    const int seq = p.seq_begin + blockIdx.y, row0 = p.cu[seq], len = p.cu[seq + 1] - row0, h = (int)blockIdx.x * kWaves + wave;
    if (len > p.short_upto || h >= p.Hq) return;
    const long long ldq = (long long)p.Hq * D, ldk = (long long)p.Hkv * D, kvo = (long long)(h / (p.Hq / p.Hkv)) * D;
    for (int r = blockIdx.z; r < len; r += gridDim.z) {
        const long long at = (row0 + r) * ldq + (long long)h * D, row = (long long)(row0 + r) * p.Hq + h;
        HeadRow<T, E> x;
        float delta;
        attn_dq_row(p.Q + at, p.dO + at, p.O + at, p.K + kvo, p.V + kvo, ldk, SeenKeys{0, 0, row0, r + 1}, D, p.scale, p.LSE[row], x, delta);
        if (lane == 0) p.delta[row] = delta;
        store_row(x, tmp[wave], p.dQ + (row0 + r) * p.ldo + (long long)h * D, D, p.scale, p.rope, p.log2_base, p.positions ? p.positions[row0 + r] : r);
    }
}
template <typename T, int E>
__global__ __launch_bounds__(kWaves * 64) void k_attn_bwd_dkv_rows(AttnPlainParams<T> p) {
    __shared__ float tmp[kWaves][64 * E];
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), lane = threadIdx.x & 63, D = p.D, G = p.Hq / p.Hkv;
    const int seq = p.seq_begin + blockIdx.y, row0 = p.cu[seq], len = p.cu[seq + 1] - row0, kv = (int)blockIdx.x * kWaves + wave;
    if (len > p.short_upto || kv >= p.Hkv) return;
    for (int r = blockIdx.z; r < len; r += gridDim.z) {
        const long long at = ((long long)(row0 + r) * p.Hkv + kv) * D, out = (row0 + r) * p.ldo + (long long)kv * D;
        HeadRow<T, E> dk, dv;
        attn_dkv_row(p.K + at, p.V + at, p.Q, p.dO, p.O, p.LSE, p.delta, p.Hq, kv * G, (kv + 1) * G, p.cu, nullptr, p.n_seqs, seq, r, D, p.scale,
                     dk, dv);
        store_row(dk, tmp[wave], p.dK + out, D, p.scale, p.rope, p.log2_base, p.positions ? p.positions[row0 + r] : r);
#pragma unroll
        for (int e = 0; e < E; ++e)
            if (lane + 64 * e < D) stf(p.dV + out + lane + 64 * e, dv.v[e]);
    }
}

// A tile kernel spends a work-group's blocks on every (sequence, head), however short: of sequences of a few tokens it takes
// less time to form a row at a time.  Up to how many tokens that is so, forward / backward in us, rows against tiles, 8000
// tokens, 8/2 heads: bf16 heads of 64 (tiles: the matrix-core kernels) 8 tokens 36 / 181 against 40 / 267, 12 tokens 47 / 227
// against 28 / 211; fp32 64 8 tokens 35 / 258 against 79 / 349, 12 tokens 48 / 293 against 55 / 299; bf16 80 16 tokens 70 /
// 341 against 175 / 455, 24 tokens 140 / 538 against 143 / 379; fp32 128 16 tokens 59 / 362 against 90 / 428; bf16 160 24
// tokens 229 / 765 against 453 / 1029.  The rows are a launch (backward: two) more where there are long sequences beside
// them, so the tiles of the short ones have to be worth it: more than per_cu work-groups for each compute unit (forward of
// one sequence of 1000 tokens and 256 of 4, 8 heads: fp32 64 83 against 169 us, bf16 64 40 against 30 us and left to the
// tiles there, 1024 of 4: 51 against 60 us).
int rows_up_to(int D, int Hq, int per_cu, int first, int n_seqs, const int* cu_host, const int* prefix, ShortRows* rows) {
    *rows = ShortRows{};
    if (prefix) return ALCH_OK;
    const int limit = D > 128 ? 24 : D <= 32 || D == 64 ? 8 : 16;
    long long n = 0, tokens = 0;
    for (int s = first; s < n_seqs; ++s) {
        const int len = cu_host[s + 1] - cu_host[s];
        if (len > 0 && len <= limit) { ++n; tokens += len; }
    }
    int n_cu = 0;
    ALCH_TRY(compute_units(&n_cu));
    if (n * Hq >= (long long)per_cu * n_cu) *rows = ShortRows{limit, (int)(tokens / (2 * n)) > 1 ? (int)(tokens / (2 * n)) : 1};
    return ALCH_OK;
}

// (forward of 64 sequences of 4 tokens, 8 heads, rows against tiles: bf16 80 12 against 19 us, fp32 64 13 and 13 us)
static int plain_per_cu(int D) { return D > 64 ? 2 : 4; }

// rows of a head start on a multiple of four elements
template <typename T>
static bool head_rows_vec(int D, std::initializer_list<const void*> ptrs) {
    bool ok = D % 4 == 0;
    for (const void* q : ptrs) ok = ok && reinterpret_cast<uintptr_t>(q) % (4 * sizeof(T)) == 0;
    return ok;
}

// f(32-column blocks of a head, whether it fills them in rows of aligned groups of four: told apart for the head sizes of
// the fp32 layers)
template <typename T, typename F>
static int with_blocks(int D, bool vec, F&& f) {
    auto g = [&](auto NB) {
        constexpr int kNB = decltype(NB)::value;
        if constexpr (std::is_same<T, float>::value && (kNB == 2 || kNB == 4))
            if (vec && D == kNB * 32) return f(NB, std::true_type{});
        f(NB, std::false_type{});
    };
    if (D <= 32) g(std::integral_constant<int, 1>{});
    else if (D <= 64) g(std::integral_constant<int, 2>{});
    else if (D <= 128) g(std::integral_constant<int, 4>{});
    else g(std::integral_constant<int, 8>{});
    ALCH_HIP_TRY(hipGetLastError());
    return ALCH_OK;
}

// f(number of sequences) for ranges of at most 65535 of them (the limit of a grid's second dimension)
template <typename T, typename F>
static void by_sequences(AttnPlainParams<T>& p, int seq_begin, F&& f) {
    for (int s = seq_begin; s < p.n_seqs; s += 65535) {
        p.seq_begin = s;
        f(p.n_seqs - s < 65535 ? p.n_seqs - s : 65535);
    }
}

template <typename T>
static AttnPlainParams<T> bwd_params(const AttnArgs& a) {
    AttnPlainParams<T> p = {};
    p.Q = (const T*)a.Q; p.K = (const T*)a.K; p.V = (const T*)a.V; p.O = (const T*)a.O; p.dO = (const T*)a.dO;
    p.LSE = const_cast<float*>(a.LSE); p.delta = a.delta;
    p.dQ = (T*)a.dQ; p.dK = (T*)a.dK; p.dV = (T*)a.dV; p.ldo = a.ld_dqkv;
    p.cu = a.cu_seqlens; p.prefix = a.prefix; p.positions = a.positions;
    p.n_seqs = a.n_seqs; p.Hq = a.Hq; p.Hkv = a.Hkv; p.D = a.D;
    p.scale = 1.f / sqrtf((float)a.D);
    p.rope = a.rope_base > 0.f;
    p.log2_base = p.rope ? log2f(a.rope_base) : 0.f;
    p.vec = head_rows_vec<T>(a.D, {a.Q, a.K, a.V, a.O, a.dO});
    p.short_upto = a.rows.up_to;
    return p;
}

// the elements of a head that a lane of a row kernel holds
template <typename F>
static int with_row(int D, F&& f) {
    if (D <= 64) f(std::integral_constant<int, 1>{});
    else if (D <= 128) f(std::integral_constant<int, 2>{});
    else f(std::integral_constant<int, 4>{});
    ALCH_HIP_TRY(hipGetLastError());
    return ALCH_OK;
}

template <typename T>
static int attn_bwd_rows_t(const AttnArgs& a, hipStream_t stream) {
    AttnPlainParams<T> p = bwd_params<T>(a);
    return with_row(a.D, [&](auto E) {
        by_sequences(p, 0, [&](int n) {
            k_attn_bwd_dq_rows<T, decltype(E)::value><<<dim3(ceil_div(a.Hq, kWaves), n, a.rows.step), kWaves * 64, 0, stream>>>(p);
            k_attn_bwd_dkv_rows<T, decltype(E)::value><<<dim3(ceil_div(a.Hkv, kWaves), n, a.rows.step), kWaves * 64, 0, stream>>>(p);
        });
    });
}
int launch_attn_bwd_rows(const AttnArgs& a, hipStream_t stream) {
    return a.dtype == ALCH_BF16 ? attn_bwd_rows_t<__bf16>(a, stream) : attn_bwd_rows_t<float>(a, stream);
}

template <typename T>
static int attn_bwd_generic_t(const AttnArgs& a, hipStream_t stream) {
    AttnPlainParams<T> p = bwd_params<T>(a);
    const int longest = longest_sequence(a.cu_seqlens_host, 0, a.n_seqs);
    if (longest <= a.rows.up_to) return ALCH_OK;
    p.blocks = ceil_div(longest, kBlk);
    int n_cu = 0;
    ALCH_TRY(compute_units(&n_cu));
    return with_blocks<T>(a.D, p.vec, [&](auto NB, auto full) {
        constexpr int kNB = decltype(NB)::value;
        constexpr bool kFull = decltype(full)::value;
        // A batch whose work-groups all find a compute unit is bound by the latency of one: both gradients in one launch,
        // delta formed where it is needed (2 x 128 tokens, 4 heads of 64: 19 us).  Beyond that the registers of the dK/dV
        // code would halve the wavefronts of the dQ work-groups.
        if constexpr (kNB <= 4)
            if ((long long)p.blocks * (a.Hq + a.Hkv) * a.n_seqs <= n_cu) {
                k_attn_bwd_plain<T, kNB, kFull><<<dim3(p.blocks * (a.Hq + a.Hkv), a.n_seqs), kWaves * 64, 0, stream>>>(p);
                return;
            }
        by_sequences(p, 0, [&](int n) {  // also writes delta, which the second kernel reads for all sequences
            k_attn_bwd_dq_plain<T, kNB, kFull><<<dim3(p.blocks * a.Hq, n), kWaves * 64, 0, stream>>>(p);
        });
        by_sequences(p, 0, [&](int n) {
            k_attn_bwd_dkv_plain<T, kNB, kFull><<<dim3(p.blocks * a.Hkv, n), kWaves * 64, 0, stream>>>(p);
        });
    });
}

int launch_attn_bwd_generic(const AttnArgs& a, hipStream_t stream) {
    if (a.T <= 0) return ALCH_OK;
    if (a.D > 256) return fail(ALCH_ERR_UNSUPPORTED, "head_dim %d > 256", a.D);
    AttnArgs b = a;
    ALCH_TRY(rows_up_to(a.D, a.Hq, plain_per_cu(a.D), 0, a.n_seqs, a.cu_seqlens_host, a.prefix, &b.rows));
    if (b.rows.up_to) ALCH_TRY(launch_attn_bwd_rows(b, stream));
    return a.dtype == ALCH_BF16 ? attn_bwd_generic_t<__bf16>(b, stream) : attn_bwd_generic_t<float>(b, stream);
}

template <typename T>
static AttnPlainParams<T> fwd_params(const void* Q, const void* K, const void* V, void* O, float* LSE, int n_seqs, const int* cu,
                                     const int* prefix, int Hq, int Hkv, int D, int short_upto) {
    AttnPlainParams<T> p = {};
    p.Q = (const T*)Q; p.K = (const T*)K; p.V = (const T*)V; p.Oout = (T*)O; p.LSE = LSE;
    p.cu = cu; p.prefix = prefix; p.n_seqs = n_seqs; p.Hq = Hq; p.Hkv = Hkv; p.D = D;
    p.scale = 1.f / sqrtf((float)D);
    p.vec = head_rows_vec<T>(D, {Q, K, V});
    p.short_upto = short_upto;
    return p;
}

template <typename T>
static int attn_fwd_rows_t(AttnPlainParams<T> p, int seq_begin, int step, hipStream_t stream) {
    return with_row(p.D, [&](auto E) {
        by_sequences(p, seq_begin, [&](int n) {
            k_attn_fwd_rows<T, decltype(E)::value><<<dim3(ceil_div(p.Hq, kWaves), n, step), kWaves * 64, 0, stream>>>(p);
        });
    });
}
int launch_attn_fwd_rows(alch_dtype dt, const void* Q, const void* K, const void* V, void* O, float* LSE, int n_seqs, const int* cu_seqlens,
                         int seq_begin, int Hq, int Hkv, int D, const ShortRows& rows, hipStream_t stream) {
    return dt == ALCH_BF16
               ? attn_fwd_rows_t(fwd_params<__bf16>(Q, K, V, O, LSE, n_seqs, cu_seqlens, nullptr, Hq, Hkv, D, rows.up_to), seq_begin, rows.step, stream)
               : attn_fwd_rows_t(fwd_params<float>(Q, K, V, O, LSE, n_seqs, cu_seqlens, nullptr, Hq, Hkv, D, rows.up_to), seq_begin, rows.step, stream);
}

template <typename T>
static int attn_fwd_generic_t(const void* Q, const void* K, const void* V, void* O, float* LSE, int n_seqs, const int* cu,
                              const int* cu_host, const int* prefix, int seq_begin, int Hq, int Hkv, int D, int short_upto, hipStream_t stream) {
    AttnPlainParams<T> p = fwd_params<T>(Q, K, V, O, LSE, n_seqs, cu, prefix, Hq, Hkv, D, short_upto);
    const int longest = longest_sequence(cu_host, seq_begin, n_seqs);
    if (longest <= short_upto) return ALCH_OK;
    p.blocks = ceil_div(longest, kBlk);
    return with_blocks<T>(D, p.vec, [&](auto NB, auto full) {
        by_sequences(p, seq_begin, [&](int n) {
            k_attn_fwd_plain<T, decltype(NB)::value, decltype(full)::value><<<dim3(p.blocks * Hq, n), kWaves * 64, 0, stream>>>(p);
        });
    });
}

int launch_attn_fwd_generic(alch_dtype dt, const void* Q, const void* K, const void* V, void* O, float* LSE, int T,
                            int n_seqs, const int* cu_seqlens, const int* cu_seqlens_host, const int* prefix,
                            int seq_begin, int Hq, int Hkv, int D, hipStream_t stream) {
    if (T - cu_seqlens_host[seq_begin] <= 0) return ALCH_OK;
    if (D > 256) return fail(ALCH_ERR_UNSUPPORTED, "head_dim %d > 256", D);
    ShortRows rows;
    ALCH_TRY(rows_up_to(D, Hq, plain_per_cu(D), seq_begin, n_seqs, cu_seqlens_host, prefix, &rows));
    if (rows.up_to) ALCH_TRY(launch_attn_fwd_rows(dt, Q, K, V, O, LSE, n_seqs, cu_seqlens, seq_begin, Hq, Hkv, D, rows, stream));
    return dt == ALCH_BF16
               ? attn_fwd_generic_t<__bf16>(Q, K, V, O, LSE, n_seqs, cu_seqlens, cu_seqlens_host, prefix, seq_begin, Hq, Hkv, D, rows.up_to, stream)
               : attn_fwd_generic_t<float>(Q, K, V, O, LSE, n_seqs, cu_seqlens, cu_seqlens_host, prefix, seq_begin, Hq, Hkv, D, rows.up_to, stream);
}

}  // namespace alch
