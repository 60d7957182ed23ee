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
// dQ 78 us, dK/dV 63 us, plus 9 us for delta and the RoPE backward; with these inside, now 21 and 31 us.
#include <initializer_list>
#include <type_traits>

#include "kernels.h"

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
    int n_seqs, seq_begin, blocks, Hq, Hkv, D;  // the grid: (head, block of 32 rows) x sequences from seq_begin on
    long long ldo;          // row stride of dQ, dK, dV
    float scale, log2_base;  // log2_base > 0: dQ and dK are rotated by minus the RoPE angle
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

// acc += A B^T over the head: rows ra (this lane's row of A) and rb (of B), both [*, D].
template <typename T, int NB>
__device__ __forceinline__ f32x16 rows_product(const T* ra, const T* rb, int D, bool vec, int half, f32x16 acc) {
#pragma unroll
    for (int nb = 0; nb < NB; ++nb) {
        f32x4 a[4], b[4];
        const bool whole = vec && nb * 32 + 32 <= D;
#pragma unroll
        for (int c = 0; c < 4; ++c) {
            const int d = nb * 32 + 8 * c + 4 * half;
            a[c] = whole ? ld4(ra + d) : head4(ra, d, D, vec);
            b[c] = whole ? ld4(rb + d) : head4(rb, d, D, vec);
        }
#pragma unroll
        for (int c = 0; c < 4; ++c)
#pragma unroll
            for (int i = 0; i < 4; ++i) acc = __builtin_amdgcn_mfma_f32_32x32x2f32(a[c][i], b[c][i], acc, 0, 0, 0);
    }
    return acc;
}
__device__ __forceinline__ int row_of(int e, int half) { return 8 * (e >> 2) + 4 * half + (e & 3); }

// Sums of the wavefronts, added in order into LDS [32 rows][kLd]; value e of block nb of a lane is element
// (row_of(e), nb*32 + lane&31), or its transpose.
template <int NB, bool kTransposed>
__device__ __forceinline__ void fold(float* buf, int ld, const f32x16 (&x)[NB], int wave, int lane, float factor) {
    for (int w = 0; w < kWaves; ++w) {
        __syncthreads();
        if (wave == w) {
#pragma unroll
            for (int nb = 0; nb < NB; ++nb)
#pragma unroll
                for (int e = 0; e < 16; ++e) {
                    const int r = row_of(e, lane >> 5), c = lane & 31;
                    float* q = kTransposed ? buf + c * ld + nb * 32 + r : buf + r * ld + nb * 32 + c;
                    const float v = x[nb][e] * factor;
                    *q = w == 0 ? v : *q + v;
                }
        }
    }
    __syncthreads();
}

// LDS [32][ld] -> rows of the output, scaled and, with log2_base > 0, rotated by minus the RoPE angle.
template <typename T>
__device__ __forceinline__ void store_rows(const float* buf, int ld, T* out, long long ldo, int rows, int D, float scale,
                                           float log2_base, const int* positions, int token0, int row0) {
    if (log2_base > 0.f) {
        const int hd = D >> 1;
        for (int q = threadIdx.x; q < rows * hd; q += kWaves * 64) {
            const int r = q / hd, k = q - r * hd;
            const int pos = positions ? positions[token0 + r] : row0 + r;
            float sn, cs;
            sincosf((float)pos * exp2f(-2.f * (float)k / (float)D * log2_base), &sn, &cs);
            const float a = buf[r * ld + k] * scale, b = buf[r * ld + k + hd] * scale;
            stf(out + (long long)r * ldo + k, a * cs + b * sn);
            stf(out + (long long)r * ldo + k + hd, b * cs - a * sn);
        }
        return;
    }
    for (int q = threadIdx.x; q < rows * D; q += kWaves * 64) {
        const int r = q / D, k = q - r * D;
        stf(out + (long long)r * ldo + k, buf[r * ld + k] * scale);
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
    // first key of block b, keys of its sequence, its first row in the batch
    __device__ __forceinline__ void at(int b, int& j0, int& keys, int& row0) const {
        const bool in_pre = b < n_pre;
        j0 = (in_pre ? b : b - n_pre) * kBlk;
        keys = in_pre ? pre_len : len;
        row0 = in_pre ? pre0 : own0;
    }
};

template <typename T, int NB>
__global__ __launch_bounds__(kWaves * 64) void k_attn_fwd_plain(AttnPlainParams<T> p) {
    constexpr int kLd = NB * 32 + 1;
    __shared__ float buf[kBlk * kLd];
    __shared__ float ml[2][kWaves][kBlk];
    const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), half = lane >> 5;
    const int seq = p.seq_begin + blockIdx.y, h = (int)blockIdx.x % p.Hq, kv = h / (p.Hq / p.Hkv), D = p.D;
    const int i0 = (p.blocks - 1 - (int)blockIdx.x / p.Hq) * kBlk;  // the longest rows first
    const KeyBlocks kb(p.cu, p.prefix, seq, i0);
    if (i0 >= kb.len) return;
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
        f32x16 S;
#pragma unroll
        for (int e = 0; e < 16; ++e) S[e] = 0.f;
        S = rows_product<T, NB>(p.K + (row0 + min(j0 + (lane & 31), keys - 1)) * ldk + (long long)kv * D, q, D, p.vec, half, S);
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
                Ot[nb] = __builtin_amdgcn_mfma_f32_32x32x2f32(d < D ? ldf(vr + d) : 0.f, S[e], Ot[nb], 0, 0, 0);
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
    fold<NB, true>(buf, kLd, Ot, wave, lane, expf(m - M) / L);
    const int rows = min(kBlk, kb.len - i0);
    store_rows(buf, kLd, p.Oout + (kb.own0 + i0) * ldq + (long long)h * D, ldq, rows, D, 1.f, 0.f, nullptr, 0, 0);
    if (wave == 0 && half == 0 && lane < rows) p.LSE[(long long)(kb.own0 + i0 + lane) * p.Hq + h] = M + logf(L);
}

template <typename T, int NB>
__global__ __launch_bounds__(kWaves * 64) void k_attn_bwd_dq_plain(AttnPlainParams<T> p) {
    constexpr int kLd = NB * 32 + 1;
    __shared__ float buf[kBlk * kLd];
    const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), half = lane >> 5;
    const int seq = p.seq_begin + blockIdx.y, h = (int)blockIdx.x % p.Hq, kv = h / (p.Hq / p.Hkv), D = p.D;
    const int i0 = (p.blocks - 1 - (int)blockIdx.x / p.Hq) * kBlk;
    const KeyBlocks kb(p.cu, p.prefix, seq, i0);
    if (i0 >= kb.len) return;
    const long long ldq = (long long)p.Hq * D, ldk = (long long)p.Hkv * D;
    const int i = min(i0 + (lane & 31), kb.len - 1);
    const long long qoff = (kb.own0 + i) * ldq + (long long)h * D, roff = (long long)(kb.own0 + i) * p.Hq + h;
    const T *q = p.Q + qoff, *go = p.dO + qoff, *o = p.O + qoff;
    // delta_i = sum_d dO O of this lane's query, half of the elements per lane
    float del = 0.f;
    for (int d = 4 * half; d < D; d += 8) {
        const f32x4 a = head4(go, d, D, p.vec), b = head4(o, d, D, p.vec);
#pragma unroll
        for (int c = 0; c < 4; ++c) del = __builtin_fmaf(a[c], b[c], del);
    }
    del += __shfl_xor(del, 32, 64);
    if (wave == 0 && half == 0 && i0 + lane < kb.len) p.delta[roff] = del;
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
        f32x16 S, dP;
#pragma unroll
        for (int e = 0; e < 16; ++e) S[e] = dP[e] = 0.f;
        S = rows_product<T, NB>(p.K + koff, q, D, p.vec, half, S);
        dP = rows_product<T, NB>(p.V + koff, go, D, p.vec, half, dP);
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
                dQ[nb] = __builtin_amdgcn_mfma_f32_32x32x2f32(S[e], d < D ? ldf(kr + d) : 0.f, dQ[nb], 0, 0, 0);
            }
        }
    }
    fold<NB, false>(buf, kLd, dQ, wave, lane, 1.f);
    store_rows(buf, kLd, p.dQ + (kb.own0 + i0) * p.ldo + (long long)h * D, p.ldo, min(kBlk, kb.len - i0), D, p.scale,
               p.log2_base, p.positions, kb.own0 + i0, i0);
}

template <typename T, int NB>
__global__ __launch_bounds__(kWaves * 64) void k_attn_bwd_dkv_plain(AttnPlainParams<T> p) {
    constexpr int kLd = NB * 32 + 1;
    __shared__ float buf[kBlk * kLd];
    const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), half = lane >> 5;
    const int seq = p.seq_begin + blockIdx.y, kv = (int)blockIdx.x % p.Hkv, G = p.Hq / p.Hkv, D = p.D;
    const int own0 = p.cu[seq], len = p.cu[seq + 1] - own0, j0 = (int)blockIdx.x / p.Hkv * kBlk;
    if (j0 >= len) return;
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
                f32x16 S, dP;
#pragma unroll
                for (int e = 0; e < 16; ++e) S[e] = dP[e] = 0.f;
                S = rows_product<T, NB>(p.Q + qoff, k, D, p.vec, half, S);
                dP = rows_product<T, NB>(p.dO + qoff, v, D, p.vec, half, dP);
#pragma unroll
                for (int e = 0; e < 16; ++e) {
                    const int i = i0 + row_of(e, half);
                    const long long roff = (long long)(row0 + min(i, n - 1)) * p.Hq + h;
                    const bool seen = i < n && (c > seq || i >= j0 + (lane & 31));
                    S[e] = seen ? expf(S[e] * p.scale - p.LSE[roff]) : 0.f;
                    dP[e] = S[e] * (dP[e] - p.delta[roff]);
                }
                const T *qh = p.Q + row0 * ldq + (long long)h * D, *gh = p.dO + row0 * ldq + (long long)h * D;
#pragma unroll
                for (int e = 0; e < 16; ++e) {
                    const long long ro = min(i0 + row_of(e, half), n - 1) * ldq;
#pragma unroll
                    for (int nb = 0; nb < NB; ++nb) {
                        const int d = nb * 32 + (lane & 31);
                        dV[nb] = __builtin_amdgcn_mfma_f32_32x32x2f32(S[e], d < D ? ldf(gh + ro + d) : 0.f, dV[nb], 0, 0, 0);
                        dK[nb] = __builtin_amdgcn_mfma_f32_32x32x2f32(dP[e], d < D ? ldf(qh + ro + d) : 0.f, dK[nb], 0, 0, 0);
                    }
                }
            }
        if (!p.prefix) break;
    }
    const int rows = min(kBlk, len - j0);
    const long long out = (own0 + j0) * p.ldo + (long long)kv * D;
    fold<NB, false>(buf, kLd, dK, wave, lane, 1.f);
    store_rows(buf, kLd, p.dK + out, p.ldo, rows, D, p.scale, p.log2_base, p.positions, own0 + j0, j0);
    fold<NB, false>(buf, kLd, dV, wave, lane, 1.f);
    store_rows(buf, kLd, p.dV + out, p.ldo, rows, D, 1.f, 0.f, nullptr, 0, 0);
}

// rows of a head start on a multiple of four elements
template <typename T>
static bool head_rows_vec(int D, std::initializer_list<const void*> ptrs) {
    bool ok = D % 4 == 0;
    for (const void* q : ptrs) ok = ok && reinterpret_cast<uintptr_t>(q) % (4 * sizeof(T)) == 0;
    return ok;
}

template <typename F>
static int with_blocks(int D, F&& f) {
    if (D > 256) return fail(ALCH_ERR_UNSUPPORTED, "head_dim %d > 256", D);
    if (D <= 32) f(std::integral_constant<int, 1>{});
    else if (D <= 64) f(std::integral_constant<int, 2>{});
    else if (D <= 128) f(std::integral_constant<int, 4>{});
    else f(std::integral_constant<int, 8>{});
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
static int attn_bwd_generic_t(const AttnArgs& a, hipStream_t stream) {
    AttnPlainParams<T> p = {};
    p.Q = (const T*)a.Q; p.K = (const T*)a.K; p.V = (const T*)a.V; p.O = (const T*)a.O; p.dO = (const T*)a.dO;
    p.LSE = const_cast<float*>(a.LSE); p.delta = a.delta;
    p.dQ = (T*)a.dQ; p.dK = (T*)a.dK; p.dV = (T*)a.dV; p.ldo = a.ld_dqkv;
    p.cu = a.cu_seqlens; p.prefix = a.prefix; p.positions = a.positions;
    p.n_seqs = a.n_seqs; p.Hq = a.Hq; p.Hkv = a.Hkv; p.D = a.D;
    p.scale = 1.f / sqrtf((float)a.D);
    p.log2_base = a.rope_base > 0.f ? log2f(a.rope_base) : 0.f;
    p.vec = head_rows_vec<T>(a.D, {a.Q, a.K, a.V, a.O, a.dO});
    p.blocks = ceil_div(a.max_seqlen, kBlk);
    if (p.blocks <= 0 || a.n_seqs <= 0) return ALCH_OK;
    return with_blocks(a.D, [&](auto NB) {
        by_sequences(p, 0, [&](int n) {  // also writes delta, which the second kernel reads for all sequences
            k_attn_bwd_dq_plain<T, decltype(NB)::value><<<dim3(p.blocks * a.Hq, n), kWaves * 64, 0, stream>>>(p);
        });
        by_sequences(p, 0, [&](int n) {
            k_attn_bwd_dkv_plain<T, decltype(NB)::value><<<dim3(p.blocks * a.Hkv, n), kWaves * 64, 0, stream>>>(p);
        });
    });
}

int launch_attn_bwd_generic(const AttnArgs& a, hipStream_t stream) {
    if (a.T <= 0) return ALCH_OK;
    return a.dtype == ALCH_BF16 ? attn_bwd_generic_t<__bf16>(a, stream) : attn_bwd_generic_t<float>(a, stream);
}

template <typename T>
static int attn_fwd_generic_t(const void* Q, const void* K, const void* V, void* O, float* LSE, int n_seqs, int max_seqlen,
                              const int* cu, const int* prefix, int seq_begin, int Hq, int Hkv, int D, hipStream_t stream) {
    AttnPlainParams<T> p = {};
    p.Q = (const T*)Q; p.K = (const T*)K; p.V = (const T*)V; p.Oout = (T*)O; p.LSE = LSE;
    p.cu = cu; p.prefix = prefix; p.n_seqs = n_seqs; p.Hq = Hq; p.Hkv = Hkv; p.D = D;
    p.scale = 1.f / sqrtf((float)D);
    p.vec = head_rows_vec<T>(D, {Q, K, V});
    p.blocks = ceil_div(max_seqlen, kBlk);
    return with_blocks(D, [&](auto NB) {
        by_sequences(p, seq_begin, [&](int n) {
            k_attn_fwd_plain<T, decltype(NB)::value><<<dim3(p.blocks * Hq, n), kWaves * 64, 0, stream>>>(p);
        });
    });
}

int launch_attn_fwd_generic(alch_dtype dt, const void* Q, const void* K, const void* V, void* O, float* LSE, int T,
                            int n_seqs, int max_seqlen, const int* cu_seqlens, const int* cu_seqlens_host, const int* prefix,
                            int seq_begin, int Hq, int Hkv, int D, hipStream_t stream) {
    if (T - cu_seqlens_host[seq_begin] <= 0 || max_seqlen <= 0) return ALCH_OK;
    return dt == ALCH_BF16
               ? attn_fwd_generic_t<__bf16>(Q, K, V, O, LSE, n_seqs, max_seqlen, cu_seqlens, prefix, seq_begin, Hq, Hkv, D, stream)
               : attn_fwd_generic_t<float>(Q, K, V, O, LSE, n_seqs, max_seqlen, cu_seqlens, prefix, seq_begin, Hq, Hkv, D, stream);
}

}  // namespace alch
