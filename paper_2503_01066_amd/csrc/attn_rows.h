// Attention a row at a time: one wavefront per query (forward, dQ) or key (dK, dV), elements lane + 64 e of a head in its
// lanes.  The tile kernels multiply the pairs above the diagonal with a probability of zero instead of leaving them out, which
// is the same for every finite number, but a NaN or an infinity in a key, a value, a query or an output gradient would reach
// rows that do not see it (0 * inf).  A tile kernel whose sums are not finite therefore forms its rows again with these, which
// visit visible pairs only.  Finite batches never come here; rows that are not finite by their own right come out so again.
// The other use is sequences too short to fill a tile of 32 keys (attn_generic.hip: rows_up_to).
#pragma once
#include "kernels.h"

namespace alch {

// NaN if any of the sums is not finite, else the old value
template <typename V>
__device__ __forceinline__ float not_finite(const V& x, float flag) {
#pragma unroll
    for (int e = 0; e < 16; ++e) flag = __builtin_fmaf(x[e], 0.f, flag);
    return flag;
}

__device__ __forceinline__ float lanes_sum(float v) {
#pragma unroll
    for (int d = 32; d > 0; d >>= 1) v += __shfl_xor(v, d, 64);
    return v;
}

template <typename T, int E>
struct HeadRow {  // elements of one row of a head, zero from D on
    float v[E];
    __device__ __forceinline__ void load(const T* row, int D) {
#pragma unroll
        for (int e = 0; e < E; ++e) {
            const int d = (int)(threadIdx.x & 63) + 64 * e;
            v[e] = d < D ? (float)row[d] : 0.f;
        }
    }
    __device__ __forceinline__ void clear() {
#pragma unroll
        for (int e = 0; e < E; ++e) v[e] = 0.f;
    }
    __device__ __forceinline__ float dot(const HeadRow& o) const {
        float s = 0.f;
#pragma unroll
        for (int e = 0; e < E; ++e) s += v[e] * o.v[e];
        return lanes_sum(s);
    }
    __device__ __forceinline__ void add(float a, const HeadRow& o) {
#pragma unroll
        for (int e = 0; e < E; ++e) v[e] += a * o.v[e];
    }
};

// The keys that query i of a sequence sees, by row of the batch: its prefix's, then own0 .. own0 + i.
struct SeenKeys {
    int pre0, pre_len, own0, n;
    __device__ __forceinline__ int row(int jj) const { return jj < pre_len ? pre0 + jj : own0 + jj - pre_len; }
};

// K, V: of the kv head
template <typename T, int E>
__device__ void attn_fwd_row(const T* q, const T* K, const T* V, long long ldk, const SeenKeys& keys, int D, float scale, HeadRow<T, E>& o,
                             float& lse) {
    HeadRow<T, E> qr;
    qr.load(q, D);
    o.clear();
    float m = -INFINITY, l = 0.f;
    for (int jj = 0; jj < keys.n; ++jj) {
        const long long at = keys.row(jj) * ldk;
        HeadRow<T, E> k, v;
        k.load(K + at, D);
        v.load(V + at, D);
        const float s = qr.dot(k) * scale, mn = fmaxf(m, s), corr = expf(m - mn), p = expf(s - mn);
        l = l * corr + p;
#pragma unroll
        for (int e = 0; e < E; ++e) o.v[e] = o.v[e] * corr + p * v.v[e];
        m = mn;
    }
#pragma unroll
    for (int e = 0; e < E; ++e) o.v[e] /= l;
    lse = m + logf(l);
}

// (without the factor scale of the result)
template <typename T, int E>
__device__ void attn_dq_row(const T* q, const T* dO, const T* O, const T* K, const T* V, long long ldk, const SeenKeys& keys, int D,
                            float scale, float lse, HeadRow<T, E>& dq, float& delta) {
    HeadRow<T, E> qr, g, o;
    qr.load(q, D);
    g.load(dO, D);
    o.load(O, D);
    delta = g.dot(o);
    dq.clear();
    for (int jj = 0; jj < keys.n; ++jj) {
        const long long at = keys.row(jj) * ldk;
        HeadRow<T, E> k, v;
        k.load(K + at, D);
        v.load(V + at, D);
        dq.add(expf(qr.dot(k) * scale - lse) * (g.dot(v) - delta), k);
    }
}

// Sums over the query heads h_first .. h_end-1 of the rows that see key j of sequence seq: the sequence's own from j on, then
// all of the sequences that name it as their prefix.  dk without the factor scale.  delta: of every row, or null (formed here).
template <typename T, int E>
__device__ void attn_dkv_row(const T* k, const T* v, const T* Q, const T* dO, const T* O, const float* LSE, const float* delta, int Hq, int h_first, int h_end,
                             const int* cu, const int* prefix, int n_seqs, int seq, int j, int D, float scale, HeadRow<T, E>& dk,
                             HeadRow<T, E>& dv) {
    HeadRow<T, E> kr, vr;
    kr.load(k, D);
    vr.load(v, D);
    dk.clear();
    dv.clear();
    for (int c = seq; c < n_seqs; ++c) {
        if (c > seq && !(prefix && prefix[c] == seq)) continue;
        for (int h = h_first; h < h_end; ++h)
            for (int i = cu[c] + (c == seq ? j : 0); i < cu[c + 1]; ++i) {
                const long long at = ((long long)i * Hq + h) * D;
                HeadRow<T, E> q, g, o;
                q.load(Q + at, D);
                g.load(dO + at, D);
                float del;
                if (delta) {
                    del = delta[(long long)i * Hq + h];
                } else {
                    o.load(O + at, D);
                    del = g.dot(o);
                }
                const float p = expf(kr.dot(q) * scale - LSE[(long long)i * Hq + h]);
                dv.add(p, g);
                dk.add(p * (vr.dot(g) - del), q);
            }
        if (!prefix) break;
    }
}

}  // namespace alch
