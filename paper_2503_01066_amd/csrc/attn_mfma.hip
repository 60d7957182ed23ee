// Matrix-core attention: the choice of kernel, and the instantiations for heads of 128 (attn_mfma_kernels.h).
#include "attn_mfma_kernels.h"

namespace alch {

// Batches of heads of 64 that the grid of the matrix-core kernels cannot hold run on the fp32-arithmetic ones, which take any.
// (Heads of 128 are refused there: they have never had another path.)
static bool head_size_fits(int D, int n_seqs, const int* cu_host) {
    return D == 128 || (D == 64 && n_seqs <= kMaxGridSeqs && longest_sequence(cu_host, 0, n_seqs) <= kMaxGridBlocks * 128);
}

bool attn_mfma_supported(const AttnArgs& a) {
    return a.dtype == ALCH_BF16 && head_size_fits(a.D, a.n_seqs, a.cu_seqlens_host) && a.T > 0 && a.ld_dqkv % 8 == 0 && aligned16(a.Q) && aligned16(a.K) &&
           aligned16(a.V) && aligned16(a.dO) && aligned16(a.O);
}

int launch_attn_bwd_mfma(const AttnArgs& a, hipStream_t stream) {
    if (a.D == 128) return attn_bwd_mfma<128>(a, stream);
    AttnArgs b = a;
    b.max_seqlen = longest_sequence(a.cu_seqlens_host, 0, a.n_seqs);
    ALCH_TRY(rows_up_to(a.D, a.Hq, kRowsPerCu, 0, a.n_seqs, a.cu_seqlens_host, a.prefix, &b.rows));
    if (b.rows.up_to) ALCH_TRY(launch_attn_bwd_rows(b, stream));
    return b.max_seqlen > b.rows.up_to ? attn_bwd_mfma_d64(b, stream) : ALCH_OK;
}

int launch_attn_fwd(alch_dtype dt, const void* Q, const void* K, const void* V, void* O, float* LSE, int T,
                    int n_seqs, int max_seqlen, const int* cu_seqlens, const int* cu_seqlens_host, const int* prefix,
                    const int* prefix_host, int seq_begin, int Hq, int Hkv, int D, hipStream_t stream) {
    if (seq_begin >= n_seqs) return ALCH_OK;
    const double pairs = attn_pairs(n_seqs - seq_begin, cu_seqlens_host + seq_begin, nullptr) +
                         (attn_pairs(n_seqs, cu_seqlens_host, prefix_host) - attn_pairs(n_seqs, cu_seqlens_host, nullptr));
    TraceScope ts(kTraceAttnFwd, 4.0 * D * Hq * pairs, 0.0, stream);
    if (dt == ALCH_BF16 && head_size_fits(D, n_seqs, cu_seqlens_host) && T > 0 && aligned16(Q) && aligned16(K) && aligned16(V) && aligned16(O)) {
        if (D == 128) return attn_fwd_mfma<128>(Q, K, V, O, LSE, n_seqs, max_seqlen, cu_seqlens, prefix, seq_begin, Hq, Hkv, 0, stream);
        const int longest = longest_sequence(cu_seqlens_host, seq_begin, n_seqs);
        ShortRows rows;
        ALCH_TRY(rows_up_to(D, Hq, kRowsPerCu, seq_begin, n_seqs, cu_seqlens_host, prefix, &rows));
        if (rows.up_to) ALCH_TRY(launch_attn_fwd_rows(dt, Q, K, V, O, LSE, n_seqs, cu_seqlens, seq_begin, Hq, Hkv, D, rows, stream));
        return longest > rows.up_to ? attn_fwd_mfma_d64(Q, K, V, O, LSE, n_seqs, longest, cu_seqlens, prefix, seq_begin, Hq, Hkv, rows.up_to, stream)
                                    : ALCH_OK;
    }
    return launch_attn_fwd_generic(dt, Q, K, V, O, LSE, T, n_seqs, cu_seqlens, cu_seqlens_host, prefix, seq_begin, Hq, Hkv, D, stream);
}

}  // namespace alch
