// Matrix-core attention: the instantiations for heads of 64 (attn_mfma_kernels.h).
#include "attn_mfma_kernels.h"

namespace alch {

int attn_bwd_mfma_d64(const AttnArgs& a, hipStream_t stream) { return attn_bwd_mfma<64>(a, stream); }

int attn_fwd_mfma_d64(const void* Q, const void* K, const void* V, void* O, float* LSE, int n_seqs, int max_seqlen,
                      const int* cu_seqlens, const int* prefix, int seq_begin, int Hq, int Hkv, int short_upto, hipStream_t stream) {
    return attn_fwd_mfma<64>(Q, K, V, O, LSE, n_seqs, max_seqlen, cu_seqlens, prefix, seq_begin, Hq, Hkv, short_upto, stream);
}

}  // namespace alch
