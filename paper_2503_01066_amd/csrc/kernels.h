// Internal launch interfaces between the translation units of libalch.
#pragma once
#include "common.h"

namespace alch {

// ---- capture/pack ----------------------------------------------------------------------
static constexpr int kMaxStreamsPerLaunch = 16;
static constexpr int kGatherGridMax = 1 << 20;  // one work-group per candidate row, capped
size_t pack_workspace_bytes(int total_tokens);
int launch_pack(const uint8_t* mask, int T, const int* cu_seqlens, int n_seqs, int n_streams,
                const alch_stream* streams, long long capacity, int* kept_index, int* cu_kept,
                int* n_kept_and_status, void* workspace, hipStream_t stream, bool traced = true);
int launch_pack_gather(int T, int n_streams, const alch_stream* streams, long long capacity, const int* kept_index,
                       const int* n_kept_and_status, hipStream_t stream, bool traced = true);

// ---- GEMM ------------------------------------------------------------------------------
// C[M,N] (+)= sum over segments of A_s(M,K_s) * B_s(K_s,N), fp32 accumulation.
//   a_kmajor: A(m,k) = A[m*lda + k]   else A(m,k) = A[k*lda + m]
//   b_kmajor: B(k,n) = B[n*ldb + k]   else B(k,n) = B[k*ldb + n]
// The output may be split along M into up to three row ranges with their own base
// pointers (rows [m_begin_i, m_begin_{i+1}) go to out[i].C, row index relative to
// m_begin_i, leading dimension ldc).
static constexpr int kMaxGemmSegs = 4;  // operand pairs summed into one product
static constexpr int kMaxGemmOuts = 3;  // row ranges of C with their own base pointers
struct GemmSeg {
    const void* A;
    const void* B;
    int K;
    long long lda, ldb;
};
struct GemmOut {
    void* C;
    int m_begin;  // first row of the product that goes to C; of a product cut by columns, the first column
    long long ldc;
    const void* B = nullptr;  // cut by columns: the right operand's part behind these columns
};
enum GemmEpilogue { kEpiNone = 0, kEpiSwigluBwd = 1 };
struct GemmDesc {
    int M = 0, N = 0;
    bool a_kmajor = true, b_kmajor = true;
    int n_seg = 0;
    GemmSeg seg[kMaxGemmSegs];
    int n_out = 0;
    GemmOut out[kMaxGemmOuts];
    int accumulate = 0;
    const void* residual = nullptr;  // with accumulate: what is added instead of the old values of C (row stride of C)
    // out[] are column ranges of the product, each with a right operand of its own (k-major, row stride of seg[0].B), one
    // operand pair: products with a common left operand in one launch
    bool by_cols = false;
    alch_dtype dtype = ALCH_BF16;
    // kEpiSwigluBwd: the product is dAct [M, N]; with G, U [M, N] (ld = ldgu) the kernel writes
    // dG to out[0].C[:, 0:N], dU to out[0].C[:, N:2N] and Act = silu(G)*U to act_out [M, N].
    int epilogue = kEpiNone;
    const void* G = nullptr;
    const void* U = nullptr;
    long long ldgu = 0;
    void* act_out = nullptr;
    // optional device-resident sizes (matrix-core kernel only): effective M = min(*m_dev, M); effective K of
    // every operand pair = min(*k_dev, K), token-major operands only.  Rows / contraction steps beyond them are neither read
    // nor written.
    const int* m_dev = nullptr;
    const int* k_dev = nullptr;
    // optional scratch (matrix-core kernel only): when the last round of tiles would leave at least half of the
    // compute units idle, every tile of that round is split along the contraction over s work-groups, which
    // write fp32 partial tiles here; a second kernel adds them in a fixed order.  kGemmSplitWsBytes always suffices.
    void* split_ws = nullptr;
    size_t split_ws_bytes = 0;
    // cut the contraction into the same parts whichever of the matrix-core kernels runs (those of the 256x256 one),
    // so that the result has the same bits: see stack_backward_impl
    bool keep_parts = false;
};
static constexpr size_t kGemmSplitWsBytes = (size_t)64 << 20;
int launch_gemm(const GemmDesc& d, hipStream_t stream);
// A data gradient and a weight gradient that do not depend on one another: whether they run as one launch, and that launch.
bool gemm_together(const GemmDesc& data, const GemmDesc& weight);
int launch_gemm_together(const GemmDesc& data, const GemmDesc& weight, hipStream_t stream);
// used by launch_gemm
bool gemm_mfma_supported(const GemmDesc& d);
bool gemm_cols_together(const GemmDesc& d);
int launch_gemm_mfma(const GemmDesc& d, hipStream_t stream);
bool gemm_mfma_together(const GemmDesc& data, const GemmDesc& weight);
int launch_gemm_mfma_together(const GemmDesc& data, const GemmDesc& weight, hipStream_t stream);
int launch_gemm_generic(const GemmDesc& d, hipStream_t stream);

// ---- row-wise kernels --------------------------------------------------------------------
// H = X * rsqrt(mean(X^2)+eps) * g   (rows of width `width`)
// rows_dev (optional, bf16 row kernel only): the row count is min(*rows_dev, T), read on the device.
int launch_rmsnorm_fwd(alch_dtype dt, const void* X, const void* g, void* H, int T, int width, float eps,
                       hipStream_t stream, const int* rows_dev = nullptr);
// dX = resid + rmsnorm_bwd(dH; X, g)   (resid may be NULL; resid_mask zeroes resid rows where mask==0);
// dg (+)= sum_t dH*X*r  (dg may be NULL).  partial: fp32 scratch [rmsnorm_bwd_blocks(T), width].
// hn_out (may be NULL): also writes the normalised rows X*r*g themselves, the operand of the weight gradients
// that follow, so that X is read once for both.
int rmsnorm_bwd_blocks(int T);
// sums (may be NULL): dg is left to a later launch_gain_sums, which adds the partial rows of up to two such calls at once;
// `partial` of the first has to stay until then.
struct GainSums {
    struct { const float* partial; void* dg; int rows; } of[2];
    int n = 0;
};
// Rows of an RMSNorm backward (see launch_rmsnorm_bwd); partial null: no gain gradient.
struct NormBwdRows {
    const void *dH, *X, *g, *resid;
    const uint8_t* resid_mask;
    void* dX;
    float* partial;
    int Trows, width;
    float eps;
    void* hn_out;
};
// fp32: a weight gradient in one launch with the RMSNorm backward, or with the sums of the gain gradients, that do not depend on
// it: whether it can be, and those launches (dg as launch_rmsnorm_bwd, left to `sums`).
bool gemm_beside_rows(const GemmDesc& weight, int width);
int launch_gemm_beside_norm(const GemmDesc& weight, NormBwdRows rows, void* dg, GainSums& sums, hipStream_t stream);
int launch_gemm_beside_gains(const GemmDesc& weight, const GainSums& sums, int width, int accumulate, hipStream_t stream);
int launch_gain_sums(alch_dtype dt, const GainSums& sums, int width, int accumulate, hipStream_t stream);
int launch_rmsnorm_bwd(alch_dtype dt, const void* dH, const void* X, const void* g, const void* resid,
                       const uint8_t* resid_mask, void* dX, void* dg, int accumulate, float* partial, int T,
                       int width, float eps, hipStream_t stream, const int* rows_dev = nullptr, void* hn_out = nullptr,
                       GainSums* sums = nullptr);
// inv[t] = rank of token t among the first *n_rows entries of index (the kept tokens, ascending), -1 if absent; of a head also
// kept_labels[r] = labels[index[r]] and chunk_rows[c] = rows of chunk c among the kept ones
int launch_kept_rows(const int* index, const int* n_rows, int* inv, int T, hipStream_t stream, const int* labels = nullptr,
                     int* kept_labels = nullptr, int n_chunks = 0, int chunk = 0, int* chunk_rows = nullptr);
// out [T, row_bytes] = src[inv[t], :] where inv[t] >= 0, zeros elsewhere; a second pair of tensors likewise
int launch_scatter_rows(const void* src, const int* inv, void* out, int T, size_t row_bytes, hipStream_t stream, const void* src2 = nullptr,
                        void* out2 = nullptr, size_t row_bytes2 = 0);
// Act = silu(G) * U
int launch_swiglu_act(alch_dtype dt, const void* G, const void* U, void* Act, long long n, hipStream_t stream);
// In-place rotary rotation of q [T, n_q, D] and k [T, n_kv, D].
int launch_rope(alch_dtype dt, void* q, int n_q, void* k, int n_kv, int T, int D, const int* positions,
                const int* cu_seqlens, int n_seqs, float base, hipStream_t stream);
// out = a with rows zeroed where mask == 0 (mask may be NULL: plain copy)
int launch_masked_copy(alch_dtype dt, const void* a, const uint8_t* mask, void* out, int T, int width,
                       hipStream_t stream);

// ---- low-rank adapters ---------------------------------------------------------------------
static constexpr int kLoraSlot = 64;       // columns of one zero-padded rank slot (rank <= 64)
static constexpr int kLoraMaxSplits = 64;  // token splits of the adapter-gradient reduction
// Y[t, 0:r] = alpha * sum_k X[t, k] * S[j*lds + k] (S is an [r, K] matrix); columns r .. slot_cols-1 of Y
// are written as zeros; r = 0 (S may be null) zero-fills the slot.  Up to three problems per launch, all
// with Trows rows, the same alpha, and outputs of row stride ldy.
struct LoraDown {
    const void* X; long long ldx; int K;
    const void* S; long long lds; int r;
    void* Y;
};
// as_problems > 0: the sums over K are cut as for so many problems, whatever else the launch holds (t2 keeps its bits).
// rows_dev (optional, matrix-core kernel only): the row count is min(*rows_dev, Trows), read on the device.
static constexpr int kDownGroups = 4;  // groups of eight rank columns of a problem
int launch_lora_down(alch_dtype dt, const LoraDown* jobs, int n_jobs, int Trows, float alpha, long long ldy,
                     int slot_cols, hipStream_t stream, int as_problems = 0, const int* rows_dev = nullptr);
int lora_down_parts(int Trows, int problems, int n_cu);  // parts that the sums over K are cut into
// C(j, n) (+)= alpha * sum_t S[t*lds + j] * X[t*ldx + n], j < r, n < N; stored C[j*ldc + n], or C[n*ldc + j]
// when transposed.  Up to kLoraUpJobs problems per launch, all with Trows rows, the same r, alpha and
// accumulate.  scratch: lora_up_scratch_bytes(r, sum of the N of the jobs) bytes of fp32 partial sums.
static constexpr int kLoraUpJobs = 6;
struct LoraUp {
    const void* S; long long lds;
    const void* X; long long ldx;
    int N;
    void* C; long long ldc;
    int transposed;
};
size_t lora_up_scratch_bytes(int rank, int n_sum);
// The sums over the splits of several such launches may be left to one launch: LoraUpSums holds them until
// launch_lora_up_sums.  launch_lora_up makes room first where the scratch, or the list, would not take its problems.
struct LoraUpJob {
    const void* S; long long lds;
    const void* X; long long ldx;
    int N, nsplit, rows_per_split;
    void* C; long long ldc;
    int transposed;
    int first_group;        // work-groups of the jobs before this one in the launch that adds the splits
    long long scratch_off;  // floats
    const int* rows_dev;    // of a row count on the device: it, and the rows of a split; splits past it were not written
    int rows_dev_split;
};
static constexpr int kLoraUpSums = 14;  // A and B of seven projections
struct LoraUpParams {
    LoraUpJob job[kLoraUpSums];
    int n_jobs, Trows, r, accumulate;
    float alpha;
    float* scratch;
};
struct LoraUpSums {
    LoraUpParams p = {};
    long long floats = 0, capacity = 0;  // of the scratch: taken, all
};
int launch_lora_up(alch_dtype dt, const LoraUp* jobs, int n_jobs, LoraUpSums& sums, hipStream_t stream);
int launch_lora_up_sums(alch_dtype dt, LoraUpSums& sums, hipStream_t stream);
// Adds a gradient whose partial sums [r/8][nsplit][8][N] a kernel will leave at scratch + sums.floats (before the call).
void add_lora_up_job(LoraUpSums& sums, const LoraUp& j, int nsplit, const int* rows_dev = nullptr, int rows_dev_split = 0);
// Both in one pass over X [Trows, K] (bf16; lora_pass.hip): T = alpha X P^T into an output slot (P [r, K], null: none; pad:
// zeros in the columns past the rank, and in all of them without P), and the gradients up[i] = Q[:, q_col .. +r]^T X, whose
// sums are left to launch_lora_up_sums.  Q and T have row stride ldq; Q holds the three slots of a row.  rows_dev: as
// launch_lora_down.
static constexpr int kPassUps = 3;
struct LoraPass {
    const void* X; long long ldx; int K;
    const void* P = nullptr; long long ldp = 0;
    void* T = nullptr;
    bool pad = false;
    bool keep_bits = false;  // T is an operand of a data gradient: summed as launch_lora_down sums these problems by themselves
    const void* Q = nullptr;
    int n_up = 0;
    struct { int q_col; void* C; long long ldc; int transposed; } up[kPassUps] = {};
};
bool lora_pass_fits(const LoraPass* jobs, int n_jobs, int Trows, const LoraUpSums& sums);
int launch_lora_pass(const LoraPass* jobs, int n_jobs, int Trows, long long ldq, float alpha, LoraUpSums& sums, hipStream_t stream,
                     const int* rows_dev = nullptr);
// A layer of bf16 under a loss mask, on its kept rows alone: their number is known to the device, and products whose size is there are the
// matrix-core kernels' alone.  What these refuse of the layer's sizes (k in pieces of 64, rows of more than 2^21 elements, operands of 2 GiB) is
// looked at ahead of anything that is enqueued; such a layer runs on all rows.
inline bool kept_rows_fit(int T, int H, int F, int QD) {
    const auto operand = [](long long rows, long long width) { return width <= 1 << 21 && rows * width * 2 < 1LL << 31; };
    return H % 64 == 0 && F % 64 == 0 && QD % 64 == 0 && operand(T, 2LL * F) && operand(T, H) && operand(T, QD) && operand(H, F) &&
           operand(F, H) && operand(H, QD);
}
// Whether a layer with adapters does so: where the rows that are left out are worth the launches that find, gather and scatter the others
// (one tile of 128 rows gets no shorter).  The host does not know how many are kept, and with most of them these launches, and products
// planned on the device, cost more than the rows are worth.  us on all rows / on the kept ones, rank 8, frozen base unless stated:
//   8B shape (4096, 14336)     0.25 of the rows kept   0.6           0.75          0.9
//     260 tokens                382 / 315              382 / 350     384 / 359     385 / 369
//     520                       492 / 380              498 / 450     504 / 476     506 / 494
//     1200                      765 / 560              816 / 755     826 / 782     831 / 1006
//     1490                      918 / 628              938 / 833     948 / 1054    959 / 1096 (all kept 951 / 1122)
//     3000                      1455 / 909             1602 / 1355   1637 / 1498   1648 / 1717
//     8000                      3336 / 1867            3664 / 3077   3714 / 3509   3756 / 3842
//   hidden 2048, ffn 8192, 1000 346 / 306              353 / 349     361 / 360     358 / 393
//     3000                      703 / 531              746 / 675     744 / 815     751 / 841
//   5120, 17920, 1000           888 / 636              910 / 885     921 / 927     929 / 1196
//     1500                      1218 / 807             1272 / 1301   1297 / 1409   1313 / 1515
//   70B shape (8192, 28672) 300 843 / 628              851 / 740     860 / 760     869 / 946
//     2000                      2750 / 1431            3016 / 2583   3087 / 2870   3111 / 3257
// Over 32 sizes a quarter of the rows comes out 1.13 to 2.0 times as fast, 0.6 0.98 to 1.44, 0.75 0.90 to 1.17, 0.9 0.78 to 1.14: this is for masks
// that leave out a third and more.  It loses most where the gradient of H2 has tiles of 128x256 for more than half of the compute units, which a
// plan on the device leaves whole.  Below the line (8B shape 130 tokens, all gradients 455 / 468 at a quarter, 200 489 / 494; hidden 2048 390 tokens 322 / 334, 520 362 / 363) there is
// nothing to gain with few kept rows either.
inline bool adapters_on_kept_rows(int T, int H, int F) { return T > 128 && (double)T * H * F >= 15e9; }
// Operand preparation: job i writes dst [rows_out, cols] = src [r, cols] (or, transpose, src [cols, r]
// transposed) followed by zero rows; src null: all zeros.
struct LoraPrepJob {
    const void* src; void* dst;
    int r, cols, rows_out, transpose;
};
struct LoraPrepParams { LoraPrepJob job[16]; };
int launch_lora_prep(alch_dtype dt, const LoraPrepParams& p, int n_jobs, hipStream_t stream);

// ---- attention ---------------------------------------------------------------------------
struct ShortRows { int up_to = 0, step = 1; };  // tokens of the longest such sequence; wavefronts that share the rows of a head
struct AttnArgs {
    alch_dtype dtype;
    int T, n_seqs, max_seqlen, Hq, Hkv, D;
    const int* cu_seqlens;       // device
    const int* cu_seqlens_host;  // host
    // shared prefixes: prefix[s] = -1 or the index of the earlier sequence whose keys and values every token
    // of s also attends to (device / host copies, both null when no sequence has a prefix)
    const int* prefix = nullptr;
    const int* prefix_host = nullptr;
    const void *Q, *K, *V, *O, *dO;  // dense [T, heads*D]
    const float* LSE;                // [T, Hq]
    float* delta;                    // scratch [2, T, Hq]: row sums of dO*O, produced inside launch_attn_bwd; the
                                     // matrix-core kernels keep LSE * log2(e) in the second half
    void *dQ, *dK, *dV;              // row stride ld_dqkv elements; dQ, dK, dV adjacent: [dQ | dK | dV] rows
    long long ld_dqkv;
    // rope_base > 0: dQ and dK come out already rotated by minus the RoPE angle (RoPE backward)
    const int* positions = nullptr;  // device [T] or null (index inside the sequence)
    float rope_base = 0.f;
    // optional: fp32 partial sums of dK, dV where the key blocks are too few or too unequal for the chip; 16-byte aligned,
    // any size (T * Hkv * 2 * D floats for each of up to 8 parts are made use of)
    void* scratch = nullptr;
    size_t scratch_bytes = 0;
    ShortRows rows;  // see rows_up_to
    bool keep_parts = false;  // as GemmDesc: key blocks are cut as by plan_dkv_parts whatever launch they are in
};
// Tokens of the longest of the sequences first .. n_seqs-1.  max_seqlen is only a bound on them, and may be any number that
// is not below it.
inline int longest_sequence(const int* cu_host, int first, int n_seqs) {
    int n = 0;
    for (int s = first; s < n_seqs; ++s) n = cu_host[s + 1] - cu_host[s] > n ? cu_host[s + 1] - cu_host[s] : n;
    return n;
}
int compute_units(int* n_cu);  // of the current device, a multiple of 8
int launch_attn_bwd(const AttnArgs& a, hipStream_t stream);
int launch_attn_bwd_generic(const AttnArgs& a, hipStream_t stream);
bool attn_mfma_supported(const AttnArgs& a);
int launch_attn_bwd_mfma(const AttnArgs& a, hipStream_t stream);
int attn_bwd_mfma_d64(const AttnArgs& a, hipStream_t stream);
int attn_fwd_mfma_d64(const void* Q, const void* K, const void* V, void* O, float* LSE, int n_seqs, int max_seqlen,
                      const int* cu_seqlens, const int* prefix, int seq_begin, int Hq, int Hkv, int short_upto, hipStream_t stream);
// Sequences too short for the tile kernels, a row at a time: up to how many tokens these take them (0: they take none), and
// the launches for them.  The tile kernels then leave them out.
int rows_up_to(int D, int Hq, int per_cu, int first, int n_seqs, const int* cu_host, const int* prefix, ShortRows* rows);
int launch_attn_bwd_rows(const AttnArgs& a, hipStream_t stream);
int launch_attn_fwd_rows(alch_dtype dt, const void* Q, const void* K, const void* V, void* O, float* LSE, int n_seqs, const int* cu_seqlens,
                         int seq_begin, int Hq, int Hkv, int D, const ShortRows& rows, hipStream_t stream);
static constexpr int kMaxPrefixSeqs = 4096;  // sequences per batch when prefixes are shared
double attn_pairs(int n_seqs, const int* cu_host, const int* prefix_host);
// forward: writes O [T,Hq*D] and LSE [T,Hq] for the query rows of sequences seq_begin .. n_seqs-1 (keys and
// values of a prefix sequence are read wherever it lies); prefix / prefix_host as in AttnArgs
int launch_attn_fwd_generic(alch_dtype dt, const void* Q, const void* K, const void* V, void* O, float* LSE, int T,
                            int n_seqs, const int* cu_seqlens, const int* cu_seqlens_host, const int* prefix,
                            int seq_begin, int Hq, int Hkv, int D, hipStream_t stream);
int launch_attn_fwd(alch_dtype dt, const void* Q, const void* K, const void* V, void* O, float* LSE, int T,
                    int n_seqs, int max_seqlen, const int* cu_seqlens, const int* cu_seqlens_host, const int* prefix,
                    const int* prefix_host, int seq_begin, int Hq, int Hkv, int D, hipStream_t stream);

// ---- LM head + cross-entropy ---------------------------------------------------------------
// n_counted[0] = #{t : labels[t] >= 0 and (mask == NULL or mask[t] != 0)}; row_loss[0..T) = 0; counted[t] (or NULL): that predicate
int launch_count_labels(const int* labels, const uint8_t* loss_mask, int T, int vocab, int* n_counted, float* row_loss, uint8_t* counted,
                        hipStream_t stream);
// One chunk of logits rows [rows, vocab] (row stride ld), in place: logits -> dlogits =
// (softmax - onehot(label)) / N for counted rows, 0 otherwise; row_loss[r] = -log softmax[label].
int launch_ce_chunk(alch_dtype dt, void* logits, long long ld, int rows, int vocab, const int* labels,
                    const uint8_t* loss_mask, const int* n_counted, float* row_loss, hipStream_t stream,
                    const int* rows_dev = nullptr);
// ---- DPO head on scored tokens (items) -----------------------------------------------------
// logp[m], logz[m] of a chunk of item logits rows
int launch_dpo_logp(alch_dtype dt, const void* logits, long long ld, int rows, int vocab, const int* labels, float* logp,
                    float* logz, hipStream_t stream);
// pi[slot] = sum of logp; z, loss, weight of every slot (w_slot [2 n_pairs]); z_out may be null
int launch_dpo_weights(const float* logp, const int* slots, const int* labels, int n_items, int vocab, const float* ref,
                       int n_pairs, float beta, float* pi, float* w_slot, float* z_out, float* loss_out, hipStream_t stream);
// a chunk of item logits rows -> their gradient, in place
int launch_dpo_grad(alch_dtype dt, void* logits, long long ld, int rows, int vocab, const int* labels, const int* slots,
                    const float* logz, const float* w_slot, int n_slots, hipStream_t stream);
// out [T, width] = 0, then out[item_row[m]] += src[m] (items sorted by row; fixed order)
int launch_dpo_scatter(alch_dtype dt, const void* src, const int* item_row, int n_items, void* out, int T, int width,
                       hipStream_t stream);

// loss_out[0] = sum(row_loss) / max(N, 1)   (fixed summation order)
int launch_finish_loss(const float* row_loss, const int* n_counted, float* loss_out, int T, hipStream_t stream);

}  // namespace alch
