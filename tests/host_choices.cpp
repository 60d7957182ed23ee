// Answers questions about the library's host-side choices, one a line of stdin (see test_host_choices.py).  No GPU call.
#include <iostream>
#include <string>

#include <vector>

#include "attn_mfma_kernels.h"
#include "gemm_mfma_common.h"

using namespace alch;

namespace alch {
int compute_units(int* n_cu) {  // in place of the library's, which asks the device
    *n_cu = 256;
    return ALCH_OK;
}
}  // namespace alch

static void* const kSome = reinterpret_cast<void*>(0x10000);  // aligned, never followed

static GemmDesc product(int M, int N, int K, bool a_kmajor, bool b_kmajor) {
    GemmDesc d;
    d.M = M; d.N = N; d.a_kmajor = a_kmajor; d.b_kmajor = b_kmajor;
    d.n_seg = d.n_out = 1;
    d.seg[0] = GemmSeg{kSome, kSome, K, a_kmajor ? K : M, b_kmajor ? K : N};
    d.out[0] = GemmOut{kSome, 0, N};
    return d;
}

int main() {
    std::string what;
    while (std::cin >> what) {
        if (what == "supported") {  // M N K a_kmajor b_kmajor, contraction length on the device
            int M, N, K, a, b, dev;
            std::cin >> M >> N >> K >> a >> b >> dev;
            GemmDesc d = product(M, N, K, a, b);
            if (dev) d.k_dev = static_cast<const int*>(kSome);
            std::cout << gemm_mfma_supported(d) << "\n";
        } else if (what == "kernel") {  // M N K a_kmajor b_kmajor, whole tiles: 1 for 128x256, 0 for 256x256
            int M, N, K, a, b;
            std::cin >> M >> N >> K >> a >> b;
            std::cout << pair_is_better(M, N, K, a, b, false, 256, 1, pair_plan(M, N, up_div(K, BK), a, 256, 0)) << "\n";
        } else if (what == "rows_beside") {  // hidden ffn T qkv of an fp32 layer: the norm beside dWd, the gain sums beside d[Wq; Wk; Wv]
            int H, F, T, qkv;
            std::cin >> H >> F >> T >> qkv;
            GemmDesc dWd = product(H, F, T, false, false), dH2 = product(T, H, F, true, false), dWqkv = product(qkv, H, T, false, false);
            dH2.n_seg = 2;
            dH2.seg[1] = dH2.seg[0];
            dWd.dtype = dH2.dtype = dWqkv.dtype = ALCH_F32;
            const bool together = (size_t)T * F >= (size_t)rmsnorm_bwd_blocks(T) * H;
            std::cout << (together && !gemm_together(dH2, dWd) && gemm_beside_rows(dWd, H)) << " " << (together && gemm_beside_rows(dWqkv, H)) << "\n";
        } else if (what == "one_pass") {  // T hidden ffn rank: the pass over Act, dG and dU, all adapters and gradients
            int T, H, F, r;
            std::cin >> T >> H >> F >> r;
            LoraPass jobs[3] = {};
            for (int i = 0; i < 3; ++i) {
                jobs[i].X = kSome; jobs[i].ldx = i ? 2 * (long long)F : F; jobs[i].K = F;
                jobs[i].P = kSome; jobs[i].ldp = F; jobs[i].T = kSome;
                jobs[i].pad = jobs[i].keep_bits = i > 0;
                jobs[i].Q = kSome;
                jobs[i].up[jobs[i].n_up++] = {0, kSome, F, 0};
            }
            LoraUpSums sums;
            sums.p.Trows = T; sums.p.r = r; sums.p.scratch = static_cast<float*>(kSome);
            sums.capacity = (long long)(lora_up_scratch_bytes(r, 2 * (H + F)) / sizeof(float));
            std::cout << lora_pass_fits(jobs, 3, T, sums) << "\n";
        } else if (what == "t_parts") {  // T problems: parts of the contraction of t2
            int T, problems;
            std::cin >> T >> problems;
            std::cout << lora_down_parts(T, problems, 256) << "\n";
        } else if (what == "kept_rows") {  // T hidden ffn, width of all query heads: a masked layer runs on its kept rows
            int T, H, F, QD;
            std::cin >> T >> H >> F >> QD;
            std::cout << kept_rows_fit(T, H, F, QD) << "\n";
        } else if (what == "adapters_pay") {  // T hidden ffn: with adapters, too
            int T, H, F;
            std::cin >> T >> H >> F;
            std::cout << adapters_on_kept_rows(T, H, F) << "\n";
        } else if (what == "rows") {  // rows N K swiglu, of several layers: data gradient with the row count on the device: its kernel
            // (0: 256x256, 1: 128x256, 2: 64x64, 3: 128x128) and the parts of its cut tiles
            int M, N, K, swiglu, several;
            std::cin >> M >> N >> K >> swiglu >> several;
            MfmaGemmParams p{};
            p.n_seg = 1; p.N = N; p.K[0] = K; p.a_kmajor = 1; p.plan_cu = 256;
            p.epilogue = swiglu ? kEpiSwigluBwd : kEpiNone;
            p.narrow = several;
            p.plan_ws = several ? 0 : (long long)kGemmSplitWsBytes;
            PairPlan plan;
            const RowsKernel kernel = device_plan(p, M, plan);
            std::cout << (int)kernel << " " << (kernel == kRowsPair ? plan.parts : 1) << "\n";
        } else if (what == "attention") {  // head size, query and key/value heads, ffn, stack of several layers, number of lengths, lengths:
            // the backward in bf16: longest sequence that the row kernels take, parts of a key block, both gradients as one launch
            int D, Hq, Hkv, F, several, n;
            std::cin >> D >> Hq >> Hkv >> F >> several >> n;
            std::vector<int> cu(n + 1, 0);
            for (int i = 0; i < n; ++i) {
                std::cin >> cu[i + 1];
                cu[i + 1] += cu[i];
            }
            AttnArgs a;
            a.dtype = ALCH_BF16; a.T = cu[n]; a.n_seqs = n; a.Hq = Hq; a.Hkv = Hkv; a.D = D;
            a.cu_seqlens_host = cu.data();
            a.scratch = kSome;
            a.scratch_bytes = (size_t)a.T * 2 * F * 2;
            a.keep_parts = several;
            if (D == 64 && rows_up_to(D, Hq, kRowsPerCu, 0, n, cu.data(), nullptr, &a.rows) != ALCH_OK) return 1;
            AttnMfmaParams p{};
            p.n_blocks = up_div(longest_sequence(cu.data(), 0, n), 128);
            bool both = false;
            int longest = 0;
            if (plan_both(a, p, both) != ALCH_OK || (!both && plan_dkv_parts(a, p, longest) != ALCH_OK)) return 1;
            std::cout << a.rows.up_to << " " << p.max_parts << " " << both << "\n";
        } else {
            return 1;
        }
    }
    return 0;
}
