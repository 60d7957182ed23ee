// Answers questions about the library's host-side choices, one a line of stdin (see test_host_choices.py).  No GPU call.
#include <iostream>
#include <string>

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
        } else if (what == "one_pass") {  // T F rank: the pass over Act, dG and dU of a layer with all adapters and gradients, hidden 64
            int T, F, r;
            std::cin >> T >> F >> r;
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
            sums.capacity = (long long)(lora_up_scratch_bytes(r, 2 * (64 + F)) / sizeof(float));
            std::cout << lora_pass_fits(jobs, 3, T, sums) << "\n";
        } else {
            return 1;
        }
    }
    return 0;
}
