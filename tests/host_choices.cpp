// Answers questions about the library's host-side choices, one a line of stdin (see test_host_choices.py).  No GPU call.
#include <iostream>
#include <string>

#include "gemm_mfma_common.h"

using namespace alch;

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
        } else {
            return 1;
        }
    }
    return 0;
}
