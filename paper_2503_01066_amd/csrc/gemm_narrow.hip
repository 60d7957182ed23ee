// bf16 data gradients of few rows, whole contractions, on the gfx950 matrix cores: products whose row count only the device knows
// and whose bits have to be those of uncut tiles (stacks of several layers, see GemmDesc::keep_parts).
//
// A few hundred kept rows of 4096 columns are 16 or 32 tiles of 128x256: most compute units idle while the others walk a vocabulary of
// 128256 alone, each at half of its rate, since no second work-group fills the gaps of the first.  Here the tile is 64x64, or 128x128
// where that would be a second one for some compute unit (see device_plan).  An element of the output is the same chain of
// 32x32x16 instructions over the contraction in any tile: the same bits.
//   * LDS bounds the loop: of a step of 64 k the reads of four wavefronts (128 bytes a cycle) and the pieces that arrive (64 a cycle)
//     are 512 cycles of a 64x64 tile beside 128 of matrix instructions, 1024 beside 512 of a 128x128 one.  With the loads held to
//     one place, 160 rows by 4096, K 128256: 399 us, 480 cycles a step; 680 rows 1054 us, 1260.
//   * Cold weights are in front of that: 692 us with nine stages in flight, however the columns lie over the XCDs and also if the
//     fragments wait at the barrier.  Whole 128x256 tiles: 1540.  Same columns, K 28672 374 -> 174, K 4096 58 -> 28 us; 680 rows
//     1607 -> 1085, 377 -> 253, 58 -> 42.
#include "gemm_mfma_common.h"

namespace alch {

template <int kT> struct NarrowTile {
    static constexpr int kRows = 64 * kT, kCols = 64 * kT;
    static constexpr int kOperand = 64 * kRows * 2;  // one operand of a stage: 64 k
    static constexpr int kStage = 2 * kOperand;
    static constexpr int kStages = kT == 1 ? 9 : 4;
    static constexpr int kLoads = 2 * kT;            // of an operand, per wavefront and stage
};
static constexpr int kNarrowLds = NarrowTile<1>::kStages * NarrowTile<1>::kStage;
static_assert(NarrowTile<2>::kStages * NarrowTile<2>::kStage <= kNarrowLds, "stages of both tiles share the LDS");

template <int kT>
__device__ __forceinline__ void narrow_tile(const MfmaGemmParams& p, int Mv, int block, char* smem) {
    using Tile = NarrowTile<kT>;
    constexpr int kStages = Tile::kStages, kLoads = Tile::kLoads, kChunks = Tile::kCols / 8;
    const int tiles_m = up_div(Mv, Tile::kRows), nt = tiles_m * up_div(p.N, Tile::kCols), per_xcd = up_div(nt, 8);
    // every XCD owns per_xcd consecutive tiles, those of the same columns next to each other: the weights come into one L2
    const int t = (block % 8) * per_xcd + block / 8;
    if (block / 8 >= per_xcd || t >= nt) return;
    const int m0 = t % tiles_m * Tile::kRows, n0 = t / tiles_m * Tile::kCols;
    const int lane = threadIdx.x & 63, half = lane >> 5;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int row0 = (wave >> 1) * 32 * kT, col0 = (wave & 1) * 32 * kT;
    const uint32_t lds_w = __builtin_amdgcn_readfirstlane((uint32_t)(uintptr_t)ALCH_LDS(smem) + (uint32_t)wave * (kLoads * 1024u));

    f32x16 acc[kT][kT];
#pragma unroll
    for (int i = 0; i < kT; ++i)
#pragma unroll
        for (int j = 0; j < kT; ++j)
#pragma unroll
            for (int e = 0; e < 16; ++e) acc[i][j][e] = 0.f;

    for (int seg = 0; seg < p.n_seg; ++seg) {
        const long long lda = p.lda[seg], ldb = p.ldb[seg];
        const int K = p.K[seg], nk = K / 64;  // (K is a multiple of 64)
        // per-lane byte offsets of a stage's loads: LDS slots of 16 bytes are filled lane-linearly, which piece a lane fetches
        // carries the bank swizzle
        uint32_t va[kLoads], vb[kLoads];
#pragma unroll
        for (int j = 0; j < kLoads; ++j) {
            const int s = (wave * kLoads + j) * 64 + lane;
            const int row = s >> 3, ca = (s & 7) ^ ((row >> 1) & 7);
            va[j] = row < Mv - m0 ? (uint32_t)((row * lda + ca * 8) * 2) : kOobOffset;
            const int k = s / kChunks, cb = (s % kChunks) ^ col_swizzle<Tile::kCols>(k);
            vb[j] = cb * 8 < p.N - n0 ? (uint32_t)((k * ldb + cb * 8) * 2) : kOobOffset;
        }
        OperandStream a, b;
        a.open(p.A[seg] + (long long)m0 * lda, p.A[seg] + (long long)(Mv - 1) * lda + K, nk, 128);
        b.open(p.B[seg] + n0, p.B[seg] + (long long)(K - 1) * ldb + p.N, nk, (int)(64 * ldb * 2));
        auto load_stage = [&](uint32_t stage) {
            i32x4 ra, rb;
            a.select(ra);
            b.select(rb);
            a.advance();
            b.advance();
#pragma unroll
            for (int j = 0; j < kLoads; ++j) dma16(ra, lds_w + stage, (uint32_t)(j * 1024), va[j]);
#pragma unroll
            for (int j = 0; j < kLoads; ++j) dma16(rb, lds_w + stage, (uint32_t)(Tile::kOperand + j * 1024), vb[j]);
        };
        // A step is one set of fragments, 64 k of the small tile, 32 of the large one.
        constexpr int kSub = kT, kSteps = 4 / kT;
        struct Frags { bf16x8 a[kSteps][kT], b[kSteps][kT]; };
        auto read = [&](Frags& f, uint32_t stage, int sub) {
#pragma unroll
            for (int s = 0; s < kSteps; ++s) {
                const int kk = sub * kSteps + s;
#pragma unroll
                for (int i = 0; i < kT; ++i) {
                    const int row = row0 + i * 32 + (lane & 31), c = (kk * 2 + half) ^ ((row >> 1) & 7);
                    f.a[s][i] = *reinterpret_cast<const bf16x8*>(smem + stage + row * 128 + c * 16);
                }
#pragma unroll
                for (int j = 0; j < kT; ++j)
                    f.b[s][j] = read_frag<false, Tile::kCols>(smem + stage + Tile::kOperand, col0 + j * 32, kk, lane);
            }
        };
        auto multiply = [&](const Frags& f, int s) {
#pragma unroll
            for (int i = 0; i < kT; ++i)
#pragma unroll
                for (int j = 0; j < kT; ++j) acc[i][j] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(f.b[s][j], f.a[s][i], acc[i][j], 0, 0, 0);
        };

        __syncthreads();  // every wave is done with the previous pair's stages
        constexpr int kAhead = kT == 1 ? kStages : kStages - 1;  // stages in flight
        // vmcnt(0), known to the compiler, with nothing on its way yet: it holds the epilogue's loads of the other tile for pending and
        // waited for all stages ahead of a fragment that takes one of their registers
        __builtin_amdgcn_s_waitcnt(0x0f70);
#pragma unroll
        for (int s = 0; s < kAhead; ++s) load_stage((uint32_t)(s * Tile::kStage));
        asm volatile("s_waitcnt vmcnt(%0)" ::"n"((kAhead - 2) * 2 * kLoads) : "memory");  // stages 0 and 1 have landed
        __syncthreads();
        auto after = [](uint32_t stage) -> uint32_t { return stage == (kStages - 1) * Tile::kStage ? 0 : stage + Tile::kStage; };
        uint32_t ahead = kT == 1 ? 2 * Tile::kStage : Tile::kStage;             // the stage that is read next
        uint32_t free_stage = kT == 1 ? 0 : (kStages - 1) * Tile::kStage;       // the stage that is loaded next
        Frags f[3];
        read(f[0], 0, 0);
        // (in this order: of 24 reads the first step waits for twelve, and then loads into stage 0 of a 64x64 tile)
        __builtin_amdgcn_sched_barrier(0);
        read(f[1], kT == 1 ? Tile::kStage : 0, kT == 1 ? 0 : 1);
        // A step's fragments were read two steps ago and have arrived when those of the step before are all that is on its way (12
        // reads); so the LDS has work through the barrier.  First step of a stage: what it reads has landed in every wave's share, and
        // the stage it loads into has had its last reader.
        auto step = [&](const Frags& now, Frags& then, int sub) __attribute__((always_inline)) {
            __builtin_amdgcn_s_waitcnt(0xcc7f);  // lgkmcnt(12), known to the compiler
            if (sub == 0) asm volatile("s_waitcnt vmcnt(%0) lgkmcnt(12)\n\ts_barrier" ::"n"((kStages - 3) * 2 * kLoads) : "memory");
            __builtin_amdgcn_sched_barrier(0);
            multiply(now, 0);
            __builtin_amdgcn_sched_barrier(0);
            if (sub == 0) {
                load_stage(free_stage);
                free_stage = after(free_stage);
            }
            read(then, ahead, sub);
            if (sub == kSub - 1) ahead = after(ahead);
#pragma unroll
            for (int s = 1; s < kSteps; ++s) multiply(now, s);
            __builtin_amdgcn_sched_barrier(0);
        };
        const int steps = nk * kSub;
        for (int u = 0;; u += 3 * kSub) {
#pragma unroll
            for (int v = 0; v < 3 * kSub; ++v) {
                if (u + v >= steps) goto steps_done;
                step(f[v % 3], f[(v + 2) % 3], v % kSub);
            }
        }
    steps_done:
        asm volatile("s_waitcnt vmcnt(0) lgkmcnt(0)" ::: "memory");
    }

    // block (i, j) holds the transposed 32x32 result: this lane owns row i*32 + (lane & 31) and columns j*32 + 8b + 4*half + 0..3
#pragma unroll
    for (int i = 0; i < kT; ++i) {
        const int m = m0 + row0 + i * 32 + (lane & 31);
        if (m >= Mv) continue;
        __bf16* C = p.C[0] + (long long)m * p.ldc[0];
#pragma unroll
        for (int j = 0; j < kT; ++j) {
            const int n = n0 + col0 + j * 32 + 4 * half;
            bf16x4 o[4];
#pragma unroll
            for (int b = 0; b < 4; ++b)
#pragma unroll
                for (int r = 0; r < 4; ++r) o[b][r] = (__bf16)acc[i][j][4 * b + r];
            if (p.epilogue == kEpiSwigluBwd) {
                bf16x4 g[4], u[4];
#pragma unroll
                for (int b = 0; b < 4; ++b)
                    if (n + 8 * b < p.N) {
                        g[b] = *reinterpret_cast<const bf16x4*>(p.G + (long long)m * p.ldgu + n + 8 * b);
                        u[b] = *reinterpret_cast<const bf16x4*>(p.U + (long long)m * p.ldgu + n + 8 * b);
                    }
#pragma unroll
                for (int b = 0; b < 4; ++b)
                    if (n + 8 * b < p.N) {
                        bf16x4 dg, du, act;
                        swiglu_gradient<4>(o[b], g[b], u[b], dg, du, act);
                        *reinterpret_cast<bf16x4*>(C + n + 8 * b) = dg;
                        *reinterpret_cast<bf16x4*>(C + p.N + n + 8 * b) = du;
                        if (p.act_out) *reinterpret_cast<bf16x4*>(p.act_out + (long long)m * p.N + n + 8 * b) = act;
                    }
                continue;
            }
#pragma unroll
            for (int b = 0; b < 4; ++b)
                if (n + 8 * b < p.N) *reinterpret_cast<bf16x4*>(C + n + 8 * b) = o[b];
        }
    }
}

__global__ __launch_bounds__(256, 1) void k_gemm_narrow_rows(MfmaGemmParams p) {
    __shared__ __attribute__((aligned(1024))) char smem[kNarrowLds];
    const int Mv = min(__builtin_amdgcn_readfirstlane(*p.m_dev), p.M);
    if (Mv <= 0) return;
    PairPlan plan;
    const RowsKernel kernel = device_plan(p, Mv, plan);
    if (kernel == kRowsNarrow64) narrow_tile<1>(p, Mv, (int)blockIdx.x, smem);
    else if (kernel == kRowsNarrow128) narrow_tile<2>(p, Mv, (int)blockIdx.x, smem);
}

int launch_gemm_narrow_rows(const MfmaGemmParams& p, int grid, hipStream_t stream) {
    k_gemm_narrow_rows<<<grid, 256, 0, stream>>>(p);
    ALCH_HIP_TRY(hipGetLastError());
    return ALCH_OK;
}

}  // namespace alch
