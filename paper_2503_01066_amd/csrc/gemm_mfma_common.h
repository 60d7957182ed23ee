// Pieces shared by the bf16 matrix-core GEMM kernels (gemm_mfma.hip, gemm_pair.hip).
#pragma once
#include <algorithm>
#include "kernels.h"

namespace alch {

typedef __attribute__((ext_vector_type(8))) __bf16 bf16x8;
typedef __attribute__((ext_vector_type(4))) __bf16 bf16x4;
typedef __attribute__((ext_vector_type(16))) float f32x16;
typedef __attribute__((ext_vector_type(4))) float f32x4;

#define ALCH_LDS(p) ((__attribute__((address_space(3))) void*)(p))

static constexpr int BK = 32;
static constexpr uint32_t kOobOffset = 0x80000000u;      // >= any num_records we set

struct MfmaGemmParams {
    int M, N, n_seg, n_out, accumulate, tiles_m, tiles_n;
    // optional device-resident sizes (row compaction decided on the device): the effective M, or the
    // effective K of every operand pair, is min(*ptr, host value)
    const int* m_dev;
    const int* k_dev;
    const __bf16* A[kMaxGemmSegs];
    const __bf16* B[kMaxGemmSegs];
    int K[kMaxGemmSegs];
    long long lda[kMaxGemmSegs], ldb[kMaxGemmSegs];
    __bf16* C[3];
    int m_begin[3];
    long long ldc[3];
    // by_cols: m_begin are columns; C[i] and B[i] (of range i, not of an operand pair) point m_begin[i] columns / rows
    // before their range, so that they are indexed with columns of the whole product
    int by_cols;
    const __bf16* residual;
    int epilogue;
    const __bf16* G;
    const __bf16* U;
    long long ldgu;
    __bf16* act_out;
    // Tiles q < q_end of every XCD's share are computed whole by the plain instantiation.  The kSplit
    // instantiation computes the tiles q_end .. of the share, split_s work-groups per tile, partial tiles
    // [tile of the split round][part][256][256] fp32 in split_ws.
    int q_end;
    float* split_ws;
    int split_s, split_per;  // parts per tile; k-tiles per part (counted over all operand pairs in order)
    int per_xcd;             // k_gemm_pair: tiles of an XCD's share
    // m_dev: k_gemm_pair plans on the device, for plan_cu compute units and plan_ws bytes of scratch (0: no tile is cut);
    // either: several kernels are launched, and those that the estimate does not choose leave at once; narrow: k_gemm_narrow_rows may be one.
    int either, narrow, plan_cu, a_kmajor, b_kmajor;
    long long plan_ws;
};

// output range that row (or column) x of the product belongs to
__device__ __forceinline__ int range_of(const MfmaGemmParams& p, int x) {
    int r = 0;
#pragma unroll
    for (int s = 1; s < 3; ++s)
        if (s < p.n_out && x >= p.m_begin[s]) r = s;
    return r;
}

typedef __attribute__((ext_vector_type(4))) int i32x4;

// 16 bytes per lane from buffer `r` at byte offset `voff` straight into LDS at
// lds_addr + lane*16.  Written as assembly so that the compiler does not order later LDS
// reads of the other pipeline stage behind it; completion is awaited with vmcnt.
// lds_off: a constant once the loop around it is unrolled (as an operand of the addition it takes no scalar register: the
// addresses of a whole ring were more of them than there are).
// s_nop: a load into LDS takes one wait state after a scalar write of m0.  The compiler puts it there for its own loads
// of this kind and does not look into assembly.
__device__ __forceinline__ void dma16(i32x4 r, uint32_t lds_addr, uint32_t lds_off, uint32_t voff) {
    asm volatile("s_add_u32 m0, %0, %3\n\ts_nop 0\n\tbuffer_load_dwordx4 %1, %2, 0 offen lds"
                 :
                 : "s"(lds_addr), "v"(voff), "s"(r), "i"(lds_off)
                 : "memory", "m0", "scc");
}

// Per-lane byte offsets (relative to the tile origin) of the 4 direct-to-LDS loads a wave
// issues for one operand tile.  LDS slot s (16-byte units) = (wave*4 + j)*64 + lane.
//   k-major tile [256 rows][32 k]: slot = row*4 + (c ^ ((row>>2)&3)), c = 16-byte chunk in the row
//   mn-major tile [32 k][256 cols]: slot = k*32 + (c ^ (4*(k&3)))
template <bool KMAJOR>
__device__ __forceinline__ void tile_offsets(uint32_t (&voff)[4], int wave, int lane, long long ld, int valid) {
#pragma unroll
    for (int j = 0; j < 4; ++j) {
        const int s = (wave * 4 + j) * 64 + lane;
        if (KMAJOR) {
            const int row = s >> 2, c = (s & 3) ^ ((row >> 2) & 3);
            voff[j] = row < valid ? (uint32_t)((row * ld + c * 8) * 2) : kOobOffset;
        } else {
            const int k = s >> 5, c = (s & 31) ^ (4 * (k & 3));
            voff[j] = c * 8 < valid ? (uint32_t)((k * ld + c * 8) * 2) : kOobOffset;
        }
    }
}

// An operand as a run of equal steps through a buffer, in scalar registers: address and bytes left, steps left.  Past the end the
// loads go to an empty buffer, so the number in flight is the same in every step.
struct OperandStream {
    uint32_t lo, hi;
    int left_bytes, left, bytes;
    __device__ __forceinline__ void open(const __bf16* first, const __bf16* end, int steps, int step_bytes) {
        const uint64_t u = (uint64_t)first;
        const long long l = (const char*)end - (const char*)first;
        lo = __builtin_amdgcn_readfirstlane((uint32_t)u);
        hi = __builtin_amdgcn_readfirstlane((uint32_t)(u >> 32) & 0xffffu);
        left_bytes = __builtin_amdgcn_readfirstlane((int)(l < 0 ? 0 : (l > 0x7fffffffLL ? 0x7fffffffLL : l)));
        left = __builtin_amdgcn_readfirstlane(steps);
        bytes = __builtin_amdgcn_readfirstlane(step_bytes);
    }
    __device__ __forceinline__ void select(i32x4& r) const {
        int n;
        asm volatile("s_cmp_gt_i32 %1, 0\n\ts_cselect_b32 %0, %2, 0" : "=&s"(n) : "s"(left), "s"(left_bytes) : "scc");
        r[0] = (int)lo; r[1] = (int)hi; r[2] = n; r[3] = 0x00020000;
    }
    __device__ __forceinline__ void advance() {
        asm volatile("s_add_u32 %0, %0, %4\n\ts_addc_u32 %1, %1, 0\n\ts_sub_i32 %2, %2, %4\n\ts_max_i32 %2, %2, 0\n\t"
                     "s_sub_i32 %3, %3, 1"
                     : "+s"(lo), "+s"(hi), "+s"(left_bytes), "+s"(left)
                     : "s"(bytes)
                     : "scc");
    }
};

// Which 16-byte piece of row k of a token-major tile lies where: rows of 512 and 256 bytes meet in the banks every second row of a
// fragment's four, rows of 128 bytes every second one, too, half as far apart.
template <int kCols> __device__ __forceinline__ int col_swizzle(int k) { return kCols == 64 ? 4 * ((k >> 1) & 1) : 4 * (k & 3); }

// Fragment (8 consecutive-k bf16 per lane for one 32-wide block of rows/cols) from an LDS tile; kCols = columns of a
// token-major tile.
template <bool KMAJOR, int kCols = 256>
__device__ __forceinline__ bf16x8 read_frag(const char* stage, int idx0 /*first row/col of the 32-block*/, int kk, int lane) {
    if (KMAJOR) {
        const int row = idx0 + (lane & 31);
        const int c = (kk * 2 + (lane >> 5)) ^ ((row >> 2) & 3);
        return *reinterpret_cast<const bf16x8*>(stage + row * 64 + c * 16);
    } else {
        const int g = lane >> 4, i = lane & 15;
        const int col = idx0 + (g & 1) * 16 + 4 * (i & 3);
        const int krow = kk * 16 + 8 * (g >> 1) + (i >> 2);  // + 4 for the second half
        const int chunk = col >> 3, sub = (col & 7) * 2;
        const char* p0 = stage + krow * (kCols * 2) + ((chunk ^ col_swizzle<kCols>(krow)) << 4) + sub;
        const char* p1 = p0 + 4 * (kCols * 2);  // krow + 4 is swizzled alike
        bf16x4 lo = __builtin_amdgcn_ds_read_tr16_b64_v4bf16((__attribute__((address_space(3))) bf16x4*)(p0));
        bf16x4 hi = __builtin_amdgcn_ds_read_tr16_b64_v4bf16((__attribute__((address_space(3))) bf16x4*)(p1));
        return __builtin_shufflevector(lo, hi, 0, 1, 2, 3, 4, 5, 6, 7);
    }
}

__device__ __forceinline__ float bf2f(__bf16 v) { return (float)v; }

// dAct = d rounded to bf16, saved g, u -> dG = dAct U s'(G), dU = dAct silu(G), Act = silu(G) U, of kN elements
template <int kN, typename V>
__device__ __forceinline__ void swiglu_gradient(const V& dv, const V& gv, const V& uv, V& dg, V& du, V& act) {
#pragma unroll
    for (int r = 0; r < kN; ++r) {
        const float g = bf2f(gv[r]), u = bf2f(uv[r]), d = bf2f(dv[r]);
        const float sg = __builtin_amdgcn_rcpf(1.f + __builtin_amdgcn_exp2f(-1.4426950408889634f * g));
        const float silu = g * sg;
        dg[r] = (__bf16)(d * u * sg * (1.f + g * (1.f - sg)));
        du[r] = (__bf16)(d * silu);
        act[r] = (__bf16)(silu * u);
    }
}

// ---- how the kernel of 128x256 tiles walks a product, and which of the two kernels takes it.  In whole numbers: products whose
// row count only the device knows are planned there, and every kernel of theirs has to come to the same answer.
static constexpr int PM = 128, PN = 256;
__host__ __device__ inline int up_div(int a, int b) { return (a + b - 1) / b; }
__host__ __device__ inline int least(int a, int b) { return a < b ? a : b; }

// A share of per_xcd tiles per XCD (of tiles_m tile rows, the last may be empty), whole up to q_end, the others in `parts` parts
// of `per` k-tiles each, with their partial tiles in split_ws.
struct PairPlan { int per_xcd, q_end, parts, per; };
// The rest of a share is cut for one work-group per compute unit (a second one
// would halve the length of the parts again and double the partial tiles: 487 x 4096 x 4096 41 us with 8 parts, 31 us with
// 4).  Tiles that leave some compute units with two work-groups and the others with one are cut as well, once every
// compute unit has a whole one: 4099 rows by 2048 are 33 tiles for the 32 units of an XCD.
__host__ __device__ inline PairPlan pair_plan(int M, int N, int nk_total, bool a_kmajor, int n_cu, long long ws_bytes) {
    const int per_xcd = up_div(up_div(M, PM) * up_div(N, PN), 8), cus = n_cu / 8;
    PairPlan plan{per_xcd, per_xcd, 1, 0};
    if (ws_bytes == 0) return plan;
    const int rem = per_xcd % cus;
    if (rem == 0) return plan;
    const int s = least(least(cus / rem, 16), nk_total / 16);
    if (s < 2 || (long long)8 * rem * s * PM * PN * (int)sizeof(float) > ws_bytes) return plan;
    plan.q_end = per_xcd - rem;
    plan.parts = s;
    plan.per = up_div(nk_total, s);
    if (a_kmajor) plan.per += plan.per & 1;  // parts start on a 64-k boundary: whole 128-byte lines of A
    return plan;
}

// The kernel whose estimated time is shorter.  Both estimates count rounds of tiles over the compute units of an XCD: so many
// us (here in units of 1e-4) for each k of the contraction and for what a tile costs
// besides, with the last round on its own.  The constants are fits to measured products of 128 .. 8192 rows,
// K 128 .. 28672, each form (data gradient, weight gradient, forward), which they reproduce to about 10 % (both kernels on 40
// products: profiles/contraction_kernels_both_sides.txt; the one taken is never more than 2 % behind the other, but for
// 487 x 4096 x 28672, a tie by the estimates: 126 and 118 us).  Of the 256x256 kernel only the forward constant was fitted again
// since its rings hold half stages; data gradients have become up to 3 % faster than theirs says:
//   256x256 tiles, one per compute unit:   0.0232 K + 11 us a round (forward 0.0222 K); a last round that is cut along K (big_parts
//                                          > 1) adds its two kernels
//   128x256 tiles, two per compute unit:   0.0265 K + 2 us a round (0.0255 K + 3 weight gradient, 0.0276 K + 6 forward);
//                                          with one per compute unit, half of that
// The second one reads 1.5 times as much from L2 per multiply-add, which the long K pays for (8192 x 4096 x 28672: 1290
// against 1505 us), and has no idle start and end of tile, nor as coarse a last round (weight gradients 14336 x 4096 x 480: 81
// against 59 us, 6144 x 4096 x 1024: 80 against 49; data gradients 487 x 4096 x 4096: 46 against 30, 6001 x 4096 x 6144: 241 against
// 228 us).
// Whole tiles of the second one fill rounds of two work-groups per compute unit, or a last one of at most one each; the
// tiles cut along K run beside that.  4099 x 2048 x 16384 is 17 tiles for the 32 compute units of an XCD, or 32 whole tiles
// of half the size and one in 16 parts: 261 against 220 us.
__host__ __device__ inline bool pair_is_better(int M, int N, long long K, bool a_kmajor, bool b_kmajor, bool swiglu, int n_cu, int big_parts,
                                               const PairPlan& plan) {
    const int cus = n_cu / 8;                             // compute units of an XCD
    const long long swiglu_split = swiglu ? 150000 : 0;  // its finish kernel also moves G, U, dG, dU, Act
    const int tiles = up_div(up_div(M, 256) * up_div(N, 256), 8);
    const long long big_k = (b_kmajor ? 222 : 232) * K;
    long long big = tiles / cus * (big_k + 110000);
    if (tiles % cus) big += big_parts > 1 ? big_k / big_parts + 330000 + swiglu_split : big_k * 9 / 10 + 110000;
    const long long pair_k = (b_kmajor ? 276 : a_kmajor ? 265 : 255) * K, pair_fixed = b_kmajor ? 60000 : a_kmajor ? 20000 : 30000;
    long long pair = plan.q_end / (2 * cus) * (pair_k + pair_fixed);
    const int rest = plan.q_end % (2 * cus), cut = plan.per_xcd - plan.q_end, s = plan.parts;
    if (rest > 0) pair += rest <= cus ? pair_k * 52 / 100 + 40000 : pair_k * 9 / 10 + pair_fixed;
    if (cut > 0) pair += (cut * s > cus ? pair_k / s + 270000 : pair_k * 52 / 100 / s + 170000) + swiglu_split;
    return pair < big;
}
// Plan and choice of a product whose row count lies on the device, for Mv rows of it.  Two rounds of 128x256 tiles at most:
// beyond that the two kernels differ by little, and the grid that leaves when the others are chosen stays at 1024
// work-groups (5 us in a profile, 2 between products).
enum RowsKernel { kRowsBig, kRowsPair, kRowsNarrow64, kRowsNarrow128 };
// Work-groups of k_gemm_narrow_rows for Mv rows
__host__ __device__ inline int narrow_grid(const MfmaGemmParams& p, int Mv, RowsKernel kernel) {
    const int tile = kernel == kRowsNarrow64 ? 64 : 128;
    return 8 * up_div(up_div(Mv, tile) * up_div(p.N, tile), 8);
}
__host__ __device__ inline RowsKernel device_plan(const MfmaGemmParams& p, int Mv, PairPlan& plan) {
    int nk = 0;
    long long K = 0;
    for (int s = 0; s < p.n_seg; ++s) {
        nk += up_div(p.K[s], BK);
        K += p.K[s];
    }
    plan = pair_plan(Mv, p.N, nk, p.a_kmajor != 0, p.plan_cu, p.plan_ws);
    const bool pair = plan.per_xcd <= 4 * (p.plan_cu / 8) &&
                      pair_is_better(Mv, p.N, K, p.a_kmajor != 0, p.b_kmajor != 0, p.epilogue == kEpiSwigluBwd, p.plan_cu, 1, plan);
    // The smallest tile of which no compute unit has two: where that is one of 64x64 or 128x128 their contraction is as long as that of a
    // 128x256 tile, and a step of 64 k takes 341 and 507 ns of 160 and 680 rows by 4096 against 770 (K 128256; a second round of the small
    // ones 290 more).  Past one round of 128x128 the wide tile is the better one: 1244 rows, K 32000 388 against 512 us.  The same line for
    // dAct, whose columns leave the narrow tiles fewer rows: 14336 columns, K 4096 60 rows 80 -> 46 us, 250 86 -> 63; 28672, K 8192 125 rows 183 -> 150.
    if (p.narrow) {
        if (narrow_grid(p, Mv, kRowsNarrow64) <= p.plan_cu) return kRowsNarrow64;
        if (narrow_grid(p, Mv, kRowsNarrow128) <= p.plan_cu) return kRowsNarrow128;
    }
    return pair ? kRowsPair : kRowsBig;
}

int launch_gemm_pair(MfmaGemmParams p, bool a_kmajor, bool b_kmajor, int tiles_m, const PairPlan& plan, float* split_ws, hipStream_t stream);
int launch_gemm_pair_rows(MfmaGemmParams p, int grid, int cut, float* split_ws, hipStream_t stream);  // m_dev, k-major A: most work-groups, cut tiles of an XCD
int launch_gemm_narrow_rows(const MfmaGemmParams& p, int grid, hipStream_t stream);  // m_dev, k-major A, token-major B
size_t pair_split_bytes(const PairPlan& plan);  // scratch of its partial tiles
int pair_grid(const PairPlan& plan);            // its work-groups
int launch_gemm_two_pairs(MfmaGemmParams data, int data_tiles_m, const PairPlan& data_plan, MfmaGemmParams weight, int weight_tiles_m,
                          const PairPlan& weight_plan, float* split_ws, hipStream_t stream);

template <int I> struct IntC { static constexpr int value = I; };

}  // namespace alch
