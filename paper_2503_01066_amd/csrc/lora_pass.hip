// Adapter products of bf16 layers on the matrix cores: the gradients of an adapter, C = S^T X over the tokens (dA = t2^T x,
// dB = dy^T t1, "up"), by themselves or in one pass with a rank-r product of the same rows, t = alpha X P^T ("down": t1 = s x A^T
// on Act, t2 = s dy B on dG and dU), so that [dG | dU] and Act, the largest activations of a layer, are read once and not twice.
//
// What bounds both kernels: HBM, behind the write-back of the product that wrote the activation.  Eight multiply-adds an
// element for either contraction are as long as the memory on the vector ALU; the matrix cores do them, from one copy of the
// rows in LDS: "down" reads them as they lie, "up" with the transposing LDS read.  Sums over the tokens are left as fp32 partial
// sums of a row block or split and added in a fixed order at the end of the layer (k_lora_up_finish): no atomics.
// 8B shape, 5120 tokens, us: [dG | dU] and Act in one pass 113 (3.9 TB/s) and 5 for the sums of t, before 213 for t and 132 for
// the gradients, dY and H2 among them; the other gradients 60 (4.5 TB/s), before 70; all adapter work of a layer 451 -> 314.
// Layers with adapters, us: 100 tokens 310 -> 283, 900 672 -> 637, 5003 2782 -> 2667, heads of 64 1000 tokens 410 -> 358.
#include <algorithm>

#include "kernels.h"

namespace alch {

typedef __attribute__((ext_vector_type(8))) __bf16 bf16x8;
typedef __attribute__((ext_vector_type(4))) __bf16 bf16x4;
typedef __attribute__((ext_vector_type(16))) float f32x16;
typedef __attribute__((ext_vector_type(4))) float f32x4;
typedef __attribute__((ext_vector_type(4))) int i32x4;
#define ALCH_LDS(p) ((__attribute__((address_space(3))) void*)(p))

static constexpr int kPassCols = 512, kPassRows = 32;  // k_lora_up_mfma: columns of a work-group, rows of a step
static constexpr int kPassProblems = 12, kPassGroups = 4;
static constexpr int kPassStage = kPassRows * kPassCols * 2, kPassQ = kPassRows * 64;  // bytes: rows of X, of the up factors
static constexpr uint32_t kPassOob = 0x80000000u;

struct LoraPassProblem {
    const __bf16* X; long long ldx; int K;
    int n_down; const __bf16* P; long long ldp;          // groups of eight rows of P [8 n_down, K]
    int n_up; const __bf16* Q; int q_col[kPassGroups];   // groups of eight columns of Q (row stride ldq), first columns
    long long up_off[kPassGroups];                       // partial sums of a group: floats from `scratch`, [split][8][K]
    long long t_off;                                     // those of "down": [part][Trows][8 n_down]
    int first;                                           // first blockIdx.x of the problem
};
struct LoraPassParams {
    LoraPassProblem pr[kPassProblems];
    int n, Trows, rows_per_split, parts;
    long long ldq;
    float* scratch;
    const int* rows_dev;  // the row count is min(*rows_dev, Trows); splits past it are not written
};

__device__ __forceinline__ i32x4 pass_rsrc(const void* p, long long bytes) {
    const uint64_t a = reinterpret_cast<uint64_t>(p);
    i32x4 r;
    r[0] = __builtin_amdgcn_readfirstlane((int)(uint32_t)a);
    r[1] = __builtin_amdgcn_readfirstlane((int)((uint32_t)(a >> 32) & 0xffffu));
    r[2] = __builtin_amdgcn_readfirstlane((int)(bytes < 0 ? 0 : bytes));
    r[3] = 0x00020000;
    return r;
}
// (s_nop: a load into LDS takes one wait state after a scalar write of m0, which the compiler does not see to in assembly)
__device__ __forceinline__ void pass_dma16(i32x4 r, uint32_t lds_addr, uint32_t voff) {
    asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tbuffer_load_dwordx4 %1, %2, 0 offen lds" ::"s"(lds_addr), "v"(voff), "s"(r)
                 : "memory", "m0");
}
// 16-byte piece c of row r of X sits at position c ^ pass_swz(r) of its row: 16 rows at one piece, and four rows at four pieces
// in a row, then lie in 16 different pieces of a 256-byte bank line
__device__ __forceinline__ int pass_swz(int row) { return ((row & 3) << 2) | ((row >> 2) & 3); }
// Operand fragment of eight consecutive rows of a token-major tile in LDS (second: four rows on)
__device__ __forceinline__ bf16x8 pass_tr(const char* first, const char* second) {
    const bf16x4 lo = __builtin_amdgcn_ds_read_tr16_b64_v4bf16((__attribute__((address_space(3))) bf16x4*)first);
    const bf16x4 hi = __builtin_amdgcn_ds_read_tr16_b64_v4bf16((__attribute__((address_space(3))) bf16x4*)second);
    return __builtin_shufflevector(lo, hi, 0, 1, 2, 3, 4, 5, 6, 7);
}
// Rows of the work-group's block or split that starts at r0 (none: nothing to do)
__device__ __forceinline__ int pass_rows(const LoraPassParams& p, long long r0, int most) {
    const int Trows = p.rows_dev ? min(__builtin_amdgcn_readfirstlane(*p.rows_dev), p.Trows) : p.Trows;
    return (int)min((long long)most, Trows - r0);
}
__device__ __forceinline__ int pass_problem(const LoraPassParams& p) {
    int at = 0;
    for (int i = 1; i < p.n; ++i)
        if ((int)blockIdx.x >= p.pr[i].first) at = i;
    return at;
}
// Offset of the lane's 16 bytes of the up factors (lane: row lane / 4, group lane % 4); groups that do not exist read zeros
__device__ __forceinline__ uint32_t pass_q_offset(const LoraPassProblem& pb, long long ldq, int lane) {
    uint32_t v = kPassOob;
#pragma unroll
    for (int g = 0; g < kPassGroups; ++g)
        if (g == (lane & 3) && g < pb.n_up) v = (uint32_t)(((lane >> 2) * ldq + pb.q_col[g]) * 2);
    return v;
}

// "up" alone.  A work-group owns 512 columns and the rows of a split, which it takes 32 at a time, one step ahead in LDS; the
// sums stay in registers.
__global__ __launch_bounds__(256, 2) void k_lora_up_mfma(LoraPassParams p) {
    __shared__ __attribute__((aligned(1024))) char smem[2 * (kPassStage + kPassQ)];
    const uint32_t lds0 = (uint32_t)(uintptr_t)ALCH_LDS(smem);
    const int lane = threadIdx.x & 63, half = lane >> 5, c = lane & 31;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const LoraPassProblem& pb = p.pr[pass_problem(p)];
    const int c0 = ((int)blockIdx.x - pb.first) * kPassCols, K = pb.K, n_up = pb.n_up;
    const long long r0 = (long long)blockIdx.y * p.rows_per_split;
    const int rows = pass_rows(p, r0, p.rows_per_split);
    if (rows <= 0) return;
    const int n = (rows + kPassRows - 1) / kPassRows;

    // loads of a step: row wave*8 + j of X each, 16 bytes a lane; the first two wavefronts also 16 rows of the up factors
    const uint32_t vq = pass_q_offset(pb, p.ldq, lane);
    const __bf16* Xb = pb.X + (r0 + wave * 8) * pb.ldx + c0;
    const __bf16* Qb = pb.Q + (r0 + wave * 16) * p.ldq;
    const int cols = min(kPassCols, K - c0);
    // (addresses are formed anew in every step from a lane number that the compiler cannot see through: kept, they spill, and the
    // reload of each waits for all loads before it)
    auto issue = [&](int i, int ln) {
        const int left = rows - i * kPassRows;
        const uint32_t st = lds0 + (uint32_t)(i & 1) * (kPassStage + kPassQ);
        const __bf16* x = Xb + (long long)i * kPassRows * pb.ldx;
#pragma unroll
        for (int j = 0; j < 8; ++j)  // past the last row or column: zeros
            pass_dma16(pass_rsrc(x + j * pb.ldx, wave * 8 + j < left ? cols * 2 : 0), st + (uint32_t)(wave * 8 + j) * 1024u,
                       (uint32_t)((ln << 4) ^ (pass_swz(wave * 8 + j) << 4)));
        if (wave < 2) {
            const int q_rows = min(left - wave * 16, 16);
            pass_dma16(pass_rsrc(Qb + (long long)i * kPassRows * p.ldq, q_rows > 0 ? ((q_rows - 1) * p.ldq + kLoraSlot * 3) * 2 : 0),
                       st + kPassStage + (uint32_t)wave * 1024u, vq);
        }
    };
    issue(0, lane);
    f32x16 up[4];
#pragma unroll
    for (int nb = 0; nb < 4; ++nb)
#pragma unroll
        for (int e = 0; e < 16; ++e) up[nb][e] = 0.f;
    for (int i = 0; i < n; ++i) {
        // the loads of step i are there and every wavefront is done with step i - 1
        asm volatile("s_waitcnt vmcnt(0) lgkmcnt(0)\n\ts_barrier" ::: "memory");
        int ln = lane;
        asm volatile("" : "+v"(ln));
        if (i + 1 < n) issue(i + 1, ln);
        const char* st = smem + (i & 1) * (kPassStage + kPassQ);
        // transposing reads: this lane's row of the 4 x 4 block of lanes, its four columns of 32
        const int row = 8 * (ln >> 5) + ((ln & 15) >> 2), col = ((ln >> 4) & 1) * 16 + 4 * (ln & 3);
        const char* q = st + kPassStage + row * 64 + col * 2;
        const char* xs = st + wave * 256 + (col & 7) * 2;
        const int at0 = row * 1024 + (((col >> 3) ^ pass_swz(row)) << 4), at1 = (row + 4) * 1024 + (((col >> 3) ^ pass_swz(row + 4)) << 4);
#pragma unroll
        for (int ks = 0; ks < 2; ++ks) {
            const bf16x8 qf = pass_tr(q + ks * 1024, q + ks * 1024 + 256);
#pragma unroll
            for (int nb = 0; nb < 4; ++nb)
                up[nb] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(qf, pass_tr(xs + ks * 16384 + (at0 ^ (nb << 6)), xs + ks * 16384 + (at1 ^ (nb << 6))),
                                                                 up[nb], 0, 0, 0);
        }
    }
    // element e of up[nb]: factor column 8 (e >> 2) + 4 half + (e & 3), column nb*32 + c of the wavefront's 128
#pragma unroll
    for (int g = 0; g < kPassGroups; ++g) {
        if (g >= n_up) break;
        float* out = p.scratch + pb.up_off[g] + ((long long)blockIdx.y * 8 + 4 * half) * K;
#pragma unroll
        for (int nb = 0; nb < 4; ++nb) {
            const int col = c0 + wave * 128 + nb * 32 + c;
            if (col < K) {
#pragma unroll
                for (int e = 0; e < 4; ++e) out[(long long)e * K + col] = up[nb][4 * g + e];
            }
        }
    }
}

// "down" and "up" in one pass.  A work-group owns kM blocks of 128 rows and one of `parts` parts of the contraction of "down",
// cut and summed exactly as k_lora_down_mfma does (t2 is an operand of the data gradients: its bits, and those of all layers below,
// stay).  It walks its part 128 columns at a time, for each the blocks of rows, one step ahead in LDS.  "down": a wavefront's
// 32 rows of a block, in registers over all columns; "up": its 32 of the 128 columns over all rows of the work-group, which leave
// as the partial sums of a split after every 128 columns.
static constexpr int kBothRows = 128, kBothCols = 128, kBothStage = kBothRows * kBothCols * 2;
template <int kM>
__global__ __launch_bounds__(256, 2) void k_lora_both(LoraPassParams p) {
    __shared__ __attribute__((aligned(1024))) char smem[2 * kBothStage + kM * kBothRows * 64];
    const uint32_t lds0 = (uint32_t)(uintptr_t)ALCH_LDS(smem);
    const int lane = threadIdx.x & 63, half = lane >> 5, c = lane & 31;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const LoraPassProblem& pb = p.pr[pass_problem(p)];
    const int part = (int)blockIdx.x - pb.first, chunks = pb.K >> 6;
    const int k0 = part * chunks / p.parts * 64, cols = (part + 1) * chunks / p.parts * 64 - k0;  // this part's columns
    const long long r0 = (long long)blockIdx.y * (kM * kBothRows);
    const int rows = pass_rows(p, r0, kM * kBothRows);
    if (rows <= 0) return;
    const int n = (cols + kBothCols - 1) / kBothCols * kM, n_down = pb.n_down, n_up = pb.n_up;
    const uint32_t q_lds = lds0 + 2 * kBothStage;

    {   // the up factors of all rows
        const uint32_t vq = pass_q_offset(pb, p.ldq, lane);
#pragma unroll
        for (int j = 0; j < 2 * kM; ++j) {
            const int row = (wave * 2 * kM + j) * 16, left = min(rows - row, 16);
            pass_dma16(pass_rsrc(pb.Q + (r0 + row) * p.ldq, left > 0 ? ((left - 1) * p.ldq + kLoraSlot * 3) * 2 : 0), q_lds + (uint32_t)row * 64u, vq);
        }
    }
    // loads of a step: rows wave*32 + 4j .. +3 of a block, 256 bytes each (past the last row or column: zeros)
    const __bf16* Xb = pb.X + (r0 + wave * 32) * pb.ldx + k0;
    uint32_t vx[4];
    int piece[4];
#pragma unroll
    for (int j = 0; j < 4; ++j) {
        piece[j] = (lane & 15) ^ ((lane >> 4) << 2) ^ j;
        vx[j] = (uint32_t)((lane >> 4) * pb.ldx * 2 + piece[j] * 16);
    }
    auto issue = [&](int i) {
        const int m = i % kM, col = i / kM * kBothCols, left = rows - m * kBothRows - wave * 32, pieces = (cols - col) / 8;
        const uint32_t st = lds0 + (uint32_t)(i & 1) * kBothStage + (uint32_t)wave * 8192u;
        const __bf16* x = Xb + (long long)m * kBothRows * pb.ldx + col;
#pragma unroll
        for (int j = 0; j < 8; ++j) {
            const int valid = min(left - 4 * j, 4);
            pass_dma16(pass_rsrc(x + (long long)(4 * j) * pb.ldx, valid > 0 ? ((valid - 1) * pb.ldx + min(kBothCols, cols - col)) * 2 : 0), st + (uint32_t)j * 1024u,
                       piece[j & 3] < pieces ? vx[j & 3] : kPassOob);
        }
    };
    // operand of "down": row c of P, k of 128 columns
    const __bf16* Pb = pb.P + (long long)c * pb.ldp + k0 + 8 * half;
    auto factors = [&](int col, bf16x8 (&f)[8]) {
#pragma unroll
        for (int kk = 0; kk < 8; ++kk) {
            bf16x8 z;
#pragma unroll
            for (int e = 0; e < 8; ++e) z[e] = (__bf16)0.f;
            f[kk] = c < 8 * n_down && col + kk * 16 < cols ? *reinterpret_cast<const bf16x8*>(Pb + col + kk * 16) : z;
        }
    };
    bf16x8 pf[8], pn[8];
    factors(0, pn);
    issue(0);
    f32x16 down[kM], up;
#pragma unroll
    for (int m = 0; m < kM; ++m)
#pragma unroll
        for (int e = 0; e < 16; ++e) down[m][e] = 0.f;
    const int row = 8 * half + ((lane & 15) >> 2), col4 = ((lane >> 4) & 1) * 16 + 4 * (lane & 3);  // transposing reads
    const char* q = smem + 2 * kBothStage + row * 64 + col4 * 2;
    const int at0 = row * 256 + (((wave * 4 + (col4 >> 3)) ^ pass_swz(row)) << 4) + (col4 & 7) * 2;
    const int at1 = (row + 4) * 256 + (((wave * 4 + (col4 >> 3)) ^ pass_swz(row + 4)) << 4) + (col4 & 7) * 2;
    const int at_down = (wave * 32 + c) * 256 + ((half ^ pass_swz(c)) << 4);
    for (int i0 = 0; i0 < n; i0 += kM) {
        const int col = i0 / kM * kBothCols;
#pragma unroll
        for (int e = 0; e < 16; ++e) up[e] = 0.f;
#pragma unroll
        for (int m = 0; m < kM; ++m) {
            const int i = i0 + m;
            // the loads of step i are there and every wavefront is done with step i - 1
            asm volatile("s_waitcnt vmcnt(0) lgkmcnt(0)\n\ts_barrier" ::: "memory");
            if (m == 0) {
#pragma unroll
                for (int kk = 0; kk < 8; ++kk) pf[kk] = pn[kk];
                if (i + kM < n) factors(col + kBothCols, pn);
            }
            if (i + 1 < n) issue(i + 1);
            const char* st = smem + (i & 1) * kBothStage;
#pragma unroll
            for (int kk = 0; kk < 8; ++kk)
                down[m] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(*reinterpret_cast<const bf16x8*>(st + (at_down ^ (kk << 5))), pf[kk], down[m], 0, 0, 0);
#pragma unroll
            for (int ks = 0; ks < 8; ++ks)
                up = __builtin_amdgcn_mfma_f32_32x32x16_bf16(pass_tr(q + (m * 8 + ks) * 1024, q + (m * 8 + ks) * 1024 + 256),
                                                             pass_tr(st + ks * 4096 + at0, st + ks * 4096 + at1), up, 0, 0, 0);
        }
        // element e of up: factor column 8 (e >> 2) + 4 half + (e & 3), column c of the wavefront's 32
        if (col + wave * 32 + c < cols) {
#pragma unroll
            for (int g = 0; g < kPassGroups; ++g) {
                if (g >= n_up) break;
                float* out = p.scratch + pb.up_off[g] + ((long long)blockIdx.y * 8 + 4 * half) * pb.K + k0 + col + wave * 32 + c;
#pragma unroll
                for (int e = 0; e < 4; ++e) out[(long long)e * pb.K] = up[4 * g + e];
            }
        }
    }
    if (c < 8 * n_down) {
#pragma unroll
        for (int m = 0; m < kM; ++m) {
            const int first = m * kBothRows + wave * 32;
            float* t = p.scratch + pb.t_off + ((long long)part * p.Trows + r0 + first) * (8 * n_down) + c;
#pragma unroll
            for (int e = 0; e < 16; ++e) {
                const int r = 8 * (e >> 2) + 4 * half + (e & 3);
                if (first + r < rows) t[(long long)r * (8 * n_down)] = down[m][e];
            }
        }
    }
}

// Sums of "down" over the parts -> eight columns of an output slot in bf16; columns past the rank of a slot as zeros (it is
// read as a zero-padded operand of a matrix-core product).  A thread owns the eight columns of one row.
struct LoraTJob {
    long long t_off; int parts, groups, group;  // parts = 0: zeros
    __bf16* out;
};
static constexpr int kTJobs = 3 * kLoraSlot / 8;
struct LoraTParams {
    LoraTJob job[kTJobs];
    int n, Trows;
    long long ldo;
    float alpha;
    const float* scratch;
    const int* rows_dev;
};
__global__ __launch_bounds__(256) void k_lora_t_finish(LoraTParams p) {
    const LoraTJob jb = p.job[blockIdx.y];
    const int row = blockIdx.x * 256 + threadIdx.x;
    if (row >= (p.rows_dev ? min(*p.rows_dev, p.Trows) : p.Trows)) return;
    f32x4 lo = {0.f, 0.f, 0.f, 0.f}, hi = lo;
    const float* t = p.scratch + jb.t_off + ((long long)row * jb.groups + jb.group) * 8;
#pragma unroll 4
    for (int s = 0; s < jb.parts; ++s) {
        const f32x4* at = reinterpret_cast<const f32x4*>(t + (long long)s * p.Trows * jb.groups * 8);
        lo += at[0];
        hi += at[1];
    }
    bf16x8 o;
#pragma unroll
    for (int e = 0; e < 8; ++e) o[e] = (__bf16)(p.alpha * (e < 4 ? lo[e & 3] : hi[e & 3]));
    *reinterpret_cast<bf16x8*>(jb.out + (long long)row * p.ldo) = o;
}

// ---- host ----------------------------------------------------------------------------------------------------------
// How a launch runs: "up" alone in splits of the rows, two work-groups to a compute unit and 64 rows to a split at least; both in
// blocks of 128 rows, or of 256 where those are more than two work-groups to a compute unit, or more splits than there may be.
// (parts of K: see k_lora_both.)
struct PassPlan {
    bool both;
    int n_up, splits, rows, parts;
    long long need_up, need_t;  // floats of scratch: the gradients' partial sums, which stay until the layer's sums, and those of "down"
};
static int plan_pass(const LoraPass* jobs, int n_jobs, int Trows, const LoraUpSums& sums, PassPlan& p) {
    const int r = sums.p.r, groups = r / 8;
    p = {};
    int slabs = 0, problems = 0, kept = 0;
    long long width = 0;  // columns of all gradients
    for (int i = 0; i < n_jobs; ++i) {
        const LoraPass& j = jobs[i];
        const int n = std::max(ceil_div(j.n_up * groups, kPassGroups), j.P ? ceil_div(groups, kPassGroups) : 0);
        slabs += ceil_div(j.K, kPassCols) * n;
        problems += n;
        p.n_up += j.n_up;
        p.both = p.both || j.P;
        if (j.P && j.keep_bits) kept += ceil_div(groups, kDownGroups);
        width += (long long)j.n_up * j.K;
    }
    int n_cu = 0;
    ALCH_TRY(compute_units(&n_cu));
    if (p.both) {
        p.parts = lora_down_parts(Trows, std::max(kept, 1), n_cu);
        p.rows = ceil_div(Trows, kBothRows) * p.parts * problems <= 2 * n_cu && ceil_div(Trows, kBothRows) <= kLoraMaxSplits ? kBothRows : 2 * kBothRows;
        for (int i = 0; i < n_jobs; ++i)
            if (jobs[i].P) p.need_t += (long long)p.parts * Trows * r;
        p.need_t += 4;  // (aligned from the end of the scratch)
    } else {
        int splits = slabs > 0 ? std::max(1, std::min(std::min(2 * n_cu / slabs, kLoraMaxSplits), ceil_div(Trows, 64))) : 1;
        while (splits > 1 && width * r * splits > sums.capacity) splits = (splits + 1) / 2;
        p.rows = ceil_div(ceil_div(Trows, splits), kPassRows) * kPassRows;
    }
    p.splits = ceil_div(Trows, p.rows);
    p.need_up = width * r * p.splits;
    return ALCH_OK;
}
// What k_lora_both takes: K is cut in chunks of 64, and the rows of a block lie within 1 GiB (offsets in 32 bits).
static bool both_takes(const LoraPass& j) { return j.K % 64 == 0 && j.ldx % 8 == 0 && j.ldp % 8 == 0 && kBothRows * j.ldx < (1LL << 29); }
bool lora_pass_fits(const LoraPass* jobs, int n_jobs, int Trows, const LoraUpSums& sums) {
    PassPlan p;
    for (int i = 0; i < n_jobs; ++i)
        if (!both_takes(jobs[i])) return false;
    return plan_pass(jobs, n_jobs, Trows, sums, p) == ALCH_OK && p.need_up + p.need_t <= sums.capacity && p.splits <= kLoraMaxSplits;
}

int launch_lora_pass(const LoraPass* jobs, int n_jobs, int Trows, long long ldq, float alpha, LoraUpSums& sums, hipStream_t stream,
                     const int* rows_dev) {
    if (Trows <= 0 || n_jobs <= 0) return ALCH_OK;
    const int r = sums.p.r, groups = r / 8;
    if (r % 8 || r <= 0 || ldq % 8) return fail(ALCH_ERR_UNSUPPORTED, "adapter product: rank must be a positive multiple of 8");
    PassPlan plan;
    ALCH_TRY(plan_pass(jobs, n_jobs, Trows, sums, plan));
    for (int i = 0; i < n_jobs; ++i)
        if (jobs[i].K % 8 || jobs[i].ldx % 8 || (plan.both && !both_takes(jobs[i])))
            return fail(ALCH_ERR_UNSUPPORTED, "adapter product: widths and strides must be multiples of 8, of a shared pass of 64");
    if (sums.p.n_jobs + plan.n_up > kLoraUpSums || sums.floats + plan.need_up + plan.need_t > sums.capacity)
        ALCH_TRY(launch_lora_up_sums(ALCH_BF16, sums, stream));
    if (plan.need_up + plan.need_t > sums.capacity) return fail(ALCH_ERR_UNSUPPORTED, "adapter product: more partial sums than scratch");
    LoraPassParams p = {};
    LoraTParams tp = {};
    p.Trows = tp.Trows = Trows;
    p.rows_per_split = plan.rows;
    p.rows_dev = tp.rows_dev = rows_dev;
    p.parts = plan.parts;
    p.ldq = tp.ldo = ldq;
    tp.alpha = alpha;
    p.scratch = sums.p.scratch;
    tp.scratch = sums.p.scratch;
    long long t_off = (sums.capacity - plan.need_t) / 4 * 4;
    double flops = 0, bytes = 0;
    int first = 0;
    for (int i = 0; i < n_jobs; ++i) {
        const LoraPass& j = jobs[i];
        const int up_groups = j.n_up * groups, down_groups = j.P ? groups : 0;
        long long up_off[kPassUps];
        for (int u = 0; u < j.n_up; ++u) {
            up_off[u] = sums.floats;
            add_lora_up_job(sums, LoraUp{nullptr, 0, j.X, j.ldx, j.K, j.up[u].C, j.up[u].ldc, j.up[u].transposed}, plan.splits,
                            rows_dev, plan.rows);
        }
        for (int g0 = 0; g0 < up_groups || g0 < down_groups; g0 += kPassGroups) {
            if (p.n == kPassProblems) return fail(ALCH_ERR_UNSUPPORTED, "adapter product: too many problems");
            LoraPassProblem& pb = p.pr[p.n++];
            pb.X = static_cast<const __bf16*>(j.X); pb.ldx = j.ldx; pb.K = j.K;
            pb.first = first;
            first += plan.both ? plan.parts : ceil_div(j.K, kPassCols);
            pb.n_down = std::max(0, std::min(down_groups - g0, kPassGroups));
            pb.P = pb.n_down > 0 ? static_cast<const __bf16*>(j.P) + (long long)g0 * 8 * j.ldp : nullptr; pb.ldp = j.ldp;
            pb.n_up = std::max(0, std::min(up_groups - g0, kPassGroups));
            pb.Q = static_cast<const __bf16*>(pb.n_up > 0 ? j.Q : j.X);  // (never read without groups)
            for (int g = 0; g < pb.n_up; ++g) {
                const int u = (g0 + g) / groups, chunk = (g0 + g) % groups;
                pb.q_col[g] = j.up[u].q_col + chunk * 8;
                pb.up_off[g] = up_off[u] + (long long)chunk * plan.splits * 8 * j.K;
            }
            if (pb.n_down > 0) {
                pb.t_off = t_off;
                for (int g = 0; g < pb.n_down; ++g)
                    tp.job[tp.n++] = LoraTJob{t_off, plan.parts, pb.n_down, g, static_cast<__bf16*>(j.T) + (g0 + g) * 8};
                t_off += (long long)plan.parts * Trows * pb.n_down * 8;
            }
            flops += rows_dev ? 0.0 : 2.0 * Trows * j.K * 8 * (pb.n_down + pb.n_up);  // (what is done only the device knows)
            bytes += rows_dev ? 0.0 : 2.0 * Trows * j.K;
        }
        for (int g = down_groups; j.pad && g < kLoraSlot / 8; ++g) tp.job[tp.n++] = LoraTJob{0, 0, 1, 0, static_cast<__bf16*>(j.T) + g * 8};
    }
    TraceScope ts(kTraceLora, flops, bytes, stream);
    const dim3 grid(first, plan.splits);
    if (p.n > 0 && !plan.both) k_lora_up_mfma<<<grid, 256, 0, stream>>>(p);
    else if (p.n > 0 && plan.rows == kBothRows) k_lora_both<1><<<grid, 256, 0, stream>>>(p);
    else if (p.n > 0) k_lora_both<2><<<grid, 256, 0, stream>>>(p);
    if (tp.n > 0) k_lora_t_finish<<<dim3(ceil_div(Trows, 256), tp.n), 256, 0, stream>>>(tp);
    ALCH_HIP_TRY(hipGetLastError());
    return ALCH_OK;
}

}  // namespace alch
