// bf16 GEMM on the gfx950 matrix cores: C[M,N] (+)= sum_s A_s(M,K_s) B_s(K_s,N), fp32 accumulate.
//
// This one kernel carries all dense contractions of the decoder-layer backward pass
// (Section 4.2 / 4.3.2 of the paper: per-layer backward from saved activations): the
// data gradients (dY.W, activation k-major x weight n-major), the weight gradients
// (dOut^T.Act, both operands token-major, contraction over tokens) and the forward
// projections (x.W^T, both k-major).
//
// Design for CDNA4:
//   * 256x256 tile per work-group, contraction in steps of 32, 4 wavefronts of 64 lanes, each owning 128x128 of the
//     tile as 4x4 MFMA 32x32x16 bf16 accumulators (256 accumulator registers per lane).
//   * Tiles are fetched HBM/L2 -> LDS with 16-byte direct-to-LDS buffer loads (no registers in between) into two rings of
//     five 16 KB stages, one per operand, that fill the 160 KB LDS.  A stage holds 32 k of 256 columns, or, of a k-major
//     operand, 64 k of 128 rows, so that every load covers whole 128-byte lines (see tile_offsets_wide).
//     A direct-to-LDS load writes lane-linearly, so the bank-conflict swizzle is applied
//     by permuting which global 16-byte chunk each lane fetches.
//   * Operands whose contraction index is contiguous in memory are read from LDS with
//     ds_read_b128; operands whose contraction index is the row (token) index are read
//     with the transposing ds_read_b64_tr_b16, so no transposed copy is ever made.
//   * Out-of-range rows/columns (ragged token counts) come back as zeros from the buffer
//     load's range check; stores are predicated.
//   * Work-groups are numbered so that each of the 8 XCDs (one L2 each) works on a
//     compact patch of output tiles.
//   * The grid is persistent, one work-group per compute unit, each walking its share of the tiles
//     round by round.  When the last round would hold tiles for at most half of the compute units, it
//     is left to a second launch (the kSplit instantiation) in which s work-groups of the same XCD
//     share a tile, each taking 1/s of the contraction and leaving an fp32 partial tile in a scratch
//     buffer; k_gemm_split_finish adds the s partials in a fixed order and writes the output
//     (deterministic, no atomics).
#include <atomic>
#include "gemm_mfma_common.h"

namespace alch {

static constexpr int BM = 256, BN = 256;
static constexpr int kStages = 5;                        // of either operand: 2 x 5 x 16 KB = the whole 160 KB LDS
static constexpr int kOperandStageBytes = 256 * BK * 2;  // 16 KB
static constexpr int kLoadsPerTile = 8;                  // direct-to-LDS instructions per wave per k-tile (A + B)
static constexpr int kGroupM = 4;                        // tile rows per raster band

// ---- the rings
// Two k-tiles (64 k) are used up together: batch b of an operand, in stage b % 5, is half b & 1 of its 64 k number b / 2.
// Of an operand whose columns are contiguous the halves are its k-tiles; of a k-major one they are rows 0-127 and 128-255,
// all 64 k of them: a k-tile takes 64 bytes of every row, and fetched by itself every 128-byte line crosses the L2 -> L1
// path twice (the 32 KB L1 has long lost it by the second time), which costs time and power.  Batches of 64 k free their
// stages two at a time, so five stages hold what 2.5 x 64 k need, and one barrier in two k-tiles is enough: batch kt + 4
// goes out in the second half of step kt and has 1.5 steps (1 us) to land if kt is odd, 2.5 if it is even.  Before, with 32 k
// a stage for B (A in three stages of 64 k x 256 rows), four and five k-tiles ahead: 8192 x 4096 x 28672, both operands
// k-major, 1458 -> 1301 us, 8192 x 14336 x 4096 751 -> 677, 3001 x 4096 x 14336 292 -> 266; a layer forward of 5003 tokens
// 2029 -> 1931 us.  The other forms, whose lines were whole before, are within 1 % of what they were.
//   slot (16-byte units) in a stage of rows = rl*8 + (c ^ ((rl>>1)&7)), rl = row & 127, c = 16-byte chunk of the
//   row's 64 k: 16 consecutive rows at one logical chunk then cover all 64 banks once (ds_read_b128).
__device__ __forceinline__ void tile_offsets_wide(uint32_t (&voff)[8], int wave, int lane, long long ld, int valid) {
#pragma unroll
    for (int h = 0; h < 2; ++h)
#pragma unroll
        for (int j = 0; j < 4; ++j) {
            const int sl = (wave * 4 + j) * 64 + lane;
            const int rl = sl >> 3, c = (sl & 7) ^ ((rl >> 1) & 7), row = h * 128 + rl;
            voff[h * 4 + j] = row < valid ? (uint32_t)((row * ld + c * 8) * 2) : kOobOffset;
        }
}

// fragment of k-tile `par` (0/1) of 64 k: rows `row` + (lane&31) of half `hi`, k = par*32 + kk*16 + 8*(lane>>5) ..+7;
// off0, off1: stages of the halves
__device__ __forceinline__ bf16x8 read_frag_wide(const char* ring, uint32_t off0, uint32_t off1, int hi, int par, int row, int kk, int lane) {
    const int rl = row + (lane & 31), c = (par * 4 + kk * 2 + (lane >> 5)) ^ ((rl >> 1) & 7);
    const uint32_t at = off1 > off0 ? off0 + (uint32_t)hi * kOperandStageBytes : hi ? off1 : off0;
    return *reinterpret_cast<const bf16x8*>(ring + at + rl * 128 + c * 16);
}

struct Frags {
    bf16x8 a[4], b[4];
};

template <typename F> __device__ __forceinline__ void static_for4(F&& f) {
    f(IntC<0>{});
    f(IntC<1>{});
    f(IntC<2>{});
    f(IntC<3>{});
}

template <bool AK, bool BKM, bool kSplit = false>
__global__ __launch_bounds__(256) void k_gemm_mfma(MfmaGemmParams p) {
    __shared__ __attribute__((aligned(1024))) char smem[2 * kStages * kOperandStageBytes];  // ring of A, ring of B
    const uint32_t lds0 = (uint32_t)(uintptr_t)ALCH_LDS(smem);
    constexpr int kU = 2 * kStages;  // steps after which the rings are back at their first stage, at an even step
    constexpr uint32_t kRing = kStages * kOperandStageBytes;
    auto stage_off = [](int b) -> uint32_t { return (uint32_t)(b % kStages) * kOperandStageBytes; };

    // ---- work-group -> output tile: XCD-contiguous chunks, banded raster inside a chunk
    // The grid is persistent (one work-group per compute unit): each work-group walks its share of
    // the tiles, so the stores of one tile drain while the next tile's loads are already in flight.
    const int Mv = p.m_dev ? min(__builtin_amdgcn_readfirstlane(*p.m_dev), p.M) : p.M;
    if (!kSplit && p.either) {
        PairPlan plan;
        if (device_plan(p, Mv, plan) != kRowsBig) return;
    }
    const int tiles_m = p.m_dev ? (Mv + BM - 1) / BM : p.tiles_m;
    const int nt = tiles_m * p.tiles_n;
    const int per_xcd = (nt + 7) / 8;
    const int lane = threadIdx.x & 63;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int wm = wave >> 1, wn = wave & 1;
    const uint32_t lds_wave = __builtin_amdgcn_readfirstlane(lds0 + (uint32_t)wave * 4096u);
    // kSplit: one tile per work-group; work-group w of an XCD takes part w / rem of tile q_end + w % rem
    const int rem = per_xcd - p.q_end;
    const int ks = kSplit ? (int)(blockIdx.x / 8) / rem : 0;
    // (q_end comes from the host's tile count; with a device-resident row count the XCD's share may be shorter)
    for (int q = kSplit ? p.q_end + (int)(blockIdx.x / 8) % rem : (int)(blockIdx.x / 8); q < (kSplit ? per_xcd : min(p.q_end, per_xcd));
         q += kSplit ? per_xcd : (int)(gridDim.x / 8)) {
    const int t = (blockIdx.x % 8) * per_xcd + q;
    if (t >= nt) break;
    const int band_tiles = kGroupM * p.tiles_n;
    const int band = t / band_tiles, in_band = t % band_tiles;
    const int band_rows = min(kGroupM, tiles_m - band * kGroupM);
    const int tm = band * kGroupM + in_band % band_rows;
    const int tn = in_band / band_rows;
    const int m0 = tm * BM, n0 = tn * BN;

    f32x16 acc[4][4];
#pragma unroll
    for (int i = 0; i < 4; ++i)
#pragma unroll
        for (int j = 0; j < 4; ++j)
#pragma unroll
            for (int e = 0; e < 16; ++e) acc[i][j][e] = 0.f;

    // (seen anew for every tile: addresses formed from it are not kept, and spilled, across the tiles' ends)
    int flane = lane;
    asm volatile("" : "+v"(flane));
    int seg_kt0 = 0;  // kSplit: k-tiles of the operand pairs before this one
    for (int seg = 0; seg < p.n_seg; ++seg) {
        const long long lda = p.lda[seg], ldb = p.ldb[seg];
        const int K = p.k_dev ? min(__builtin_amdgcn_readfirstlane(*p.k_dev), p.K[seg]) : p.K[seg];
        int nk = (K + BK - 1) / BK;
        const char *pa, *pb, *enda, *endb;
        long long stepa, stepb;
        if (AK) {
            pa = (const char*)(p.A[seg] + (long long)m0 * lda);
            enda = (const char*)(p.A[seg] + (long long)(Mv - 1) * lda + K);
            stepa = BK * 2;
        } else {
            pa = (const char*)(p.A[seg] + m0);
            enda = (const char*)(p.A[seg] + (long long)(K - 1) * lda + Mv);
            stepa = (long long)BK * lda * 2;
        }
        if (BKM) {
            const __bf16* B = p.B[p.by_cols ? range_of(p, n0) : seg];
            pb = (const char*)(B + (long long)n0 * ldb);
            endb = (const char*)(B + (long long)(p.N - 1) * ldb + K);
            stepb = BK * 2;
        } else {
            pb = (const char*)(p.B[seg] + n0);
            endb = (const char*)(p.B[seg] + (long long)(K - 1) * ldb + p.N);
            stepb = (long long)BK * ldb * 2;
        }
        if (kSplit) {  // this work-group's share [ks*per, (ks+1)*per) of the k-tiles of all pairs, cut to this pair
            const int lo = min(max(ks * p.split_per - seg_kt0, 0), nk), hi = min(max((ks + 1) * p.split_per - seg_kt0, 0), nk);
            seg_kt0 += nk;
            if (hi <= lo) continue;
            nk = hi - lo;
            pa += (long long)lo * stepa;
            pb += (long long)lo * stepb;
        }
        uint32_t va[AK ? 8 : 4], vb[BKM ? 8 : 4];
        if constexpr (AK) tile_offsets_wide(va, wave, flane, lda, Mv - m0);
        else tile_offsets<false>(va, wave, flane, lda, Mv - m0);
        if constexpr (BKM) tile_offsets_wide(vb, wave, flane, ldb, p.N - n0);
        else tile_offsets<false>(vb, wave, flane, ldb, p.N - n0);

        // Loads of the next k-tile go out one instruction at a time between MFMAs (a burst of
        // eight would hold the wave at the issue stage while the texture path drains).  Past the
        // last tile the same loads are issued against an empty buffer (they fetch nothing and
        // write zeros nobody reads), so the outstanding-load count is the same in every iteration.
        // The stream state (tile base address, bytes left in the operand) is kept in scalar registers
        // and advanced with scalar instructions, off the vector pipeline that feeds the MFMAs.
        uint32_t a_lo, a_hi, b_lo, b_hi;
        int a_rem, b_rem;
        {
            const uint64_t ua = (uint64_t)pa, ub = (uint64_t)pb;
            const long long la = enda - pa, lb = endb - pb;
            a_lo = __builtin_amdgcn_readfirstlane((uint32_t)ua);
            a_hi = __builtin_amdgcn_readfirstlane((uint32_t)(ua >> 32) & 0xffffu);
            a_rem = __builtin_amdgcn_readfirstlane((int)(la < 0 ? 0 : (la > 0x7fffffffLL ? 0x7fffffffLL : la)));
            b_lo = __builtin_amdgcn_readfirstlane((uint32_t)ub);
            b_hi = __builtin_amdgcn_readfirstlane((uint32_t)(ub >> 32) & 0xffffu);
            b_rem = __builtin_amdgcn_readfirstlane((int)(lb < 0 ? 0 : (lb > 0x7fffffffLL ? 0x7fffffffLL : lb)));
        }
        const int sa_step = __builtin_amdgcn_readfirstlane((int)stepa);
        const int sb_step = __builtin_amdgcn_readfirstlane((int)stepb);
        i32x4 ra, rb;
        // The loads of a step read through the descriptors ra, rb; an exhausted stream gets an empty buffer.  The stream of a
        // k-major operand moves by 128 bytes (64 k) after every second batch (the increment alternates 0, 128).
        int a_left = nk, a_inc = AK ? 0 : sa_step, b_left = nk, b_inc = BKM ? 0 : sb_step;
        auto select = [](i32x4& r, uint32_t lo, uint32_t hi, int bytes, int left) {
            int n;
            asm volatile("s_cmp_gt_i32 %1, 0\n\ts_cselect_b32 %0, %2, 0" : "=&s"(n) : "s"(left), "s"(bytes) : "scc");
            r[0] = (int)lo; r[1] = (int)hi; r[2] = n; r[3] = 0x00020000;
        };
        auto advance = [](uint32_t& lo, uint32_t& hi, int& bytes, int& left, int step) {
            asm volatile("s_add_u32 %0, %0, %4\n\ts_addc_u32 %1, %1, 0\n\ts_sub_i32 %2, %2, %4\n\ts_max_i32 %2, %2, 0\n\t"
                         "s_sub_i32 %3, %3, 1"
                         : "+s"(lo), "+s"(hi), "+s"(bytes), "+s"(left)
                         : "s"(step)
                         : "scc");
        };
        // in four pieces, each short enough to hide behind a matrix product
        auto open_step = [&](auto piece) {
            constexpr int q = decltype(piece)::value;
            if constexpr (q == 0) select(ra, a_lo, a_hi, a_rem, a_left);
            if constexpr (q == 1) {
                advance(a_lo, a_hi, a_rem, a_left, a_inc);
                if constexpr (AK) asm volatile("s_sub_i32 %0, 128, %0" : "+s"(a_inc) : : "scc");
            }
            if constexpr (q == 2) select(rb, b_lo, b_hi, b_rem, b_left);
            if constexpr (q == 3) {
                advance(b_lo, b_hi, b_rem, b_left, b_inc);
                if constexpr (BKM) asm volatile("s_sub_i32 %0, 128, %0" : "+s"(b_inc) : : "scc");
            }
        };
        auto open_a = [&]() { open_step(IntC<0>{}); open_step(IntC<1>{}); };
        auto open_b = [&]() { open_step(IntC<2>{}); open_step(IntC<3>{}); };
        // loads of batch `b`
#define ALCH_DMA_A(b, j) dma16(ra, lds_wave, stage_off(b) + (uint32_t)(j) * 1024u, va[(AK ? ((b) & 1) * 4 : 0) + (j)])
#define ALCH_DMA_B(b, j) dma16(rb, lds_wave, kRing + stage_off(b) + (uint32_t)(j) * 1024u, vb[(BKM ? ((b) & 1) * 4 : 0) + (j)])
#define ALCH_MFMA(F, i, j) acc[i][j] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(F.b[j], F.a[i], acc[i][j], 0, 0, 0)
#define ALCH_SB() __builtin_amdgcn_sched_barrier(0)
        // fragment reads of k-tile `st`
        auto frag_a = [&](int st, int kk, int i) -> bf16x8 {
            if constexpr (AK) return read_frag_wide(smem, stage_off(st / 2 * 2), stage_off(st / 2 * 2 + 1), wm, st & 1, i * 32, kk, flane);
            else return read_frag<false>(smem + stage_off(st), wm * 128 + i * 32, kk, flane);
        };
        auto frag_b = [&](int st, int kk, int i) -> bf16x8 {
            const char* ring = smem + kRing;
            if constexpr (BKM) return read_frag_wide(ring, stage_off(st / 2 * 2), stage_off(st / 2 * 2 + 1), wn, st & 1, i * 32, kk, flane);
            else return read_frag<false>(ring + stage_off(st), wn * 128 + i * 32, kk, flane);
        };
#define ALCH_RA(F, st, kk, i) F.a[i] = frag_a(st, kk, i)
#define ALCH_RB(F, st, kk, i) F.b[i] = frag_b(st, kk, i)

        // all waves are done with the previous segment's stages before they are refilled
        __syncthreads();
        // batches 0..3 of both; k-tile 0 needs the first two, the 16 loads behind them may still be in flight
#pragma unroll
        for (int b = 0; b < 4; ++b) {
            open_a();
            open_b();
#pragma unroll
            for (int j = 0; j < 4; ++j) { ALCH_DMA_A(b, j); ALCH_DMA_B(b, j); }
        }
        asm volatile("s_waitcnt vmcnt(%0)" ::"n"(2 * kLoadsPerTile) : "memory");
        __syncthreads();
        Frags f0, f1;
#pragma unroll
        for (int i = 0; i < 4; ++i) { ALCH_RA(f0, 0, 0, i); ALCH_RB(f0, 0, 0, i); }
        // One wavefront to a SIMD: whatever stands between two matrix products and takes longer than one of them is time in
        // which the matrix cores idle (on operands of zeros, which the power cap lets run, a k-tile took 1262 cycles of 1024).
        // So a step ends in a branch out of the loop alone, in straight line with the next one, where the compiler knows
        // which fragments are on their way and waits for those that a product needs instead of for all; the descriptors
        // of the next loads are formed in pieces between products of the first half; and LDS addresses are constants added
        // to one base.  Before, with 22 scalar instructions behind the barrier and a wait for all fragments: step 8b 6400,
        // now 6245 us; layer backward over 2 x 3001 tokens 6687 -> 6486 us; layer forward of 5003 tokens 2066 -> 2015 us.
        for (int kt = 0;; kt += kU) {
#pragma unroll
            for (int s = 0; s < kU; ++s) {
                if ((!(AK || BKM) || s % 2 == 0) && kt + s >= nk) goto steps_done;  // (k-major operands: whole pairs of k-tiles)
                const int st = s, stn = (s + 1) % kU;
                // ---- first half: MFMAs on k 0..15 of this stage, fragment reads for k 16..31.  Their order goes to
                // and fro over the columns, so that two in a row always share a fragment: the power cap sets the
                // clock, and an operand that stays draws less (registers alone, random operands: both operands
                // new 1770, rows of four in one direction 1793, to and fro 1808 TFLOP/s; layer forward of 5003
                // tokens 2022 -> 2013 us, preference step 8371 -> 8346 us).
                ALCH_SB();
                ALCH_RA(f1, st, 1, 0); ALCH_RA(f1, st, 1, 1); ALCH_MFMA(f0, 0, 0); ALCH_MFMA(f0, 0, 1); ALCH_SB();
                ALCH_RA(f1, st, 1, 2); ALCH_RA(f1, st, 1, 3); ALCH_MFMA(f0, 0, 2); ALCH_MFMA(f0, 0, 3); ALCH_SB();
                ALCH_RB(f1, st, 1, 0); ALCH_RB(f1, st, 1, 1); ALCH_MFMA(f0, 1, 3); ALCH_MFMA(f0, 1, 2); ALCH_SB();
                ALCH_RB(f1, st, 1, 2); ALCH_RB(f1, st, 1, 3); ALCH_MFMA(f0, 1, 1); ALCH_MFMA(f0, 1, 0); ALCH_SB();
                ALCH_MFMA(f0, 2, 0); ALCH_SB(); open_step(IntC<0>{}); ALCH_SB();
                ALCH_MFMA(f0, 2, 1); ALCH_SB(); open_step(IntC<1>{}); ALCH_SB();
                ALCH_MFMA(f0, 2, 2); ALCH_SB(); open_step(IntC<2>{}); ALCH_SB();
                ALCH_MFMA(f0, 2, 3); ALCH_SB(); open_step(IntC<3>{}); ALCH_SB();
                ALCH_MFMA(f0, 3, 3); ALCH_MFMA(f0, 3, 2); ALCH_MFMA(f0, 3, 1); ALCH_MFMA(f0, 3, 0);
                ALCH_SB();
                // odd steps: the batches of k-tiles kt+s+1 and kt+s+2 have landed (this wave's share: what may still be in
                // flight is the batch that step s-1 issued), and this wave's reads of k-tiles kt+s-1 and kt+s are done
                if (s % 2) asm volatile("s_waitcnt vmcnt(%0) lgkmcnt(0)\n\ts_barrier" ::"n"(kLoadsPerTile) : "memory");
                // ---- second half: MFMAs on k 16..31, loads of batch s + 4, fragment reads of the next k-tile
                ALCH_SB();
                ALCH_DMA_A(s + 4, 0); ALCH_RA(f0, stn, 0, 0); ALCH_RA(f0, stn, 0, 1); ALCH_MFMA(f1, 0, 0); ALCH_MFMA(f1, 0, 1); ALCH_SB();
                ALCH_DMA_A(s + 4, 1); ALCH_RA(f0, stn, 0, 2); ALCH_RA(f0, stn, 0, 3); ALCH_MFMA(f1, 0, 2); ALCH_MFMA(f1, 0, 3); ALCH_SB();
                ALCH_DMA_A(s + 4, 2); ALCH_RB(f0, stn, 0, 0); ALCH_MFMA(f1, 1, 3); ALCH_MFMA(f1, 1, 2); ALCH_SB();
                ALCH_DMA_A(s + 4, 3); ALCH_RB(f0, stn, 0, 1); ALCH_MFMA(f1, 1, 1); ALCH_MFMA(f1, 1, 0); ALCH_SB();
                ALCH_DMA_B(s + 4, 0); ALCH_RB(f0, stn, 0, 2); ALCH_MFMA(f1, 2, 0); ALCH_MFMA(f1, 2, 1); ALCH_SB();
                ALCH_DMA_B(s + 4, 1); ALCH_RB(f0, stn, 0, 3); ALCH_MFMA(f1, 2, 2); ALCH_MFMA(f1, 2, 3); ALCH_SB();
                ALCH_DMA_B(s + 4, 2); ALCH_MFMA(f1, 3, 3); ALCH_MFMA(f1, 3, 2); ALCH_SB();
                ALCH_DMA_B(s + 4, 3); ALCH_MFMA(f1, 3, 1); ALCH_MFMA(f1, 3, 0); ALCH_SB();
            }
        }
    steps_done:
        asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
#undef ALCH_DMA_A
#undef ALCH_DMA_B
#undef ALCH_MFMA
#undef ALCH_SB
#undef ALCH_RA
#undef ALCH_RB
    }

    if constexpr (kSplit) {
        // fp32 partial tile, row-major [256][256]: block (i, j) holds (see below) row i*32 + (lane&31) and, in
        // registers 4b..4b+3, columns j*32 + 8b + 4*(lane>>5) + 0..3 of the wave's 128x128 quarter
        float* ws = p.split_ws + ((size_t)(((blockIdx.x % 8) * rem + (q - p.q_end)) * p.split_s + ks)) * (BM * BN) +
                    (wm * 128 + (lane & 31)) * BN + wn * 128 + 4 * (lane >> 5);
        static_for4([&](auto ic) {
            constexpr int i = decltype(ic)::value;
#pragma unroll
            for (int j = 0; j < 4; ++j)
#pragma unroll
                for (int b = 0; b < 4; ++b) {
                    f32x4 v;
#pragma unroll
                    for (int r = 0; r < 4; ++r) v[r] = acc[i][j][4 * b + r];
                    *reinterpret_cast<f32x4*>(ws + i * 32 * BN + j * 32 + 8 * b) = v;
                }
        });
    } else {
    // ---- epilogue.  The MFMAs were issued with the operand roles swapped, so block (i, j) holds
    // the transposed 32x32 result: this lane owns output row m = .. + i*32 + (lane&31) and, in
    // registers 4b..4b+3, the four consecutive columns n = .. + j*32 + 8b + 4*(lane>>5) + 0..3.
    const bool cols = BKM && p.by_cols;
    const int oseg = range_of(p, cols ? n0 : m0);
    __bf16* __restrict__ C = p.C[oseg];
    const long long ldc = p.ldc[oseg];
    const int mrel0 = cols ? m0 : m0 - p.m_begin[oseg];
    const int m_end = (!cols && oseg + 1 < p.n_out ? min(p.m_begin[oseg + 1], Mv) : Mv);
    const int half = lane >> 5;

    if (!p.accumulate) {
        // Stage the wave's 128x128 bf16 result through the (now idle) pipeline LDS so that it leaves
        // as whole 256-byte row segments: 8-byte LDS writes, 16-byte LDS reads, 16-byte global stores.
        constexpr int kRowStride = 256;  // chunks XOR-ed with the row: 8-byte writes 2-way, 16-byte reads conflict-free
        char* stage = smem + wave * (128 * kRowStride);
        __syncthreads();  // every wave's loads have landed and every wave is done reading the pipeline
        static_for4([&](auto ic) {
            constexpr int i = decltype(ic)::value;
            char* row = stage + (i * 32 + (lane & 31)) * kRowStride;
#pragma unroll
            for (int j = 0; j < 4; ++j)
#pragma unroll
                for (int b = 0; b < 4; ++b) {
                    bf16x4 o;
#pragma unroll
                    for (int r = 0; r < 4; ++r) o[r] = (__bf16)acc[i][j][4 * b + r];
                    *reinterpret_cast<bf16x4*>(row + ((((4 * j + b) ^ (lane & 15)) << 4) | (half << 3))) = o;
                }
        });
        // (a wave reads back only what it wrote itself: no barrier needed in between)
        const int n = n0 + wn * 128 + (lane & 15) * 8;
        if (p.epilogue == kEpiSwigluBwd) {
            // G and U rows (read once, never again: non-temporal loads keep them out of the way of the operand
            // panels in L2) are fetched eight row-steps at a time before any store is issued: the
            // compiler may not move a load above a store it cannot prove disjoint, and one round trip
            // to memory per row-step would leave the epilogue bound by latency.
            constexpr int kBatch = 8;
#pragma unroll 1
            for (int q0 = 0; q0 < 32; q0 += kBatch) {
                bf16x8 g8[kBatch], u8[kBatch];
#pragma unroll
                for (int k = 0; k < kBatch; ++k) {
                    const int m = m0 + wm * 128 + 4 * (q0 + k) + (lane >> 4);
                    if (m < Mv && n < p.N) {
                        g8[k] = __builtin_nontemporal_load(reinterpret_cast<const bf16x8*>(p.G + (long long)m * p.ldgu + n));
                        u8[k] = __builtin_nontemporal_load(reinterpret_cast<const bf16x8*>(p.U + (long long)m * p.ldgu + n));
                    }
                }
#pragma unroll
                for (int k = 0; k < kBatch; ++k) {
                    const int rl = 4 * (q0 + k) + (lane >> 4);
                    const int m = m0 + wm * 128 + rl;
                    const bf16x8 d8 = *reinterpret_cast<const bf16x8*>(stage + rl * kRowStride + (((lane & 15) ^ (rl & 15)) << 4));
                    if (m < Mv && n < p.N) {
                        bf16x8 dg8, du8, a8;
                        swiglu_gradient<8>(d8, g8[k], u8[k], dg8, du8, a8);
                        *reinterpret_cast<bf16x8*>(C + (long long)m * ldc + n) = dg8;
                        *reinterpret_cast<bf16x8*>(C + (long long)m * ldc + p.N + n) = du8;
                        if (p.act_out) *reinterpret_cast<bf16x8*>(p.act_out + (long long)m * p.N + n) = a8;
                    }
                }
            }
        } else {
#pragma unroll 8
            for (int qq = 0; qq < 32; ++qq) {
                const int rl = 4 * qq + (lane >> 4);
                const int ml = wm * 128 + rl;
                const bf16x8 d8 = *reinterpret_cast<const bf16x8*>(stage + rl * kRowStride + (((lane & 15) ^ (rl & 15)) << 4));
                if (m0 + ml < m_end && n < p.N) *reinterpret_cast<bf16x8*>(C + (long long)(mrel0 + ml) * ldc + n) = d8;
            }
        }
    } else {
        // accumulate: C = round(acc + C) with the sum in fp32, straight from the accumulators.  The old
        // values of a 32-row block are all fetched before its first store (see the note on loads above).
        static_for4([&](auto ic) {
            constexpr int i = decltype(ic)::value;
            const int ml = wm * 128 + i * 32 + (lane & 31);
            __bf16* row = C + (long long)(mrel0 + ml) * ldc;
            const __bf16* old_row = BKM && p.residual ? p.residual + (long long)(m0 + ml) * ldc : row;
            const bool row_ok = m0 + ml < m_end;
            bf16x4 old[4][4];
#pragma unroll
            for (int j = 0; j < 4; ++j)
#pragma unroll
                for (int b = 0; b < 4; ++b) {
                    const int nn = n0 + wn * 128 + j * 32 + 8 * b + 4 * half;
                    if (row_ok && nn < p.N) old[j][b] = *reinterpret_cast<const bf16x4*>(old_row + nn);
                }
#pragma unroll
            for (int j = 0; j < 4; ++j)
#pragma unroll
                for (int b = 0; b < 4; ++b) {
                    const int nn = n0 + wn * 128 + j * 32 + 8 * b + 4 * half;
                    if (row_ok && nn < p.N) {
                        bf16x4 o;
#pragma unroll
                        for (int r = 0; r < 4; ++r) o[r] = (__bf16)(acc[i][j][4 * b + r] + bf2f(old[j][b][r]));
                        *reinterpret_cast<bf16x4*>(row + nn) = o;
                    }
                }
        });
    }
    }  // plain epilogue
    }  // tiles of this work-group
}

// Sum of the partial tiles of the split round -> output.  blockIdx.x: tile of that round (same tile numbering as
// the GEMM kernel), blockIdx.y: slab of 16 rows; a thread handles four consecutive columns of four rows.
__global__ __launch_bounds__(256) void k_gemm_split_finish(MfmaGemmParams p, int per_xcd, int nt) {
    const int rem = per_xcd - p.q_end;
    const int t = (blockIdx.x / rem) * per_xcd + p.q_end + blockIdx.x % rem;
    if (t >= nt) return;
    const int band_tiles = kGroupM * p.tiles_n;
    const int band = t / band_tiles, in_band = t % band_tiles;
    const int band_rows = min(kGroupM, p.tiles_m - band * kGroupM);
    const int m0 = (band * kGroupM + in_band % band_rows) * BM, n0 = (in_band / band_rows) * BN;
    const bool cols = p.by_cols;
    const int oseg = range_of(p, cols ? n0 : m0);
    __bf16* __restrict__ C = p.C[oseg];
    const long long ldc = p.ldc[oseg];
    const int mrel0 = cols ? m0 : m0 - p.m_begin[oseg];
    const int m_end = (!cols && oseg + 1 < p.n_out ? min(p.m_begin[oseg + 1], p.M) : p.M);
    const __bf16* old_rows = p.residual ? p.residual + (long long)m0 * ldc : C + (long long)mrel0 * ldc;
    const float* ws = p.split_ws + (size_t)blockIdx.x * p.split_s * (BM * BN);
    const int col = 4 * (threadIdx.x & 63), n = n0 + col;
    if (n >= p.N) return;  // (N is a multiple of 8: a thread's four columns are all inside or all outside)
    const int r0 = blockIdx.y * 16 + (threadIdx.x >> 6);
    if (p.epilogue == kEpiSwigluBwd) {
        // the summed product is dAct (rounded to bf16 as the fused epilogue of the unsplit kernel does); with the
        // saved G, U: dG = dAct U s'(G), dU = dAct silu(G), Act = silu(G) U
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            const int m = m0 + r0 + 4 * i;
            if (m >= p.M) continue;
            f32x4 v = {0.f, 0.f, 0.f, 0.f};
            for (int k = 0; k < p.split_s; ++k) v += *reinterpret_cast<const f32x4*>(ws + (size_t)k * (BM * BN) + (r0 + 4 * i) * BN + col);
            const bf16x4 g4 = *reinterpret_cast<const bf16x4*>(p.G + (long long)m * p.ldgu + n);
            const bf16x4 u4 = *reinterpret_cast<const bf16x4*>(p.U + (long long)m * p.ldgu + n);
            bf16x4 d4, dg4, du4, a4;
#pragma unroll
            for (int e = 0; e < 4; ++e) d4[e] = (__bf16)v[e];
            swiglu_gradient<4>(d4, g4, u4, dg4, du4, a4);
            *reinterpret_cast<bf16x4*>(C + (long long)m * ldc + n) = dg4;
            *reinterpret_cast<bf16x4*>(C + (long long)m * ldc + p.N + n) = du4;
            if (p.act_out) *reinterpret_cast<bf16x4*>(p.act_out + (long long)m * p.N + n) = a4;
        }
        return;
    }
    f32x4 v[4];
    bf16x4 old[4];
#pragma unroll
    for (int i = 0; i < 4; ++i) {  // all loads first
        const int r = r0 + 4 * i;
        v[i] = f32x4{0.f, 0.f, 0.f, 0.f};
        if (m0 + r < m_end) {
            for (int k = 0; k < p.split_s; ++k) v[i] += *reinterpret_cast<const f32x4*>(ws + (size_t)k * (BM * BN) + r * BN + col);
            if (p.accumulate) old[i] = *reinterpret_cast<const bf16x4*>(old_rows + (long long)r * ldc + n);
        }
    }
#pragma unroll
    for (int i = 0; i < 4; ++i) {
        const int r = r0 + 4 * i;
        if (m0 + r < m_end) {
            bf16x4 o;
#pragma unroll
            for (int e = 0; e < 4; ++e) o[e] = (__bf16)(p.accumulate ? v[i][e] + bf2f(old[i][e]) : v[i][e]);
            *reinterpret_cast<bf16x4*>(C + (long long)(mrel0 + r) * ldc + n) = o;
        }
    }
}

bool gemm_mfma_supported(const GemmDesc& d) {
    if (d.dtype != ALCH_BF16 || d.M <= 0 || d.N <= 0 || d.n_seg < 1 || d.n_seg > kMaxGemmSegs || d.n_out < 1 || d.n_out > 3)
        return false;
    for (int s = 0; s < d.n_seg; ++s) {
        const GemmSeg& g = d.seg[s];
        if (g.K <= 0 || !aligned16(g.A) || !aligned16(g.B) || g.lda % 8 || g.ldb % 8) return false;
        if ((d.a_kmajor || d.b_kmajor) && (g.K % 64 || d.k_dev)) return false;  // no k tail on k-major operands
        if (!d.a_kmajor && d.M % 8) return false;
        if (!d.b_kmajor && d.N % 8) return false;
        if (d.N % 8) return false;  // 16-byte output stores
        if (g.lda > (1 << 21) || g.ldb > (1 << 21)) return false;  // tile extent must stay below 2 GiB
        // the kernel tracks the bytes left in an operand in a signed 32-bit scalar
        const long long a_rows = d.a_kmajor ? d.M : g.K, b_rows = d.b_kmajor ? d.N : g.K;
        if (a_rows * g.lda * 2 >= (1LL << 31) || b_rows * g.ldb * 2 >= (1LL << 31)) return false;
    }
    for (int o = 0; o < d.n_out; ++o) {
        if (d.out[o].ldc % 8 || !aligned16(d.out[o].C)) return false;
        if (d.out[o].m_begin % BM) return false;  // (a tile is as wide as it is high)
        if (d.by_cols && (!aligned16(d.out[o].B) || !d.b_kmajor || d.n_seg != 1 || d.epilogue != kEpiNone)) return false;
        if (o == 0 && d.out[o].m_begin != 0) return false;
        if (o > 0 && d.out[o].m_begin <= d.out[o - 1].m_begin) return false;
    }
    if (d.residual && (!d.accumulate || !d.b_kmajor || d.n_out != 1 || !aligned16(d.residual))) return false;
    if (d.epilogue == kEpiSwigluBwd && (d.n_out != 1 || d.accumulate || d.ldgu % 8 || (d.act_out && !aligned16(d.act_out)) || !aligned16(d.G) || !aligned16(d.U))) return false;
    return true;
}

// How the 256x256 kernel walks a product: tiles q < q_end of every XCD's share whole, the rest in `parts` parts of
// `per` k-tiles each.
struct BigPlan { int q_end, parts, per; };
static BigPlan big_plan(const MfmaGemmParams& p, bool kmajor, int n_cu, size_t ws_bytes) {
    const int per_xcd = ceil_div(ceil_div(p.M, BM) * ceil_div(p.N, BN), 8), wgx = n_cu / 8;
    const int full_q = per_xcd / wgx * wgx, rem = per_xcd - full_q;
    BigPlan b{per_xcd, 1, 0};
    int nk_total = 0;
    for (int s = 0; s < p.n_seg; ++s) nk_total += ceil_div(p.K[s], BK);
    // Split of the last round (see the header): host-known sizes and a contraction long enough that every part
    // still runs the pipeline for a while (the finish kernel carries the SwiGLU-gradient epilogue if there is one).  A
    // product with tiles for at most half of the compute units (a short batch) has no other round: every tile is split.
    if (ws_bytes > 0 && !p.m_dev && !p.k_dev && rem > 0 && 2 * rem <= wgx) {
        int s = wgx / rem < 16 ? wgx / rem : 16;
        if (s > nk_total / 16) s = nk_total / 16;
        if (s > 1 && (size_t)8 * rem * s * BM * BN * sizeof(float) <= ws_bytes) {
            b.q_end = full_q;
            b.parts = s;
            b.per = ceil_div(nk_total, s);
            if (kmajor) b.per += b.per & 1;  // parts are whole 64 k, which the loop takes k-major operands in
        }
    }
    return b;
}

// Column ranges run as one product, unless their bits are to stay and a product of one of them, or of all, is cut along
// the contraction: what is cut depends on the number of tiles.
bool gemm_cols_together(const GemmDesc& d) {
    if (!d.keep_parts) return true;
    int n_cu = 0;
    if (compute_units(&n_cu) != ALCH_OK) return false;
    MfmaGemmParams p{};
    p.M = d.M;
    p.n_seg = 1;
    p.K[0] = d.seg[0].K;
    p.m_dev = d.m_dev;
    const size_t ws_bytes = aligned16(d.split_ws) && d.split_ws ? d.split_ws_bytes : 0;
    for (int s = -1; s < d.n_out; ++s) {
        p.N = s < 0 ? d.N : (s + 1 < d.n_out ? d.out[s + 1].m_begin : d.N) - d.out[s].m_begin;
        if (big_plan(p, d.a_kmajor || d.b_kmajor, n_cu, ws_bytes).parts > 1) return false;
    }
    return true;
}

int compute_units(int* n_cu) {
    static constexpr int kDevices = 64;
    static std::atomic<int> known[kDevices] = {};  // by device: those of a process need not be alike (partitions)
    int dev = 0;
    ALCH_HIP_TRY(hipGetDevice(&dev));
    const bool kept = dev >= 0 && dev < kDevices;
    int n = kept ? known[dev].load(std::memory_order_relaxed) : 0;
    if (n == 0) {
        int v = 0;
        ALCH_HIP_TRY(hipDeviceGetAttribute(&v, hipDeviceAttributeMultiprocessorCount, dev));
        n = v > 8 ? v / 8 * 8 : 8;
        if (kept) known[dev].store(n, std::memory_order_relaxed);
    }
    *n_cu = n;
    return ALCH_OK;
}

// A product as either kernel would run it, and which of them does.
struct MfmaProduct {
    MfmaGemmParams p;
    int n_cu, pair_tiles_m;
    size_t ws_bytes;
    float* split_ws;
    BigPlan big;
    PairPlan pair;
    bool as_pair;
};
static int plan_product(const GemmDesc& d, MfmaProduct& out) {
    MfmaGemmParams& p = out.p;
    p.M = d.M;
    p.N = d.N;
    p.n_seg = d.n_seg;
    p.n_out = d.n_out;
    p.accumulate = d.accumulate;
    p.m_dev = d.m_dev;
    p.k_dev = d.k_dev;
    p.tiles_m = ceil_div(d.M, BM);
    p.tiles_n = ceil_div(d.N, BN);
    for (int s = 0; s < kMaxGemmSegs; ++s) {
        const bool on = s < d.n_seg;
        p.A[s] = on ? static_cast<const __bf16*>(d.seg[s].A) : nullptr;
        p.B[s] = on ? static_cast<const __bf16*>(d.seg[s].B) : nullptr;
        p.K[s] = on ? d.seg[s].K : 0;
        p.lda[s] = on ? d.seg[s].lda : 0;
        p.ldb[s] = on ? d.seg[s].ldb : 0;
    }
    for (int s = 0; s < kMaxGemmOuts; ++s) {
        const bool oo = s < d.n_out;
        p.C[s] = oo ? static_cast<__bf16*>(d.out[s].C) : nullptr;
        p.m_begin[s] = oo ? d.out[s].m_begin : 0x7fffffff;
        p.ldc[s] = oo ? d.out[s].ldc : 0;
    }
    p.by_cols = d.by_cols;
    p.residual = static_cast<const __bf16*>(d.residual);
    if (d.by_cols)  // (as numbers: what is indexed lies in the range)
        for (int s = 0; s < d.n_out; ++s) {
            p.B[s] = reinterpret_cast<const __bf16*>(reinterpret_cast<uintptr_t>(d.out[s].B) -
                                                     (uintptr_t)d.out[s].m_begin * (uintptr_t)d.seg[0].ldb * 2);
            p.C[s] = reinterpret_cast<__bf16*>(reinterpret_cast<uintptr_t>(d.out[s].C) - (uintptr_t)d.out[s].m_begin * 2);
        }
    p.epilogue = d.epilogue;
    p.G = static_cast<const __bf16*>(d.G);
    p.U = static_cast<const __bf16*>(d.U);
    p.ldgu = d.ldgu;
    p.act_out = static_cast<__bf16*>(d.act_out);
    const int nt = p.tiles_m * p.tiles_n;
    ALCH_TRY(compute_units(&out.n_cu));
    out.split_ws = aligned16(d.split_ws) ? static_cast<float*>(d.split_ws) : nullptr;
    const size_t ws_bytes = out.ws_bytes = out.split_ws ? d.split_ws_bytes : 0;
    out.big = big_plan(p, d.a_kmajor || d.b_kmajor, out.n_cu, ws_bytes);
    int nk_total = 0;
    long long K = 0;
    for (int s = 0; s < p.n_seg; ++s) {
        nk_total += ceil_div(p.K[s], BK);
        K += p.K[s];
    }
    p.either = 0;
    p.plan_cu = out.n_cu;
    p.a_kmajor = d.a_kmajor;
    p.b_kmajor = d.b_kmajor;
    p.plan_ws = d.keep_parts ? 0 : (long long)ws_bytes;
    p.narrow = d.keep_parts && d.m_dev && d.a_kmajor && !d.b_kmajor && !d.accumulate && d.n_out == 1;
    const bool swiglu = p.epilogue == kEpiSwigluBwd;
    // m_dev: launch_device_rows.  k_dev: whole tiles, of the kernel that is the faster one with half of the tokens kept (its
    // tiles are the same for any count, and the lengths where the choice turns lie close together)
    if (p.m_dev || p.k_dev) {
        out.pair = pair_plan(p.M, p.N, nk_total, d.a_kmajor, out.n_cu, 0);
        out.pair_tiles_m = ceil_div(p.M, BM / 2);
        out.as_pair = !p.m_dev && !d.a_kmajor && !d.b_kmajor && pair_is_better(p.M, p.N, K / 2, d.a_kmajor, d.b_kmajor, swiglu, out.n_cu, 1, out.pair);
        return ALCH_OK;
    }
    // (a 256x256 tile is two tiles of the other kernel, numbered in the same order)
    out.pair = d.keep_parts ? PairPlan{2 * ceil_div(nt, 8), 2 * out.big.q_end, out.big.parts, out.big.per}
                            : pair_plan(p.M, p.N, nk_total, d.a_kmajor, out.n_cu, (long long)ws_bytes);
    out.pair_tiles_m = d.keep_parts ? 2 * p.tiles_m : ceil_div(p.M, BM / 2);
    out.as_pair = pair_is_better(p.M, p.N, K, d.a_kmajor, d.b_kmajor, swiglu, out.n_cu, out.big.parts, out.pair);
    return ALCH_OK;
}

static void launch_big(const MfmaGemmParams& p, int grid, hipStream_t stream) {
    if (p.a_kmajor && p.b_kmajor) k_gemm_mfma<true, true><<<grid, 256, 0, stream>>>(p);
    else if (p.a_kmajor) k_gemm_mfma<true, false><<<grid, 256, 0, stream>>>(p);
    else if (!p.b_kmajor) k_gemm_mfma<false, false><<<grid, 256, 0, stream>>>(p);
    else k_gemm_mfma<false, true><<<grid, 256, 0, stream>>>(p);
}

// A product whose row count lies on the device (the rows that a loss mask keeps): every kernel that some count of rows up to M
// calls for is launched, and reads the count.  With 256x256 tiles alone, whole, a few hundred kept rows left most compute
// units without work and the others with all of a long contraction: the gradient of H2 of 175 kept rows (4096 columns, K 28672)
// was 474 us on 16 busy compute units.  Layers of 4096/14336 with a quarter of the rows kept: 700 tokens 1022 -> 509 us, 1500 tokens
// 1210 -> 748, 5003 tokens and a tenth of them 1825 -> 1292; where the 256x256 tiles stay (hidden 8192, 8192 tokens) 8854 and 8889: the
// launches that leave are 28 us of a profile.  (In stacks of several layers the narrow tiles are a third one, 5 us for each of four products where
// the rows are too many for them: two layers, 0.6 of 4000 tokens 7461 -> 7488 us, 0.25 of 8000 9782 -> 9797.)
static int launch_device_rows(MfmaProduct& m, hipStream_t stream) {
    MfmaGemmParams& p = m.p;
    int pair_most = 0, cut_most = 0, narrow_most = 0;
    bool any_big = false;
    const int step = p.narrow ? PM / 2 : PM;  // rows of the smallest tile: the plan is the same in between
    for (int rows = step; rows < p.M + step; rows += step) {
        PairPlan plan;
        const RowsKernel kernel = device_plan(p, std::min(rows, p.M), plan);
        if (kernel == kRowsNarrow64 || kernel == kRowsNarrow128) {
            narrow_most = std::max(narrow_most, narrow_grid(p, std::min(rows, p.M), kernel));
            continue;
        }
        if (kernel == kRowsBig || !p.a_kmajor) {
            any_big = true;
            continue;
        }
        pair_most = std::max(pair_most, pair_grid(plan));
        if (plan.parts > 1) cut_most = std::max(cut_most, plan.per_xcd - plan.q_end);
    }
    p.either = (int)any_big + (pair_most > 0) + (narrow_most > 0) > 1;
    if (any_big) {
        const int nt = p.tiles_m * p.tiles_n;
        p.q_end = ceil_div(nt, 8);
        p.split_ws = nullptr;
        p.split_s = 1;
        launch_big(p, std::min(ceil_div(nt, 8) * 8, m.n_cu), stream);
    }
    if (pair_most > 0) ALCH_TRY(launch_gemm_pair_rows(p, pair_most, cut_most, m.split_ws, stream));
    if (narrow_most > 0) ALCH_TRY(launch_gemm_narrow_rows(p, narrow_most, stream));
    ALCH_HIP_TRY(hipGetLastError());
    return ALCH_OK;
}

int launch_gemm_mfma(const GemmDesc& d, hipStream_t stream) {
    MfmaProduct m;
    ALCH_TRY(plan_product(d, m));
    if (d.m_dev) return launch_device_rows(m, stream);
    if (m.as_pair) return launch_gemm_pair(m.p, d.a_kmajor, d.b_kmajor, m.pair_tiles_m, m.pair, m.split_ws, stream);
    MfmaGemmParams& p = m.p;
    const BigPlan& plan = m.big;
    float* split_ws = m.split_ws;
    const int n_cu = m.n_cu, nt = p.tiles_m * p.tiles_n;
    const int grid = ceil_div(nt, 8) * 8 < n_cu ? ceil_div(nt, 8) * 8 : n_cu;
    const int per_xcd = ceil_div(nt, 8), rem = per_xcd - plan.q_end;
    p.q_end = plan.q_end;
    p.split_ws = plan.parts > 1 ? split_ws : nullptr;
    p.split_s = plan.parts;
    p.split_per = plan.per;
    const int grid_split = 8 * rem * p.split_s;
    if (p.q_end > 0) launch_big(p, grid, stream);
    if (p.split_s > 1) {
        if (d.a_kmajor && d.b_kmajor) k_gemm_mfma<true, true, true><<<grid_split, 256, 0, stream>>>(p);
        else if (d.a_kmajor) k_gemm_mfma<true, false, true><<<grid_split, 256, 0, stream>>>(p);
        else if (!d.b_kmajor) k_gemm_mfma<false, false, true><<<grid_split, 256, 0, stream>>>(p);
        else k_gemm_mfma<false, true, true><<<grid_split, 256, 0, stream>>>(p);
    }
    if (p.split_s > 1) k_gemm_split_finish<<<dim3(8 * rem, BM / 16), 256, 0, stream>>>(p, per_xcd, nt);
    ALCH_HIP_TRY(hipGetLastError());
    return ALCH_OK;
}

// Whether a data gradient and a weight gradient run as one launch: where the data gradient is at most one round of work-groups.
// One of two rounds, its last one cut, leaves nothing to fill, and the weight gradient behind it takes from the caches
// what the launch after both reads (hidden 5120, ffn 17920, 5003 tokens: layer 6346 us apart, 6463 together).
static bool plan_together(const GemmDesc& data, const GemmDesc& weight, MfmaProduct& a, MfmaProduct& b) {
    if (data.split_ws != weight.split_ws || !gemm_mfma_supported(data) || !gemm_mfma_supported(weight)) return false;
    if (!data.a_kmajor || data.b_kmajor || weight.a_kmajor || weight.b_kmajor) return false;
    if (plan_product(data, a) != ALCH_OK || plan_product(weight, b) != ALCH_OK) return false;
    return a.as_pair && b.as_pair && pair_grid(a.pair) <= 2 * a.n_cu &&
           pair_split_bytes(a.pair) + pair_split_bytes(b.pair) <= std::min(data.split_ws_bytes, weight.split_ws_bytes);
}
bool gemm_mfma_together(const GemmDesc& data, const GemmDesc& weight) {
    MfmaProduct a, b;
    return plan_together(data, weight, a, b);
}
int launch_gemm_mfma_together(const GemmDesc& data, const GemmDesc& weight, hipStream_t stream) {
    MfmaProduct a, b;
    if (!plan_together(data, weight, a, b)) return fail(ALCH_ERR_UNSUPPORTED, "products that do not run together");
    return launch_gemm_two_pairs(a.p, a.pair_tiles_m, a.pair, b.p, b.pair_tiles_m, b.pair, a.split_ws, stream);
}

}  // namespace alch
