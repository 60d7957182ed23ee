// bf16 GEMM on the gfx950 matrix cores, two work-groups per compute unit: the kernel for products whose tiles are short
// or few.  Same contract as k_gemm_mfma (gemm_mfma.hip).  A row count that only the
// device knows is planned there: every work-group, and the finish kernel, forms the same plan from it.
//
//   * 128x256 tile per work-group, 4 wavefronts of 64x128 each (128 accumulator registers), at most 256 registers and
//     80 KB of LDS, so that two work-groups share a compute unit: while one waits for its first loads, writes its tile or
//     meets its barrier, the other one keeps the matrix cores busy.  The persistent 256x256 kernel has nothing to put
//     there; its loop reads a third less from LDS and L2 per multiply-add, which is why it stays the better one for
//     products of many long tiles.
//   * HBM/L2 -> LDS by 16-byte direct-to-LDS buffer loads, three stages of 32 k; a k-major A is staged in two
//     super-stages of 64 k (whole 128-byte lines) beside three stages of B, exactly 80 KB.
//   * Tiles beyond q_end of an XCD's share are cut along the contraction: split_s work-groups leave fp32 partial tiles,
//     k_gemm_pair_finish adds them in a fixed order and writes the output (deterministic, no atomics).
#include "gemm_mfma_common.h"

namespace alch {

static constexpr int kPairGroupM = 8;  // tile rows per raster band

// Epilogue of 64 x 128 results in the accumulators of a wavefront: block (i, j) holds the transposed 32x32 result, this
// lane owns output row i*32 + (lane&31) and, in registers 4b..4b+3, columns j*32 + 8b + 4*(lane>>5) + 0..3.  The results
// pass through 16 KB of LDS of the wavefront's own so that they leave as 16-byte pieces of 256-byte row segments.
static constexpr int kSuper = 16384, kAStage = 8192, kBStage = 16384;
template <bool kWide> static constexpr int kPairLds = kWide ? 2 * kSuper + 3 * kBStage : 3 * (kAStage + kBStage);

// Plan and row count of a product; kRows: from the row count on the device (false: nothing to do).
template <bool kRows>
__device__ __forceinline__ bool the_plan(const MfmaGemmParams& p, PairPlan& plan, int& Mv, int& tiles_m) {
    plan = PairPlan{p.per_xcd, p.q_end, p.split_s, p.split_per};
    Mv = p.M;
    tiles_m = p.tiles_m;
    if constexpr (kRows) {
        Mv = min(__builtin_amdgcn_readfirstlane(*p.m_dev), p.M);
        const bool pair = device_plan(p, Mv, plan) == kRowsPair;
        tiles_m = up_div(Mv, PM);
        return Mv > 0 && (!p.either || pair);
    }
    return true;
}

// Work-group `block` of the product's grid.
template <bool AK, bool BKM, bool kRows = false>
__device__ __forceinline__ void pair_tile(const MfmaGemmParams& p, int block, char* smem) {
    constexpr bool kWide = AK;
    constexpr int kU = kWide ? 12 : 3;  // steps after which every ring is back at its first stage
    const uint32_t lds0 = (uint32_t)(uintptr_t)ALCH_LDS(smem);
    auto a_off = [](int st) -> uint32_t { return kWide ? (uint32_t)((st / 2) % 2) * kSuper : (uint32_t)(st % 3) * (kAStage + kBStage); };
    auto b_off = [](int st) -> uint32_t {
        return kWide ? 2 * kSuper + (uint32_t)(st % 3) * kBStage : (uint32_t)(st % 3) * (kAStage + kBStage) + kAStage;
    };
    const int lane = threadIdx.x & 63;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int wm = wave >> 1, wn = wave & 1;
    const uint32_t lds_a = __builtin_amdgcn_readfirstlane(lds0 + (uint32_t)wave * 2048u);
    const uint32_t lds_b = __builtin_amdgcn_readfirstlane(lds0 + (uint32_t)wave * 4096u);

    // ---- work-group -> tile (and part of its contraction): every XCD owns per_xcd consecutive tiles
    PairPlan plan;
    int Mv, tiles_m;
    if (!the_plan<kRows>(p, plan, Mv, tiles_m)) return;
    const int nt = tiles_m * p.tiles_n, per_xcd = plan.per_xcd;
    const int in_xcd = block / 8;
    const bool whole = in_xcd < plan.q_end;
    const int rem = per_xcd - plan.q_end;
    if (kRows && !whole && (rem == 0 || in_xcd >= plan.q_end + rem * plan.parts)) return;  // (grids for any number of rows)
    const int q = whole ? in_xcd : plan.q_end + (in_xcd - plan.q_end) % rem;
    const int ks = whole ? 0 : (in_xcd - plan.q_end) / rem;
    const int t = (block % 8) * per_xcd + q;
    if (q >= per_xcd || t >= nt) return;
    const int band_tiles = kPairGroupM * p.tiles_n;
    const int band = t / band_tiles, in_band = t % band_tiles;
    const int band_rows = min(kPairGroupM, tiles_m - band * kPairGroupM);
    const int m0 = (band * kPairGroupM + in_band % band_rows) * PM, n0 = (in_band / band_rows) * PN;
    if (m0 >= Mv) return;

    f32x16 acc[2][4];
#pragma unroll
    for (int i = 0; i < 2; ++i)
#pragma unroll
        for (int j = 0; j < 4; ++j)
#pragma unroll
            for (int e = 0; e < 16; ++e) acc[i][j][e] = 0.f;

    int seg_kt0 = 0;  // k-tiles of the operand pairs before this one
    for (int seg = 0; seg < p.n_seg; ++seg) {
        const long long lda = p.lda[seg], ldb = p.ldb[seg];
        int K = p.K[seg];
        if constexpr (!AK && !BKM)  // (weight gradients)
            if (p.k_dev) K = min(__builtin_amdgcn_readfirstlane(*p.k_dev), K);
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
        if (!whole) {  // this work-group's share [ks*per, (ks+1)*per) of the k-tiles of all pairs, cut to this pair
            const int lo = min(max(ks * plan.per - seg_kt0, 0), nk), hi = min(max((ks + 1) * plan.per - seg_kt0, 0), nk);
            seg_kt0 += nk;
            if (hi <= lo) continue;
            nk = hi - lo;
            pa += (long long)lo * stepa;
            pb += (long long)lo * stepb;
        }
        // per-lane byte offsets of the loads of one step (LDS slots of 16 bytes are filled lane-linearly; which piece a
        // lane fetches carries the bank swizzle)
        uint32_t va[kWide ? 4 : 2], vb[4];
        if constexpr (kWide) {
#pragma unroll
            for (int j = 0; j < 4; ++j) {
                const int sl = (wave * 4 + j) * 64 + lane, row = sl >> 3, c = (sl & 7) ^ ((row >> 1) & 7);
                va[j] = row < Mv - m0 ? (uint32_t)((row * lda + c * 8) * 2) : kOobOffset;
            }
        } else {
#pragma unroll
            for (int j = 0; j < 2; ++j) {
                const int sl = (wave * 2 + j) * 64 + lane, k = sl >> 4, c = (sl & 15) ^ (4 * (k & 3));
                va[j] = c * 8 < Mv - m0 ? (uint32_t)((k * lda + c * 8) * 2) : kOobOffset;
            }
        }
        tile_offsets<BKM>(vb, wave, lane, ldb, p.N - n0);

        // Stream state in scalar registers: address and bytes left of either operand, tiles left.  Past the end the
        // loads go to an empty buffer, so the number in flight is the same in every step.
        const uint64_t ua = (uint64_t)pa, ub = (uint64_t)pb;
        const long long la = enda - pa, lb = endb - pb;
        uint32_t a_lo = __builtin_amdgcn_readfirstlane((uint32_t)ua), a_hi = __builtin_amdgcn_readfirstlane((uint32_t)(ua >> 32) & 0xffffu);
        uint32_t b_lo = __builtin_amdgcn_readfirstlane((uint32_t)ub), b_hi = __builtin_amdgcn_readfirstlane((uint32_t)(ub >> 32) & 0xffffu);
        int a_rem = __builtin_amdgcn_readfirstlane((int)(la < 0 ? 0 : (la > 0x7fffffffLL ? 0x7fffffffLL : la)));
        int b_rem = __builtin_amdgcn_readfirstlane((int)(lb < 0 ? 0 : (lb > 0x7fffffffLL ? 0x7fffffffLL : lb)));
        int a_left = kWide ? (nk + 1) / 2 : nk, b_left = nk;
        const int sa_step = __builtin_amdgcn_readfirstlane(kWide ? 128 : (int)stepa), sb_step = __builtin_amdgcn_readfirstlane((int)stepb);
        i32x4 ra, rb;
        auto select = [](i32x4& r, uint32_t lo, uint32_t hi, int left_bytes, int left) {
            int n;
            asm volatile("s_cmp_gt_i32 %1, 0\n\ts_cselect_b32 %0, %2, 0" : "=&s"(n) : "s"(left), "s"(left_bytes) : "scc");
            r[0] = (int)lo; r[1] = (int)hi; r[2] = n; r[3] = 0x00020000;
        };
        auto advance = [](uint32_t& lo, uint32_t& hi, int& left_bytes, int& left, int step) {
            asm volatile("s_add_u32 %0, %0, %4\n\ts_addc_u32 %1, %1, 0\n\ts_sub_i32 %2, %2, %4\n\ts_max_i32 %2, %2, 0\n\t"
                         "s_sub_i32 %3, %3, 1"
                         : "+s"(lo), "+s"(hi), "+s"(left_bytes), "+s"(left)
                         : "s"(step)
                         : "scc");
        };
        auto select_a = [&]() { select(ra, a_lo, a_hi, a_rem, a_left); };
        auto select_b = [&]() { select(rb, b_lo, b_hi, b_rem, b_left); };
        auto advance_a = [&]() { advance(a_lo, a_hi, a_rem, a_left, sa_step); };
        auto advance_b = [&]() { advance(b_lo, b_hi, b_rem, b_left, sb_step); };
        auto open_a = [&]() { select_a(); advance_a(); };
        auto open_b = [&]() { select_b(); advance_b(); };
        // the loads of tile `st` (A: of the super-stage that holds it)
        auto load_a = [&](int st, int j) { dma16(ra, kWide ? lds_b : lds_a, a_off(st) + (uint32_t)j * 1024u, va[j]); };
        auto load_b = [&](int st, int j) { dma16(rb, lds_b, b_off(st) + (uint32_t)j * 1024u, vb[j]); };
        auto frag_a = [&](int st, int kk, int i) -> bf16x8 {
            if constexpr (kWide) {
                const int row = wm * 64 + i * 32 + (lane & 31), c = ((st & 1) * 4 + kk * 2 + (lane >> 5)) ^ ((row >> 1) & 7);
                return *reinterpret_cast<const bf16x8*>(smem + a_off(st) + row * 128 + c * 16);
            } else {
                return read_frag<false, PM>(smem + a_off(st), wm * 64 + i * 32, kk, lane);
            }
        };
        auto frag_b = [&](int st, int kk, int j) -> bf16x8 { return read_frag<BKM>(smem + b_off(st), wn * 128 + j * 32, kk, lane); };
        struct Frags { bf16x8 a[2], b[4]; };
#define ALCH_SB() __builtin_amdgcn_sched_barrier(0)
#define ALCH_MM(F, i, j) acc[i][j] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(F.b[j], F.a[i], acc[i][j], 0, 0, 0)

        __syncthreads();  // every wave is done with the previous pair's stages
        if constexpr (kWide) {  // as steps -3, -2, -1 of the loop below issue them
            open_a(); open_b();
#pragma unroll
            for (int j = 0; j < 4; ++j) load_a(0, j);
#pragma unroll
            for (int j = 0; j < 4; ++j) load_b(0, j);
            open_b();
#pragma unroll
            for (int j = 0; j < 4; ++j) load_b(1, j);
            open_a(); open_b();
#pragma unroll
            for (int j = 0; j < 4; ++j) load_a(2, j);
#pragma unroll
            for (int j = 0; j < 4; ++j) load_b(2, j);
        } else {
#pragma unroll
            for (int s = 0; s < 3; ++s) {
                open_a(); open_b();
#pragma unroll
                for (int j = 0; j < 2; ++j) load_a(s, j);
#pragma unroll
                for (int j = 0; j < 4; ++j) load_b(s, j);
            }
        }
        asm volatile("s_waitcnt vmcnt(12)" ::: "memory");  // tile 0 has landed
        __syncthreads();
        Frags f0, f1;
#pragma unroll
        for (int i = 0; i < 2; ++i) f0.a[i] = frag_a(0, 0, i);
#pragma unroll
        for (int j = 0; j < 4; ++j) f0.b[j] = frag_b(0, 0, j);
        for (int kt = 0;; kt += kU) {
#pragma unroll
            for (int s = 0; s < kU; ++s) {
                if (kt + s >= nk) goto steps_done;
                const int sn = (s + 1) % kU;
                // k 0..15 of the tile; fragments of k 16..31 (two products in a row share a fragment, see gemm_mfma.hip)
                ALCH_SB();
                f1.a[0] = frag_a(s, 1, 0); f1.b[0] = frag_b(s, 1, 0); ALCH_MM(f0, 0, 0); ALCH_MM(f0, 0, 1); ALCH_SB();
                f1.b[1] = frag_b(s, 1, 1); f1.a[1] = frag_a(s, 1, 1); ALCH_MM(f0, 1, 1); ALCH_MM(f0, 1, 0); ALCH_SB();
                f1.b[2] = frag_b(s, 1, 2); f1.b[3] = frag_b(s, 1, 3); ALCH_MM(f0, 1, 2); ALCH_SB();
                if (!kWide || s % 2) select_a();
                ALCH_SB(); ALCH_MM(f0, 1, 3); ALCH_SB();
                if (!kWide || s % 2) advance_a();
                ALCH_SB(); ALCH_MM(f0, 0, 3); ALCH_SB();
                select_b();
                ALCH_SB(); ALCH_MM(f0, 0, 2); ALCH_SB();
                advance_b();
                // tile s+1 has landed (this wave's share: what may still be in flight is what step s-1 issued), and
                // this wave's reads of tile s are done
                asm volatile("s_waitcnt vmcnt(%0) lgkmcnt(0)\n\ts_barrier" ::"n"(kWide ? (s % 2 ? 4 : 8) : 6) : "memory");
                // k 16..31; loads of tile s+3 into the stage of tile s, fragments of tile s+1
                ALCH_SB();
                if (kWide && s % 2) { load_a(s + 3, 0); load_a(s + 3, 1); }
                if (!kWide) load_a(s, 0);
                f0.a[0] = frag_a(sn, 0, 0); f0.b[0] = frag_b(sn, 0, 0); ALCH_MM(f1, 0, 0); ALCH_MM(f1, 0, 1); ALCH_SB();
                if (kWide && s % 2) { load_a(s + 3, 2); load_a(s + 3, 3); }
                if (!kWide) load_a(s, 1);
                f0.b[1] = frag_b(sn, 0, 1); f0.a[1] = frag_a(sn, 0, 1); ALCH_MM(f1, 1, 1); ALCH_MM(f1, 1, 0); ALCH_SB();
                load_b(s, 0); load_b(s, 1);
                f0.b[2] = frag_b(sn, 0, 2); f0.b[3] = frag_b(sn, 0, 3); ALCH_MM(f1, 1, 2); ALCH_MM(f1, 1, 3); ALCH_SB();
                load_b(s, 2); load_b(s, 3);
                ALCH_MM(f1, 0, 3); ALCH_MM(f1, 0, 2); ALCH_SB();
            }
        }
    steps_done:
        asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
#undef ALCH_SB
#undef ALCH_MM
    }

    const int half = lane >> 5;
    if (!whole) {
        float* ws = p.split_ws + ((size_t)(((block % 8) * rem + (q - plan.q_end)) * plan.parts + ks)) * (PM * PN) +
                    (wm * 64 + (lane & 31)) * PN + wn * 128 + 4 * half;
#pragma unroll
        for (int i = 0; i < 2; ++i)
#pragma unroll
            for (int j = 0; j < 4; ++j)
#pragma unroll
                for (int b = 0; b < 4; ++b) {
                    f32x4 v;
#pragma unroll
                    for (int r = 0; r < 4; ++r) v[r] = acc[i][j][4 * b + r];
                    *reinterpret_cast<f32x4*>(ws + i * 32 * PN + j * 32 + 8 * b) = v;
                }
        return;
    }
    const bool cols = BKM && p.by_cols;
    const int oseg = range_of(p, cols ? n0 : m0);
    __bf16* __restrict__ C = p.C[oseg];
    const long long ldc = p.ldc[oseg];
    const int mrel0 = cols ? m0 : m0 - p.m_begin[oseg];
    const int m_end = (!cols && oseg + 1 < p.n_out ? min(p.m_begin[oseg + 1], Mv) : Mv);
    char* stage = smem + wave * 16384;
    const int n = n0 + wn * 128 + (lane & 15) * 8;
    __syncthreads();  // every wave's loads have landed and every wave is done reading the pipeline
    if (p.accumulate) {
        const __bf16* old_rows = BKM && p.residual ? p.residual + (long long)m0 * ldc : C + (long long)mrel0 * ldc;
        // C = round(acc + C), the sum in fp32: 32 rows at a time through LDS as fp32 [32][128], 16-byte pieces XOR-ed with
        // the row, all old values of a pass requested before its first store
#pragma unroll
        for (int i = 0; i < 2; ++i) {
            char* row = stage + (lane & 31) * 512;
#pragma unroll
            for (int j = 0; j < 4; ++j)
#pragma unroll
                for (int b = 0; b < 4; ++b) {
                    f32x4 v;
#pragma unroll
                    for (int r = 0; r < 4; ++r) v[r] = acc[i][j][4 * b + r];
                    *reinterpret_cast<f32x4*>(row + (((8 * j + 2 * b + half) ^ (lane & 15)) << 4)) = v;
                }
            bf16x8 old[8];
#pragma unroll
            for (int k = 0; k < 8; ++k) {
                const int ml = wm * 64 + i * 32 + 4 * k + (lane >> 4);
                if (m0 + ml < m_end && n < p.N) old[k] = *reinterpret_cast<const bf16x8*>(old_rows + (long long)ml * ldc + n);
            }
#pragma unroll
            for (int k = 0; k < 8; ++k) {
                const int rl = 4 * k + (lane >> 4), ml = wm * 64 + i * 32 + rl;
                const f32x4 lo = *reinterpret_cast<const f32x4*>(stage + rl * 512 + (((2 * (lane & 15)) ^ (rl & 15)) << 4));
                const f32x4 hi = *reinterpret_cast<const f32x4*>(stage + rl * 512 + (((2 * (lane & 15) + 1) ^ (rl & 15)) << 4));
                if (m0 + ml < m_end && n < p.N) {
                    bf16x8 o;
#pragma unroll
                    for (int e = 0; e < 8; ++e) o[e] = (__bf16)((e < 4 ? lo[e & 3] : hi[e & 3]) + bf2f(old[k][e]));
                    *reinterpret_cast<bf16x8*>(C + (long long)(mrel0 + ml) * ldc + n) = o;
                }
            }
        }
        return;
    }
    // bf16 [64][128] of the wavefront, 16-byte pieces XOR-ed with the row
#pragma unroll
    for (int i = 0; i < 2; ++i) {
        char* row = stage + (i * 32 + (lane & 31)) * 256;
#pragma unroll
        for (int j = 0; j < 4; ++j)
#pragma unroll
            for (int b = 0; b < 4; ++b) {
                bf16x4 o;
#pragma unroll
                for (int r = 0; r < 4; ++r) o[r] = (__bf16)acc[i][j][4 * b + r];
                *reinterpret_cast<bf16x4*>(row + ((((4 * j + b) ^ (lane & 15)) << 4) | (half << 3))) = o;
            }
    }
    if (p.epilogue == kEpiSwigluBwd) {
        constexpr int kBatch = 8;
#pragma unroll
        for (int q0 = 0; q0 < 16; q0 += kBatch) {
            bf16x8 g8[kBatch], u8[kBatch];
#pragma unroll
            for (int k = 0; k < kBatch; ++k) {
                const int m = m0 + wm * 64 + 4 * (q0 + k) + (lane >> 4);
                if (m < Mv && n < p.N) {
                    g8[k] = __builtin_nontemporal_load(reinterpret_cast<const bf16x8*>(p.G + (long long)m * p.ldgu + n));
                    u8[k] = __builtin_nontemporal_load(reinterpret_cast<const bf16x8*>(p.U + (long long)m * p.ldgu + n));
                }
            }
#pragma unroll
            for (int k = 0; k < kBatch; ++k) {
                const int rl = 4 * (q0 + k) + (lane >> 4);
                const int m = m0 + wm * 64 + rl;
                const bf16x8 d8 = *reinterpret_cast<const bf16x8*>(stage + rl * 256 + (((lane & 15) ^ (rl & 15)) << 4));
                if (m < Mv && n < p.N) {
                    bf16x8 dg8, du8, a8;
                    swiglu_gradient<8>(d8, g8[k], u8[k], dg8, du8, a8);
                    *reinterpret_cast<bf16x8*>(C + (long long)m * ldc + n) = dg8;
                    *reinterpret_cast<bf16x8*>(C + (long long)m * ldc + p.N + n) = du8;
                    if (p.act_out) *reinterpret_cast<bf16x8*>(p.act_out + (long long)m * p.N + n) = a8;
                }
            }
        }
        return;
    }
#pragma unroll 8
    for (int k = 0; k < 16; ++k) {
        const int rl = 4 * k + (lane >> 4), ml = wm * 64 + rl;
        const bf16x8 d8 = *reinterpret_cast<const bf16x8*>(stage + rl * 256 + (((lane & 15) ^ (rl & 15)) << 4));
        if (m0 + ml < m_end && n < p.N) *reinterpret_cast<bf16x8*>(C + (long long)(mrel0 + ml) * ldc + n) = d8;
    }
}

template <bool AK, bool BKM>
__global__ __launch_bounds__(256, 2) void k_gemm_pair(MfmaGemmParams p) {
    __shared__ __attribute__((aligned(1024))) char smem[kPairLds<AK>];
    pair_tile<AK, BKM>(p, (int)blockIdx.x, smem);
}

// With the row count on the device: kernels of their own, since a plan to be formed first, or looked at and left, is 0.4 us a
// launch (801 tokens of hidden 2048, 8 launches: 359 / 362 us).
template <bool BKM>
__global__ __launch_bounds__(256, 2) void k_gemm_pair_rows(MfmaGemmParams p) {
    __shared__ __attribute__((aligned(1024))) char smem[kPairLds<true>];
    pair_tile<true, BKM, true>(p, (int)blockIdx.x, smem);
}

// A data gradient and a weight gradient that does not depend on it, the one with the longer tiles in the first n_first
// work-groups.  Of a short batch the one has a work-group per compute unit, or fewer, that read cold weights, the other many
// short ones that write cold gradients: they fill each other's gaps, and neither waits for the other's last round.  Every tile
// and part of a tile is the one of a launch of its own: the same bits.  Layer backward, us, three launches of two products
// against six of one: heads of 64 100 tokens 183 / 200, 3001 894 / 925; 8B shape 100 tokens 343 / 370, 487 622 / 636, 2300
// 1933 / 1978.  Nine shapes at 11 to 20 sizes from 32 to 8192 tokens: 1 % slower at one (hidden 5120, 1800 tokens).
// Longer tiles first: hidden 256, ffn 14336, 5120 tokens, dO's 640 short tiles in front of 224 long ones 177 us, behind them
// 109, two launches 112.
__global__ __launch_bounds__(256, 2) void k_gemm_two_pairs(MfmaGemmParams data, MfmaGemmParams weight, int n_first, int weight_first) {
    __shared__ __attribute__((aligned(1024))) char smem[kPairLds<true>];
    const bool first = (int)blockIdx.x < n_first;
    const int block = first ? (int)blockIdx.x : (int)blockIdx.x - n_first;
    if (first != (weight_first != 0)) pair_tile<true, false>(data, block, smem);
    else pair_tile<false, false>(weight, block, smem);
}

// Sum of the partial tiles -> output.  blockIdx.x % 8: XCD of the tile, blockIdx.x / 8: split tile of its share,
// blockIdx.y: slab of 16 rows; a thread handles eight consecutive columns of two rows.
template <bool kRows>
__global__ __launch_bounds__(256) void k_gemm_pair_finish(MfmaGemmParams p) {
    PairPlan plan;
    int Mv, tiles_m;
    if (!the_plan<kRows>(p, plan, Mv, tiles_m)) return;
    const int per_xcd = plan.per_xcd, nt = tiles_m * p.tiles_n;
    const int rem = per_xcd - plan.q_end;
    const int xcd = blockIdx.x % 8, j = blockIdx.x / 8;
    const int t = xcd * per_xcd + plan.q_end + j;
    if (j >= rem || t >= nt) return;
    const int band_tiles = kPairGroupM * p.tiles_n;
    const int band = t / band_tiles, in_band = t % band_tiles;
    const int band_rows = min(kPairGroupM, tiles_m - band * kPairGroupM);
    const int m0 = (band * kPairGroupM + in_band % band_rows) * PM, n0 = (in_band / band_rows) * PN;
    const bool cols = p.by_cols;
    const int oseg = range_of(p, cols ? n0 : m0);
    __bf16* __restrict__ C = p.C[oseg];
    const long long ldc = p.ldc[oseg];
    const int mrel0 = cols ? m0 : m0 - p.m_begin[oseg];
    const int m_end = (!cols && oseg + 1 < p.n_out ? min(p.m_begin[oseg + 1], Mv) : Mv);
    const float* ws = p.split_ws + (size_t)(xcd * rem + j) * plan.parts * (PM * PN);
    const int col = 8 * (threadIdx.x & 31), n = n0 + col;
    if (n >= p.N) return;  // (N is a multiple of 8)
#pragma unroll
    for (int i = 0; i < 2; ++i) {
        const int r = blockIdx.y * 16 + i * 8 + (threadIdx.x >> 5), m = m0 + r;
        if (m >= m_end) continue;
        f32x4 lo = {0.f, 0.f, 0.f, 0.f}, hi = lo;
#pragma unroll 4
        for (int k = 0; k < plan.parts; ++k) {
            const float* w = ws + (size_t)k * (PM * PN) + r * PN + col;
            lo += *reinterpret_cast<const f32x4*>(w);
            hi += *reinterpret_cast<const f32x4*>(w + 4);
        }
        bf16x8 o;
        if (p.epilogue == kEpiSwigluBwd) {
            const bf16x8 g8 = *reinterpret_cast<const bf16x8*>(p.G + (long long)m * p.ldgu + n);
            const bf16x8 u8 = *reinterpret_cast<const bf16x8*>(p.U + (long long)m * p.ldgu + n);
#pragma unroll
            for (int e = 0; e < 8; ++e) o[e] = (__bf16)(e < 4 ? lo[e & 3] : hi[e & 3]);
            bf16x8 dg8, du8, a8;
            swiglu_gradient<8>(o, g8, u8, dg8, du8, a8);
            *reinterpret_cast<bf16x8*>(C + (long long)m * ldc + n) = dg8;
            *reinterpret_cast<bf16x8*>(C + (long long)m * ldc + p.N + n) = du8;
            if (p.act_out) *reinterpret_cast<bf16x8*>(p.act_out + (long long)m * p.N + n) = a8;
            continue;
        }
        __bf16* dst = C + (long long)(mrel0 + r) * ldc + n;
        bf16x8 old;
        if (p.accumulate) old = *reinterpret_cast<const bf16x8*>(p.residual ? p.residual + (long long)m * ldc + n : dst);
#pragma unroll
        for (int e = 0; e < 8; ++e) {
            const float v = e < 4 ? lo[e & 3] : hi[e & 3];
            o[e] = (__bf16)(p.accumulate ? v + bf2f(old[e]) : v);
        }
        *reinterpret_cast<bf16x8*>(dst) = o;
    }
}

static void set_pair_plan(MfmaGemmParams& p, int tiles_m, const PairPlan& plan, float* split_ws) {
    p.tiles_m = tiles_m;
    p.tiles_n = ceil_div(p.N, PN);
    p.per_xcd = plan.per_xcd;
    p.q_end = plan.q_end;
    p.split_s = plan.parts;
    p.split_per = plan.per;
    p.split_ws = split_ws;
}
// Steps of 32 k of its longest work-group
static int pair_steps(const MfmaGemmParams& p, const PairPlan& plan) {
    int steps = 0;
    for (int s = 0; s < p.n_seg; ++s) steps += ceil_div(p.K[s], BK);
    return plan.q_end > 0 ? steps : plan.per;
}
int pair_grid(const PairPlan& plan) { return 8 * (plan.q_end + (plan.per_xcd - plan.q_end) * plan.parts); }
static void finish_pair(const MfmaGemmParams& p, hipStream_t stream) {
    if (p.split_s > 1) k_gemm_pair_finish<false><<<dim3(8 * (p.per_xcd - p.q_end), PM / 16), 256, 0, stream>>>(p);
}

int launch_gemm_pair(MfmaGemmParams p, bool a_kmajor, bool b_kmajor, int tiles_m, const PairPlan& plan, float* split_ws, hipStream_t stream) {
    set_pair_plan(p, tiles_m, plan, split_ws);
    const int grid = pair_grid(plan);
    if (a_kmajor && b_kmajor) k_gemm_pair<true, true><<<grid, 256, 0, stream>>>(p);
    else if (a_kmajor) k_gemm_pair<true, false><<<grid, 256, 0, stream>>>(p);
    else if (b_kmajor) k_gemm_pair<false, true><<<grid, 256, 0, stream>>>(p);
    else k_gemm_pair<false, false><<<grid, 256, 0, stream>>>(p);
    finish_pair(p, stream);
    ALCH_HIP_TRY(hipGetLastError());
    return ALCH_OK;
}

size_t pair_split_bytes(const PairPlan& plan) {
    return plan.parts > 1 ? (size_t)8 * (plan.per_xcd - plan.q_end) * plan.parts * PM * PN * sizeof(float) : 0;
}

int launch_gemm_two_pairs(MfmaGemmParams data, int data_tiles_m, const PairPlan& data_plan, MfmaGemmParams weight, int weight_tiles_m,
                          const PairPlan& weight_plan, float* split_ws, hipStream_t stream) {
    set_pair_plan(data, data_tiles_m, data_plan, split_ws);
    set_pair_plan(weight, weight_tiles_m, weight_plan, split_ws + pair_split_bytes(data_plan) / sizeof(float));
    const int n_data = pair_grid(data_plan), n_weight = pair_grid(weight_plan);
    const bool weight_first = pair_steps(weight, weight_plan) > pair_steps(data, data_plan);
    k_gemm_two_pairs<<<n_data + n_weight, 256, 0, stream>>>(data, weight, weight_first ? n_weight : n_data, weight_first);
    finish_pair(data, stream);
    finish_pair(weight, stream);
    ALCH_HIP_TRY(hipGetLastError());
    return ALCH_OK;
}

int launch_gemm_pair_rows(MfmaGemmParams p, int grid, int cut, float* split_ws, hipStream_t stream) {
    p.tiles_n = ceil_div(p.N, PN);
    p.split_ws = split_ws;
    if (p.b_kmajor) k_gemm_pair_rows<true><<<grid, 256, 0, stream>>>(p);
    else k_gemm_pair_rows<false><<<grid, 256, 0, stream>>>(p);
    if (cut > 0) k_gemm_pair_finish<true><<<dim3(8 * cut, PM / 16), 256, 0, stream>>>(p);
    ALCH_HIP_TRY(hipGetLastError());
    return ALCH_OK;
}

}  // namespace alch
