// Causal grouped-query attention on the gfx950 matrix cores, head_dim 128 or 64 (kD), bf16: the kernels and
// their launch functions.  Each head size is instantiated by a source file of its own.
//
// Backward from the saved record (Section 4.1 of the paper: the prompt's Q, K, V stay on the
// GPU after prefill; Section 4.2: the layer's backward consumes them).  Probabilities are
// rebuilt from saved Q, K and LSE, never stored: p_ij = exp(q_i.k_j/sqrt(D) - LSE_i), j <= i.
//
// Two kernels, no atomics, deterministic:
//   dK/dV kernel: a work-group owns 128 keys of one (sequence, kv head) -- 32 per wavefront,
//     their K and V fragments held in registers -- and streams 64-query tiles of Q and dO of
//     every query head of the group through LDS (direct-to-LDS loads, four stages, software pipelined).
//       S = Q K^T, dP = dO V^T            (tile rows from LDS with ds_read_b128)
//       P, dS in the accumulator layout feed straight back as the left operand of
//       dV += P^T dO, dK += dS^T Q        (dO, Q rows read with the transposing LDS read)
//   dQ kernel: a work-group owns 128 queries of one (sequence, query head) and streams 64-key
//     tiles of K and V:  S^T = K Q^T, dP^T = V dO^T, dQ += dS K.
// The LDS tile is [rows][kD] bf16 with the 16-byte chunk index XOR-ed by a function of the row
// that makes both the row-major and the transposing reads bank-conflict free.
//
// Heads of 64 run the same schedule with half as many matrix instructions per score element, so they are bound by the
// vector port (exponentials and conversions) rather than by the matrix pipes.  They took kernels of a wavefront per row
// before, whose every (row, key) pair costs two six-step lane reductions and which held probabilities and dS in fp32.  That
// precision is kept: P and dS enter the second contractions as sums of two bf16 numbers each (2^-17 of the value is lost, the
// results are bf16), the forward's LSE is formed to fp32 rounding and RoPE angles take the accurate sine and cosine.  Against
// 64 bits (4096 tokens) the errors of O, dQ, dK, dV are those of rounding the exact values to bf16 to four digits (1.61e-3 ..
// 1.68e-3; P and dS in one bf16 number: 2.06e-3 .. 2.32e-3), that of the LSE 4.6e-8.  5 sequences, 4099 tokens, 32/8 heads:
// dQ 7043 -> 65 us, dK/dV 7630 -> 131 us and 7 us for the sum of its parts (one bf16 number: 53 and 103 us), delta and RoPE
// backward (29 us) inside these.  Heads of 128 round P and dS to bf16 once.
#pragma once
#include <algorithm>
#include <type_traits>
#include "attn_rows.h"

namespace alch {

typedef __attribute__((ext_vector_type(8))) __bf16 bf16x8;
typedef __attribute__((ext_vector_type(4))) __bf16 bf16x4;
typedef __attribute__((ext_vector_type(16))) float f32x16;
typedef __attribute__((ext_vector_type(4))) float f32x4;
typedef __attribute__((ext_vector_type(4))) int i32x4;

#define ALCH_LDS(p) ((__attribute__((address_space(3))) void*)(p))

static constexpr int kTileRows = 64;  // rows of a streamed tile
template <int kD> struct AttnTile {
    static_assert(kD == 128 || kD == 64, "");
    static constexpr int kRowBytes = kD * 2;
    static constexpr int kBytes = kTileRows * kRowBytes;   // 16 KB / 8 KB
    static constexpr int kStageBytes = 2 * kBytes + 1024;  // two tiles + two 64-float vectors (padded)
    static constexpr int kKK = kD / 16;                    // 16-wide steps of a contraction over the head
    static constexpr int kNB = kD / 32;                    // 32-wide column blocks of a head
    static constexpr int kLoads = kD / 32;                 // 1 KB direct-to-LDS loads per wavefront and tile
    static constexpr bool kTwo = kD == 64;                 // probabilities and dS as two bf16 numbers each (see the head)
};
static constexpr float kLog2e = 1.4426950408889634f;
static constexpr int kMinPartTiles = 8;  // tiles a part of a key block has at least
static constexpr int kRowsPerCu = 16;    // see rows_up_to
static constexpr int kMaxGridSeqs = 65535, kMaxGridBlocks = 65535;  // of 128 tokens: limits of a grid's second and third dimension

struct AttnMfmaParams {
    const __bf16 *Q, *K, *V, *O, *dO;
    const float* LSE;
    float* delta;  // written by the dQ kernel (row sums of dO*O), read by the dK/dV kernel
    float* lse2;   // LSE * log2(e), written by the dQ kernel for the dK/dV kernel (its exponent is one fused multiply-add)
    __bf16 *dQ, *dK, *dV;
    const int* cu;
    const int* prefix;     // null, or per sequence: -1 / the earlier sequence whose keys it also attends to
    int n_seqs, short_upto;  // sequences of up to so many tokens are not these kernels'
    const int* positions;  // RoPE positions per token, or null: index inside the sequence
    int Hq, Hkv;
    long long ldq, ldk, ldo;  // row strides (elements) of Q/dO, K/V, and of the outputs
    float scale;
    int rope;              // rotate dQ, dK by minus the RoPE angle before they are stored
    float rope_log2_base;
    // dK/dV: key blocks of up to n_blocks per sequence; a block whose query stream is longer than part_len tiles is cut
    // over the query heads of the group into up to max_parts work-groups, which leave fp32 partial sums
    // [part][T][Hkv][dK | dV] in `partial` (max_parts 1: none is)
    int T, n_blocks, max_parts, part_len;
    float* partial;
};

// Work-groups that share a key block whose query stream has `tiles` tiles per head, and how many heads each takes.
__device__ __forceinline__ int dkv_parts(const AttnMfmaParams& p, int G, int tiles, int& heads) {
    const int want = min(p.max_parts, (G * tiles + p.part_len - 1) / p.part_len);
    heads = (G + max(want, 1) - 1) / max(want, 1);
    return (G + heads - 1) / heads;
}
// The sequences that name `seq` as their prefix and have a row, looked for by a wavefront, 64 candidates at a time (one at a
// time, a key block of a batch of 600 sequences spent most of its time on this).  Every lane takes part.
struct PrefixSeqs {
    int first, last;     // of them (last -1: none)
    int tiles, ragged;   // 64-query tiles per head of all, and how many of those are not whole
    int base, row0, n;   // the 64 looked at now: lane i holds the first row and the rows of sequence base + i, 0 if it is none of them
};
__device__ __forceinline__ void prefix_window(const AttnMfmaParams& p, int seq, int base, int& row0, int& n) {
    const int i = base + (int)(threadIdx.x & 63), c = min(i, p.n_seqs - 1);
    const int named = p.prefix[c], end = p.cu[c + 1];
    row0 = p.cu[c];
    n = i < p.n_seqs && named == seq ? end - row0 : 0;
}
__device__ __forceinline__ PrefixSeqs prefix_seqs(const AttnMfmaParams& p, int seq) {
    PrefixSeqs s{p.n_seqs, -1, 0, 0, seq + 1, 0, 0};
    int row0, n;
    prefix_window(p, seq, seq + 1, row0, n);
    for (int base = seq + 1; base < p.n_seqs; base += 64) {
        int row0_next, n_next;
        prefix_window(p, seq, base + 64, row0_next, n_next);  // (on its way while these are counted)
        const unsigned long long bits = __ballot(n > 0);
        if (bits) {
            if (s.last < 0) {
                s.first = base + __builtin_ctzll(bits);
                s.base = base; s.row0 = row0; s.n = n;
            }
            s.last = base + 63 - __builtin_clzll(bits);
            s.ragged += __popcll(__ballot(n % kTileRows != 0));
            s.tiles += (n + kTileRows - 1) / kTileRows;
        }
        row0 = row0_next; n = n_next;
    }
    int sum = 0;
    for (int b = 0; __ballot(s.tiles >> b != 0); ++b) sum += __popcll(__ballot(s.tiles >> b & 1)) << b;
    s.tiles = sum;
    return s;
}
// The next one behind sequence c that has whole tiles, or one that is not whole (n_seqs: none)
__device__ __forceinline__ int prefix_next(const AttnMfmaParams& p, int seq, PrefixSeqs& s, int c, bool whole) {
    for (c = max(c + 1, s.first); c <= s.last; c = s.base + 64) {
        if (c < s.base || c >= s.base + 64) {
            s.base = c;
            prefix_window(p, seq, c, s.row0, s.n);
        }
        const unsigned long long bits = (whole ? __ballot(s.n >= kTileRows) : __ballot(s.n % kTileRows != 0)) >> (c - s.base);
        if (bits) return c + __builtin_ctzll(bits);
    }
    return p.n_seqs;
}

template <int kD> __device__ __forceinline__ float rope_theta(int d, float log2_base) {
    const float x = -(float)d * (2.0f / kD) * log2_base;
    return AttnTile<kD>::kTwo ? exp2f(x) : __builtin_amdgcn_exp2f(x);
}
template <int kD> __device__ __forceinline__ void rope_sincos(float angle, float& sn, float& cs) {
    if (AttnTile<kD>::kTwo) sincosf(angle, &sn, &cs);
    else __sincosf(angle, &sn, &cs);
}
// RoPE backward on one accumulator set: block nb of the lower half holds element d = nb*32 + (lane&31) of a head,
// block nb + kNB/2 its partner d + kD/2; x'[d] = x[d] cos a + x[d+kD/2] sin a, x'[d+kD/2] = x[d+kD/2] cos a - x[d] sin a
// with a = pos * base^(-2d/kD).
template <int kD>
__device__ __forceinline__ void rope_backward_rows(f32x16 (&x)[AttnTile<kD>::kNB], const AttnMfmaParams& p, int seq_start, int row0,
                                                  int len, int lane) {
    const int half = lane >> 5;
#pragma unroll
    for (int nb = 0; nb < AttnTile<kD>::kNB / 2; ++nb) {
        const float theta = rope_theta<kD>(nb * 32 + (lane & 31), p.rope_log2_base);
#pragma unroll
        for (int e = 0; e < 16; ++e) {
            const int r = row0 + 8 * (e >> 2) + 4 * half + (e & 3);
            const int pos = (p.positions && r < len) ? p.positions[seq_start + r] : r;
            float sn, cs;
            rope_sincos<kD>((float)pos * theta, sn, cs);
            const float a = x[nb][e], b = x[nb + AttnTile<kD>::kNB / 2][e];
            x[nb][e] = a * cs + b * sn;
            x[nb + AttnTile<kD>::kNB / 2][e] = b * cs - a * sn;
        }
    }
}

// The same for one row of a head of 64, element `lane` per lane
template <int kD>
__device__ __forceinline__ float rope_backward_row(float x, const AttnMfmaParams& p, int seq_start, int row, int lane) {
    if (!p.rope) return x;
    const int pos = p.positions ? p.positions[seq_start + row] : row;
    float sn, cs;
    rope_sincos<kD>((float)pos * rope_theta<kD>(lane & 31, p.rope_log2_base), sn, cs);
    const float other = __shfl_xor(x, 32, 64);
    return lane < 32 ? x * cs + other * sn : x * cs - other * sn;
}

__device__ __forceinline__ i32x4 rsrc_of(const void* p, long long bytes) {
    const uint32_t n = bytes <= 0 ? 0u : (bytes > 0x7fffffffLL ? 0x7fffffffu : (uint32_t)bytes);
    const uint64_t a = reinterpret_cast<uint64_t>(p);
    i32x4 r;
    r[0] = __builtin_amdgcn_readfirstlane((int)(uint32_t)a);
    r[1] = __builtin_amdgcn_readfirstlane((int)((uint32_t)(a >> 32) & 0xffffu));
    r[2] = __builtin_amdgcn_readfirstlane((int)n);
    r[3] = 0x00020000;
    return r;
}
// (s_nop: a load into LDS takes one wait state after a scalar write of m0, which the compiler does not see to in assembly)
__device__ __forceinline__ void dma16(i32x4 r, uint32_t lds_addr, uint32_t voff) {
    asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tbuffer_load_dwordx4 %1, %2, 0 offen lds" ::"s"(lds_addr), "v"(voff), "s"(r)
                 : "memory", "m0");
}
__device__ __forceinline__ void dma4(i32x4 r, uint32_t lds_addr, uint32_t voff) {
    asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tbuffer_load_dword %1, %2, 0 offen lds" ::"s"(lds_addr), "v"(voff), "s"(r)
                 : "memory", "m0");
}

// chunk swizzle of the [rows][kD] tile, 16-byte chunks.  The row-major reads want 16 consecutive rows at one chunk on
// 16 different 16-byte slots of the 256-byte bank line, the transposing reads want four consecutive rows at four
// neighbouring chunks on 16 different ones.  128 elements: a row is one bank line of 16 chunks.  64 elements: two rows
// share a line, the low row bit picks the half and the other three pick one of its 8 chunks.
template <int kD>
__device__ __forceinline__ int swz(int row) {
    if (kD == 128) return ((row & 3) << 2) | ((row >> 2) & 3);
    return (((row >> 1) & 1) << 2) | ((row >> 2) & 3);
}

// Per-lane byte offsets of one wave's share (a quarter of the loads) of a 64-row tile of rows `ld` elements apart.
template <int kD>
__device__ __forceinline__ void tile_voffsets(uint32_t (&voff)[AttnTile<kD>::kLoads], long long ld, int wave, int lane) {
    constexpr int kChunks = kD / 8;
#pragma unroll
    for (int j = 0; j < AttnTile<kD>::kLoads; ++j) {
        const int slot = (wave * AttnTile<kD>::kLoads + j) * 64 + lane;
        const int row = slot / kChunks, c = (slot % kChunks) ^ swz<kD>(row);
        voff[j] = (uint32_t)((row * ld + c * 8) * 2);
    }
}
// The loads themselves: tile rows start at `base`, `rows_valid` rows exist (the rest read as zero).
template <int kD>
__device__ __forceinline__ void issue_rows_tile(const __bf16* base, long long ld, int rows_valid, uint32_t lds_addr,
                                                int wave, const uint32_t (&voff)[AttnTile<kD>::kLoads]) {
    const i32x4 r = rsrc_of(base, rows_valid > 0 ? ((long long)(rows_valid - 1) * ld + kD) * 2 : 0);
#pragma unroll
    for (int j = 0; j < AttnTile<kD>::kLoads; ++j)
        dma16(r, lds_addr + (uint32_t)(wave * AttnTile<kD>::kLoads + j) * 1024u, voff[j]);
}
// LDS read addresses.  Every fragment address of a [rows][kD] tile is a per-lane constant combined
// with compile-time terms, so the lane parts are computed once per kernel:
//   d-fragments (k = d):   byte = row0*kRowBytes + (lane_d ^ (kk << 5)),       lane_d from frag_d_lane()
//   row-fragments (k = row): byte = (row0 + 16*ks)*kRowBytes + (lane_r ^ (nb << 6)), lane_r from frag_rows_lane()
// where row0 is a multiple of 32 (XOR and ADD commute with it).
template <int kD>
__device__ __forceinline__ uint32_t frag_d_lane(int lane) {
    const int row = lane & 31;
    return (uint32_t)(row * AttnTile<kD>::kRowBytes + (((lane >> 5) ^ swz<kD>(row)) << 4));
}
// second = 0: tile rows 4*(g>>1) + (i>>2); second = 1: eight rows further down
template <int kD>
__device__ __forceinline__ uint32_t frag_rows_lane(int lane, int second) {
    const int g = lane >> 4, i = lane & 15;
    const int col = (g & 1) * 16 + 4 * (i & 3);
    const int r = 4 * (g >> 1) + (i >> 2) + 8 * second;
    return (uint32_t)(r * AttnTile<kD>::kRowBytes + (((col >> 3) ^ swz<kD>(r)) << 4) + (col & 7) * 2);
}
__device__ __forceinline__ bf16x8 lds_frag_d(const char* tile, uint32_t lane_d, int kk) {
    return *reinterpret_cast<const bf16x8*>(tile + (lane_d ^ (uint32_t)(kk << 5)));
}
template <int kD>
__device__ __forceinline__ bf16x8 lds_frag_rows(const char* tile, uint32_t lane_r0, uint32_t lane_r1, int ks, int nb) {
    const char* t = tile + ks * 16 * AttnTile<kD>::kRowBytes;
    bf16x4 lo = __builtin_amdgcn_ds_read_tr16_b64_v4bf16((__attribute__((address_space(3))) bf16x4*)(t + (lane_r0 ^ (uint32_t)(nb << 6))));
    bf16x4 hi = __builtin_amdgcn_ds_read_tr16_b64_v4bf16((__attribute__((address_space(3))) bf16x4*)(t + (lane_r1 ^ (uint32_t)(nb << 6))));
    return __builtin_shufflevector(lo, hi, 0, 1, 2, 3, 4, 5, 6, 7);
}

// Accumulator elements 8 ks .. 8 ks + 7 as the bf16 operand of the next contraction.  kTwo: as a sum of two bf16 numbers, the
// rounded value and the rounded rest, which carries 16 bits of the fp32 value at the price of a second matrix instruction.
template <bool kTwo> struct Operand;
template <> struct Operand<false> { bf16x8 hi; };
template <> struct Operand<true> { bf16x8 hi, lo; };
template <bool kTwo>
__device__ __forceinline__ void pack8(Operand<kTwo>& o, const f32x16& v, int ks) {
#pragma unroll
    for (int e = 0; e < 8; ++e) {
        o.hi[e] = (__bf16)v[8 * ks + e];
        if constexpr (kTwo) o.lo[e] = (__bf16)(v[8 * ks + e] - (float)o.hi[e]);
    }
}

// 16-byte global load of an operand fragment held in registers for the whole kernel:
// rows row0 + (lane&31) of a [rows, ld] matrix (column offset already in base), zero beyond rows_valid
__device__ __forceinline__ bf16x8 global_frag_d(const __bf16* base, long long ld, int row0, int rows_valid, int kk, int lane) {
    const int row = row0 + (lane & 31);
    bf16x8 z;
#pragma unroll
    for (int e = 0; e < 8; ++e) z[e] = (__bf16)0.f;
    if (row >= rows_valid) return z;
    return *reinterpret_cast<const bf16x8*>(base + (long long)row * ld + kk * 16 + 8 * (lane >> 5));
}

// ---------------------------------------------------------------------------------------------
// dK / dV
// kPrefix: sequences may name an earlier sequence as their prefix.  The key block then also meets, after the
// queries of its own sequence (causal), every query of every sequence that names this one (no mask but the
// ends of the sequences).
// kv: key/value head, z: part and key block, smem: four stages.
template <int kD, bool kPrefix>
__device__ __forceinline__ void attn_dkv_block(const AttnMfmaParams& p, const int kv, const int seq, const int z, char* smem) {
    constexpr int kTileBytes = AttnTile<kD>::kBytes, kStageBytes = AttnTile<kD>::kStageBytes, kRowBytes = AttnTile<kD>::kRowBytes;
    constexpr int kKK = AttnTile<kD>::kKK, kNB = AttnTile<kD>::kNB, kLoads = AttnTile<kD>::kLoads;
    const uint32_t lds0 = (uint32_t)(uintptr_t)ALCH_LDS(smem);
    // Work-groups are handed out in order of z first, so it counts the work down: a key block
    // with `rem` blocks of queries at or after it costs rem units, and the heaviest of all sequences
    // and heads start first (longest-processing-time-first keeps the last compute units busy).
    const int seq_start = p.cu[seq], len = p.cu[seq + 1] - seq_start;
    if (len <= p.short_upto) return;
    const int part = z / p.n_blocks;
    const int rem = p.n_blocks - (z - part * p.n_blocks), kb = (len + 127) / 128 - rem;
    if (kb < 0) return;
    // this work-group's query heads h_first .. h_end-1: the group's, or a part of them
    const int qt0 = (kb * 128) / kTileRows;
    const int nqt = (len + kTileRows - 1) / kTileRows - qt0;
    const int G = p.Hq / p.Hkv;
    int head_tiles = nqt;
    PrefixSeqs named{};
    if constexpr (kPrefix) {
        named = prefix_seqs(p, seq);
        head_tiles += named.tiles;
    }
    int part_heads;
    const int parts = dkv_parts(p, G, head_tiles, part_heads);
    if (part >= parts) return;
    const int h_first = kv * G + part * part_heads, h_end = min(h_first + part_heads, kv * G + G);
    const int lane = threadIdx.x & 63, half = lane >> 5;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int j0 = kb * 128 + wave * 32;  // this wave's first key (index inside the sequence)

    // K, V fragments of the wave's 32 keys stay in registers
    const __bf16* Kb = p.K + (long long)seq_start * p.ldk + kv * kD;
    const __bf16* Vb = p.V + (long long)seq_start * p.ldk + kv * kD;
    bf16x8 kf[kKK], vf[kKK];
#pragma unroll
    for (int kk = 0; kk < kKK; ++kk) {
        kf[kk] = global_frag_d(Kb, p.ldk, j0, len, kk, lane);
        vf[kk] = global_frag_d(Vb, p.ldk, j0, len, kk, lane);
    }
    f32x16 dK[kNB], dV[kNB];
#pragma unroll
    for (int n = 0; n < kNB; ++n)
#pragma unroll
        for (int e = 0; e < 16; ++e) dK[n][e] = dV[n][e] = 0.f;

    const uint32_t lane_d = frag_d_lane<kD>(lane), lane_r0 = frag_rows_lane<kD>(lane, 0), lane_r1 = frag_rows_lane<kD>(lane, 1);
    uint32_t voff[kLoads];
    tile_voffsets<kD>(voff, p.ldq, wave, lane);
    const int n_it = (h_end - h_first) * head_tiles;
    const float sl2 = p.scale * kLog2e;

    // The tile stream: for the key block's own sequence and then (kPrefix) every sequence that names it as
    // prefix, for every query head of the group, the 64-query tiles qt_first .. qt_end-1 of that sequence.
    // The stream is ordered in passes over the heads of the group: first the (at most two) tiles of every head that
    // meet the diagonal of the key block, which need the causal mask, last the others, which need none -- rows and
    // keys past the end of the sequence are zero-filled by the loads, so they contribute exactly nothing to rows that
    // are stored.  kPrefix: between the two, still masked, the last tiles past the diagonal that are not whole; fewer than
    // four that need no mask take it, too (the other loop's code has to be fetched for them).
    // n_mask iterations take the masked code.  (Prefix batches, with the mask on all tiles and responses looked for one by one
    // -> so, 32/8 heads of 128, two responses to a prompt, us: 4 prompts of 1024 tokens, responses of 128 194 -> 157; 4 of
    // 2048, 64 401 -> 333; one of 500, 40 35 -> 35, sixteen of them 76 -> 74; 40 of 64, 32 148 -> 93; 200 of 40, 20 1822 -> 470.
    // Heads of 64: 185 -> 155, 388 -> 323, 33.5 -> 34.8, 75 -> 78, 144 -> 93, 1812 -> 468.)
    const int n_diag = min(2, nqt);
    const int n_tail = kPrefix ? named.ragged + (nqt > n_diag && len % kTileRows != 0 ? 1 : 0) : 0;
    int n_mask = (h_end - h_first) * (n_diag + n_tail);
    if (kPrefix && n_it - n_mask < 4) n_mask = n_it;
    struct Cursor {
        int c, row0, n;         // sequence of the queries, its first row in the batch, its length
        int qt_first, qt_end;   // its tiles that this key block meets in the current pass
        int h, qt;              // query head and tile of the current position
        int pass;               // kPrefix: 0 the diagonal, 1 tiles that are not whole, 2 all others
    };
    auto advance = [&](Cursor& q) {
        if (++q.qt < q.qt_end) return;
        q.qt = q.qt_first;
        if (++q.h < h_end) return;
        q.h = h_first;
        if constexpr (!kPrefix) {
            if (q.qt_first == qt0 && nqt > n_diag) {  // second pass: the tiles past the diagonal
                q.qt_first = q.qt = qt0 + n_diag;
                q.qt_end = qt0 + nqt;
            }
        }
        if constexpr (kPrefix) {
            int c = q.c, pass = q.pass;
            for (;;) {
                c = pass == 0 ? p.n_seqs : prefix_next(p, seq, named, c, pass == 2);  // (of the diagonal the sequence itself is all)
                const bool own = c >= p.n_seqs;
                if (own) {
                    if (pass == 2) break;
                    pass = pass == 0 && n_tail > 0 ? 1 : 2;
                    c = seq;
                }
                const int row0 = own ? seq_start : __builtin_amdgcn_readlane(named.row0, c - named.base);
                const int n = own ? len : __builtin_amdgcn_readlane(named.n, c - named.base);
                const int lo = own ? qt0 + n_diag : 0, whole = n / kTileRows;
                const int first = pass == 1 ? max(whole, lo) : lo, end = pass == 1 ? whole + (n % kTileRows != 0) : whole;
                if (first < end) {
                    q.c = c; q.row0 = row0; q.n = n; q.pass = pass;
                    q.qt_first = q.qt = first; q.qt_end = end;
                    break;
                }
            }
        }
        // (past the end of the stream the cursor wraps; its tiles are then loaded with zero extent)
    };
    // Software pipeline over the tile stream, four LDS stages (tile t in stage t & 3).  Entering iteration
    // `it`, of tile `it` (two blocks of 32 queries) the wave holds P, dS of block 0 packed to bf16 and the raw
    // scores S = Q K^T, dP = dO V^T of block 1.  The iteration waits for its own loads of tile it+1 (issued two
    // iterations ago) and meets the other waves (every wave is then past its reads of tile it-1, whose stage
    // receives tile it+3), then runs kGroups (16, or 8 for heads of 64) groups of four matrix instructions:
    //   first half:  dV += P^T dO, dK += dS^T Q of block 0   |  S, dP of block 0 of tile it+1
    //   second half: the same for block 1                     |  S, dP of block 1 of tile it+1
    // Every matrix instruction is followed by its share of everything else, pinned in place (a wave issues in
    // order, so vector work only overlaps a matrix instruction that was issued before it): the six LDS reads of
    // the group two ahead, half of the exp/mask/dS work of two score elements (four for heads of 64; block 1 of
    // tile `it` during the first half, block 0 of tile it+1 during the second), one of the direct-to-LDS loads of tile it+3,
    // the LSE / delta rows the coming groups need, and once per iteration the stream bookkeeping and the
    // buffer descriptors of the tile the next iteration loads.  Beyond the end of the stream the loads are
    // issued with zero extent: they move nothing and keep every wave's count of outstanding loads the same.
    f32x16 S1, dP1;         // raw scores of block 1 of the current tile
    constexpr bool kTwo = AttnTile<kD>::kTwo;
    Operand<kTwo> pf0[2], dsf0[2]; // P, dS of block 0 of the current tile
    const int jl = j0 + (lane & 31);  // this lane's key
    const unsigned live_own = (unsigned)max(len - jl, 0);
    // P, dS of accumulator elements e0 .. e0+n-1 of one block, in place.  Element e is query row
    // i = i0 + 8*(e>>2) + 4*half + (e&3) against key column jl.  Pairs above the diagonal (jl > i) and rows
    // or keys past the end of the sequence get exponent -inf, i.e. p = 0 exactly: with rel = i - jl that
    // is one unsigned test, rel >= max(len - jl, 0).  Queries of a sequence that names this one as prefix
    // see every key: rel = i and the bound is that sequence's length (0 for a key past the end).
    // l, d: LSE and delta of the block's 16 rows of this lane.
    struct Meta { int ibase, sub; unsigned live; };  // first query row of a tile; what rel subtracts; the bound
    auto meta_of = [&](const Cursor& q) {
        Meta m;
        m.ibase = q.qt * kTileRows;
        if (!kPrefix || q.c == seq) { m.sub = jl; m.live = live_own; }
        else { m.sub = 0; m.live = jl < len ? (unsigned)q.n : 0u; }
        return m;
    };
    auto softmax_part = [&](f32x16& s, f32x16& dp, const f32x4 (&l)[4], const f32x4 (&d)[4], const Meta& m, int blk, int e0, int n) {
        const int rel0 = m.ibase + blk * 32 + 4 * half - (kPrefix ? m.sub : jl);
        const unsigned live = kPrefix ? m.live : live_own;
#pragma unroll
        for (int e = e0; e < e0 + n; ++e) {
            const unsigned rel = (unsigned)(rel0 + 8 * (e >> 2) + (e & 3));
            float arg = __builtin_fmaf(s[e], sl2, -l[e >> 2][e & 3]);
            arg = rel >= live ? -INFINITY : arg;
            const float pr = __builtin_amdgcn_exp2f(arg);
            s[e] = pr;
            dp[e] = pr * (dp[e] - d[e >> 2][e & 3]);
        }
    };
    auto load_row_scalars = [&](const char* stage, int ib, f32x4 (&l)[4], f32x4 (&d)[4]) {
        const float* lse_s = reinterpret_cast<const float*>(stage + 2 * kTileBytes);
#pragma unroll
        for (int b = 0; b < 4; ++b) {
            l[b] = *reinterpret_cast<const f32x4*>(lse_s + ib * 32 + 8 * b + 4 * half);
            d[b] = *reinterpret_cast<const f32x4*>(lse_s + 64 + ib * 32 + 8 * b + 4 * half);
        }
    };

    // Buffer descriptors of one tile's loads (Q rows, dO rows, and for the first two waves LSE / delta).
    struct LoadDesc { i32x4 q, dO, sc; };
    auto desc_of = [&](const Cursor& q, bool live) {
        const int rows = live ? q.n - q.qt * kTileRows : 0;
        const long long ext = rows > 0 ? ((long long)(rows - 1) * p.ldq + kD) * 2 : 0;
        const long long row = (long long)(q.row0 + q.qt * kTileRows);
        LoadDesc d;
        d.q = rsrc_of(p.Q + row * p.ldq + q.h * kD, ext);
        d.dO = rsrc_of(p.dO + row * p.ldq + q.h * kD, ext);
        d.sc = rsrc_of((wave == 0 ? p.lse2 : p.delta) + row * p.Hq + q.h,
                       (rows > 0 && wave < 2) ? ((long long)(rows - 1) * p.Hq + 1) * 4 : 0);
        return d;
    };
    // LDS address of the row-scalar load of this wave: LSE (wave 0), delta (wave 1); the other two waves issue the
    // same instruction with zero extent into the stage's padding, so every wave has kTileLoads loads per tile in flight
    const uint32_t sc_lds = 2 * kTileBytes + (wave < 2 ? (uint32_t)wave * 256u : 512u + (uint32_t)(wave - 2) * 256u);
    const uint32_t sc_voff = (uint32_t)(lane * p.Hq * 4);
    auto issue_tile = [&](const LoadDesc& d, uint32_t st) {
#pragma unroll
        for (int j = 0; j < kLoads; ++j) dma16(d.q, st + (uint32_t)(wave * kLoads + j) * 1024u, voff[j]);
#pragma unroll
        for (int j = 0; j < kLoads; ++j) dma16(d.dO, st + kTileBytes + (uint32_t)(wave * kLoads + j) * 1024u, voff[j]);
        dma4(d.sc, st + sc_lds, sc_voff);
    };
    // Four LDS stages, tile t in stage t & 3; iteration `it` works on tiles it and it+1 and loads tile it+3.
    Cursor q_ld{seq, seq_start, len, qt0, qt0 + n_diag, h_first, qt0, 0};
    Meta m_cur = meta_of(q_ld);
    issue_tile(desc_of(q_ld, 0 < n_it), lds0);
    advance(q_ld);
    Meta m_nxt = meta_of(q_ld);
    issue_tile(desc_of(q_ld, 1 < n_it), lds0 + kStageBytes);
    advance(q_ld);
    Meta m_nn = meta_of(q_ld);
    issue_tile(desc_of(q_ld, 2 < n_it), lds0 + 2 * kStageBytes);
    advance(q_ld);  // now at tile 3, the one iteration 0 loads
    Meta m_n3 = meta_of(q_ld);
    LoadDesc dsc = desc_of(q_ld, 3 < n_it);
    advance(q_ld);
    constexpr int kTileLoads = 2 * kLoads + 1;
    asm volatile("s_waitcnt vmcnt(%0)" ::"n"(2 * kTileLoads) : "memory");
    __syncthreads();
    f32x4 l1[4], d1[4];  // LSE, delta of block 1 of the current tile
    {   // tile 0: scores of both blocks, P and dS of block 0
        f32x16 S0, dP0;
#pragma unroll
        for (int e = 0; e < 16; ++e) S0[e] = dP0[e] = S1[e] = dP1[e] = 0.f;
#pragma unroll
        for (int kk = 0; kk < kKK; ++kk) {
            S0 = __builtin_amdgcn_mfma_f32_32x32x16_bf16(lds_frag_d(smem, lane_d, kk), kf[kk], S0, 0, 0, 0);
            dP0 = __builtin_amdgcn_mfma_f32_32x32x16_bf16(lds_frag_d(smem + kTileBytes, lane_d, kk), vf[kk], dP0, 0, 0, 0);
            S1 = __builtin_amdgcn_mfma_f32_32x32x16_bf16(lds_frag_d(smem + 32 * kRowBytes, lane_d, kk), kf[kk], S1, 0, 0, 0);
            dP1 = __builtin_amdgcn_mfma_f32_32x32x16_bf16(lds_frag_d(smem + kTileBytes + 32 * kRowBytes, lane_d, kk), vf[kk], dP1, 0, 0, 0);
        }
        f32x4 l[4], d[4];
        load_row_scalars(smem, 0, l, d);
        softmax_part(S0, dP0, l, d, m_cur, 0, 0, 16);
#pragma unroll
        for (int ks = 0; ks < 2; ++ks) {
            pack8(pf0[ks], S0, ks);
            pack8(dsf0[ks], dP0, ks);
        }
        load_row_scalars(smem, 1, l1, d1);
    }

#define ALCH_SB __builtin_amdgcn_sched_barrier(0)
    struct Frags { bf16x8 rdo, rq, dq, ddo; };
    auto iteration = [&](auto masked_tag, int it) __attribute__((always_inline)) {
        constexpr bool kMasked = decltype(masked_tag)::value;
        const char* tq = smem + (uint32_t)(it & 3) * kStageBytes;
        const char* tdo = tq + kTileBytes;
        const char* nq = smem + (uint32_t)((it + 1) & 3) * kStageBytes;
        const char* ndo = nq + kTileBytes;
        const uint32_t st3 = lds0 + (uint32_t)((it + 3) & 3) * kStageBytes;

        ALCH_SB;
        asm volatile("s_waitcnt vmcnt(%0)" ::"n"(kTileLoads) : "memory");  // tile it+1 has landed (tile it+2 may still be on its way)
        __syncthreads();
        ALCH_SB;

        f32x4 ln[4], dn[4];  // LSE, delta of block 0 of the next tile
        // group g works on block g / kHalf, on the 16 rows (g / kNB) % 2 of it and its column block g % kNB
        constexpr int kGroups = 4 * kNB, kHalf = kGroups / 2;
        constexpr int kElems = 16 / kHalf;  // score elements per group: 2, or 4 for heads of 64
        Frags fr[3];
        auto ld_rdo = [&](int g) { fr[g % 3].rdo = lds_frag_rows<kD>(tdo + (g / kHalf) * 32 * kRowBytes, lane_r0, lane_r1, (g / kNB) & 1, g % kNB); };
        auto ld_rq = [&](int g) { fr[g % 3].rq = lds_frag_rows<kD>(tq + (g / kHalf) * 32 * kRowBytes, lane_r0, lane_r1, (g / kNB) & 1, g % kNB); };
        auto ld_d = [&](int g) {
            const int kk = g % kHalf;
            fr[g % 3].dq = lds_frag_d(nq + (g / kHalf) * 32 * kRowBytes, lane_d, kk);
            fr[g % 3].ddo = lds_frag_d(ndo + (g / kHalf) * 32 * kRowBytes, lane_d, kk);
        };
        ld_rdo(0); ld_rq(0); ld_d(0);
        ld_rdo(1); ld_rq(1); ld_d(1);
        f32x16 Sn0, dPn0, Sn1, dPn1;  // scores of the next tile
        Operand<kTwo> pf1[2], dsf1[2], pfn[2], dsfn[2];
        Meta m_n4;
        LoadDesc dsc_next;
        // One element of the softmax gradient in two halves, each pinned where it is written so that it is issued
        // between two matrix instructions: h1 = masked exponent -> probability, h2 = dS = p (dP - delta).
        {
            auto sm_h1 = [&](f32x16& sc, const f32x4 (&l)[4], const Meta& m, int blk, int e) {
                float arg = __builtin_fmaf(sc[e], sl2, -l[e >> 2][e & 3]);
                if constexpr (kMasked) {
                    const int rel0 = m.ibase + blk * 32 + 4 * half - (kPrefix ? m.sub : jl);
                    const unsigned live = kPrefix ? m.live : live_own;
                    const unsigned rel = (unsigned)(rel0 + 8 * (e >> 2) + (e & 3));
                    arg = rel >= live ? -INFINITY : arg;
                }
                float pr = __builtin_amdgcn_exp2f(arg);
                asm volatile("" : "+v"(pr));
                sc[e] = pr;
            };
            auto sm_h2 = [&](const f32x16& sc, f32x16& dp, const f32x4 (&d)[4], int e) {
                float t = sc[e] * (dp[e] - d[e >> 2][e & 3]);
                asm volatile("" : "+v"(t));
                dp[e] = t;
            };
#pragma unroll
            for (int g = 0; g < kGroups; ++g) {
                const int ib = g / kHalf, ks = (g / kNB) & 1, nb = g % kNB, kk = g % kHalf;
                const int e0 = kElems * (g % kHalf), e1 = e0 + kElems / 2, e2 = e0 + kElems;
                const Frags& f = fr[g % 3];
                const Operand<kTwo>& pg = ib == 0 ? pf0[ks] : pf1[ks];
                const Operand<kTwo>& dsg = ib == 0 ? dsf0[ks] : dsf1[ks];
                auto h1 = [&](int b, int n) __attribute__((always_inline)) {
#pragma unroll
                    for (int e = b; e < n; ++e) {
                        if (ib == 0) sm_h1(S1, l1, m_cur, 1, e); else sm_h1(Sn0, ln, m_nxt, 0, e);
                    }
                };
                auto h2 = [&](int b, int n) __attribute__((always_inline)) {
#pragma unroll
                    for (int e = b; e < n; ++e) {
                        if (ib == 0) sm_h2(S1, dP1, d1, e); else sm_h2(Sn0, dPn0, dn, e);
                    }
                };
                // slot 0
                if (g + 2 < kGroups) ld_rdo(g + 2);
                h1(e0, e1);
                ALCH_SB;
                dV[nb] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(pg.hi, f.rdo, dV[nb], 0, 0, 0);
                ALCH_SB;
                if constexpr (kTwo) {
                    h1(e1, e2);
                    ALCH_SB;
                    dV[nb] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(pg.lo, f.rdo, dV[nb], 0, 0, 0);
                    ALCH_SB;
                }
                // slot 1
                if (g + 2 < kGroups) ld_rq(g + 2);
                if constexpr (kTwo) h2(e0, e1); else h1(e1, e2);
                ALCH_SB;
                dK[nb] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(dsg.hi, f.rq, dK[nb], 0, 0, 0);
                ALCH_SB;
                if constexpr (kTwo) {
                    h2(e1, e2);
                    ALCH_SB;
                    dK[nb] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(dsg.lo, f.rq, dK[nb], 0, 0, 0);
                    ALCH_SB;
                }
                // slot 2
                if (g + 2 < kGroups) ld_d(g + 2);
                if constexpr (!kTwo) h2(e0, e2);
                ALCH_SB;
                if (g == 0) {
#pragma unroll
                    for (int e = 0; e < 16; ++e) Sn0[e] = dPn0[e] = 0.f;
                }
                if (g == kHalf) {
#pragma unroll
                    for (int e = 0; e < 16; ++e) Sn1[e] = dPn1[e] = 0.f;
                }
                if (ib == 0) Sn0 = __builtin_amdgcn_mfma_f32_32x32x16_bf16(f.dq, kf[kk], Sn0, 0, 0, 0);
                else Sn1 = __builtin_amdgcn_mfma_f32_32x32x16_bf16(f.dq, kf[kk], Sn1, 0, 0, 0);
                ALCH_SB;
                // slot 3: the loads of tile it+3, the row scalars the next groups need, the stream bookkeeping, packs
                if (g < kLoads) dma16(dsc.q, st3 + (uint32_t)(wave * kLoads + g) * 1024u, voff[g % kLoads]);
                else if (g < 2 * kLoads) dma16(dsc.dO, st3 + kTileBytes + (uint32_t)(wave * kLoads + g - kLoads) * 1024u, voff[g % kLoads]);
                else if (g == 2 * kLoads) dma4(dsc.sc, st3 + sc_lds, sc_voff);
                if (g < 4) {       // LSE, delta of block 0 of tile it+1 (used from group kHalf on)
                    const float* sc_n = reinterpret_cast<const float*>(nq + 2 * kTileBytes);
                    ln[g] = *reinterpret_cast<const f32x4*>(sc_n + 8 * g + 4 * half);
                    dn[g] = *reinterpret_cast<const f32x4*>(sc_n + 64 + 8 * g + 4 * half);
                }
                if (g >= kGroups - 4) {  // LSE, delta of block 1 of tile it+1 (used by the next iteration's first half)
                    constexpr int kLast = kGroups - 4;
                    const float* sc_n = reinterpret_cast<const float*>(nq + 2 * kTileBytes);
                    l1[g - kLast] = *reinterpret_cast<const f32x4*>(sc_n + 32 + 8 * (g - kLast) + 4 * half);
                    d1[g - kLast] = *reinterpret_cast<const f32x4*>(sc_n + 64 + 32 + 8 * (g - kLast) + 4 * half);
                }
                if (g == kHalf + 1) {  // position and descriptors of tile it+4, which the next iteration loads
                    m_n4 = meta_of(q_ld);
                    dsc_next = desc_of(q_ld, it + 4 < n_it);
                    advance(q_ld);
                }
                auto pack = [&](Operand<kTwo>& po, Operand<kTwo>& dso, const f32x16& pr, const f32x16& ds, int k) __attribute__((always_inline)) {
                    pack8(po, pr, k);
                    pack8(dso, ds, k);
                    asm volatile("" : "+v"(po.hi), "+v"(dso.hi));
                    if constexpr (kTwo) asm volatile("" : "+v"(po.lo), "+v"(dso.lo));
                };
                if (g == kHalf / 2 - 1) pack(pf1[0], dsf1[0], S1, dP1, 0);
                if (g == kHalf - 1) pack(pf1[1], dsf1[1], S1, dP1, 1);
                if (g == kHalf + kHalf / 2 - 1) pack(pfn[0], dsfn[0], Sn0, dPn0, 0);
                if (g == kGroups - 1) pack(pfn[1], dsfn[1], Sn0, dPn0, 1);
                ALCH_SB;
                if (ib == 0) dPn0 = __builtin_amdgcn_mfma_f32_32x32x16_bf16(f.ddo, vf[kk], dPn0, 0, 0, 0);
                else dPn1 = __builtin_amdgcn_mfma_f32_32x32x16_bf16(f.ddo, vf[kk], dPn1, 0, 0, 0);
                ALCH_SB;
            }
        }
        // hand over to the next iteration
        S1 = Sn1; dP1 = dPn1;
#pragma unroll
        for (int ks = 0; ks < 2; ++ks) { pf0[ks] = pfn[ks]; dsf0[ks] = dsfn[ks]; }
        m_cur = m_nxt; m_nxt = m_nn; m_nn = m_n3; m_n3 = m_n4;
        dsc = dsc_next;
    };
    {
        int it = 0;
        for (; it < n_mask && it < n_it; ++it) iteration(std::true_type{}, it);
        for (; it < n_it; ++it) iteration(std::false_type{}, it);
    }
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");

    if constexpr (kTwo) {
        float flag = 0.f;
#pragma unroll
        for (int nb = 0; nb < kNB; ++nb) flag = not_finite(dV[nb], not_finite(dK[nb], flag));
        if (__any(!(flag == 0.f))) {  // formed again from the visible pairs alone (attn_rows.h)
            for (int j = j0; j < min(j0 + 32, len); ++j) {
                HeadRow<__bf16, 1> dk, dv;
                attn_dkv_row(Kb + (long long)j * p.ldk, Vb + (long long)j * p.ldk, p.Q, p.dO, p.O, p.LSE, p.delta, p.Hq, h_first, h_end, p.cu,
                             kPrefix ? p.prefix : nullptr, p.n_seqs, seq, j, kD, p.scale, dk, dv);
                if (parts > 1) {
                    float* row = p.partial + (((long long)part * p.T + seq_start + j) * p.Hkv + kv) * (2 * kD);
                    row[lane] = dk.v[0];
                    row[kD + lane] = dv.v[0];
                } else {
                    const long long at = (long long)(seq_start + j) * p.ldo + kv * kD + lane;
                    p.dK[at] = (__bf16)(rope_backward_row<kD>(dk.v[0], p, seq_start, j, lane) * p.scale);
                    p.dV[at] = (__bf16)dv.v[0];
                }
            }
            return;
        }
    }
    // accumulator element e of block nb: key row j0 + 8*(e>>2) + 4*half + (e&3), column nb*32 + (lane&31)
    if (parts > 1) {
        float* ws = p.partial + (((long long)part * p.T + seq_start) * p.Hkv + kv) * (2 * kD) + (lane & 31);
#pragma unroll
        for (int nb = 0; nb < kNB; ++nb)
#pragma unroll
            for (int e = 0; e < 16; ++e) {
                const int j = j0 + 8 * (e >> 2) + 4 * half + (e & 3);
                if (j < len) {
                    float* row = ws + (long long)j * p.Hkv * (2 * kD) + nb * 32;
                    row[0] = dK[nb][e];
                    row[kD] = dV[nb][e];
                }
            }
        return;
    }
    if (p.rope) rope_backward_rows<kD>(dK, p, seq_start, j0, len, lane);
    __bf16* dKb = p.dK + (long long)seq_start * p.ldo + kv * kD;
    __bf16* dVb = p.dV + (long long)seq_start * p.ldo + kv * kD;
#pragma unroll
    for (int nb = 0; nb < kNB; ++nb)
#pragma unroll
        for (int e = 0; e < 16; ++e) {
            const int j = j0 + 8 * (e >> 2) + 4 * half + (e & 3);
            if (j < len) {
                const long long off = (long long)j * p.ldo + nb * 32 + (lane & 31);
                dKb[off] = (__bf16)(dK[nb][e] * p.scale);
                dVb[off] = (__bf16)dV[nb][e];
            }
        }
}

template <int kD, bool kPrefix>
__global__ __launch_bounds__(256) void k_attn_bwd_dkv_mfma(AttnMfmaParams p) {
    __shared__ __attribute__((aligned(1024))) char smem[4 * AttnTile<kD>::kStageBytes];
    attn_dkv_block<kD, kPrefix>(p, blockIdx.x, blockIdx.y, blockIdx.z, smem);
}

// Sum of the partial dK, dV of the key blocks that were cut (in the order of the parts), RoPE backward, one rounding.
// blockIdx.z: 32 keys of a sequence; kD / 4 threads to a row, four columns of the lower half of dK and their partners
// or eight of dV each.
template <int kD, bool kPrefix>
__global__ __launch_bounds__(256) void k_dkv_finish(AttnMfmaParams p) {
    const int seq = blockIdx.y, kv = blockIdx.x;
    const int seq_start = p.cu[seq], len = p.cu[seq + 1] - seq_start;
    const int row0 = (int)blockIdx.z * 32, kb = row0 / 128;
    if (row0 >= len || len <= p.short_upto) return;
    int tiles = (len + kTileRows - 1) / kTileRows - 2 * kb;
    if constexpr (kPrefix) tiles += prefix_seqs(p, seq).tiles;
    int heads;
    const int parts = dkv_parts(p, p.Hq / p.Hkv, tiles, heads);
    if (parts < 2) return;
    constexpr int kRowThreads = kD / 4;
    const int c = (int)threadIdx.x % kRowThreads;
    const bool is_k = c < kRowThreads / 2;
    // columns c0 .. c0+3 and c1 .. c1+3 of [dK | dV]
    const int c0 = is_k ? 4 * c : kD + 8 * (c - kRowThreads / 2), c1 = is_k ? c0 + kD / 2 : c0 + 4;
    const long long pitch = (long long)p.T * p.Hkv * (2 * kD);
    for (int r = row0 + (int)threadIdx.x / kRowThreads; r < min(row0 + 32, len); r += 256 / kRowThreads) {
        const float* src = p.partial + ((long long)(seq_start + r) * p.Hkv + kv) * (2 * kD);
        f32x4 a = {0.f, 0.f, 0.f, 0.f}, b = a;
        for (int k = 0; k < parts; ++k) {
            a += *reinterpret_cast<const f32x4*>(src + k * pitch + c0);
            b += *reinterpret_cast<const f32x4*>(src + k * pitch + c1);
        }
        if (is_k) {
            if (p.rope) {
                const int pos = p.positions ? p.positions[seq_start + r] : r;
#pragma unroll
                for (int e = 0; e < 4; ++e) {
                    float sn, cs;
                    rope_sincos<kD>((float)pos * rope_theta<kD>(c0 + e, p.rope_log2_base), sn, cs);
                    const float x = a[e], y = b[e];
                    a[e] = x * cs + y * sn;
                    b[e] = y * cs - x * sn;
                }
            }
            a *= p.scale;
            b *= p.scale;
        }
        __bf16* dst = (is_k ? p.dK : p.dV) + (long long)(seq_start + r) * p.ldo + kv * kD - (is_k ? 0 : kD);
        bf16x4 oa, ob;
#pragma unroll
        for (int e = 0; e < 4; ++e) { oa[e] = (__bf16)a[e]; ob[e] = (__bf16)b[e]; }
        *reinterpret_cast<bf16x4*>(dst + c0) = oa;
        *reinterpret_cast<bf16x4*>(dst + c1) = ob;
    }
}

// ---------------------------------------------------------------------------------------------
// dQ
// h: query head, z of n_z: query block, smem: two stages; kWrite: leaves delta and LSE * log2(e) for dK/dV.
template <int kD, bool kWrite>
__device__ __forceinline__ void attn_dq_block(const AttnMfmaParams& p, const int h, const int seq, const int z, const int n_z, char* smem) {
    constexpr int kTileBytes = AttnTile<kD>::kBytes, kStageBytes = AttnTile<kD>::kStageBytes, kRowBytes = AttnTile<kD>::kRowBytes;
    constexpr int kKK = AttnTile<kD>::kKK, kNB = AttnTile<kD>::kNB, kLoads = AttnTile<kD>::kLoads;
    const uint32_t lds0 = (uint32_t)(uintptr_t)ALCH_LDS(smem);
    // (one request for both tables: work-groups of a block or two are a chain of such requests)
    const int* table = p.prefix ? p.prefix : p.cu;
    const int seq_start = p.cu[seq], len = p.cu[seq + 1] - seq_start, named = table[seq], pre = p.prefix ? named : -1;
    // z is the slowest index, so it counts down the keys that a query block meets: its own blocks up to the
    // diagonal and those of its prefix.  By its own blocks alone the responses on a long prompt, the heaviest of all, start
    // last.  As many ranks as the longest sequence has blocks: what lies beyond shares the last ones, and the grid
    // holds no work-group more than without prefixes.  (32/8 heads of 128, two responses to a prompt, us by own blocks / with a
    // rank for every count of keys / so: one prompt of 2048 tokens, responses of 40 132 / 98 / 98; 4 of 1024, 128 142 / 128 /
    // 125; 4 of 1024, 16 137 / 134 / 124; 4 of 300, 100 57 / 56 / 47; 6 of 100, 100 39 / 44 / 41.)
    int qb = n_z - 1 - z, pre_start = 0, pre_len = 0;
    if (pre >= 0) {
        pre_start = p.cu[pre];
        pre_len = p.cu[pre + 1] - pre_start;
        qb -= min((pre_len + 127) / 128, n_z - (len + 127) / 128);
    }
    if (qb < 0 || qb * 128 >= len || len <= p.short_upto) return;
    const int lane = threadIdx.x & 63, half = lane >> 5;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int kv = h / (p.Hq / p.Hkv);
    const int i0 = qb * 128 + wave * 32;  // this wave's first query

    const uint32_t lane_d = frag_d_lane<kD>(lane), lane_r0 = frag_rows_lane<kD>(lane, 0), lane_r1 = frag_rows_lane<kD>(lane, 1);
    uint32_t voff[kLoads];
    tile_voffsets<kD>(voff, p.ldk, wave, lane);
    // key tiles: all tiles of the prefix sequence (if any), then own tiles 0 .. the last one that holds a
    // key <= the work-group's last query
    const int npt = (pre_len + kTileRows - 1) / kTileRows;
    const int last_q = min(qb * 128 + 127, len - 1);
    const int n_it = npt + last_q / kTileRows + 1;
    const float sl2 = p.scale * kLog2e;
    // Buffer descriptors of a tile from scalar arithmetic alone: base of the sequence's K / V plus the tile's byte
    // offset, extent = what is left of the sequence (rows past its end read as zero), both below 2 GiB.
    const long long kv_off = (long long)kv * kD;
    const unsigned long long baseK_own = reinterpret_cast<unsigned long long>(p.K + (long long)seq_start * p.ldk + kv_off);
    const unsigned long long baseV_own = reinterpret_cast<unsigned long long>(p.V + (long long)seq_start * p.ldk + kv_off);
    const unsigned long long baseK_pre = reinterpret_cast<unsigned long long>(p.K + (long long)pre_start * p.ldk + kv_off);
    const unsigned long long baseV_pre = reinterpret_cast<unsigned long long>(p.V + (long long)pre_start * p.ldk + kv_off);
    const unsigned tile_bytes = (unsigned)(kTileRows * p.ldk * 2);   // distance of two tiles
    struct TileSrc { i32x4 k, v; };
    auto desc = [&](unsigned long long base, int rows) {
        const unsigned n = rows > 0 ? (unsigned)(((long long)(min(rows, kTileRows) - 1) * p.ldk + kD) * 2) : 0u;
        i32x4 r;
        r[0] = __builtin_amdgcn_readfirstlane((int)(unsigned)base);
        r[1] = __builtin_amdgcn_readfirstlane((int)((unsigned)(base >> 32) & 0xffffu));
        r[2] = __builtin_amdgcn_readfirstlane((int)n);
        r[3] = 0x00020000;
        return r;
    };
    auto tile_src = [&](int it) {
        const bool in_pre = it < npt;
        const int tile = in_pre ? it : it - npt;
        const int rows = it < n_it ? (in_pre ? pre_len : len) - tile * kTileRows : 0;  // past the last tile: nothing moves
        const unsigned long long off = (unsigned long long)tile * tile_bytes;
        TileSrc t;
        t.k = desc((in_pre ? baseK_pre : baseK_own) + off, rows);
        t.v = desc((in_pre ? baseV_pre : baseV_own) + off, rows);
        return t;
    };
    // load j of a wave's share of tile `it`: kLoads 1 KB pieces of the K tile, kLoads of the V tile
    auto issue_piece = [&](const TileSrc& t, int it, int j) {
        const uint32_t st = lds0 + (uint32_t)(it & 1) * kStageBytes + (j < kLoads ? 0u : (uint32_t)kTileBytes);
        dma16(j < kLoads ? t.k : t.v, st + (uint32_t)(wave * kLoads + j % kLoads) * 1024u, voff[j % kLoads]);
    };
    {   // the first tile is on its way while the Q, dO and O fragments below are fetched
        const TileSrc t0 = tile_src(0);
#pragma unroll
        for (int j = 0; j < 2 * kLoads; ++j) issue_piece(t0, 0, j);
    }
    const __bf16* Qb = p.Q + (long long)seq_start * p.ldq + h * kD;
    const __bf16* dOb = p.dO + (long long)seq_start * p.ldq + h * kD;
    bf16x8 qf[kKK], gf[kKK];
#pragma unroll
    for (int kk = 0; kk < kKK; ++kk) {
        qf[kk] = global_frag_d(Qb, p.ldq, i0, len, kk, lane);
        gf[kk] = global_frag_d(dOb, p.ldq, i0, len, kk, lane);
    }
    const int i = i0 + (lane & 31);  // this lane's query (accumulator column)
    const bool i_ok = i < len;
    const float lse2 = i_ok ? p.LSE[(long long)(seq_start + i) * p.Hq + h] * kLog2e : 0.f;
    if (kWrite && i_ok && half == 0) p.lse2[(long long)(seq_start + i) * p.Hq + h] = lse2;
    // delta_i = sum_d dO[i,d] O[i,d]: each lane holds half of the elements of its query's dO row
    float del = 0.f;
    {
        const __bf16* Ob = p.O + (long long)seq_start * p.ldq + h * kD;
#pragma unroll
        for (int kk = 0; kk < kKK; ++kk) {
            const bf16x8 of = global_frag_d(Ob, p.ldq, i0, len, kk, lane);
#pragma unroll
            for (int e = 0; e < 8; ++e) del += (float)of[e] * (float)gf[kk][e];
        }
        del += __shfl_xor(del, 32, 64);
        if (kWrite && i_ok && half == 0) p.delta[(long long)(seq_start + i) * p.Hq + h] = del;
    }
    const float ndel = -del;
    f32x16 dQ[kNB];
#pragma unroll
    for (int n = 0; n < kNB; ++n)
#pragma unroll
        for (int e = 0; e < 16; ++e) dQ[n][e] = 0.f;

    for (int it = 0; it < n_it; ++it) {
        asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
        __syncthreads();
        {   // the loads of tile it+1 (two waves share a SIMD: while this one queues its loads the other computes)
            const TileSrc tn = tile_src(it + 1);
#pragma unroll
            for (int j = 0; j < 2 * kLoads; ++j) issue_piece(tn, it + 1, j);
        }
        const char* tk = smem + (it & 1) * kStageBytes;
        const char* tv = tk + kTileBytes;
        // keys of this tile count from 0 inside their own sequence; key j is visible to query i when
        // j <= lim: the last prefix key for a prefix tile, i itself (the diagonal) for an own tile
        const bool in_pre = it < npt;
        const int jt = (in_pre ? it : it - npt) * kTileRows;
        const int lim = in_pre ? pre_len - 1 : i, lim0 = in_pre ? pre_len - 1 : i0;
#pragma unroll
        for (int jb = 0; jb < 2; ++jb) {
            const int j0 = jt + jb * 32;
            // a 32-key block wholly above this wavefront's diagonal contributes nothing: skipped (the other
            // wavefronts of the work-group, further down the diagonal, still need the tile)
            if (!in_pre && j0 > i0 + 31) continue;
            const char* bk = tk + jb * 32 * kRowBytes;
            const char* bv = tv + jb * 32 * kRowBytes;
            // transposed: rows = keys, columns = queries.  dP starts from -delta (every element of a lane belongs
            // to the lane's query), so the accumulator comes out as dP - delta
            f32x16 St, dPt;
#pragma unroll
            for (int e = 0; e < 16; ++e) { St[e] = 0.f; dPt[e] = ndel; }
#pragma unroll
            for (int kk = 0; kk < kKK; ++kk) {
                St = __builtin_amdgcn_mfma_f32_32x32x16_bf16(lds_frag_d(bk, lane_d, kk), qf[kk], St, 0, 0, 0);
                dPt = __builtin_amdgcn_mfma_f32_32x32x16_bf16(lds_frag_d(bv, lane_d, kk), gf[kk], dPt, 0, 0, 0);
            }
#pragma unroll
            for (int e = 0; e < 16; ++e) {
                const float pr = __builtin_amdgcn_exp2f(__builtin_fmaf(St[e], sl2, -lse2));
                dPt[e] = pr * dPt[e];
            }
            if (!i_ok || j0 + 31 > lim0) {
#pragma unroll
                for (int e = 0; e < 16; ++e) {
                    const int j = j0 + 8 * (e >> 2) + 4 * half + (e & 3);
                    if (!i_ok || j > lim) dPt[e] = 0.f;
                }
            }
#pragma unroll
            for (int ks = 0; ks < 2; ++ks) {
                // left operand dS[i][j]: row i = lane&31 (this lane's query), k <-> key rows of the accumulator
                Operand<AttnTile<kD>::kTwo> dsf;
                pack8(dsf, dPt, ks);
#pragma unroll
                for (int nb = 0; nb < kNB; ++nb) {
                    const bf16x8 kr = lds_frag_rows<kD>(bk, lane_r0, lane_r1, ks, nb);
                    dQ[nb] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(dsf.hi, kr, dQ[nb], 0, 0, 0);
                    if constexpr (AttnTile<kD>::kTwo) dQ[nb] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(dsf.lo, kr, dQ[nb], 0, 0, 0);
                }
            }
        }
    }

    if constexpr (AttnTile<kD>::kTwo) {
        float flag = 0.f;
#pragma unroll
        for (int nb = 0; nb < kNB; ++nb) flag = not_finite(dQ[nb], flag);
        if (__any(!(flag == 0.f))) {
            for (int r = i0; r < min(i0 + 32, len); ++r) {
                const long long at = (long long)(seq_start + r) * p.ldq + h * kD;
                HeadRow<__bf16, 1> x;
                float del_again;
                attn_dq_row(p.Q + at, p.dO + at, p.O + at, p.K + kv_off, p.V + kv_off, p.ldk, SeenKeys{pre_start, pre_len, seq_start, pre_len + r + 1},
                            kD, p.scale, p.LSE[(long long)(seq_start + r) * p.Hq + h], x, del_again);
                p.dQ[(long long)(seq_start + r) * p.ldo + h * kD + lane] = (__bf16)(rope_backward_row<kD>(x.v[0], p, seq_start, r, lane) * p.scale);
            }
            return;
        }
    }
    if (p.rope) rope_backward_rows<kD>(dQ, p, seq_start, i0, len, lane);
    __bf16* dQb = p.dQ + (long long)seq_start * p.ldo + h * kD;
#pragma unroll
    for (int nb = 0; nb < kNB; ++nb)
#pragma unroll
        for (int e = 0; e < 16; ++e) {
            const int ii = i0 + 8 * (e >> 2) + 4 * half + (e & 3);
            if (ii < len) dQb[(long long)ii * p.ldo + nb * 32 + (lane & 31)] = (__bf16)(dQ[nb][e] * p.scale);
        }
}

template <int kD>
__global__ __launch_bounds__(256, 2) void k_attn_bwd_dq_mfma(AttnMfmaParams p) {
    __shared__ __attribute__((aligned(1024))) char smem[2 * AttnTile<kD>::kStageBytes];
    attn_dq_block<kD, true>(p, blockIdx.x, blockIdx.y, blockIdx.z, gridDim.z, smem);
}

// ---------------------------------------------------------------------------------------------
// Short batches: both gradients in one launch, behind one that forms delta and LSE * log2(e).  A work-group of either is a chain of
// latencies of 12 to 35 us, and where all of both find a compute unit the second need not wait for the first.  All launches of it, with
// delta (5 us) and the sums of cut key blocks (6 to 10): one sequence of 201 tokens, 32/8 heads of 128 57 -> 32 us, 487 tokens 68 -> 49; heads of 64
// 260 tokens 46 -> 28, 100 tokens 39 -> 23.  Layer backward of the 8B shape 201 tokens 425 -> 395 us, 487 636 -> 614; hidden 2048 260 tokens
// 230 -> 209, 100 181 -> 162.
template <int kD>
__global__ __launch_bounds__(256) void k_both_gradients_mfma(AttnMfmaParams p, int n_dkv) {
    __shared__ __attribute__((aligned(1024))) char smem[4 * AttnTile<kD>::kStageBytes];
    const int b = (int)blockIdx.x;
    if (b < n_dkv) {
        attn_dkv_block<kD, false>(p, b % p.Hkv, b / p.Hkv % p.n_seqs, b / (p.Hkv * p.n_seqs), smem);
    } else {
        const int q = b - n_dkv;
        attn_dq_block<kD, false>(p, q % p.Hq, q / p.Hq % p.n_seqs, q / (p.Hq * p.n_seqs), p.n_blocks, smem);
    }
}
// Two lanes to a row of a head, which add in the order of attn_dq_block: the same bits.
template <int kD>
__global__ __launch_bounds__(256) void k_row_delta(AttnMfmaParams p) {
    const long long at = (long long)blockIdx.x * 128 + (threadIdx.x >> 1);  // row of the batch and head
    const int half = threadIdx.x & 1;
    const bool ok = at < (long long)p.T * p.Hq;
    const long long off = (ok ? at / p.Hq * p.ldq + at % p.Hq * kD : 0) + 8 * half;
    float del = 0.f;
#pragma unroll
    for (int kk = 0; kk < AttnTile<kD>::kKK; ++kk) {
        const bf16x8 of = *reinterpret_cast<const bf16x8*>(p.O + off + kk * 16), gf = *reinterpret_cast<const bf16x8*>(p.dO + off + kk * 16);
#pragma unroll
        for (int e = 0; e < 8; ++e) del += (float)of[e] * (float)gf[e];
    }
    del += __shfl_xor(del, 1, 64);
    if (ok && half == 0) {
        p.delta[at] = del;
        p.lse2[at] = p.LSE[at] * kLog2e;
    }
}

// ---------------------------------------------------------------------------------------------
// forward: O = softmax_causal(Q K^T / sqrt(D)) V and LSE, the step of the prefill that produces the
// O and LSE members of the record.  A work-group owns 128 queries of one (sequence, head), 32 per
// wavefront with their Q fragments in registers, and streams 64-key tiles of K and V through LDS.
// Scores are formed transposed (rows = keys, columns = queries) so that a lane owns one query: its
// running maximum, normaliser and the rescaling of its output column are per-lane scalars, and P
// in the accumulator layout is directly the right operand of O^T += V^T P^T.
struct AttnFwdParams {
    const __bf16 *Q, *K, *V;
    __bf16* O;
    float* LSE;
    const int* cu;
    const int* prefix;  // as in the backward
    int seq_begin;      // first sequence whose queries are computed
    int short_upto;     // as in the backward
    int Hq, Hkv;
    long long ldq, ldk;
    float scale;
};

template <int kD>
__global__ __launch_bounds__(256, 2) void k_attn_fwd_mfma(AttnFwdParams p) {
    constexpr int kTileBytes = AttnTile<kD>::kBytes, kStageBytes = AttnTile<kD>::kStageBytes, kRowBytes = AttnTile<kD>::kRowBytes;
    constexpr int kKK = AttnTile<kD>::kKK, kNB = AttnTile<kD>::kNB, kLoads = AttnTile<kD>::kLoads;
    __shared__ __attribute__((aligned(1024))) char smem[2 * kStageBytes];
    const uint32_t lds0 = (uint32_t)(uintptr_t)ALCH_LDS(smem);
    const int seq = p.seq_begin + blockIdx.y, h = blockIdx.x;
    const int seq_start = p.cu[seq], len = p.cu[seq + 1] - seq_start;
    // heaviest (last) query blocks of every sequence and head first: blockIdx.z is the slowest index
    const int qb = (int)gridDim.z - 1 - (int)blockIdx.z;
    if (qb * 128 >= len || len <= p.short_upto) return;
    const int lane = threadIdx.x & 63, half = lane >> 5;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int kv = h / (p.Hq / p.Hkv);
    const int i0 = qb * 128 + wave * 32;

    const __bf16* Qb = p.Q + (long long)seq_start * p.ldq + h * kD;
    bf16x8 qf[kKK];
#pragma unroll
    for (int kk = 0; kk < kKK; ++kk) qf[kk] = global_frag_d(Qb, p.ldq, i0, len, kk, lane);
    const int i = i0 + (lane & 31);
    f32x16 Ot[kNB];  // O^T: block nb holds d = nb*32 + 8b + 4*half + r (register 4b+r) of query i
#pragma unroll
    for (int n = 0; n < kNB; ++n)
#pragma unroll
        for (int e = 0; e < 16; ++e) Ot[n][e] = 0.f;
    float m2 = -INFINITY, l = 0.f;  // running max (log2 domain) and normaliser of this lane's half of the keys
    float m_raw = -INFINITY;        // heads of 64: the running max of the raw scores (m2 is it, scaled and rounded)
    bool rows_again = false;

    const uint32_t lane_d = frag_d_lane<kD>(lane), lane_r0 = frag_rows_lane<kD>(lane, 0), lane_r1 = frag_rows_lane<kD>(lane, 1);
    uint32_t voff[kLoads];
    tile_voffsets<kD>(voff, p.ldk, wave, lane);
    // key tiles: all tiles of the prefix sequence (if any), then the own tiles up to the diagonal; one
    // running maximum and normaliser cover both, so O and LSE are those of the joint softmax
    const int pre = p.prefix ? p.prefix[seq] : -1;
    const int pre_start = pre >= 0 ? p.cu[pre] : 0, pre_len = pre >= 0 ? p.cu[pre + 1] - pre_start : 0;
    const int npt = (pre_len + kTileRows - 1) / kTileRows;
    const int last_q = min(qb * 128 + 127, len - 1);
    const int n_it = npt + last_q / kTileRows + 1;
    const float sl2 = p.scale * kLog2e;

    auto issue = [&](int it) {
        const bool in_pre = it < npt;
        const int row_first = (in_pre ? it : it - npt) * kTileRows;
        const int rows_valid = (in_pre ? pre_len : len) - row_first;
        const long long row = (long long)((in_pre ? pre_start : seq_start) + row_first);
        const uint32_t st = lds0 + (uint32_t)(it & 1) * kStageBytes;
        issue_rows_tile<kD>(p.K + row * p.ldk + kv * kD, p.ldk, rows_valid, st, wave, voff);
        issue_rows_tile<kD>(p.V + row * p.ldk + kv * kD, p.ldk, rows_valid, st + kTileBytes, wave, voff);
    };

    issue(0);
    for (int it = 0; it < n_it; ++it) {
        asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
        __syncthreads();
        if (it + 1 < n_it) issue(it + 1);
        const char* tk = smem + (it & 1) * kStageBytes;
        const char* tv = tk + kTileBytes;
        const bool in_pre = it < npt;
        const int jt = (in_pre ? it : it - npt) * kTileRows;  // first key of the tile inside its own sequence
        const int lim = in_pre ? pre_len - 1 : i;             // last key of the tile's sequence this query sees
        if (!in_pre && jt > i0 + 31) continue;  // wholly above this wave's diagonal
        f32x16 St[2];
#pragma unroll
        for (int jb = 0; jb < 2; ++jb) {
#pragma unroll
            for (int e = 0; e < 16; ++e) St[jb][e] = 0.f;
#pragma unroll
            for (int kk = 0; kk < kKK; ++kk)
                St[jb] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(lds_frag_d(tk + jb * 32 * kRowBytes, lane_d, kk), qf[kk], St[jb], 0, 0, 0);
        }
        // scores; heads of 128 take them to the log2 domain here, heads of 64 inside the exponent, where it costs no rounding
        constexpr bool kTwo = AttnTile<kD>::kTwo;
        if constexpr (!kTwo) {
#pragma unroll
            for (int jb = 0; jb < 2; ++jb)
#pragma unroll
                for (int e = 0; e < 16; ++e) St[jb][e] *= sl2;
        }
        // masked: key j = jt + jb*32 + 8b + 4*half + r must satisfy j <= lim
        if (jt + 63 > (in_pre ? pre_len - 1 : i0)) {
#pragma unroll
            for (int jb = 0; jb < 2; ++jb)
#pragma unroll
                for (int e = 0; e < 16; ++e)
                    if (jt + jb * 32 + 8 * (e >> 2) + 4 * half + (e & 3) > lim) St[jb][e] = -INFINITY;
        }
        float mx = kTwo ? m_raw : m2;
        const float m_old = mx;
#pragma unroll
        for (int jb = 0; jb < 2; ++jb)
#pragma unroll
            for (int e = 0; e < 16; ++e) mx = fmaxf(mx, St[jb][e]);
        mx = fmaxf(mx, __shfl_xor(mx, 32, 64));  // both halves of the wave share the query
        // The vector port bounds the kernel, so the sums are rescaled only where a maximum of the wavefront moved (with the tiles
        // above its diagonal left out: 6 sequences of 5003 tokens, 32/8 heads of 128 82 -> 74 us, 2 of 4096 394 -> 351, heads of
        // 64 283 -> 248, same bits).  A reference that was left behind by up to 2^8, so that hardly a tile rescales, gave another
        // 5 %, and O 2-15 % further from 64 bits: the largest probability of a row is one here, which no rounding changes.
        float alpha = 1.f;
        if (__any(mx > m_old)) {
            if (kTwo) {
                m_raw = mx;
                mx *= sl2;
                asm("" : "+v"(mx));  // (the rounded product everywhere: fused into the differences below, each tile would rescale by its rounding)
            }
            alpha = __builtin_amdgcn_exp2f(m2 - mx);  // 0 on the first tile (m2 = -inf), keys 0.. always valid
            m2 = mx;
#pragma unroll
            for (int n = 0; n < kNB; ++n)
#pragma unroll
                for (int e = 0; e < 16; ++e) Ot[n][e] *= alpha;
        }
        float sum = 0.f;
#pragma unroll
        for (int jb = 0; jb < 2; ++jb)
#pragma unroll
            for (int e = 0; e < 16; ++e) {
                const float pr = __builtin_amdgcn_exp2f(kTwo ? __builtin_fmaf(St[jb][e], sl2, -m2) : St[jb][e] - m2);
                St[jb][e] = pr;
                sum += pr;
            }
        l = l * alpha + sum;
#pragma unroll
        for (int jb = 0; jb < 2; ++jb)
#pragma unroll
            for (int ks = 0; ks < 2; ++ks) {
                Operand<kTwo> pf;  // right operand P^T: column = this lane's query, k <-> key rows
                pack8(pf, St[jb], ks);
#pragma unroll
                for (int nb = 0; nb < kNB; ++nb) {
                    const bf16x8 vr = lds_frag_rows<kD>(tv + jb * 32 * kRowBytes, lane_r0, lane_r1, ks, nb);
                    Ot[nb] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(vr, pf.hi, Ot[nb], 0, 0, 0);
                    if constexpr (kTwo) Ot[nb] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(vr, pf.lo, Ot[nb], 0, 0, 0);
                }
            }
    }
    l += __shfl_xor(l, 32, 64);
    if constexpr (AttnTile<kD>::kTwo) {
        float flag = 0.f;
#pragma unroll
        for (int nb = 0; nb < kNB; ++nb) flag = not_finite(Ot[nb], flag);
        rows_again = __any(!(flag == 0.f));
        if (rows_again)
            for (int r = i0; r < min(i0 + 32, len); ++r) {
                HeadRow<__bf16, 1> o;
                float lse_again;
                attn_fwd_row(Qb + (long long)r * p.ldq, p.K + kv * kD, p.V + kv * kD, p.ldk, SeenKeys{pre_start, pre_len, seq_start, pre_len + r + 1},
                             kD, p.scale, o, lse_again);
                p.O[(long long)(seq_start + r) * p.ldq + h * kD + lane] = (__bf16)o.v[0];
            }
    }
    if (i < len) {
        const float inv = 1.f / l;
        __bf16* orow = p.O + (long long)(seq_start + i) * p.ldq + h * kD;
        if (!rows_again)
#pragma unroll
        for (int nb = 0; nb < kNB; ++nb)
#pragma unroll
            for (int b = 0; b < 4; ++b) {
                bf16x4 o;
#pragma unroll
                for (int r = 0; r < 4; ++r) o[r] = (__bf16)(Ot[nb][4 * b + r] * inv);
                *reinterpret_cast<bf16x4*>(orow + nb * 32 + 8 * b + 4 * half) = o;
            }
        if (half == 0) {
            const long long row = (long long)(seq_start + i) * p.Hq + h;
            if (AttnTile<kD>::kTwo) p.LSE[row] = (float)((double)m2 * 0.6931471805599453 + (double)logf(l));  // (m2 as the exponents had it)
            else p.LSE[row] = (m2 + __builtin_amdgcn_logf(l)) * 0.6931471805599453f;
        }
    }
}

// Which key blocks the dK/dV kernel cuts (max_parts 1: none), and the longest sequence.  A compute unit holds one
// work-group, at about 2 us a tile and 11 us besides, so a launch of few work-groups lasts as long as its longest one:
// blocks beyond 1.2 even shares of all tiles are cut.  The second kernel and the partial sums take 9 us: at least ten
// tiles have to come off the longest block.  With more work-groups than compute units by an eighth the dispatcher, which
// hands them out in a fixed order over the shader engines, fills the chip no better with parts than without.  Measured
// (dK/dV and the sum of the parts, 32/8 heads of 128): one sequence of 512 tokens 62 -> 39 us, 1024 119 -> 54 us, 2048
// 230 -> 159 us, 1239 + 1057 + 705 146 -> 113 us, 4 x 1024 153 -> 144 us; not cut: 8 x 512 96 us (cut: 99), 6001 tokens
// in 7 sequences 166 us (cut: 172 .. 208).  Heads of 64, 5 sequences of 4099 tokens 115 -> 103 us.
inline int plan_dkv_parts(const AttnArgs& a, AttnMfmaParams& p, int& longest) {
    p.max_parts = 1;
    p.part_len = 1 << 30;
    p.partial = nullptr;
    const int G = a.Hq / a.Hkv;
    const size_t part_bytes = (size_t)a.T * a.Hkv * 2 * a.D * sizeof(float);
    const int* cu = a.cu_seqlens_host;
    int child[kMaxPrefixSeqs];  // tiles of the sequences that name this one (batches with prefixes have no more sequences)
    if (a.prefix_host) {
        std::fill(child, child + a.n_seqs, 0);
        for (int s = 0; s < a.n_seqs; ++s)
            if (a.prefix_host[s] >= 0) child[a.prefix_host[s]] += ceil_div(cu[s + 1] - cu[s], kTileRows);
    }
    long long total = 0, most = 0, n_blocks = 0;
    for (int s = 0; s < a.n_seqs; ++s) {
        const int len = cu[s + 1] - cu[s];
        if (len == 0) continue;
        longest = std::max(longest, len);
        const long long tiles = ceil_div(len, kTileRows), blocks = ceil_div(len, 128), more = a.prefix_host ? child[s] : 0;
        total += blocks * (tiles + more) - blocks * (blocks - 1);  // sum over its blocks of tiles - 2 kb + more
        most = std::max(most, tiles + more);
        n_blocks += blocks;
    }
    int n_cu = 0;
    ALCH_TRY(compute_units(&n_cu));
    const long long part_len = std::max<long long>(total * G * a.Hkv * 6 / 5 / n_cu, kMinPartTiles);
    if (!a.scratch || part_bytes == 0 || n_blocks * a.Hkv > n_cu + n_cu / 8 || most * G < part_len + 10) return ALCH_OK;
    const int max_parts = (int)std::min<size_t>(std::min(G, 8), a.scratch_bytes / part_bytes);
    if (max_parts < 2 || (long long)p.n_blocks * max_parts > kMaxGridBlocks) return ALCH_OK;
    p.max_parts = max_parts;
    p.part_len = (int)part_len;
    p.partial = static_cast<float*>(a.scratch);
    return ALCH_OK;
}

// Whether both gradients run as one launch (k_both_gradients_mfma): where every work-group of both finds a compute unit, and the
// launch and those behind it come out shorter than one behind the other.  The gain has run out where the units do: layers, 70B shape 320 tokens
// 1524 -> 1504 us, 384 (the last) 1607 -> 1593, 5120/17920 512 880 -> 858, 640 (the last) 1026 -> 1028, 8B shape 640 706 -> 695, 768 (the last) 799 ->
// 795, hidden 2048 640 322 -> 308, 768 (the last) 350 -> 352.  Key blocks are cut as finely as the units that are left
// allow, into parts of two tiles at least, if five tiles or more come off the longest: 10 us for the 9 of the sums.  (Parts of four, if eight
// come off -> so, layers, us: heads of 64, 100 tokens 169 -> 159, 3 sequences of 100 216 -> 210; 8B shape 128 tokens 332 -> 328, 150 362 -> 354,
// 2 sequences of 125 405 -> 399; 201 and 256 tokens as before.)
inline int plan_both(const AttnArgs& a, AttnMfmaParams& p, bool& both) {
    both = false;
    if (a.prefix) return ALCH_OK;
    int n_cu = 0;
    ALCH_TRY(compute_units(&n_cu));
    const int* cu = a.cu_seqlens_host;
    const int G = a.Hq / a.Hkv;
    long long blocks = 0;
    int longest = 0;
    for (int s = 0; s < a.n_seqs; ++s) {
        const int len = cu[s + 1] - cu[s];
        blocks += ceil_div(len, 128);
        if (blocks * (a.Hq + a.Hkv) > n_cu) return ALCH_OK;
        longest = std::max(longest, len);
    }
    AttnMfmaParams apart = p, one = p;
    // work-groups of both, and tiles of the longest of dK/dV (as dkv_parts)
    struct Size { long long groups; int tiles; };
    const auto size = [&](const AttnMfmaParams& q) {
        Size z{blocks * a.Hq, 0};
        for (int s = 0; s < a.n_seqs; ++s) {
            const int len = cu[s + 1] - cu[s];
            for (int kb = 0; kb * 128 < len; ++kb) {
                const int tiles = ceil_div(len, kTileRows) - 2 * kb;
                const int want = (int)std::min<long long>(q.max_parts, ((long long)G * tiles + q.part_len - 1) / q.part_len);
                const int heads = ceil_div(G, std::max(want, 1));
                z.groups += ceil_div(G, heads) * a.Hkv;
                z.tiles = std::max(z.tiles, heads * tiles);
            }
        }
        return z;
    };
    int unused = 0;
    ALCH_TRY(plan_dkv_parts(a, apart, unused));
    const Size before = size(apart);
    Size now = before;
    one.n_blocks = ceil_div(longest, 128);
    one.max_parts = apart.max_parts; one.part_len = apart.part_len; one.partial = apart.partial;
    if (!a.keep_parts) {
        one.max_parts = 1;
        one.part_len = 1 << 30;
        now = size(one);
        const size_t part_bytes = (size_t)a.T * a.Hkv * 2 * a.D * sizeof(float);
        const int max_parts = a.scratch && part_bytes ? (int)std::min<size_t>(std::min(G, 8), a.scratch_bytes / part_bytes) : 1;
        for (int part_len = 2; max_parts > 1 && part_len + 5 <= now.tiles; ++part_len) {
            AttnMfmaParams q = one;
            q.max_parts = max_parts;
            q.part_len = part_len;
            const Size z = size(q);
            if (z.groups > n_cu) continue;
            if (z.tiles + 5 > now.tiles) break;
            q.partial = static_cast<float*>(a.scratch);
            one = q;
            now = z;
            break;
        }
    }
    // us (see plan_dkv_parts; dQ: 2.5 a tile and 10; delta: 5)
    const int sums = 9, dq = 10 + 5 * ceil_div(longest, kTileRows) / 2;
    const int together = 5 + std::max(dq, 11 + 2 * now.tiles) + (one.max_parts > 1 ? sums : 0);
    const int behind = dq + 11 + 2 * before.tiles + (apart.max_parts > 1 ? sums : 0);
    if (now.groups > n_cu || together >= behind) return ALCH_OK;
    both = true;
    p = one;
    return ALCH_OK;
}

template <int kD>
int attn_bwd_mfma(const AttnArgs& a, hipStream_t stream) {
    AttnMfmaParams p{};
    p.Q = (const __bf16*)a.Q; p.K = (const __bf16*)a.K; p.V = (const __bf16*)a.V; p.dO = (const __bf16*)a.dO;
    p.O = (const __bf16*)a.O; p.LSE = a.LSE; p.delta = a.delta; p.lse2 = a.delta + (size_t)a.T * a.Hq;
    p.positions = a.positions; p.rope = a.rope_base > 0.f; p.rope_log2_base = p.rope ? log2f(a.rope_base) : 0.f;
    p.dQ = (__bf16*)a.dQ; p.dK = (__bf16*)a.dK; p.dV = (__bf16*)a.dV;
    p.cu = a.cu_seqlens; p.prefix = a.prefix; p.n_seqs = a.n_seqs; p.Hq = a.Hq; p.Hkv = a.Hkv;
    p.ldq = (long long)a.Hq * a.D; p.ldk = (long long)a.Hkv * a.D; p.ldo = a.ld_dqkv;
    p.scale = 1.0f / sqrtf((float)a.D);
    const int nb = (int)(((long long)a.max_seqlen + 127) / 128);
    if (nb <= 0 || a.n_seqs <= 0) return ALCH_OK;
    if (nb > kMaxGridBlocks || a.n_seqs > kMaxGridSeqs) return fail(ALCH_ERR_UNSUPPORTED, "attention: more than 65535 sequences or 128-token blocks");
    p.T = a.T;
    p.n_blocks = nb;
    p.short_upto = a.rows.up_to;
    bool both;
    ALCH_TRY(plan_both(a, p, both));
    if (both) {
        const int n_dkv = a.Hkv * a.n_seqs * p.n_blocks * p.max_parts, n_dq = a.Hq * a.n_seqs * p.n_blocks;
        k_row_delta<kD><<<(unsigned)ceil_div((long long)a.T * a.Hq, 128LL), 256, 0, stream>>>(p);
        if (n_dkv + n_dq > 0) k_both_gradients_mfma<kD><<<n_dkv + n_dq, 256, 0, stream>>>(p, n_dkv);
        if (p.max_parts > 1) k_dkv_finish<kD, false><<<dim3(a.Hkv, a.n_seqs, p.n_blocks * 4), 256, 0, stream>>>(p);
        ALCH_HIP_TRY(hipGetLastError());
        return ALCH_OK;
    }
    int longest = 0;
    ALCH_TRY(plan_dkv_parts(a, p, longest));
    const bool cut = p.max_parts > 1;
    k_attn_bwd_dq_mfma<kD><<<dim3(a.Hq, a.n_seqs, nb), 256, 0, stream>>>(p);   // also writes delta
    const dim3 grid(a.Hkv, a.n_seqs, nb * p.max_parts), grid_finish(a.Hkv, a.n_seqs, ceil_div(longest, 32));
    if (a.prefix) {
        k_attn_bwd_dkv_mfma<kD, true><<<grid, 256, 0, stream>>>(p);
        if (cut) k_dkv_finish<kD, true><<<grid_finish, 256, 0, stream>>>(p);
    } else {
        k_attn_bwd_dkv_mfma<kD, false><<<grid, 256, 0, stream>>>(p);
        if (cut) k_dkv_finish<kD, false><<<grid_finish, 256, 0, stream>>>(p);
    }
    ALCH_HIP_TRY(hipGetLastError());
    return ALCH_OK;
}

template <int kD>
int attn_fwd_mfma(const void* Q, const void* K, const void* V, void* O, float* LSE, int n_seqs, int max_seqlen,
                  const int* cu_seqlens, const int* prefix, int seq_begin, int Hq, int Hkv, int short_upto, hipStream_t stream) {
    AttnFwdParams p;
    p.short_upto = short_upto;
    p.Q = (const __bf16*)Q; p.K = (const __bf16*)K; p.V = (const __bf16*)V; p.O = (__bf16*)O; p.LSE = LSE;
    p.cu = cu_seqlens; p.prefix = prefix; p.seq_begin = seq_begin;
    p.Hq = Hq; p.Hkv = Hkv; p.ldq = (long long)Hq * kD; p.ldk = (long long)Hkv * kD;
    p.scale = 1.0f / sqrtf((float)kD);
    const int nb = (int)(((long long)max_seqlen + 127) / 128);
    if (nb <= 0 || n_seqs <= 0) return ALCH_OK;
    if (nb > kMaxGridBlocks || n_seqs > kMaxGridSeqs) return fail(ALCH_ERR_UNSUPPORTED, "attention: more than 65535 sequences or 128-token blocks");
    k_attn_fwd_mfma<kD><<<dim3(Hq, n_seqs - seq_begin, nb), 256, 0, stream>>>(p);
    ALCH_HIP_TRY(hipGetLastError());
    return ALCH_OK;
}

}  // namespace alch
