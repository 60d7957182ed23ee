// Capture/pack: mask scan and row gather (Section 4.1 of the paper: only the tokens of the
// prefill that are to be trained on are recorded; Section 5: one record per layer).
//
// Batches of up to 4096 tokens take one launch for scan and gather.  The scan of longer ones is one kernel for batches
// of up to 262,144 tokens, and beyond that four small kernels over the byte mask (per-block popcount, scan of the block
// counts, index fill, per-sequence counts) with the block counts in caller-provided scratch; the gather runs one
// work-group per kept row, moving 16 bytes per lane per access.  Everything is bit-exact and
// deterministic: the output order is the ascending token order.
#include "common.h"
#include "kernels.h"

namespace alch {

static constexpr int kTokPerThread = 16;
static constexpr int kScanThreads = 256;
static constexpr int kTokPerBlock = kTokPerThread * kScanThreads;  // 4096
// Up to so many rows a call of at most 4096 tokens has a work-group per row and stream instead of one per row.  Six streams,
// whole call: 250 rows 19.3 against 19.5 us, 500 rows 21.1 against 19.9, 2000 rows 59.3 against 58.3.
static constexpr int kSmallRows = 256;

// 0x80 in every byte of w that is not zero
__device__ __forceinline__ uint32_t nonzero_flags(uint32_t w) { return (((w & 0x7f7f7f7fu) + 0x7f7f7f7fu) | w) & 0x80808080u; }

__device__ __forceinline__ int nonzero_bytes16(const uint8_t* __restrict__ mask, int t0, int T, uint32_t& bits) {
    // bits: bit i set <=> mask[t0+i] != 0 (tokens beyond T count as dropped)
    bits = 0;
    if (t0 + kTokPerThread <= T) {
        uint4 v = *reinterpret_cast<const uint4*>(mask + t0);
        uint32_t w[4] = {v.x, v.y, v.z, v.w};
#pragma unroll
        for (int i = 0; i < 4; ++i)  // the flags of four bytes, moved together by one multiplication
            bits |= ((((nonzero_flags(w[i]) >> 7) * 0x01020408u) >> 24) & 0xfu) << (4 * i);
    } else {
        for (int i = 0; i < kTokPerThread; ++i)
            if (t0 + i < T && mask[t0 + i] != 0) bits |= 1u << i;
    }
    return __popc(bits);
}

__device__ __forceinline__ int wave_inclusive_scan(int v) {
    const int lane = threadIdx.x & 63;
#pragma unroll
    for (int d = 1; d < 64; d <<= 1) {
        int o = __shfl_up(v, d, 64);
        if (lane >= d) v += o;
    }
    return v;
}

// Exclusive scan of one int per thread over a block of kScanThreads; returns the exclusive
// prefix, writes the block total to `total`.
__device__ __forceinline__ int block_exclusive_scan(int v, int& total) {
    __shared__ int wave_sum[kScanThreads / 64];
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    int inc = wave_inclusive_scan(v);
    if (lane == 63) wave_sum[wave] = inc;
    __syncthreads();
    int before = 0, tot = 0;
#pragma unroll
    for (int w = 0; w < kScanThreads / 64; ++w) {
        int s = wave_sum[w];
        if (w < wave) before += s;
        tot += s;
    }
    total = tot;
    __syncthreads();
    return before + inc - v;
}

__global__ __launch_bounds__(kScanThreads) void k_pack_count(const uint8_t* __restrict__ mask, int T,
                                                             int* __restrict__ block_counts) {
    uint32_t bits;
    int c = nonzero_bytes16(mask, (blockIdx.x * kScanThreads + threadIdx.x) * kTokPerThread, T, bits);
    int total;
    block_exclusive_scan(c, total);
    if (threadIdx.x == 0) block_counts[blockIdx.x] = total;
}

// One block: exclusive scan of the block counts in place -> block offsets; n_kept and overflow flag.
__global__ __launch_bounds__(kScanThreads) void k_pack_scan_blocks(int* __restrict__ block_counts, int nblocks,
                                                                   int* __restrict__ n_kept_and_status,
                                                                   long long capacity) {
    int carry = 0;
    for (int base = 0; base < nblocks; base += kScanThreads) {
        int i = base + threadIdx.x;
        int v = i < nblocks ? block_counts[i] : 0;
        int total;
        int ex = block_exclusive_scan(v, total);
        if (i < nblocks) block_counts[i] = carry + ex;
        carry += total;
    }
    if (threadIdx.x == 0) {
        n_kept_and_status[0] = carry;
        n_kept_and_status[1] = (long long)carry > capacity ? 1 : 0;
    }
}

__global__ __launch_bounds__(kScanThreads) void k_pack_fill(const uint8_t* __restrict__ mask, int T,
                                                            const int* __restrict__ block_offsets,
                                                            int* __restrict__ kept_index, long long capacity) {
    uint32_t bits;
    const int t0 = (blockIdx.x * kScanThreads + threadIdx.x) * kTokPerThread;
    int c = nonzero_bytes16(mask, t0, T, bits);
    int total;
    long long pos = (long long)block_offsets[blockIdx.x] + block_exclusive_scan(c, total);
    while (bits) {
        int i = __ffs(bits) - 1;
        bits &= bits - 1;
        if (pos < capacity) kept_index[pos] = t0 + i;
        ++pos;
    }
}

// One wave per sequence boundary: cu_kept[s] = kept tokens before token cu_seqlens[s].
__global__ __launch_bounds__(64) void k_pack_cu(const uint8_t* __restrict__ mask, const int* __restrict__ cu_seqlens,
                                                int n_bounds, const int* __restrict__ block_offsets, int nblocks,
                                                const int* __restrict__ n_kept_and_status,
                                                int* __restrict__ cu_kept) {
    const int s = blockIdx.x;
    if (s >= n_bounds) return;
    const int end = cu_seqlens[s];
    const int blk = end / kTokPerBlock;
    int count = 0;
    for (int t = blk * kTokPerBlock + threadIdx.x; t < end; t += 64) count += mask[t] != 0;
#pragma unroll
    for (int d = 32; d > 0; d >>= 1) count += __shfl_down(count, d, 64);
    if (threadIdx.x == 0) cu_kept[s] = (blk < nblocks ? block_offsets[blk] : n_kept_and_status[0]) + count;
}

// ---- the whole scan in one launch, for batches of up to kOneLaunchTokens tokens ------------------------
// One work-group per 4096 tokens.  Each counts all of the mask before its tokens by itself (the masks of a prefill batch
// are tens of kilobytes, read from L2), so that nothing is handed from one to the next; then it writes the indices of its
// kept tokens and cu_kept of the sequence boundaries among them.  Bound by latency: the last work-group's loads, four in
// flight.  70,001 tokens: 22 -> 6 us against one work-group for the whole mask, 32,768: 9.5 -> 8 us.  Every work-group
// reads what lies before it, so at some length the four launches of the general path are the shorter way.
static constexpr int kOneLaunchTokens = 1 << 18;

__global__ __launch_bounds__(kScanThreads) void k_pack_scan(const uint8_t* __restrict__ mask, int T,
                                                            const int* __restrict__ cu_seqlens, int n_bounds,
                                                            int* __restrict__ kept_index, int* __restrict__ cu_kept,
                                                            int* __restrict__ n_kept_and_status, long long capacity) {
    __shared__ int prefix[kScanThreads];            // kept tokens before each thread's sixteen
    __shared__ unsigned short kept_bits[kScanThreads];  // and which of these are kept
    const int tid = threadIdx.x, block0 = blockIdx.x * kTokPerBlock, t0 = block0 + tid * kTokPerThread;
    int count = 0;
#pragma unroll 4
    for (int b = 0; b < (int)blockIdx.x; ++b) {
        const uint4 v = *reinterpret_cast<const uint4*>(mask + b * kTokPerBlock + tid * kTokPerThread);
        count += __popc(nonzero_flags(v.x)) + __popc(nonzero_flags(v.y)) + __popc(nonzero_flags(v.z)) + __popc(nonzero_flags(v.w));
    }
    uint32_t bits;
    const int own = nonzero_bytes16(mask, t0, T, bits);
    int before, total;
    block_exclusive_scan(count, before);
    int ex = before + block_exclusive_scan(own, total);
    prefix[tid] = ex;
    kept_bits[tid] = (unsigned short)bits;
    if (tid == 0 && blockIdx.x == gridDim.x - 1) {
        n_kept_and_status[0] = before + total;
        n_kept_and_status[1] = (long long)(before + total) > capacity ? 1 : 0;
    }
    __syncthreads();
    // boundaries among this work-group's tokens; what lies at or behind the end of the last one's is its own too
    for (int s = tid; s < n_bounds; s += kScanThreads) {
        const int end = cu_seqlens[s];
        if (end / kTokPerBlock != (int)blockIdx.x && !(blockIdx.x == gridDim.x - 1 && end >= block0 + kTokPerBlock)) continue;
        int c = before + total;
        if (end < block0 + kTokPerBlock) {
            const int owner = (end - block0) / kTokPerThread;
            c = prefix[owner] + __popc(kept_bits[owner] & ((1u << ((end - block0) % kTokPerThread)) - 1u));
        }
        cu_kept[s] = c;
    }
    while (bits) {
        const int i = __ffs(bits) - 1;
        bits &= bits - 1;
        if (ex < capacity) kept_index[ex] = t0 + i;
        ++ex;
    }
}

// ---- gather ---------------------------------------------------------------------------

typedef unsigned int u32x4 __attribute__((ext_vector_type(4)));

struct GatherArgs {
    const char* src[kMaxStreamsPerLaunch];
    char* dst[kMaxStreamsPerLaunch];
    unsigned long long row_bytes[kMaxStreamsPerLaunch];
    unsigned long long src_stride[kMaxStreamsPerLaunch];
    int n;
};

// Row t of stream k to row r of its destination, by the whole work-group.
template <typename V>
__device__ __forceinline__ void copy_row(const GatherArgs& a, int k, long long t, long long r) {
    constexpr unsigned long long kStep = 256ull * sizeof(V);
    const unsigned long long rb = a.row_bytes[k];
    const char* __restrict__ s = a.src[k] + (unsigned long long)t * a.src_stride[k];
    char* __restrict__ d = a.dst[k] + (unsigned long long)r * rb;
    unsigned long long off = (unsigned long long)threadIdx.x * sizeof(V);
    // two independent accesses in flight per lane; non-temporal both ways (nothing is reused)
    for (; off + kStep < rb; off += 2 * kStep) {
        V v0 = __builtin_nontemporal_load(reinterpret_cast<const V*>(s + off));
        V v1 = __builtin_nontemporal_load(reinterpret_cast<const V*>(s + off + kStep));
        __builtin_nontemporal_store(v0, reinterpret_cast<V*>(d + off));
        __builtin_nontemporal_store(v1, reinterpret_cast<V*>(d + off + kStep));
    }
    for (; off < rb; off += kStep) {
        V v = __builtin_nontemporal_load(reinterpret_cast<const V*>(s + off));
        __builtin_nontemporal_store(v, reinterpret_cast<V*>(d + off));
    }
}

// One work-group per kept row (the grid is sized for the most rows the call can produce; work-groups
// beyond n_kept leave at once).  Letting the hardware dispatcher hand out rows measured faster than a
// persistent grid: the rows of the wide streams are long enough to keep every lane busy.
template <typename V>
__global__ __launch_bounds__(256) void k_pack_gather(GatherArgs a, const int* __restrict__ kept_index,
                                                     const int* __restrict__ n_kept_and_status,
                                                     long long capacity) {
    long long n_rows = n_kept_and_status[0];
    if (n_rows > capacity) n_rows = capacity;
    for (long long r = blockIdx.x; r < n_rows; r += gridDim.x)
        for (int k = 0; k < a.n; ++k) copy_row<V>(a, k, kept_index[r], r);
}

// Scan and gather of a batch of at most 4096 tokens in one launch: every work-group finds its row's token in the mask by
// itself (a 16-byte load a thread and a block scan, about 1 us), the first one writes the counts.  One prompt of 317
// tokens, 79 of them kept: bound by launches and by the chain of loads of a row, so blockIdx.y may deal out the streams
// of a row.
template <typename V>
__global__ __launch_bounds__(kScanThreads) void k_pack_small(GatherArgs a, const uint8_t* __restrict__ mask, int T,
                                                             const int* __restrict__ cu_seqlens, int n_bounds,
                                                             int* __restrict__ kept_index, int* __restrict__ cu_kept,
                                                             int* __restrict__ n_kept_and_status, long long capacity) {
    __shared__ int token;
    __shared__ int prefix[kScanThreads];
    __shared__ unsigned short kept_bits[kScanThreads];
    uint32_t bits;
    const int tid = threadIdx.x, c = nonzero_bytes16(mask, tid * kTokPerThread, T, bits);
    int total;
    const int ex = block_exclusive_scan(c, total), r = blockIdx.x;
    const bool first = blockIdx.x == 0 && blockIdx.y == 0;
    if (first) {
        prefix[tid] = ex;
        kept_bits[tid] = (unsigned short)bits;
    }
    if (r >= ex && r < ex + c) {
        for (int i = ex; i < r; ++i) bits &= bits - 1;
        token = tid * kTokPerThread + __ffs(bits) - 1;
        if (blockIdx.y == 0 && r < capacity) kept_index[r] = token;
    }
    __syncthreads();
    if (first) {
        if (tid == 0) {
            n_kept_and_status[0] = total;
            n_kept_and_status[1] = (long long)total > capacity ? 1 : 0;
        }
        for (int s = tid; s < n_bounds; s += kScanThreads) {
            const int end = cu_seqlens[s], owner = end / kTokPerThread;
            int n = total;
            if (owner < kScanThreads) n = prefix[owner] + __popc(kept_bits[owner] & ((1u << (end % kTokPerThread)) - 1u));
            cu_kept[s] = n;
        }
    }
    if (r >= total || r >= capacity) return;
    for (int k = blockIdx.y; k < a.n; k += gridDim.y) copy_row<V>(a, k, token, r);
}

size_t pack_workspace_bytes(int total_tokens) {
    int nblocks = ceil_div(total_tokens > 0 ? total_tokens : 1, kTokPerBlock);
    return round_up((size_t)nblocks * sizeof(int), 256) + 256;
}

// Streams base .. of a call, at most kMaxStreamsPerLaunch of them; false: some row is not made of aligned 16-byte pieces.
static bool gather_args(GatherArgs& a, int n_streams, const alch_stream* streams, int base) {
    a.n = n_streams - base < kMaxStreamsPerLaunch ? n_streams - base : kMaxStreamsPerLaunch;
    bool vec16 = true;
    for (int k = 0; k < a.n; ++k) {
        const alch_stream& s = streams[base + k];
        a.src[k] = static_cast<const char*>(s.src);
        a.dst[k] = static_cast<char*>(s.dst);
        a.row_bytes[k] = s.row_bytes;
        a.src_stride[k] = s.src_row_stride_bytes;
        vec16 = vec16 && aligned16(s.src) && aligned16(s.dst) && s.row_bytes % 16 == 0 && s.src_row_stride_bytes % 16 == 0;
    }
    return vec16;
}

int launch_pack(const uint8_t* mask, int T, const int* cu_seqlens, int n_seqs, int n_streams,
                const alch_stream* streams, long long capacity, int* kept_index, int* cu_kept,
                int* n_kept_and_status, void* workspace, hipStream_t stream, bool traced) {
    int* block_offsets = static_cast<int*>(workspace);
    const int nblocks = T > 0 ? ceil_div(T, kTokPerBlock) : 0;
    const long long max_rows = (long long)T < capacity ? (long long)T : capacity;
    if (T <= kTokPerBlock && max_rows > 0 && n_streams > 0 && n_streams <= kMaxStreamsPerLaunch) {
        double row_bytes_rw = 0;
        for (int k = 0; k < n_streams; ++k) row_bytes_rw += 2.0 * (double)streams[k].row_bytes;
        TraceScope ts(traced ? kTracePackGather : kTraceRowOps, 0.0, row_bytes_rw, stream);
        GatherArgs a;
        const bool vec16 = gather_args(a, n_streams, streams, 0);
        const dim3 grid((unsigned)max_rows, max_rows <= kSmallRows ? n_streams : 1);
        if (vec16)
            k_pack_small<u32x4><<<grid, kScanThreads, 0, stream>>>(a, mask, T, cu_seqlens, n_seqs + 1, kept_index, cu_kept,
                                                                   n_kept_and_status, capacity);
        else
            k_pack_small<unsigned int><<<grid, kScanThreads, 0, stream>>>(a, mask, T, cu_seqlens, n_seqs + 1, kept_index, cu_kept,
                                                                          n_kept_and_status, capacity);
        ALCH_HIP_TRY(hipGetLastError());
        return ALCH_OK;
    }
    if (T <= kOneLaunchTokens) {
        TraceScope ts(traced ? kTracePackScan : kTraceRowOps, 0.0, (double)T + 4.0 * (n_seqs + 1), stream);
        k_pack_scan<<<nblocks > 0 ? nblocks : 1, kScanThreads, 0, stream>>>(mask, T, cu_seqlens, n_seqs + 1, kept_index, cu_kept,
                                                                            n_kept_and_status, capacity);
    } else {
        TraceScope ts(traced ? kTracePackScan : kTraceRowOps, 0.0, (double)T + 4.0 * (n_seqs + 1), stream);
        k_pack_count<<<nblocks, kScanThreads, 0, stream>>>(mask, T, block_offsets);
        k_pack_scan_blocks<<<1, kScanThreads, 0, stream>>>(block_offsets, nblocks, n_kept_and_status, capacity);
        k_pack_fill<<<nblocks, kScanThreads, 0, stream>>>(mask, T, block_offsets, kept_index, capacity);
        k_pack_cu<<<n_seqs + 1, 64, 0, stream>>>(mask, cu_seqlens, n_seqs + 1, block_offsets, nblocks,
                                                  n_kept_and_status, cu_kept);
    }
    ALCH_HIP_TRY(hipGetLastError());
    return launch_pack_gather(T, n_streams, streams, capacity, kept_index, n_kept_and_status, stream, traced);
}

// The gather alone, from an index and a row count already on the device.
int launch_pack_gather(int T, int n_streams, const alch_stream* streams, long long capacity, const int* kept_index,
                       const int* n_kept_and_status, hipStream_t stream, bool traced) {
    if (T == 0 || capacity == 0) return ALCH_OK;

    // traced bytes of the gather: per kept row (read once + written once); the row count is on the device
    double row_bytes_rw = 0;
    for (int k = 0; k < n_streams; ++k) row_bytes_rw += 2.0 * (double)streams[k].row_bytes;
    TraceScope ts(traced ? kTracePackGather : kTraceRowOps, 0.0, row_bytes_rw, stream);

    long long max_rows = (long long)T < capacity ? (long long)T : capacity;
    int grid = (int)(max_rows < (long long)kGatherGridMax ? max_rows : (long long)kGatherGridMax);
    for (int base = 0; base < n_streams; base += kMaxStreamsPerLaunch) {
        GatherArgs a;
        if (gather_args(a, n_streams, streams, base))
            k_pack_gather<u32x4><<<grid, 256, 0, stream>>>(a, kept_index, n_kept_and_status, capacity);
        else
            k_pack_gather<unsigned int><<<grid, 256, 0, stream>>>(a, kept_index, n_kept_and_status, capacity);
    }
    ALCH_HIP_TRY(hipGetLastError());
    return ALCH_OK;
}

}  // namespace alch
