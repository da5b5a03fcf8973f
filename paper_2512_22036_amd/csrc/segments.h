// Segment-descriptor engine kernels: variable-size segments described by (offset, size) lists.
#ifndef FUSCO_CSRC_SEGMENTS_H
#define FUSCO_CSRC_SEGMENTS_H

#include "common.h"
#include "movers.h"

namespace {

// ------------------------------------------------------------------------------------------
// Segment-descriptor engine: segments of any size (multiples of 16 bytes) described by
// (offset, size) lists.  The active segment of a stream position is found from the cumulative
// bytes, as in the paper's dense descriptor arrays.
// ------------------------------------------------------------------------------------------
constexpr int kScanThreads = 256;
constexpr int kScanItems = 8;                            // descriptors per thread
constexpr int kScanChunk = kScanThreads * kScanItems;    // descriptors per workgroup
// Up to kScanSingleMax descriptors are scanned by one workgroup (3000: 3.7 us, 4.1 by two; 6000: 7.4 us), up to kScanDirectMax in one
// launch of workgroups that have kScanDirectThreads x kScanDirectItems each, more in two launches.
constexpr int kScanSingleThreads = 1024, kScanSingleMax = 3 * kScanSingleThreads;
constexpr int kScanDirectThreads = 1024, kScanDirectItems = 2, kScanDirectChunk = kScanDirectThreads * kScanDirectItems;
constexpr int kScanDirectMax = 32768;
constexpr int kSegThreads = 256;        // threads of a workgroup of the copy kernel
constexpr int kSegPieceBytes = 4096;    // stream bytes handled by one of its waves
constexpr int kSegUnits = kSegPieceBytes / 16 / kWave;   // 16-byte units per thread
constexpr int kSegBlockBytes = kSegThreads / kWave * kSegPieceBytes;   // stream bytes handled by a workgroup
constexpr int kSegRunBytes = 8 * kSegBlockBytes;                       // consecutive bytes taken by one XCD
// With slices a workgroup adds what it has written to the slice's counter, and additions to one counter follow one another some 150 ns
// apart: 64 workgroups of 256 threads per MiB kept a slice open longer than its bytes.  Slices in whole blocks of workgroups of kSegWideThreads are taken by
// those: of kSegWideSlice and more, streams below kSegWideBytes aside, and of kSegWideShort and more in streams of kSegWideLong and more.  Pack, us, 256 / 512 / 1024
// threads: slices of 1 MiB, 0.3 MB 6.4 / 6.6 / 7.3, 21 MB 20.7 / 15.0 / 16.2, 36 MB 28.8 / 21.8 / 21.4, 286 MB 125 / 115 / 115, of 4 MiB 286 MB 158 / 121 / 116, of
// 256 KiB 411 MB 176 / 170 / 178, of 32 KiB 36 MB 18.4 / 19.0 / 18.8.  256 / 512 threads over the same buffers, and over buffers that change: slices of 256 KiB 6 MB
// 9.4 / 9.3, 9.5 / 9.4, 12 MB 10.8 / 9.5, 11.2 / 10.4, 40 MB 20.5 / 19.5, 24.1 / 23.8; of 128 KiB 18 MB 10.5 / 11.6, 12.7 / 13.6, 40 MB 19.3 / 19.6, 23.4 / 23.9, 100
// MB 40.4 / 39.5, 45.3 / 44.5, 250 MB 96.4 / 94.5, 107.3 / 104.5; of 64 KiB 18 MB 10.3 / 11.4, 12.8 / 13.6, 40 MB 18.9 / 19.7, 23.1 / 23.6, 100 MB 39.6 / 39.5, 44.7 /
// 44.5.  (A counter per wave: 286 MB 280; two blocks by one workgroup, whose second lookups wait behind the first stores: 161.)
constexpr int kSegWideThreads = 2 * kSegThreads, kSegWideBlockBytes = 2 * kSegBlockBytes;
constexpr uint64_t kSegWideSlice = (uint64_t)256 << 10, kSegWideShort = (uint64_t)64 << 10, kSegWideBytes = (uint64_t)2 << 20, kSegWideLong = (uint64_t)64 << 20;
inline bool segments_wide(uint64_t stream_capacity, uint64_t slice_bytes)
{
    if (slice_bytes < kSegWideShort || slice_bytes % kSegWideBlockBytes != 0) return false;
    return stream_capacity >= (slice_bytes >= kSegWideSlice ? kSegWideBytes : kSegWideLong);
}
// Streams of more than this are written with non-temporal stores, smaller ones with plain stores, which leave them in the
// memory-side cache for whoever reads them.  Unpack and a pass that reads the result, other buffers in every turn, us, non-temporal
// / plain: 4 MB 9.7 / 9.6, 14 MB 17.5 / 16.2, 57 MB 59.4 / 53.2, 115 MB 110.6 / 101.0, 172 MB 162.1 / 161.0, 230 MB 213 / 216,
// 287 MB 263 / 268; pack alike.  (Without the reader 5.6 / 5.1, 8.2 / 9.0, 24.9 / 24.6, 46.9 / 50.8, 69.7 / 76.2, 92 / 100, 115 / 124.)
constexpr uint64_t kSegStreamBytes = (uint64_t)128 << 20;

// Size of descriptor i: 0 beyond n, and for a descriptor whose offset or size is not a multiple of 16, which is counted in bad.
__device__ __forceinline__ uint64_t scan_size(const fusco_segment *desc, int64_t i, int64_t n, int &bad)
{
    if (i >= n) return 0;
    const fusco_segment d = desc[i];
    if (!((d.offset | d.size) & 15u)) return d.size;
    ++bad;
    return 0;
}

// Sizes of the thread's `items` (<= kScanItems) consecutive descriptors from index i0 on; returns their sum.
__device__ __forceinline__ uint64_t scan_load(const fusco_segment *desc, int64_t n, int64_t i0, int items,
                                              uint64_t (&size)[kScanItems], int &bad)
{
    uint64_t sum = 0;
#pragma unroll
    for (int q = 0; q < kScanItems; ++q) {
        size[q] = q < items ? scan_size(desc, i0 + q, n, bad) : 0;
        sum += size[q];
    }
    return sum;
}

// Cumulative bytes, first of two launches (left out where one does): the bytes of every chunk of
// kScanChunk descriptors are left at cum[end of the chunk] with bit 0 set.  All true cumulative values are
// multiples of 16, so the second launch can tell such a chunk total from a finished entry.
__global__ __launch_bounds__(kScanThreads) void segments_total_kernel(const fusco_segment *desc, int64_t n, uint64_t *cum,
                                                                     int32_t *status)
{
    __shared__ uint64_t part[kScanThreads / kWave];
    const int tid = threadIdx.x;
    const int64_t c0 = (int64_t)blockIdx.x * kScanChunk;
    uint64_t sum = 0;
#pragma unroll
    for (int q = 0; q < kScanItems; ++q) {
        const int64_t i = c0 + q * kScanThreads + tid;
        if (i >= n) continue;
        const fusco_segment d = desc[i];
        if (!((d.offset | d.size) & 15u)) sum += d.size;
    }
    for (int d = kWave / 2; d > 0; d >>= 1) sum += __shfl_down(sum, d, kWave);
    if ((tid & (kWave - 1)) == 0) part[tid / kWave] = sum;
    __syncthreads();
    if (tid == 0) {
        for (int w = 1; w < kScanThreads / kWave; ++w) sum += part[w];
        const int64_t end = min(c0 + kScanChunk, n);
        cum[end] = sum | 1u;
        if (blockIdx.x == 0) *status = 0;
    }
}

// cum[0] = 0, cum[i + 1] = cum[i] + size of segment i; a descriptor whose offset or size is not a
// multiple of 16 is counted in *status and takes part with size 0.  One workgroup per chunk of kScanChunk descriptors.
// The bytes before the chunk come from the entries at the ends of the earlier chunks, each of which holds either that
// chunk's own bytes (bit 0 set) or, once its workgroup has been there, the cumulative value; either will do, so
// nobody waits: the workgroup takes the nearest finished entry and adds the totals between it and itself.
// Bound by latency: one workgroup that walked the whole list took 69 us for 40000 descriptors and 385 us for 200000,
// the two launches take 10 and 11 us.  SINGLE: one workgroup covers the list.
template <bool SINGLE>
__global__ __launch_bounds__(SINGLE ? kScanSingleThreads : kScanThreads) void segments_scan_kernel(const fusco_segment *desc,
                                                                                                  int64_t n, uint64_t *cum,
                                                                                                  int32_t *status)
{
    __shared__ uint64_t part[(SINGLE ? kScanSingleThreads : kScanThreads) / kWave];
    __shared__ unsigned long long before;
    __shared__ int finished, bad_total;
    const int tid = threadIdx.x, lane = tid & (kWave - 1), wave = tid / kWave;
    // a single workgroup spreads the list over all its threads (3000 descriptors: 3.5 us, 5.2 us with eight per thread)
    const int items = SINGLE ? (int)((n + kScanSingleThreads - 1) / kScanSingleThreads) : kScanItems;
    const int64_t c0 = (int64_t)blockIdx.x * kScanChunk, i0 = c0 + (int64_t)tid * items;
    if (tid == 0) {
        before = 0;
        finished = -1;
        bad_total = 0;
    }
    // the ends of the nearest earlier chunks are on their way together with the descriptors
    uint64_t near = 0;
    if (!SINGLE && tid < (int)blockIdx.x) near = __hip_atomic_load(cum + (blockIdx.x - tid) * (int64_t)kScanChunk, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    uint64_t size[kScanItems];
    int bad = 0;
    const uint64_t sum = scan_load(desc, n, i0, items, size, bad);
    uint64_t incl = sum;
    for (int d = 1; d < kWave; d <<= 1) {
        const uint64_t up = __shfl_up(incl, d, kWave);
        if (lane >= d) incl += up;
    }
    if (lane == kWave - 1) part[wave] = incl;
    __syncthreads();
    if (bad) atomicAdd(&bad_total, bad);
    if constexpr (!SINGLE) {
        // windows of the kScanThreads nearest earlier chunks, until a finished entry or the first chunk is in one
        for (int64_t hi = blockIdx.x; hi > 0; hi -= kScanThreads) {
            const int64_t j = hi - 1 - tid;   // thread 0 has the nearest chunk
            uint64_t v = 0;
            if (j >= 0) {
                v = hi == blockIdx.x ? near : __hip_atomic_load(cum + (j + 1) * kScanChunk, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
                if (!(v & 1u)) atomicMax(&finished, kScanThreads - 1 - tid);
            }
            __syncthreads();
            const int nearest = finished < 0 ? kScanThreads : kScanThreads - 1 - finished;
            if (j >= 0 && tid <= nearest) atomicAdd(&before, (unsigned long long)(v & ~(uint64_t)1));
            __syncthreads();
            if (nearest < kScanThreads) break;
        }
    }
    __syncthreads();
    uint64_t run = before + incl - sum;
    for (int w = 0; w < wave; ++w) run += part[w];
#pragma unroll
    for (int q = 0; q < kScanItems; ++q) {
        run += size[q];
        if (q < items && i0 + q < n) __hip_atomic_store(cum + i0 + q + 1, run, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    }
    if (blockIdx.x == 0 && tid == 0) cum[0] = 0;
    if (tid == 0) {
        if constexpr (SINGLE) *status = bad_total;
        else if (bad_total) atomicAdd(status, bad_total);
    }
}

// The same in one launch: a workgroup adds up all descriptors before its own instead of taking sums that an earlier launch has
// left, and the last one, which reads the whole list, counts the invalid ones.  One launch / two, us:
// 6000 descriptors 4.5 / 7.4 (one workgroup 7.4), 10000 5.0 / 7.8, 20000 6.5 / 8.3, 30000 7.7 / 8.5, 40000 9.1 / 8.7.
__global__ __launch_bounds__(kScanDirectThreads) void segments_scan_direct_kernel(const fusco_segment *desc, int n, uint64_t *cum,
                                                                                 int32_t *status)
{
    constexpr int kWaves = kScanDirectThreads / kWave, kAhead = 8;   // kAhead: descriptors that a thread requests at a time
    __shared__ uint64_t part[kWaves], earlier[kWaves];
    __shared__ int bad_part[kWaves];
    const int tid = threadIdx.x, lane = tid & (kWave - 1), wave = tid / kWave;
    const int c0 = blockIdx.x * kScanDirectChunk, i0 = c0 + tid * kScanDirectItems;
    uint64_t size[kScanDirectItems], before = 0;
    int bad = 0;
#pragma unroll
    for (int q = 0; q < kScanDirectItems; ++q) size[q] = scan_size(desc, i0 + q, n, bad);
    for (int i = tid; i < c0; i += kAhead * kScanDirectThreads) {
        uint64_t s[kAhead];
#pragma unroll
        for (int q = 0; q < kAhead; ++q) s[q] = scan_size(desc, i + q * kScanDirectThreads, c0, bad);
#pragma unroll
        for (int q = 0; q < kAhead; ++q) before += s[q];
    }
    uint64_t sum = 0;
#pragma unroll
    for (int q = 0; q < kScanDirectItems; ++q) sum += size[q];
    uint64_t incl = sum;
    for (int d = 1; d < kWave; d <<= 1) {
        const uint64_t up = __shfl_up(incl, d, kWave);
        if (lane >= d) incl += up;
        before += __shfl_xor(before, d, kWave);
        bad += __shfl_xor(bad, d, kWave);
    }
    if (lane == kWave - 1) {
        part[wave] = incl;
        earlier[wave] = before;
        bad_part[wave] = bad;
    }
    __syncthreads();
    uint64_t run = incl - sum;
    int bad_total = 0;
    for (int w = 0; w < kWaves; ++w) {
        run += earlier[w] + (w < wave ? part[w] : 0);
        bad_total += bad_part[w];
    }
#pragma unroll
    for (int q = 0; q < kScanDirectItems; ++q) {
        run += size[q];
        if (i0 + q < n) cum[i0 + q + 1] = run;
    }
    if (tid == 0) {
        if (blockIdx.x == 0) cum[0] = 0;
        if (blockIdx.x == gridDim.x - 1) *status = bad_total;
    }
}

__global__ __launch_bounds__(256) void fill_u32_kernel(uint32_t *p, int64_t n, uint32_t v)
{
    const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i < n) p[i] = v;
}

struct SegCopyArgs {
    const char *src;
    char *dst;
    const fusco_segment *src_desc, *dst_desc;   // nullptr: that side is the contiguous stream
    const uint64_t *cum;
    int64_t n;
    uint64_t src_bytes, dst_bytes;
    uint64_t limit;   // whole blocks of kSegBlockBytes that cover the stream's capacity: nothing behind them is copied
    uint64_t slice_bytes;
    uint32_t *slice_fill;
    int32_t *status;
};

// One workgroup per 16 KiB of the stream (wide ones per 32 KiB), one wave per 4 KiB of it: the wave finds the segment of its first byte by
// probing 64 cumulative entries at a time (three dependent loads for 40000 segments, where halving takes
// sixteen), then reads the next 64 segments' ends and offsets in one go and looks its units up in them.
// An XCD takes runs of neighbouring blocks: what it writes on a contiguous side are runs of 128 KiB.
// Bound by memory once the search is short.  Measured, 287 MB in 40000 segments of 16 B to 14 KiB: pack 176 -> 106 us
// (5.4 TB/s read and written), pack with 1 MiB slices 193 -> 124 us, unpack 178 -> 115 us.  A unit's load is issued as
// soon as its segment is known: all four together take 119 and 125 us.  8 KiB a wave take 117 and 124 us, 2 KiB 117 us each.
// STREAM: non-temporal stores, which the L2 still merges into whole lines at the segments' ragged edges (write-through ones
// 139 us in the unpack); for streams that the memory-side cache would not keep for their reader (kSegStreamBytes).
template <bool SLICES, bool STREAM, int THREADS>
__global__ __launch_bounds__(THREADS) void segments_copy_kernel(SegCopyArgs a)
{
    constexpr uint32_t kBlockBytes = THREADS / kWave * kSegPieceBytes;
    __shared__ uint64_t s_src[THREADS], s_dst[THREADS];
    __shared__ int s_end[THREADS], s_valid[THREADS];
    const int lane = threadIdx.x & (kWave - 1), wave = threadIdx.x / kWave;
    // workgroup b runs on XCD b mod 8; the blocks after the last whole round of runs are taken in order
    constexpr uint32_t run = kSegRunBytes / kBlockBytes, round = kXcds * run;
    uint32_t block = blockIdx.x;
    if (block < gridDim.x / round * round) {
        const uint32_t in = block % round;
        block += (in % kXcds) * run + in / kXcds - in;
    }
    const uint64_t base = (uint64_t)block * kBlockBytes;
    const uint64_t piece = base + (uint64_t)wave * kSegPieceBytes;
    // the first probes of the search below are on their way together with the stream's size
    int64_t lo = 0, hi = a.n, step = (a.n + kWave - 1) / kWave;
    uint64_t probe = a.cum[min(lane * step, hi)];
    const uint64_t total = min(a.cum[a.n], a.limit);
    if (base >= total) return;
    __shared__ int skipped_total, waves_done;
    if constexpr (SLICES) {
        if (threadIdx.x == 0) skipped_total = waves_done = 0;
        __syncthreads();
    }
    uint64_t *src_at = s_src + wave * kWave, *dst_at = s_dst + wave * kWave;
    int *end = s_end + wave * kWave, *valid = s_valid + wave * kWave;
    u32x4 v[kSegUnits];
    uint64_t to[kSegUnits];
    bool ok[kSegUnits];
    int skipped = 0;
#pragma unroll
    for (int r = 0; r < kSegUnits; ++r) ok[r] = false;
    if (piece < total) {
        // 64 segments or fewer that hold the wave's first byte: cum[lo] <= piece < cum[hi]
        while (hi - lo > kWave) {
            const int c = __builtin_popcountll(__builtin_amdgcn_ballot_w64(lo + lane * step < hi && probe <= piece));
            lo += (max(c, 1) - 1) * step;   // lane 0 probes cum[lo]: c >= 1 for cumulative entries that ascend from 0
            hi = min(lo + step, hi);
            step = (hi - lo + kWave - 1) / kWave;
            probe = a.cum[min(lo + lane * step, hi)];
        }
        // Windows of 64 segments [w, w + 64), the first one starting at byte `begin`; stream positions from here on
        // are relative to the wave's piece.
        const int bytes = (int)min((uint64_t)kSegPieceBytes, total - piece);
        uint64_t begin = __shfl(probe, 0, kWave);
        int first = 0;   // units below this position belong to an earlier window
        // The lookup of a unit ends at a q with end[q - 1] <= pos < end[q], whatever the list holds, so for q > 0 segment w + q
        // covers the unit and its entries were written for this window.  q == 0 rests on begin <= piece + pos, which
        // ascending cumulative bytes from 0 give; with sizes whose sum wraps around 2^64 (a negative int64) the search may end
        // elsewhere, and the units before `begin` are skipped.
        if (begin > piece) {
            first = (int)min(begin - piece, (uint64_t)kSegPieceBytes);
#pragma unroll
            for (int r = 0; r < kSegUnits; ++r)
                if ((r * kWave + lane) * 16 < min(first, bytes)) ++skipped;
        }
        for (int64_t w = lo;; w += kWave) {
            const int64_t i = w + lane;
            const uint64_t e = a.cum[min(i + 1, a.n)];
            uint64_t b = __shfl_up(e, 1, kWave);
            if (lane == 0) b = begin;
            const int e_rel = e <= piece ? 0 : (int)min(e - piece, (uint64_t)kSegPieceBytes);
            wave_lds_order();
            end[lane] = e_rel;
            if (i < a.n && e > piece && b < piece + bytes) {   // the wave's bytes touch this segment: its offsets are read
                const uint64_t so = a.src_desc ? a.src_desc[i].offset : b, dofs = a.dst_desc ? a.dst_desc[i].offset : b;
                // bytes of the segment, from its start, that lie inside both buffers; none for an offset that is
                // misaligned or outside (nothing below can wrap: the offset is inside the buffer)
                uint64_t room = 0;
                if (!((so | dofs) & 15u) && a.src_bytes >= 16 && so <= a.src_bytes - 16 && a.dst_bytes >= 16 &&
                    dofs <= a.dst_bytes - 16)
                    room = min(min(a.src_bytes - so, a.dst_bytes - dofs) & ~(uint64_t)15, e - b);
                const uint64_t good = b + room;
                valid[lane] = good <= piece ? 0 : (int)min(good - piece, (uint64_t)kSegPieceBytes);
                src_at[lane] = so - b + piece;
                dst_at[lane] = dofs - b + piece;
            }
            wave_lds_order();
            const int last = __shfl(e_rel, kWave - 1, kWave);
            // the segment of the window's first unit; often it reaches past the wave's bytes, and no unit needs the lookup
            // (one segment of 1 MiB: 3.5 us, 4.1 us with it)
            const uint64_t open = ~__builtin_amdgcn_ballot_w64(e_rel <= first);
            const int q_first = open ? __builtin_ctzll(open) : 0;
            const bool single = open && __builtin_amdgcn_readlane(e_rel, q_first) >= bytes;
#pragma unroll
            for (int r = 0; r < kSegUnits; ++r) {
                const int pos = (r * kWave + lane) * 16;
                if (pos < first || pos >= last || pos >= bytes) continue;   // another window's, or beyond the stream
                int q = single ? q_first : 0;   // entries of `end` that are <= pos: at most 63, because pos < last
                if (!single) {
#pragma unroll
                    for (int h = kWave / 2; h > 0; h >>= 1)
                        if (end[q + h - 1] <= pos) q += h;
                }
                if (pos >= valid[q]) {
                    ++skipped;
                    continue;
                }
                ok[r] = true;
                to[r] = dst_at[q] + (uint64_t)pos;
                v[r] = load16_stream((const u32x4 *)(a.src + src_at[q] + (uint64_t)pos));
            }
            first = max(first, last);
            begin = __shfl(e, kWave - 1, kWave);
            if (last >= bytes || w + kWave >= a.n) break;
        }
    }
#pragma unroll
    for (int r = 0; r < kSegUnits; ++r) {
        if (!ok[r]) continue;
        if constexpr (SLICES) store16_system((u32x4 *)(a.dst + to[r]), v[r]);
        else put16<STREAM>((u32x4 *)(a.dst + to[r]), v[r]);
    }
    if (skipped) atomicAdd(a.status, skipped);
    if constexpr (SLICES) {
        // A slice counts bytes only once they are in memory: the stores above are write-through at
        // system scope (sc0 sc1), every wave waits for its own to complete, and the last one of the workgroup
        // adds the bytes that the workgroup has really written (skipped units are left out, so a slice with
        // holes never reaches its size) with a system-scope atomic.  (A device-wide release fence
        // would do too, but it writes back the whole L2 of the XCD each time.)  In wide workgroups nobody waits for the last wave (in
        // narrow ones it makes no difference: 124.7 with two barriers, 123.6 without, small slices 18.4 and 18.7).
        asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
        if (skipped) atomicAdd(&skipped_total, skipped);
        bool last;
        if constexpr (THREADS > kSegThreads) {
            wave_lds_order();   // LDS serves a wave's additions in order: the last wave to arrive finds everybody's skipped units
            last = lane == 0 && atomicAdd(&waves_done, 1) == THREADS / kWave - 1;
        } else {
            __syncthreads();
            last = threadIdx.x == 0;
        }
        if (last) {
            __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "workgroup");   // the skipped units are read behind the count of waves, also by the compiler
            const uint64_t left = total - base;
            const uint32_t mine = (uint32_t)(left < kBlockBytes ? left : kBlockBytes);
            __hip_atomic_fetch_add(a.slice_fill + base / a.slice_bytes, mine - 16u * (uint32_t)skipped_total,
                                   __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_SYSTEM);
        }
    }
}

}   // namespace

#endif
