// Host side: argument checks shared by the entry points, kernel launch helpers, per-call timing events.
#ifndef FUSCO_CSRC_LAUNCH_H
#define FUSCO_CSRC_LAUNCH_H

#include "common.h"
#include "planner.h"
#include "movers.h"
#include "segments.h"
#include "probes.h"

namespace {

bool aligned16(const void *p) { return ((uintptr_t)p & 15u) == 0; }

// odd multiplier close to frac * n that shares no factor with n: i -> i * mul mod n is a bijection of
// [0, n) that sends neighbours far apart
uint32_t coprime_near(uint32_t n, double frac)
{
    if (n < 3) return 1u;
    uint32_t m = (uint32_t)((double)n * frac) | 1u;
    for (;; m += 2) {
        uint32_t x = n, y = m % n;
        while (y) { const uint32_t r = x % y; x = y; y = r; }
        if (x == 1 && m % n != 0) return m % n;
    }
}

int round_up(int v, int m) { return (v + m - 1) / m * m; }

int launch_status()
{
    return hipGetLastError() == hipSuccess ? FUSCO_OK : FUSCO_ERR_HIP;
}

// Events armed by fusco_probe_time_next_call for the calling thread (null when not armed), and their
// hand-over to the call that consumes them.
thread_local hipEvent_t g_time_start = nullptr, g_time_stop = nullptr;

struct ArmedEvents {
    hipEvent_t start, stop;
    ArmedEvents() : start(g_time_start), stop(g_time_stop)
    {
        g_time_start = nullptr;
        g_time_stop = nullptr;
    }
};

// Kernel launch that can carry a start and a stop event of its own: hipExtLaunchKernelGGL records them
// from the dispatch's own timestamps, without the barrier that a stream event puts between kernels.
template <typename K, typename A>
void launch(K kernel, dim3 grid, dim3 block, hipStream_t s, const A &a, hipEvent_t e0 = nullptr, hipEvent_t e1 = nullptr)
{
    if (e0 || e1) hipExtLaunchKernelGGL(kernel, grid, block, 0, s, e0, e1, 0, a);
    else hipLaunchKernelGGL(kernel, grid, block, 0, s, a);
}

// the same for kernels with several arguments; `lds` bytes of dynamic LDS (which the kernels do not use: asking
// for it caps the number of workgroups a compute unit holds at once)
template <typename K, typename... A>
void launch_args(K kernel, dim3 grid, dim3 block, size_t lds, hipStream_t s, hipEvent_t e0, hipEvent_t e1, A... args)
{
    if (e0 || e1) hipExtLaunchKernelGGL(kernel, grid, block, (unsigned)lds, s, e0, e1, 0, args...);
    else hipLaunchKernelGGL(kernel, grid, block, (unsigned)lds, s, args...);
}

// just over half of a compute unit's 160 KiB of LDS, which is handed out in 128 blocks of 1280 bytes
constexpr size_t kOverHalfLds = (size_t)65 * 1280;

// Dynamic LDS that lets `wgs` workgroups share a compute unit's LDS (2 <= wgs <= 15; 13 comes out as 14; for kernels without LDS
// of their own); 0 for no cap.
inline size_t lds_for_occupancy(int wgs)
{
    if (wgs < 2 || wgs > 15) return 0;
    return (size_t)(128 / wgs) * 1280;
}

// Inputs of fewer bytes are bound by latency, larger ones by memory (combine_kernel's JU, workgroup shapes, stores).
constexpr size_t kCombineLatencyBoundBytes = (size_t)64 << 20;

// Workgroup shape of combine_kernel for rows of C chunks: as many column segments as 1024 threads need, the
// threads spread evenly over them (1280 chunks: two workgroups of 640 threads, not 1024 + 256).
inline void combine_shape(int C, int &threads, int &segs)
{
    segs = (C + 1023) / 1024;
    if (segs < 1) segs = 1;
    threads = round_up((C + segs - 1) / segs, kWave);
}

// The same for inputs bound by latency.  Fewer than 512 segments of 128 threads leave compute units without work: rows of more than 256
// chunks are then cut into segments of 64 threads.  With more, rows of more than 512 chunks are cut into segments of 128, which get going
// sooner than workgroups of 16 waves and finish more evenly.  Segments of 64 / 128 / the whole row, bf16 to bf16, us:
// - rows of 14 KiB 4 tokens x 8 2.4 / 2.4 / 3.6, 64 x 8 3.2 / 3.1 / 4.5, 128 x 8 4.2 / 4.3 / 5.1, 512 x 8 11.5 / 11.5 / 11.6, 1000 x 4
//   12.7 / 12.5 / 13.1, 3500 x 1 16.4 / 16.3 / 19.0; of 520 chunks 60 x 8 2.9 / 3.1 / 3.7, 400 x 8 6.4 / 6.3 / 6.9;
// - of 512 chunks 32 x 8 2.7 / 2.7 / 3.1, 1000 x 2 5.4 / 5.2 / 5.2; of 448 100 x 8 3.0 / 3.1 / 3.5, 400 x 8 5.8 / 5.7 / 5.8; of 360
//   1537 x 6 to fp32 11.5 / 11.2 / 11.2; of 256 100 x 8 2.9 / 2.8 / 2.9.
inline void combine_shape_latency(int N, int C, int &threads, int &segs)
{
    combine_shape(C, threads, segs);
    const bool few = (int64_t)N * ((C + 127) / 128) < 512;
    if (C <= (few ? 256 : 512)) return;
    threads = few ? 64 : 128;
    segs = (C + threads - 1) / threads;
}

template <bool Y_BF16, bool OUT_BF16, int JU, bool WIDENED = Y_BF16 && !OUT_BF16 && JU == 1>
void launch_combine_as(const CombineArgs &a, dim3 grid, dim3 block, OutStores stores, hipStream_t s, hipEvent_t e0, hipEvent_t e1)
{
    // Stores differ in speed alone.  Inputs bound by latency are written through or plain, inputs bound by memory (two rows WIDENED) never plain (out_stores).
    if constexpr (JU > 0 && JU <= 4) {
        if (stores == kOutThroughStream) return launch(combine_kernel<Y_BF16, OUT_BF16, JU, kOutThroughStream, false, WIDENED>, grid, block, s, a, e0, e1);
        if (stores == kOutNonTemporal) return launch(combine_kernel<Y_BF16, OUT_BF16, JU, kOutNonTemporal, false, WIDENED>, grid, block, s, a, e0, e1);
    }
    if constexpr (!(WIDENED && JU == 2)) {
        if (stores == kOutPlain) return launch(combine_kernel<Y_BF16, OUT_BF16, JU, kOutPlain, false, WIDENED>, grid, block, s, a, e0, e1);
    }
    launch(combine_kernel<Y_BF16, OUT_BF16, JU, kOutThrough, false, WIDENED>, grid, block, s, a, e0, e1);
}

// Rows in flight.  Bound by latency: eight, four from 16 MiB on (us, 64 tokens x 8 x 14 KiB 3.1 / 3.5, 512 x 8 12.0 / 11.7, 2000 x 8 x 4
// KiB 13.4 / 13.0), for 24 and more entries, several rounds of them, from 32 MiB on (506 x 24 x 1600 B of fp32 5.2 / 6.4, 633 x 24 x 1504 B
// 6.3 / 7.4); one entry per token takes one, and two entries, as three and four of 32 MiB and more, two with the slots as scalars
// (four in lanes / that: 4096 x 2 x 2 KiB 5.6 / 5.5, 1500 x 4 x 8 KiB 11.6 / 11.2, 1000 x 4 x 14 KiB 13.4 / 13.2, but 1537 x 6 x 5760 B
// 13.8 / 14.3).  Bound by memory: one, of two entries per token both.  One row a wave takes many waves to keep memory busy: two rows below
// 32768 waves, four of the chip's fills (one / two: 1200 x 8 x 8 KiB, 9600 waves, 17.9 / 16.2; 600 x 8 x 16 KiB, 9600, 20.9 / 19.1; 11426 x
// 6 x 1152 B, 22852, 20.2 / 17.5; 13512 x 8 x 1104 B, 27024, 34.0 / 29.7; 5691 x 7 x 4096 B, 22764, 31.5 / 32.0; 6193 x 8 x 5968 B to fp32,
// 37158, 69.3 / 70.2), four below 4096 (1000 x 64 x 2 KiB, 2000 waves, 42.6 / 21.7).  Many entries keep a wave busy longer and want one
// already from 16384 waves on (1417 x 24 x 15 KiB of fp32, 21972, 88.0 / 92.0; 5614 x 24 x 3984 B, 22456, 93.4 / 96.6).
constexpr int64_t kCombineFewWaves = 4096, kCombineManyWaves = 32768, kCombineManyWavesLong = 16384;
constexpr int kCombineLongK = 16, kCombineVeryLongK = 24;   // entries from which a wave is busy long
// Three and more fp32 rows per token are spaced (kSpacedRows) from these sizes to kCombineLatencyBoundBytes, us, back to back / spaced: 753
// tokens x 6 x 1600 B (7 MiB) 2.9 / 2.7, 256 x 7 x 5824 B 3.4 / 3.1; smaller 37 x 7 x 11 KiB 2.5 / 2.6, 12 x 12 x 27 KiB 2.8 / 3.1.  More
// than eight of them take two rounds, and waiting for the first costs: 121 x 24 x 13 KiB (36 MiB) 7.7 / 8.2, 541 x 16 x 2912 B (24 MiB) 5.9
// / 6.1, but 581 x 12 x 6912 B (46 MiB) 10.6 / 9.9, 626 x 64 x 1344 B (51 MiB) 14.7 / 12.9.  Two rows as above (893 x 2 x 15 KiB 7.6 / 8.1;
// 1642 x 2 x 4192 B 5.8 / 5.2).
constexpr size_t kCombineSpacedBytes = (size_t)4 << 20, kCombineSpacedManyBytes = (size_t)42 << 20;

template <bool Y_BF16, bool OUT_BF16>
void launch_combine(CombineArgs a, int N, OutStores stores, hipStream_t s, hipEvent_t e0, hipEvent_t e1)
{
    const size_t bytes = (size_t)N * (size_t)a.k * (size_t)a.C * 16;
    const bool latency = bytes < kCombineLatencyBoundBytes;
    int threads;
    if (latency) combine_shape_latency(N, a.C, threads, a.segs);
    else combine_shape(a.C, threads, a.segs);
    a.n_rows = N;
    const dim3 grid((unsigned)N * (unsigned)a.segs), block((unsigned)threads);
    const int64_t waves = (int64_t)N * ((a.C + kWave - 1) / kWave);
    const int64_t many = a.k >= kCombineLongK ? kCombineManyWavesLong : kCombineManyWaves;
    const bool two = latency ? a.k == 2 || (a.k <= 4 && bytes >= kCombineLatencyBoundBytes / 2)
                             : a.k == 2 || (waves >= kCombineFewWaves && waves < many);
    if constexpr (!Y_BF16) {
        if (latency && a.k >= 3 && bytes >= (a.k <= 8 ? kCombineSpacedBytes : kCombineSpacedManyBytes))
            return launch_combine_as<Y_BF16, OUT_BF16, kSpacedRows>(a, grid, block, stores, s, e0, e1);
    }
    if constexpr (Y_BF16 && !OUT_BF16) {
        if (a.k == 2 && !latency) return launch_combine_as<Y_BF16, OUT_BF16, 2, true>(a, grid, block, stores, s, e0, e1);
    }
    if (a.k == 1)
        launch_combine_as<Y_BF16, OUT_BF16, 1>(a, grid, block, stores, s, e0, e1);
    else if (two)
        launch_combine_as<Y_BF16, OUT_BF16, 2>(a, grid, block, stores, s, e0, e1);
    else if (!latency && waves >= many)
        launch_combine_as<Y_BF16, OUT_BF16, 1>(a, grid, block, stores, s, e0, e1);
    else if (latency && bytes < (a.k >= kCombineVeryLongK ? kCombineLatencyBoundBytes / 2 : kCombineLatencyBoundBytes / 4))
        launch_combine_as<Y_BF16, OUT_BF16, 8>(a, grid, block, stores, s, e0, e1);
    else
        launch_combine_as<Y_BF16, OUT_BF16, 4>(a, grid, block, stores, s, e0, e1);
}

// dst[r] = src[index(r)] for n_rows destination rows of C chunks (see gather_rows_kernel)
template <bool STREAM_LOAD>
void launch_gather(const void *src, void *dst, const int32_t *idx1, const int32_t *idx2, const int32_t *n_rows_dev,
                   int n_rows, int C, hipStream_t s)
{
    if (n_rows <= 0 || C <= 0) return;
    GatherArgs a;
    a.src = (const u32x4 *)src; a.dst = (u32x4 *)dst;
    a.idx1 = idx1; a.idx2 = idx2; a.n_rows_dev = n_rows_dev; a.C = C;
    const int cpt = C >= 512 ? 4 : (C >= 128 ? 2 : 1);
    int threads = round_up((C + cpt - 1) / cpt, kWave);
    if (threads > 256) threads = 256;
    const int segs = (C + threads * cpt - 1) / (threads * cpt);
    const dim3 grid((unsigned)n_rows, (unsigned)segs), block((unsigned)threads);
    switch (cpt) {
    case 1: hipLaunchKernelGGL((gather_rows_kernel<1, STREAM_LOAD>), grid, block, 0, s, a); break;
    case 2: hipLaunchKernelGGL((gather_rows_kernel<2, STREAM_LOAD>), grid, block, 0, s, a); break;
    default: hipLaunchKernelGGL((gather_rows_kernel<4, STREAM_LOAD>), grid, block, 0, s, a); break;
    }
}

void launch_copy(void *dst, const void *src, size_t bytes, hipStream_t s)
{
    const size_t n = bytes / 16;
    if (n == 0) return;
    hipLaunchKernelGGL(probe_copy_kernel, dim3((unsigned)((n + 255) / 256)), dim3(256), 0, s, (u32x4 *)dst,
                       (const u32x4 *)src, n);
}

// `empty`: the layout has no tokens, so the tensors hold no rows and may be NULL
// walk_rows: rows the combine walks over (tokens, or send rows); the launch needs a workgroup per row and column segment
int combine_check(const void *d_y, int y_dtype, const float *d_w, const void *d_out, int out_dtype, int32_t H,
                  bool empty, int64_t walk_rows)
{
    if (H <= 0 || (!empty && (!d_y || !d_w || !d_out))) return FUSCO_ERR_INVALID_ARG;
    if ((y_dtype != FUSCO_BF16 && y_dtype != FUSCO_F32) || (out_dtype != FUSCO_BF16 && out_dtype != FUSCO_F32))
        return FUSCO_ERR_UNSUPPORTED;
    const size_t y_row = (size_t)H * (y_dtype == FUSCO_BF16 ? 2 : 4);
    if (y_row % 16 != 0 || y_row / 16 > kMaxRowChunks) return FUSCO_ERR_INVALID_ARG;
    if (!aligned16(d_y) || !aligned16(d_out) || ((uintptr_t)d_w & 3u)) return FUSCO_ERR_INVALID_ARG;
    int threads, segs;
    combine_shape((int)(y_row / 16), threads, segs);
    if (walk_rows * segs > 0x7fffffff) return FUSCO_ERR_INVALID_ARG;
    return FUSCO_OK;
}

// Where the combine walk starts.  Right after a dispatch of the same tokens the memory-side cache (256 MB)
// still holds the rows written for the last tokens.  Measured on MI355X (8192 tokens x 8 rows of 14 KiB): a
// walk that starts about 110-220 MiB of rows before the end, goes up to the last token and then wraps to
// token 0 is 7 us (2 %) faster than a walk from the last token down, and 25 us faster than one from token 0
// up.  That holds after a dispatch that writes with plain stores (the token walk); the tiled dispatch's
// streaming stores leave nothing in that cache, and when y comes from somewhere else the order makes no
// difference either.
constexpr size_t kRecentRowBytes = (size_t)160 << 20;

int combine_first_row(int N, int k, size_t row_bytes)
{
    const size_t per_token = (size_t)k * row_bytes;
    const size_t recent = kRecentRowBytes / (per_token ? per_token : 1);
    return recent >= (size_t)N ? 0 : N - (int)recent;
}

// Whether rows of row_bytes from p on consist of whole 64-byte units.  A write-through store that covers a part of such a
// unit goes to memory as a partial write: rows of 14352 B 297 us in the tiled dispatch against 228 us with stores that
// the L2 merges, rows of 8208 B 161 against 113 us; for whole units write-through is the faster one in a step
// (14336 B: 380 against 401 us with combine, 14400 B: 388 against 413 us).
bool whole_units(const void *p, size_t row_bytes) { return (((uintptr_t)p | row_bytes) & 63u) == 0; }

// Stores of the token walk where nothing but one plane of the expert tensor is written, up to the size of the memory-side cache (bit 2 of dispatch_kernel's
// MODE).  What plain stores leave dirty in the L2s is written back when the kernel ends, up to 32 MB that then go to memory with nothing else
// on its way; rows written through go there at once, and the memory-side cache keeps them.  But rows that the L2s hold are also read from there: where source and
// rows together are not much larger than the L2s, a loop over the same buffers whose reader follows at once loses by rows written through.  So they are from
// kThroughBytes of both on.  Plain / through, us, dispatch and the combine of the rows over the same buffers, the same over changing buffers, and those with
// a combine of another tensor:
// - one entry per token: 2400 x 8 KiB (37 MiB of both) 14.1 / 15.3, 16.2 / 16.0, 18.9 / 18.5; 2900 x 8 KiB (45) 16.5 / 16.9, 18.3 / 17.8, 21.1 / 20.5; 7000 x 4 KiB (55)
//   20.0 / 19.6, 21.3 / 21.3, 25.2 / 24.9; 5000 x 7 KiB (68) 26.1 / 23.2, 26.4 / 25.8, 30.2 / 29.7; 15616 x 7 KiB 65.9 / 64.3, 67.0 / 65.5, 81.4 / 78.8;
// - two and three, rows of whole lines (128 bytes): 4096 x 2 x 2 KiB (24) 9.6 / 11.5, 11.7 / 11.0, 12.9 / 12.7; 2048 x 2 x 6 KiB (36) 13.0 / 13.9, 14.6 / 14.3, 16.9 /
//   16.8; 2048 x 2 x 8 KiB (48) 18.2 / 18.5, 18.7 / 18.0, 21.3 / 21.0; 3000 x 2 x 7 KiB (62) 24.2 / 22.9, 22.4 / 21.8, 27.5 / 27.3; 3200 x 3 x 4 KiB (50) 19.9 / 18.4,
//   19.8 / 19.4, 22.4 / 22.4; 24291 x 2 x 4 KiB 102 / 100, 103 / 102, 105 / 103.  Behind a matrix product that reads the rows it is even up to 40 MiB and 1-4 % ahead
//   from there on.  Rows in other units 20720 x 2 x 5744 B 141 / 151; the tensor 16 bytes past a unit 20720 x 2 x 5760 B 129 / 140, 6128 x 3 x 4 KiB 43.5 / 49.7,
//   64 bytes past a line 126 / 124, 41.0 / 40.8;
// - rows that are no whole units gain where they are read next and lose where other memory is, one entry per token: 6000 x 8208 B 45.9 / 43.8, 47.1 / 47.7, 48.2 / 50.3;
//   18000 x 8208 B 111 / 108, 112 / 109, 121 / 125; 14000 x 14352 B 150 / 145, 150 / 145, 153 / 160; 15616 x 7024 B 78.4 / 76.8, 80.0 / 78.3, 84.8 / 81.6: left plain;
// - more entries come out even or lose: 9515 x 4 x 1 KiB 20.1 / 20.5, 4990 x 6 x 512 B 11.6 / 12.0, 2827 x 8 x 1344 B 15.5 / 15.7.
constexpr size_t kThroughBytes = (size_t)50 << 20;
inline bool walk_through(int k, const void *rows, size_t row, size_t source, size_t written)
{
    if (k > 3 || source + written < kThroughBytes) return false;
    return whole_units(rows, row) && (k == 1 || row % 128 == 0);
}

// Stores of the fused plan + dispatch, whose workgroups write a token's k rows (or a column segment of them, `group` bytes) one after the other: written
// through from kFusedThroughBytes of rows on; below, the end of a small kernel is sooner reached than memory.  us, plain / through, alone, with a combine of another
// tensor and with the combine of the rows: 128 x 8 x 7 KiB + 224 B 5.3 / 4.7, 9.8 / 9.1 (second); 219 x 8 x 11 KiB 7.4 / 6.3, 13.6 / 11.8, 13.1 / 12.5; 114 x 8 x 50 KiB 11.8 /
// 9.6, 22.4 / 20.8, 21.9 / 21.5; 155 x 4 x 3584 B (2.1 MiB) 3.8 / 3.6, 6.5 / 6.2, 7.2 / 7.1; 124 x 8 x 1 KiB (1 MiB) 3.6 / 3.7.
// A workgroup that writes much does so at one store's latency after the other, and few of them do not hide it: groups of more than kFusedThroughShort
// only from kFusedThroughTokens on, rows of partial units from kFusedThroughTokensCut on.  Kernel times with the combine of the rows and of another tensor, buffers
// that change: 18 x 8 x 16 KiB 8.2 / 8.9, 8.0 / 8.3; 32 x 8 x 16 KiB 8.2 / 8.7, 8.2 / 8.4; 64 x 8 x 16 KiB 9.0 / 8.7, 9.1 / 8.8; 14 x 16 x 10.5 KiB 8.7 / 9.8, 8.4 / 9.2;
// 52 x 16 x 10.5 KiB 10.4 / 10.1, 10.6 / 10.6; 24 x 8 x 32 KiB 10.4 / 10.9, 10.3 / 10.8; 10 x 24 x 8 KiB 9.8 / 10.8, 44 x 24 x 8 KiB 11.8 / 11.7; groups of 84 KiB
// 24 x 8 x 10.5 KiB 8.2 / 8.1, 8.1 / 7.9; partial units 40 x 8 x 10400 B 8.4 / 8.9, 8.3 / 8.2, 18 x 8 x 15040 B 8.2 / 8.8, 8.0 / 8.2, 80 x 8 x 15040 B 9.7 / 9.4, 9.7 / 9.2.
// Not groups of more than kFusedThroughMost (24 x 16 x 32704 B 8.3 / 9.4, 15 x 33 x 24640 B 13.3 / 15.0; 80 x 16 x 23200 B 10.8 / 9.3), nor rows that are no whole units
// from kFusedThroughCutBytes on (154 x 8 x 65232 B 16.7 / 16.2, 35.1 / 36.1, 36.6 / 42.8; 912 x 1 x 14816 B 8.7 / 8.0, 16.7 / 16.1, 16.8 / 16.1).
constexpr size_t kFusedThroughBytes = (size_t)2 << 20, kFusedThroughCutBytes = (size_t)16 << 20;
constexpr size_t kFusedThroughShort = (size_t)96 << 10, kFusedThroughMost = (size_t)384 << 10;
constexpr int kFusedThroughTokens = 48, kFusedThroughTokensCut = 64;
inline bool fused_through(int N, size_t written, size_t group, bool whole)
{
    if (written < kFusedThroughBytes || group > kFusedThroughMost) return false;
    if (!whole) return written < kFusedThroughCutBytes && N >= kFusedThroughTokensCut;
    return group <= kFusedThroughShort || N >= kFusedThroughTokens;
}

// Stores of combine's output rows.
// Large outputs of inputs that are bound by memory go past the memory-side cache: what write-through and plain stores leave
// dirty there costs the reads of the kernels around them more than it saves.  Steps with the experts' output in a tensor of
// its own and other buffers in every step, written through / non-temporal / both at once, us: 8192 tokens x 8 rows of
// 14 KiB 378.9 / 367.3 / 365.1, 16384 x 8 x 8 KiB 433.5 / 426.4 / 426.0, 32768 x 8 x 14 KiB 1467 / 1437 / 1437.  (A loop over
// the same buffers whose x and output fit that cache together prefers to leave the output there: 340.7 / 347.0 / 344.7 at
// 8192 x 8 x 14 KiB; 402 / 394 / 394 and 1461 / 1431 / 1429 at the other two.)
// Where input and output together are at most kReadBackBytes, half that cache, the output stays there for the operation
// that reads it next.  60 steps and trainings of random shapes, each alone and with an addition behind it that reads the
// output, other buffers in every turn, time past the cache / written through: up to 100 MiB of both 1.02-1.06 with the
// reader (one 8 MiB output of 65 MiB: 51.5 / 49.1 us; 20 MiB of 80 MiB: 54.7 / 51.5), 0.96-1.02 without; 100-128 MiB 0.99-1.08
// and 0.94-1.03; 128-160 MiB 0.99-1.06 and 0.92-1.00; 160-190 MiB 0.98-1.05 and 0.92-1.00.  Larger: 8192 tokens x 8 x 14 KiB
// 423 / 436 us with the reader, 371 / 380 without.
// Rows that are not whole units gain from the cache like the others; past it they are not written through (8192 x 8 x
// 14352 B: combine 199 us written through, 209 us plain, 178 us non-temporal).
// Outputs of inputs below kCombineLatencyBoundBytes: written through where a wave's stores cover whole units, plain otherwise.
constexpr size_t kReadBackBytes = (size_t)128 << 20;

OutStores out_stores(size_t y_bytes, const void *out, size_t rows, size_t row_bytes)
{
    const bool whole = whole_units(out, row_bytes);
    if (y_bytes < kCombineLatencyBoundBytes) return whole ? kOutThrough : kOutPlain;
    if (y_bytes + rows * row_bytes <= kReadBackBytes) return kOutThrough;
    return whole ? kOutThroughStream : kOutNonTemporal;
}

// Stores of the two-hop combine's partial rows, summed from bf16 rows (not in turn; in turn and from fp32 rows they are plain: in turn 2099 tokens x 4
// x 2704 B 12.2 us plain, 15.1 through, from fp32 3989 x 8 x 8544 B 120 and 138).  Written through they leave the L2 while the call still
// reads; the memory-side cache keeps them for whoever reads them.  us, plain / through, and with a pass that reads them:
// - rows of whole 64-byte units 175 x 8 x 4736 B 6.4 / 4.7, 20.2 / 18.8; 503 x 8 x 6720 B 13.8 / 12.4, 30.3 / 29.8; 4096 x 8 x 8 KiB 126 / 120, 213 / 209; 6000 x
//   6 x 10 KiB 165 / 158, 281 / 274;
// - others, whose ends go to memory as partial writes, up to kPartialCutBytes of input 78 x 8 x 7568 B 5.0 / 4.1, 481 x 8 x 4784 B 9.3 / 9.0, beyond it 911 x 4
//   x 8096 B 15.7 / 16.8, 1543 x 6 x 12752 B 73 / 83.
// From kPartialStreamBytes of input on, partial rows of several times that cache, they go past it: what they leave there costs the next call
// more than it gives a reader of the rows.  Written through / past the cache, us, the two hops and a pass that reads the partial rows; plan, both tensors and two hops; both:
// 4096 x 8 x 14 KiB on 8 devices 382 / 379, 370 / 359, 536 / 533; 8192 x 8 x 8 KiB 432 / 422, 409 / 393, 605 / 594; 13924 x 8 x 5504 B 498 / 492, 518 / 486, 729 / 724;
// 10000 x 6 x 8 KiB 436 / 431, 435 / 416, 624 / 611; 16384 x 4 x 7 KiB 457 / 452, 467 / 455, 666 / 662; 6849 x 8 x 9 KiB on 16 477 / 474, 469 / 452, 678 / 681; 5000 x 8
// x 12 KiB on 4 295 / 290, 334 / 317, 450 / 445; 12000 x 8 x 14 KiB (1.3 GiB) 1105 / 1089, 1025 / 1043, 1511 / 1504.
constexpr size_t kPartialCutBytes = (size_t)20 << 20, kPartialStreamBytes = (size_t)400 << 20;

inline OutStores partial_stores(size_t y_bytes, const void *partial, size_t row_bytes)
{
    if (!whole_units(partial, row_bytes)) return y_bytes < kPartialCutBytes ? kOutThrough : kOutPlain;
    return y_bytes < kPartialStreamBytes ? kOutThrough : kOutThroughStream;
}

// Two-hop combine, by the bytes of its input and the waves of its launch.
// Up to 11 MiB latency counts: a token's rows are requested at once (at once / in turn, us, rows of 14 KiB x 8: 4 tokens 4.2 / 4.7, 128 8.7
// / 10.6).  From there on so many rows of bf16 are in flight that memory is faster with fewer: an entry is looked up and its row requested
// when the row before it is there.  That takes enough waves, 4500 or, one to a token, 3000 (11-20 MiB: 3720 x 6 x 864 B, 3720 waves, 11.4 /
// 10.6; 2523 x 8 x 880 B, 2523, 9.8 / 11.1; 2430 x 3 x 1648 B, 4860 waves, 10.0 / 8.9; 3061 x 4 x 1296 B, 6122, 11.2 / 9.9; 4096 x 2 x 2
// KiB to fp32, 8192, 16.9 / 15.7; 443 x 4 x 7696 B, 3544, 8.7 / 9.6) or 20 MiB (700 x 8 x 6704 B, 4900, 24.1 / 17.7; 300 x 8 x 14 KiB 21.0
// / 15.9); with 16384 waves they are in each other's way whatever they do, and at once is faster again (8192 x 8 x 1264 B, 16384, 34.8 /
// 39.7; 8531 x 5 x 1920 B, 17062, 28.7 / 32.3), as it is where a token leaves a single partial row (one device, 3403 x 5 x 736 B 6.6 / 7.9,
// 3590 x 5 x 2256 B 13.6 / 14.9).
// From 20 MiB on wide rows are faster one by one, their entry looked up as they are added: of 144 chunks and more up to 64 MiB, of 400 and more
// beyond (in turn / one by one: 2000 x 4 x 4 KiB on 64 devices 17.3 / 16.5, 2668 x 5 x 3696 B on 8 29.7 / 27.5, 3084 x 5 x 2432 B on 64 23.9 /
// 23.6, 1200 x 8 x 7 KiB on 64, 66 MiB, 48.7 / 45.4; but 5632 x 6 x 1680 B on 8 35.0 / 37.7, 3967 x 6 x 2224 B on 16 33.2 / 33.5, 2652 x 8 x
// 4304 B on 8, 87 MiB, 62.1 / 66.4; below 20 MiB 1008 x 3 x 6128 B on 2 9.9 / 11.9).
// fp32 rows, half the elements, are faster at once than in turn (4443 x 3 x 5184 B, 66 MiB, 22.7 / 26.7), but with fewer
// than 7000 waves of 20 to 64 MiB still faster one by one (at once / one by one / in turn: 383 x 7 x 11 KiB 13.7 / 11.4 / 14.9, 572 x 8 x
// 7328 B 13.1 / 11.6 / 14.6, 227 x 8 x 27.7 KiB 18.4 / 16.5 / 18.2).
// Up to 48 MiB rows are cut into segments of up to 256 threads (4 tokens 5.5 / 6.6 with whole rows, 300 16.1 / 17.6, 500 24.6 / 24.3), but
// not rows of little more than one (277 chunks: 1040 x 7 x 4432 B 19.6 in segments of 256 and 21 chunks, 15.9 whole). Inputs of 96 MiB and
// more are bound by memory.  Where a token's rows leave at least two partial rows, a compute unit gets about 16 waves, 12 for six and more
// bf16 rows (two_hop_workgroups), which keep enough in flight by requesting their rows at once; dynamic LDS that the kernel does not use
// keeps further workgroups out.  us, no cap / capped: 8910 x 4 x 7024 B on 8 devices (2 workgroups of 7 waves) 160 / 147, 12000 x 4 x 9 KiB
// on 4 (2 of 9; 1: 232) 227 / 214, 12679 x 4 x 9.8 KiB on 2 (2 of 10; 1: 230) 217 / 210, 3242 x 8 x 6032 B on 8 (2 of 6) 90 / 83, 7116 x 4
// x 10 KiB on 16 (1 of 11) 210 / 196, 4096 x 8 x 14 KiB on 8 (1 of 14) 228 / 224, fp32 8152 x 5 x 5792 B on 16 112 / 106.  Not on one
// device (6309 x 8 x 7264 B 96 / 105, 4240 x 6 x 10.7 KiB 70 / 78) nor for three rows on few devices or in fp32 (108219 x 3 x 1104 B on 2
// 211 / 238, 33482 x 3 x 3200 B of fp32 on 4 120 / 128; bf16 on 8, 26723 x 3 x 4000 B, 211 / 200).  One or two narrow rows are taken in
// turn here too (53067 x 1 x 4 KiB 247 / 236, 128196 x 2 x 1536 B 257 / 250; wider ones at once, 40696 x 2 x 4208 B 172 / 175).
constexpr int kTwoHopWholeChunks = 352;
constexpr size_t kTwoHopSmallBytes = (size_t)48 << 20, kTwoHopInTurnBytes = (size_t)11 << 20, kTwoHopBusyBytes = (size_t)20 << 20;
constexpr size_t kTwoHopCappedBytes = (size_t)96 << 20;
constexpr int64_t kTwoHopSomeWaves = 4500, kTwoHopManyWaves = 16384, kTwoHopFewWavesF32 = 7000;
constexpr int kTwoHopSomeTokens = 3000;
constexpr int kTwoHopNarrowChunks = 256, kTwoHopWideChunks = 144, kTwoHopWiderChunks = 400;

template <bool Y_BF16, bool OUT_BF16, TwoHopRows ROWS, OutStores PARTIAL>
void launch_two_hop_with(const TwoHopArgs &a, dim3 grid, dim3 block, size_t lds, OutStores stores, hipStream_t s)
{
    const hipEvent_t none = nullptr;
    // Stores differ in speed alone.  Outputs of the smaller inputs never go past the memory-side cache, those of the larger ones always (out_stores).
    constexpr bool kLatencyBound = !Y_BF16 && ROWS == kRowsOneByOne, kPastCache = PARTIAL == kOutThroughStream;
    if constexpr (!kLatencyBound) {
        if (stores == kOutThroughStream)
            return launch_args(combine_two_hop_kernel<Y_BF16, OUT_BF16, kOutThroughStream, ROWS, PARTIAL>, grid, block, lds, s, none, none, a);
        if (kPastCache || stores == kOutNonTemporal)
            return launch_args(combine_two_hop_kernel<Y_BF16, OUT_BF16, kOutNonTemporal, ROWS, PARTIAL>, grid, block, lds, s, none, none, a);
    }
    if constexpr (!kPastCache) {
        if (stores == kOutPlain) return launch_args(combine_two_hop_kernel<Y_BF16, OUT_BF16, kOutPlain, ROWS, PARTIAL>, grid, block, lds, s, none, none, a);
        launch_args(combine_two_hop_kernel<Y_BF16, OUT_BF16, kOutThrough, ROWS, PARTIAL>, grid, block, lds, s, none, none, a);
    }
}

template <bool Y_BF16, bool OUT_BF16, TwoHopRows ROWS>
void launch_two_hop_as(const TwoHopArgs &a, dim3 grid, dim3 block, size_t lds, OutStores stores, OutStores partial, hipStream_t s)
{
    if constexpr (Y_BF16 && ROWS != kRowsInTurn) {
        if (partial == kOutThrough) return launch_two_hop_with<Y_BF16, OUT_BF16, ROWS, kOutThrough>(a, grid, block, lds, stores, s);
        if constexpr (ROWS == kRowsAtOnce)   // rows of so large an input are not taken one by one
            if (partial == kOutThroughStream) return launch_two_hop_with<Y_BF16, OUT_BF16, ROWS, kOutThroughStream>(a, grid, block, lds, stores, s);
    }
    launch_two_hop_with<Y_BF16, OUT_BF16, ROWS, kOutPlain>(a, grid, block, lds, stores, s);
}

// Workgroups of `waves` waves per compute unit where their number is capped: up to 16 waves, but at least two workgroups of up to 10 waves;
// up to 12 for six and more bf16 rows, and a single workgroup from 7 waves on (one / two of 7: 8192 x 8 x 7 KiB on 8 devices 232 / 224 us,
// but 4096 x 8 x 7 KiB 115 / 118 and 7404 x 8 x 7152 B on 16 259 / 267; of 8: 8192 x 8 x 8 KiB on 16 281 / 290).
inline int two_hop_workgroups(int waves, bool y_bf16, int k)
{
    if (y_bf16 && k >= 6) return std::max(12 / waves, 1);
    return std::max(16 / waves, waves <= 10 ? 2 : 1);
}

template <bool Y_BF16, bool OUT_BF16>
void launch_two_hop(const TwoHopArgs &a, int N, int D, OutStores stores, hipStream_t s)
{
    const size_t bytes = (size_t)N * (size_t)a.k * (size_t)a.C * 16;
    const OutStores partial = Y_BF16 ? partial_stores(bytes, a.partial, (size_t)a.C * 32) : kOutPlain;
    const int64_t waves = (int64_t)N * ((a.C + kWave - 1) / kWave);
    const int segs = bytes >= kTwoHopSmallBytes ? (a.C + 1023) / 1024 : a.C <= kTwoHopWholeChunks ? 1 : (a.C + 255) / 256;
    const int threads = round_up((a.C + segs - 1) / segs, kWave);
    const dim3 grid((unsigned)N, (unsigned)segs), block((unsigned)threads);
    if constexpr (Y_BF16) {
        const bool in_turn = bytes >= kTwoHopCappedBytes ? a.k <= 2 && a.C <= kTwoHopNarrowChunks
                                                         : D >= 2 && bytes >= kTwoHopInTurnBytes && waves < kTwoHopManyWaves &&
                                                               (waves >= kTwoHopSomeWaves || N >= kTwoHopSomeTokens || bytes >= kTwoHopBusyBytes);
        const bool wide = bytes >= kTwoHopBusyBytes && a.C >= (bytes < kCombineLatencyBoundBytes ? kTwoHopWideChunks : kTwoHopWiderChunks);
        if (in_turn && wide) return launch_two_hop_as<Y_BF16, OUT_BF16, kRowsOneByOne>(a, grid, block, 0, stores, partial, s);
        if (in_turn) return launch_two_hop_as<Y_BF16, OUT_BF16, kRowsInTurn>(a, grid, block, 0, stores, partial, s);
    } else {
        if (bytes >= kTwoHopBusyBytes && bytes < kCombineLatencyBoundBytes && waves < kTwoHopFewWavesF32)
            return launch_two_hop_as<Y_BF16, OUT_BF16, kRowsOneByOne>(a, grid, block, 0, stores, partial, s);
    }
    size_t lds = 0;
    if (bytes >= kTwoHopCappedBytes && D >= 2 && (a.k >= 4 || (Y_BF16 && a.k == 3 && D >= 4))) {
        const int wgs = two_hop_workgroups(threads / kWave, Y_BF16, a.k);
        lds = wgs == 1 ? kOverHalfLds : (size_t)(128 / wgs) * 1280;
    }
    launch_two_hop_as<Y_BF16, OUT_BF16, kRowsAtOnce>(a, grid, block, lds, stores, partial, s);
}

// out[t] = sum_j w[t, j] * y[pair_slot[t * k + j]] for N tokens; arguments already checked
void combine_launch(const int32_t *pair_slot, int N, int k, const void *d_y, int y_dtype, const float *d_w,
                    void *d_out, int out_dtype, int32_t H, hipStream_t s, hipEvent_t e0 = nullptr,
                    hipEvent_t e1 = nullptr)
{
    CombineArgs a;
    a.y = (const u32x4 *)d_y;
    a.w = d_w;
    a.out = d_out;
    a.pair_slot = pair_slot;
    a.k = k;
    a.pair_send_row = nullptr; a.send_src = nullptr; a.n_rows_dev = nullptr;
    a.C = (int32_t)((size_t)H * (y_dtype == FUSCO_BF16 ? 2 : 4) / 16);
    a.first = combine_first_row(N, k, (size_t)a.C * 16);
    const OutStores how = out_stores((size_t)N * (size_t)k * (size_t)a.C * 16, d_out, (size_t)N, (size_t)H * (out_dtype == FUSCO_BF16 ? 2 : 4));
    if (y_dtype == FUSCO_BF16 && out_dtype == FUSCO_BF16) launch_combine<true, true>(a, N, how, s, e0, e1);
    else if (y_dtype == FUSCO_BF16) launch_combine<true, false>(a, N, how, s, e0, e1);
    else if (out_dtype == FUSCO_BF16) launch_combine<false, true>(a, N, how, s, e0, e1);
    else launch_combine<false, false>(a, N, how, s, e0, e1);
}

}   // namespace

#endif
