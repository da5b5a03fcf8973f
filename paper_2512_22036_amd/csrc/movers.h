// Mover kernels: fused gather-pack (dispatch), weighted combine, their two-hop and staged variants.
#ifndef FUSCO_CSRC_MOVERS_H
#define FUSCO_CSRC_MOVERS_H

#include "common.h"
#include "planner.h"

namespace {

// ------------------------------------------------------------------------------------------
// Movers.  A row is fetched or written whole by the waves of one workgroup within a short time.
// Measured on MI355X at 14 KiB rows: scattered row reads come close to the streaming read rate
// (6.4-6.6 of 7.2 TB/s), scattered row writes do not (5.2-5.4 of 6.9 TB/s), and what the write
// rate depends on is which XCD writes which neighbouring addresses.  Combine therefore walks the
// tokens (its scattered side is the reads), and dispatch writes in the planner's transfer order
// where it can (dispatch_tiled_kernel) and walks the tokens otherwise (dispatch_kernel).
// ------------------------------------------------------------------------------------------
__device__ __forceinline__ u32x4 load16_stream(const u32x4 *p) { return __builtin_nontemporal_load(p); }

// 16-byte / 8-byte write-through stores at device scope (sc1): the data leaves the L2 of the XCD for
// memory instead of lingering there.  Used for the token-ordered output of combine, which is never
// read again by this kernel.
// The s_nop supplies the wait states gfx9 needs between a store of more than 8 bytes and a
// following VALU write to its data registers; the compiler adds them for its own stores but
// cannot see into this statement.
__device__ __forceinline__ void store16_through(u32x4 *p, u32x4 v)
{
    asm volatile("global_store_dwordx4 %0, %1, off sc1\n\ts_nop 1" ::"v"(p), "v"(v) : "memory");
}
__device__ __forceinline__ void store8_through(u32x2 *p, u32x2 v)
{
    asm volatile("global_store_dwordx2 %0, %1, off sc1\n\ts_nop 1" ::"v"(p), "v"(v) : "memory");
}
// Write-through and non-temporal together (sc1 nt): the tiled dispatch's destination rows.  Measured against
// the plain non-temporal store at 8192 tokens x 8 rows of 14 KiB: 169 us instead of 174 us in a loop over the same
// buffers, 160 us instead of 174 us after other traffic has gone through the memory-side cache, never slower.
__device__ __forceinline__ void store16_through_stream(u32x4 *p, u32x4 v)
{
    asm volatile("global_store_dwordx4 %0, %1, off sc1 nt\n\ts_nop 1" ::"v"(p), "v"(v) : "memory");
}
__device__ __forceinline__ void store8_through_stream(u32x2 *p, u32x2 v)
{
    asm volatile("global_store_dwordx2 %0, %1, off sc1 nt\n\ts_nop 1" ::"v"(p), "v"(v) : "memory");
}
// The same at system scope (sc0 sc1): for data that another agent may read once a flag says so.
__device__ __forceinline__ void store16_system(u32x4 *p, u32x4 v)
{
    asm volatile("global_store_dwordx4 %0, %1, off sc0 sc1\n\ts_nop 1" ::"v"(p), "v"(v) : "memory");
}

// Dispatch: the row is held in registers between the single read and the k (+ wire) writes.
// Slot lookups depend only on blockIdx, so they are scalar loads.
struct DispatchArgs {
    const u32x4 *x, *x_aux;
    u32x4 *expert_buf, *expert_aux, *send_buf, *send_aux;
    const int32_t *pair_slot, *pair_send_row;
    const uint8_t *pair_first;
    const int32_t *slot_token, *tile_slots;   // tiled mode: transfer order of every tile
    int32_t tile_cap;                         // entries per tile in tile_slots
    int32_t tile_tokens;                      // tokens per tile
    int32_t N;                                // tokens in all
    int32_t segs;                             // workgroups per row: a row longer than a workgroup covers is cut into columns
    int32_t seg_chunks;                       // 16-byte chunks per column segment (the last one may be shorter)
    int32_t k;
    int32_t C, Ca;   // 16-byte chunks per row in the main and in the aux plane
    int32_t write_expert, write_wire;
    const int32_t *send_off;                  // tiled mode with the wire tensor: first send row of every device
    int32_t D;
    int32_t through, through_aux;   // tiled mode: expert rows (of the main and of the aux plane) start on 64-byte boundaries
};

constexpr int kTiledMinTiles = 2 * kXcds;                 // fewer tiles would leave XCDs idle
constexpr size_t kTiledMaxTileBytes = (size_t)3840 << 10; // source rows of one tile must fit a 4 MB L2
constexpr size_t kSourceChunkBytes = (size_t)128 << 20;   // source rows of one chunk: half the 256 MB memory-side cache
constexpr size_t kCacheBytes = (size_t)256 << 20;         // the memory-side cache
constexpr size_t kTiledShortRowBytes = 8192;              // rows below this are tiled only with a small source tensor

// Loads and stores of the token walk (MODE of dispatch_kernel: bit 0 cached loads, bit 1 non-temporal stores, bit 2 stores through the L2).
// Non-temporal stores go past the memory-side cache (a read that follows such a write runs at the cold rate,
// 5.7 TB/s for 256 MB, instead of 4.2 TB/s on rows that sit dirty in that cache); plain stores leave the rows
// there, which is what a reader of a tensor of up to 256 MB wants.  With non-temporal stores a source tensor
// that fits that cache is read with plain cached loads and stays there from one call to the next, since
// nothing the kernel writes displaces it (8192 tokens x 8 rows of 14 KiB: 187 us instead of 208 us; non-temporal
// loads together with non-temporal stores take 215 us there); a larger one is read with non-temporal loads
// (32768 tokens x 2 rows of 8 KiB: 138 us, against 168 us with cached loads).  walk_mode in fusco.hip chooses.
template <bool STREAM>
__device__ __forceinline__ void put16(u32x4 *p, u32x4 v)
{
    if constexpr (STREAM) __builtin_nontemporal_store(v, p);
    else *p = v;
}

// Bit 2: rows written through the L2 at once, instead of being written back when the kernel ends.
template <int MODE>
__device__ __forceinline__ void put_row(u32x4 *p, u32x4 v)
{
    if constexpr (MODE & 4) store16_through(p, v);
    else put16<(MODE & 2) != 0>(p, v);
}

template <int CPT, int MODE>
__global__ __launch_bounds__(256) void dispatch_kernel(DispatchArgs a)
{
    // workgroup = (token, column segment), segments of one row next to each other in launch order, so that a
    // row longer than one workgroup covers is still read and written as a whole within a short time
    const int t = blockIdx.x / (uint32_t)a.segs, seg = blockIdx.x - (uint32_t)t * a.segs;
    const int Ct = a.C + a.Ca;
    const int c_end = min(Ct, (seg + 1) * a.seg_chunks);   // this segment: chunks [seg * seg_chunks, c_end)
    const int c0 = seg * a.seg_chunks + threadIdx.x;
    u32x4 v[CPT];
#pragma unroll
    for (int i = 0; i < CPT; ++i) {
        const int c = c0 + i * blockDim.x;
        const u32x4 *src = c < a.C ? a.x + (size_t)t * a.C + c : a.x_aux + (size_t)t * a.Ca + (c - a.C);
        if (c < c_end) v[i] = (MODE & 1) ? *src : load16_stream(src);
    }
    const int32_t *slots = a.pair_slot + (size_t)t * a.k;
    if (a.write_expert) {
        for (int j = 0; j < a.k; ++j) {
            const int slot = slots[j];
            if (slot < 0) continue;
#pragma unroll
            for (int i = 0; i < CPT; ++i) {
                const int c = c0 + i * blockDim.x;
                if (c >= c_end) continue;
                if (c < a.C) put_row<MODE>(a.expert_buf + (size_t)slot * a.C + c, v[i]);
                else put_row<MODE>(a.expert_aux + (size_t)slot * a.Ca + (c - a.C), v[i]);
            }
        }
    }
    if (a.write_wire) {
        const int32_t *rows = a.pair_send_row + (size_t)t * a.k;
        const uint8_t *first = a.pair_first + (size_t)t * a.k;
        for (int j = 0; j < a.k; ++j) {
            if (!first[j]) continue;
            const int row = rows[j];
#pragma unroll
            for (int i = 0; i < CPT; ++i) {
                const int c = c0 + i * blockDim.x;
                if (c >= c_end) continue;
                if (c < a.C) put_row<MODE>(a.send_buf + (size_t)row * a.C + c, v[i]);
                else put_row<MODE>(a.send_aux + (size_t)row * a.Ca + (c - a.C), v[i]);
            }
        }
    }
}

// The token walk of few workgroups: the token's slots (and send rows) come into the lanes of a wave with one load, and its rows are stored
// without a wait between them.  In dispatch_kernel a slot is looked up when its row is stored, and that load waits for the stores before it
// (loads and stores share a counter): every workgroup has one row on its way at a time.  With few workgroups the waits are what the call
// takes (with them / here, us: 300 tokens x 8 x 14 KiB 9.3 / 7.7, 500 11.7 / 10.1, 400 x 8 x 4.1 KiB in two planes 5.3 / 4.2, 700 x 8 x 2
// KiB 5.1 / 3.8); where there are many, memory is faster with fewer rows being written at a time (8192 x 8 x 2 KiB 29.2 / 30.4, 4000 x 4 x
// 4.1 KiB in two planes 14.3 / 15.7, 32768 x 4 x 7 KiB 229 / 232).  Between 1024 and 4000 workgroups short rows are still faster this way
// and long ones are not (2443 x 8 x 496 B 7.9 / 5.5, 2181 x 10 x 1504 B 7.5 / 6.8, 1058 x 4 x 1568 B 3.3 / 2.9, but 3244 x 8 x 3 KiB 13.7 /
// 14.8, 1838 x 8 x 8.4 KiB 30.5 / 31.6, 1487 x 6 x 12.5 KiB 26.5 / 28.6): the line is where none is slower.
constexpr uint64_t kWalkEagerGroups = 1024;

// The same for send rows alone, by workgroups (a row may take several), tokens, entries, devices and 16-byte chunks of a row; with the
// waits / without, us.  Without them are faster:
// - up to 1200 workgroups (1120 tokens x 6 x 4176 B on 4 devices 5.8 / 5.3; 1417 x 8 x 10.5 KiB on 16 23.5 / 26.1);
// - rows of up to 1.5 KiB, where the look-ups count (24723 x 8 x 432 B on 8 25.4 / 19.2, 22730 x 8 x 1296 B on 16 81.8 / 66.9, 6294 x 8 x 1424 B
//   on 4 11.8 / 10.1; 15757 x 16 x 832 B on 8 22.1 / 23.2), of up to 2 KiB from 6000 tokens on (53347 x 8 x 1696 B on 16, two hops, 540 / 490,
//   8983 x 10 x 2016 B on 4 19.3 / 15.1, 29171 x 10 x 1568 B on 8 71.4 / 73.2; 3729 x 8 x 1760 B on 16 10.0 / 11.4);
// - few rows of many entries (27147 x 6 x 1488 B on two 30.0 / 21.3, 1108 x 8 x 3824 B on two 4.2 / 3.6), longer ones from 3000 workgroups on
//   (2748 x 10 x 19 KiB on one, 5496 workgroups, 23.7 / 19.5, 3344 x 16 x 8 KiB on two 16.6 / 15.3; 2100 x 8 x 10 KiB on one 9.5 / 10.0);
// - rows of 12 to 16 KiB of 4000 tokens and more (4400 x 8 x 13.7 KiB on 16 110 / 104, 10356 x 8 x 12.9 KiB on 8 198 / 189);
// - of tokens with one entry those of 4800 B and more (9367 x 4896 B 17.7 / 16.4; 7476 x 2864 B 10.0 / 10.5, 6931 x 704 B 4.2 / 4.5).
// The others are faster with them (13477 x 8 x 3 KiB on 8 58.7 / 61.9, 2191 x 8 x 6 KiB on 8 14.0 / 15.6, 1787 x 2 x 10.3 KiB on one 8.2 / 9.4,
// 1350 x 8 x 8.5 KiB on two 8.5 / 9.0, 27369 x 2 x 19 KiB on 8 300 / 309).
inline bool eager_send_rows(uint64_t groups, int N, int k, int D, int chunks)
{
    if (groups <= 1200) return true;
    if (k == 1) return chunks >= 300;
    if (chunks <= 96 || (chunks <= 128 && N >= 6000)) return true;
    if (k >= 3 * D && (chunks <= 256 || groups >= 3000)) return true;
    return chunks >= 768 && chunks <= 1024 && N >= 4000;
}

template <int CPT, int MODE>
__global__ __launch_bounds__(256) void dispatch_eager_kernel(DispatchArgs a)
{
    const int t = blockIdx.x / (uint32_t)a.segs, seg = blockIdx.x - (uint32_t)t * a.segs;
    const int c_end = min(a.C + a.Ca, (seg + 1) * a.seg_chunks);
    const int c0 = seg * a.seg_chunks + threadIdx.x;
    // entry j's slot and send row in lane j; -1: none
    const int lane = threadIdx.x & (kWave - 1);
    int my_slot = -1, my_row = -1;
    if (lane < a.k) {
        const size_t p = (size_t)t * a.k + lane;
        if (a.write_expert) my_slot = a.pair_slot[p];
        if (a.write_wire && a.pair_first[p]) my_row = a.pair_send_row[p];
    }
    u32x4 v[CPT];
#pragma unroll
    for (int i = 0; i < CPT; ++i) {
        const int c = min(c0 + i * (int)blockDim.x, c_end - 1);   // no branch between the loads: threads past the segment read its last chunk
        const u32x4 *src = a.x + (size_t)t * a.C + c;
        if (c >= a.C) src = a.x_aux + (size_t)t * a.Ca + (c - a.C);
        v[i] = (MODE & 1) ? *src : load16_stream(src);
    }
    const auto store_all = [&](int mine, u32x4 *rows, u32x4 *rows_aux) {
        for (uint64_t left = __builtin_amdgcn_ballot_w64(mine >= 0); left; left &= left - 1) {
            const int row = __builtin_amdgcn_readlane(mine, __builtin_ctzll(left));
#pragma unroll
            for (int i = 0; i < CPT; ++i) {
                const int c = c0 + i * blockDim.x;
                u32x4 *dst = rows + (size_t)row * a.C + c;
                if (c >= a.C) dst = rows_aux + (size_t)row * a.Ca + (c - a.C);
                if (c < c_end) put16<(MODE & 2) != 0>(dst, v[i]);
            }
        }
    };
    store_all(my_slot, a.expert_buf, a.expert_aux);
    store_all(my_row, a.send_buf, a.send_aux);
}

// Dispatch in transfer order (the tile_slots list of the planner): one workgroup per destination row.  The
// hardware hands workgroups to the 8 XCDs in turn, so workgroup b = 8 i + x runs on XCD x; it takes entry
// i mod cap of tile x + 8 (i / cap).  An XCD therefore works through whole tiles, one after the other, and
// inside a tile it writes expert by expert: the rows of one expert are neighbours in memory, written by one
// XCD within a short time.  Every source row is needed k times by the tile; it comes from memory once and
// from the XCD's L2 afterwards (plain cached loads; a tile's source rows, or the column segment of them that
// a pass moves, fit the L2).  The rows are written with non-temporal write-through stores
// (store16_through_stream): they do not displace the source rows from the L2 - the fabric counters show
// every source row fetched 1.03 times, against 1.4 times with plain non-temporal stores - and they go past
// the memory-side cache, which the next reader of memory would otherwise have to clean first and which so
// keeps a source tensor that fits it from one call to the next.  The reads are hidden completely: the kernel
// runs at the rate of its write pattern, and that rate goes up when fewer rows are being written at a time.
// The launch therefore caps the workgroups per compute unit for long rows (tiled_workgroups_per_cu: dynamic LDS
// that the kernel does not use).  Measured on MI355X at 8192 tokens x 8 rows of 14 KiB, source tensor in the
// memory-side cache / cold in memory: 8 workgroups per compute unit 164 / 203 us, 5 workgroups 151 / 222 us,
// 5 workgroups with PULL 157 / 178 us.  The token walk takes 205 us with non-temporal loads and plain stores
// and 187 us with cached loads and non-temporal stores.
// PULL: the first tile_tokens workgroups of a pass also read one source row of the tile each (see below).
// AUX: the second plane exists.  A chunk's source and destination are picked by address selection, not by
// branching, so that the loads of a thread are issued back to back (a branch per chunk costs 3 % here).
// WIRE: the per-device receive tensors are written too.  After its pairs a tile has one entry
// per device and token, device by device: the send rows of a tile's tokens on a device are neighbours, so an XCD writes
// runs of up to tile_tokens rows, from source rows that are still in its L2; an entry whose token has no row on the
// device does nothing.  4096 tokens x 8 rows of 14 KiB on 8 devices (21700 send rows), both tensors: 143 us, 157 us by
// the token walk; in a step 392 against 417 us.
// The launch covers the tiles [tile_base, tile_base + tiles_here).
template <int CPT, bool AUX, bool PULL, bool WIRE>
__global__ __launch_bounds__(256) void dispatch_tiled_kernel(DispatchArgs a, uint32_t tile_base, uint32_t tiles_here)
{
    // a tile is worked through a.segs times, once per column segment of the rows (one pass for rows that a
    // workgroup covers): the L2 then only has to hold that segment of the tile's source rows
    const uint32_t b = blockIdx.x, x = b & (kXcds - 1), i = b / kXcds;
    const uint32_t pairs = (uint32_t)a.tile_cap;
    const uint32_t entries = WIRE ? pairs + (uint32_t)a.D * (uint32_t)a.tile_tokens : pairs;
    const uint32_t per_tile = entries * (uint32_t)a.segs;
    const uint32_t round = i / per_tile, w = i - round * per_tile;
    const uint32_t pass = w / entries, r = w - pass * entries;
    const uint32_t local = x + kXcds * round;
    if (local >= tiles_here) return;
    const uint32_t tile = tile_base + local;
    const bool wire = WIRE && r >= pairs;
    // destination row, in the expert or in the wire tensor, and source token; -1: nothing to move
    int row = -1, t = 0;
    if (!wire) {
        row = a.tile_slots[(size_t)tile * a.tile_cap + r];
    } else {
        const uint32_t q = r - pairs, d = q / (uint32_t)a.tile_tokens;
        t = (int)(tile * (uint32_t)a.tile_tokens + (q - d * (uint32_t)a.tile_tokens));
        if (t < a.N) {
            // the token's entry for the device, by the device's range of send rows
            const int lo = a.send_off[d], hi = a.send_off[d + 1];
            const int32_t *rows = a.pair_send_row + (size_t)t * a.k;
            for (int j = 0; j < a.k; ++j) {
                const int s = rows[j];
                row = s >= lo && s < hi ? s : row;
            }
        }
    }
    u32x4 *const out = wire ? a.send_buf : a.expert_buf, *const out_aux = wire ? a.send_aux : a.expert_aux;
    const int Ct = AUX ? a.C + a.Ca : a.C;
    // PULL: the first tile_tokens workgroups of a pass also read one source row of the tile each (the segment
    // of it that this pass moves) and drop it.  All of the tile's source rows are then on their way to the L2
    // while the tile's first entries are written, instead of every first use of a row waiting for memory in its
    // own workgroup: with few workgroups per compute unit that wait is what a cold source tensor costs.
    const int tp = (int)(tile * (uint32_t)a.tile_tokens + r);
    const bool pull = PULL && r < (uint32_t)a.tile_tokens && tp < a.N;
    // which segment a pass moves rotates with the token: the segments in use during a pass then lie at different
    // offsets in their rows, and rows whose size is a power of two do not all fall on the same sets of the L2
    const auto segment = [&](int token) { return a.segs > 1 ? (pass + (uint32_t)token) % (uint32_t)a.segs : 0u; };
    // A thread requests the chunks of its own row one after the other, each when the one before has arrived, and a plain dispatch
    // requests the pulled row before them: a workgroup then spends longer on its loads and fewer of them are storing at any
    // moment.  Steps with the chunks requested at once / one after the other, us: 8192 x 8 x 14 KiB 377 / 363, in two planes of 7.2 KiB
    // 277 / 273, 32768 x 8 x 14 KiB 1452 / 1407.  With the receive tensors the pulled row comes last, and threads past the
    // segment's end read its last chunk with the others instead of branching around it (4096 x 8 x 14 KiB 376; 380 as above).
    const auto load = [&](u32x4 (&v)[CPT], int token, uint32_t seg, bool own) {
        const int c_end = min(Ct, (int)(seg + 1) * a.seg_chunks), c0 = seg * a.seg_chunks + threadIdx.x;
#pragma unroll
        for (int q = 0; q < CPT; ++q) {
            const int at = c0 + q * (int)blockDim.x, c = WIRE ? min(at, c_end - 1) : at;
            const u32x4 *src = a.x + (size_t)token * a.C + c;
            if (AUX && c >= a.C) src = a.x_aux + (size_t)token * a.Ca + (c - a.C);
            if (!WIRE && c >= c_end) continue;
            v[q] = *src;
            if (own) __builtin_amdgcn_s_waitcnt(0x0f70);   // vmcnt(0)
        }
    };
    u32x4 v[CPT], p[CPT];
    uint32_t seg = 0;
    if (!WIRE && pull) load(p, tp, segment(tp), false);
    if (row >= 0) {
        if (!wire) t = a.slot_token[row];
        seg = segment(t);
        load(v, t, seg, true);
    }
    const auto store = [&] {
        const int c_end = min(Ct, (int)(seg + 1) * a.seg_chunks), c0 = seg * a.seg_chunks + threadIdx.x;
#pragma unroll
        for (int q = 0; q < CPT; ++q) {
            const int c = c0 + q * blockDim.x;
            u32x4 *dst = out + (size_t)row * a.C + c;
            if (AUX && c >= a.C) dst = out_aux + (size_t)row * a.Ca + (c - a.C);
            if (c >= c_end) continue;
            if (AUX && c >= a.C ? a.through_aux : a.through) store16_through_stream(dst, v[q]);
            else __builtin_nontemporal_store(v[q], dst);
        }
    };
    if (WIRE && pull) load(p, tp, segment(tp), false);
    if (row >= 0) store();
    if (!pull) return;
#pragma unroll
    for (int q = 0; q < CPT; ++q) asm volatile("" ::"v"(p[q]));   // the value is not used: only the read matters
}

// Reads n 16-byte units once, 4 KiB per workgroup in address order, and drops them: afterwards they sit in the
// memory-side cache.  The tiled dispatch of a source tensor larger than half that cache runs it over the source rows
// of the next chunk of tiles, so that they reach memory as one sequential burst of reads, with no writes in
// flight, instead of trickling out between the writes (measured at 32 Ki tokens of 14 KiB, chunks of 32 tiles:
// 760 us instead of 824 us; as part of the tiled kernel's own launch the reads did not help).
__global__ __launch_bounds__(256) void touch_kernel(const u32x4 *src, size_t n)
{
    const size_t i = (size_t)blockIdx.x * 256 + threadIdx.x;
    if (i >= n) return;
    const u32x4 v = src[i];
    asm volatile("" ::"v"(v));   // the value is not used: only the read matters
}

// Planner and dispatch in one launch for inputs of a single planner tile (decode-sized batches, where dependent
// launches cost more than the work).  Workgroup 0 writes the counts, the next a.small_groups workgroups the
// descriptors (plan_small_kernel's work), and one workgroup per token finds the slots of its own pairs and moves its
// row there; none waits for another.  The row is requested before the slots are worked out, so that its latency hides
// behind that.  Bound by the chain routing -> slots -> stores of one workgroup.  Kernel time, k = 8, 4 / 128 tokens of
// 7392 B (two planes, D = 64) and 256 tokens of 4 KiB (D = 8): 5.0 / 6.6 / 7.3 us; 5.8 / 7.9 / 8.2 us with the
// descriptors written by the tokens' own workgroups after their rows; 9.9 / 11.4 / 13.0 us with counters and scans over
// the keys in every workgroup.
// A row longer than a workgroup holds is cut into column segments, each with a workgroup (blockIdx.y) that finds the
// slots for itself.  k = 8, against one workgroup that loops over its row after the first 32 KiB: 4 tokens of 128 KiB
// 20.6 -> 6.3 us, 1 MiB 198 -> 11; 128 tokens of 40 KiB 14.5 -> 10.8 us, 128 KiB 47 -> 31; 256 tokens of 64 KiB 35.6 -> 31.0 us.
// (Finding the slots twice costs more than it gives for many tokens of little more than 32 KiB: 500 tokens with k = 4 of 33 KiB
// 16.0 -> 20.4 us, 64 KiB 37.2 -> 34.1 us.)
// CPT: 16-byte chunks of the row (or of its segment) per thread, as few as cover it; AUX: the second plane exists.  Chosen at
// compile time because every store of a slot is a branch of its own otherwise: CPT 4 and both planes always / as here, k = 8, us: 4
// tokens of 14 KiB 4.9 / 3.9, of 7392 B in two planes 4.5 / 4.2, 128 tokens 7.1 / 6.2 and 5.7 / 5.4; 1000 x 2 x 1 KiB 9.2 / 7.8.
constexpr int kFusedChunks = 4;   // most chunks per thread held in registers across the planning: 32 KiB a workgroup

// What a token's workgroup needs first are arguments of their own: they are all read at the start of the kernel, where members of a
// structure were read branch by branch, each after a wait (4 tokens of 14 KiB 3.85 -> 3.5 us, 128 tokens 6.1 -> 5.9).
struct FusedRows {
    u32x4 *expert_buf, *expert_aux;
};

// plan_dispatch_four_kernel: 80 scalar registers at most.  With more a SIMD holds seven of its eight waves, and a compute unit three
// workgroups instead of four.  Calls of a little more than 3 x 256 workgroups then take a second round of them (us, three / four: 682
// tokens x 3 x 16 KiB, 939 workgroups, 12.4 / 9.9; 800 x 2 x 12 KiB, 1001, 9.9 / 8.3; with CPT 4 682 x 3 x 20 KiB 14.5 / 11.3, 300 x 6 x 40
// KiB 18.0 / 16.2, 2048 x 1 x 32 KiB 27.2 / 24.9).  The registers are missed by calls of few tokens with many entries (3 x 33 x 1 KiB 6.3 /
// 6.6), and of more than 1024 workgroups memory is faster with fewer of them writing (1024 x 2 x 16 KiB, 1281 workgroups, 12.0 / 14.4).
constexpr int kFusedThree = 3 * 256, kFusedFour = 4 * 256;   // workgroups that are resident at once

template <int CPT, bool AUX, bool THROUGH>
__device__ __forceinline__ void plan_dispatch(SmallLds &s, const int32_t *A, const u32x4 *x, const u32x4 *x_aux, int32_t N, int32_t k, uint32_t k_magic,
                                              int32_t small_groups, int32_t C, int32_t Ca, int32_t seg_chunks, FusedRows m, PlanArgs a)
{
    a.A = A;
    a.N = N;
    a.k = k;
    a.k_magic = k_magic;
    a.small_groups = small_groups;
    const int b = blockIdx.x, seg = blockIdx.y;
    if (b <= a.small_groups) {
        if (seg != 0) return;
        const int p0 = (b - 1) * kSmallPairs;
        if (b == 0) small_counts(s, a);
        else small_place(s, a, p0, min(kSmallPairs, a.N * a.k - p0));
        return;
    }
    const int tid = threadIdx.x;
    const int t = b - 1 - a.small_groups;
    const int c0 = seg * seg_chunks + tid, c_end = min(C + Ca, (seg + 1) * seg_chunks);
    // source and destination of a chunk by address selection: c counts on from the main row's chunks into the aux row's
    const u32x4 *src = x + (size_t)t * C, *src_aux = x_aux + (size_t)t * Ca - C;
    u32x4 v[CPT];
#pragma unroll
    for (int i = 0; i < CPT; ++i) {
        const int c = c0 + i * kSmallThreads;
        if (c < c_end) v[i] = load16_stream((!AUX || c < C ? src : src_aux) + c);
    }
    const int slots = small_slots(s, a, t * a.k, a.k);
    for (int j = 0; j < a.k; ++j) {
        const int slot = __builtin_amdgcn_readlane(slots, j);
        if (slot < 0) continue;
        u32x4 *dst = m.expert_buf + (size_t)slot * C, *dst_aux = m.expert_aux + (size_t)slot * Ca - C;
#pragma unroll
        for (int i = 0; i < CPT; ++i) {
            const int c = c0 + i * kSmallThreads;
            if (c >= c_end) continue;
            if (AUX && c >= C) dst_aux[c] = v[i];   // rows of scales: short, and rarely whole units
            else if (THROUGH) store16_through(dst + c, v[i]);
            else dst[c] = v[i];
        }
    }
}

// THROUGH: the rows are written through instead of plain: the write-back at the kernel's end is spread over the kernel, as in the token walk.
#define FUSCO_PLAN_DISPATCH(NAME, ATTRIBUTE)                                                                                                          \
    template <int CPT, bool AUX, bool THROUGH>                                                                                                        \
    __global__ __launch_bounds__(kSmallThreads) ATTRIBUTE void NAME(const int32_t *A, const u32x4 *x, const u32x4 *x_aux, int32_t N, int32_t k,       \
                                                                    uint32_t k_magic, int32_t small_groups, int32_t C, int32_t Ca, int32_t seg_chunks, \
                                                                    FusedRows m, PlanArgs a)                                                          \
    {                                                                                                                                                 \
        __shared__ SmallLds s;                                                                                                                        \
        plan_dispatch<CPT, AUX, THROUGH>(s, A, x, x_aux, N, k, k_magic, small_groups, C, Ca, seg_chunks, m, a);                                                \
    }
FUSCO_PLAN_DISPATCH(plan_dispatch_kernel, )
FUSCO_PLAN_DISPATCH(plan_dispatch_four_kernel, __attribute__((amdgpu_num_sgpr(80))))
#undef FUSCO_PLAN_DISPATCH

// Stores of combine's output rows (out_stores chooses).  A template argument of the kernels: with a choice between the four
// at every store the two-hop combine of 4 tokens x 8 rows of 14 KiB took 7.4 us instead of 6.1, of 256 tokens of 5.6 KiB 12.2
// instead of 10.8 us, the combine of 2048 x 1 x 8 KiB 7.8 instead of 7.5 us.
enum OutStores : int32_t { kOutThrough, kOutThroughStream, kOutNonTemporal, kOutPlain };

template <OutStores HOW, typename V>
__device__ __forceinline__ void put_out(V *p, V v)
{
    if constexpr (HOW == kOutThrough) {
        if constexpr (sizeof(V) == 16) store16_through(p, v);
        else store8_through(p, v);
    } else if constexpr (HOW == kOutThroughStream) {
        if constexpr (sizeof(V) == 16) store16_through_stream(p, v);
        else store8_through_stream(p, v);
    } else if constexpr (HOW == kOutNonTemporal) {
        __builtin_nontemporal_store(v, p);
    } else {
        *p = v;
    }
}

__device__ __forceinline__ float bf16_lo(uint32_t u) { return __uint_as_float(u << 16); }
__device__ __forceinline__ float bf16_hi(uint32_t u) { return __uint_as_float(u & 0xFFFF0000u); }

// fp32 -> bfloat16 bits, round to nearest even, NaN kept quiet
__device__ __forceinline__ uint32_t to_bf16(float f)
{
    const uint32_t u = __float_as_uint(f);
    if ((u & 0x7FFFFFFFu) > 0x7F800000u) return (u >> 16) | 0x40u;
    return (u + 0x7FFFu + ((u >> 16) & 1u)) >> 16;
}

// The 16 bytes of a row of C chunks that a thread takes, c: the thread's number in the row.  WIDENED, for rows of bf16 that become rows of
// fp32, twice as long: 8 bytes in each half of the wave's 1 KiB, so that the 16 bytes of floats stored for each lie next to the
// neighbour lanes' and a store of the wave covers 1 KiB of whole lines.  Read in one piece, the floats have to be exchanged between lanes
// (put_floats) before their stores cover whole lines; that is the better one where loads and not stores are what counts.  A thread past
// the row reads the row's last bytes and stores nothing.
// Stores that covered every other 64 bytes of their lines had to meet in the L2: the two-hop combine of 4096 tokens x 8 x 14 KiB wrote its
// partial rows plain in 226 us, through in 247, past the cache in 296; now 222, 217 and 215 (through and past the cache).
struct WidenedPart {
    int at[2];    // units of 8 bytes of the row of bf16, which are chunks of the row of floats
    bool in[2];
    __device__ __forceinline__ WidenedPart(int c, int C)
    {
        const int u = (c & ~(kWave - 1)) * 2 + (c & (kWave - 1));
#pragma unroll
        for (int h = 0; h < 2; ++h) {
            in[h] = u + h * kWave < 2 * C;
            at[h] = min(u + h * kWave, 2 * C - 1);
        }
    }
    __device__ __forceinline__ u32x4 load(const u32x4 *row) const
    {
        const u32x2 lo = __builtin_nontemporal_load((const u32x2 *)row + at[0]), hi = __builtin_nontemporal_load((const u32x2 *)row + at[1]);
        return u32x4{lo[0], lo[1], hi[0], hi[1]};
    }
    // the thread's sums in the output's row, as floats or rounded to bf16
    template <OutStores HOW>
    __device__ __forceinline__ void store_f32(u32x4 *row, const float (&f)[8]) const
    {
#pragma unroll
        for (int h = 0; h < 2; ++h) {
            const u32x4 o = {__float_as_uint(f[4 * h]), __float_as_uint(f[4 * h + 1]), __float_as_uint(f[4 * h + 2]), __float_as_uint(f[4 * h + 3])};
            if (in[h]) put_out<HOW>(row + at[h], o);
        }
    }
    template <OutStores HOW>
    __device__ __forceinline__ void store_bf16(u32x2 *row, const float (&f)[8]) const
    {
#pragma unroll
        for (int h = 0; h < 2; ++h) {
            const u32x2 o = {to_bf16(f[4 * h]) | to_bf16(f[4 * h + 1]) << 16, to_bf16(f[4 * h + 2]) | to_bf16(f[4 * h + 3]) << 16};
            if (in[h]) put_out<HOW>(row + at[h], o);
        }
    }
};

// The same for rows whose sums keep their place: chunk c.
struct PlainPart {
    int c;
    bool in[1];
    __device__ __forceinline__ PlainPart(int c_, int C) : c(c_), in{c_ < C} {}
    __device__ __forceinline__ u32x4 load(const u32x4 *row) const { return load16_stream(row + c); }
};
template <bool WIDENED>
using Part = std::conditional_t<WIDENED, WidenedPart, PlainPart>;

// The eight floats of chunk c of a bf16 row, as chunks 2 c and 2 c + 1 of an fp32 row of n chunks.  Stored as they are, the lanes of a
// wave would write every other 16 bytes twice.  Exchanged inside quads of lanes, each of the two stores covers whole 64-byte units; unless the
// stores are plain and meet in the L2, the second store of even quads and the first one of odd quads change places, and each covers
// lines of 128 bytes (combine to fp32 rows, in 64 / 128 bytes, us: 10911 tokens x 4 x 13.4 KiB 157 / 147, 2469 x 2 x 1536 B 5.1 / 4.3, 5030 x 8 x
// 5760 B 52.0 / 50.9).  Every lane of the wave takes part, also those whose chunk lies past the row.
template <OutStores HOW>
__device__ __forceinline__ void put_floats(u32x4 *row, int c, int n, const float (&f)[8])
{
    u32x4 quad[2];
#pragma unroll
    for (int q = 0; q < 4; ++q) {
        const int lo = (int)__float_as_uint(f[q]), hi = (int)__float_as_uint(f[4 + q]);
        // lane j of a quad gets chunk j of the quad's first (second) four: the half j mod 2 of lane j / 2 (2 + j / 2)
        const int lo0 = __builtin_amdgcn_update_dpp(0, lo, 0x50, 0xf, 0xf, true), hi0 = __builtin_amdgcn_update_dpp(0, hi, 0x50, 0xf, 0xf, true);
        const int lo1 = __builtin_amdgcn_update_dpp(0, lo, 0xFA, 0xf, 0xf, true), hi1 = __builtin_amdgcn_update_dpp(0, hi, 0xFA, 0xf, 0xf, true);
        quad[0][q] = (uint32_t)((c & 1) ? hi0 : lo0);
        quad[1][q] = (uint32_t)((c & 1) ? hi1 : lo1);
    }
    if constexpr (HOW == kOutPlain) {
#pragma unroll
        for (int h = 0; h < 2; ++h) {
            const int at = (c & ~3) * 2 + h * 4 + (c & 3);
            if (at < n) put_out<HOW>(row + at, quad[h]);
        }
        return;
    }
    u32x4 o[2];
#pragma unroll
    for (int q = 0; q < 4; ++q) {
        o[0][q] = (uint32_t)__builtin_amdgcn_update_dpp((int)quad[0][q], (int)quad[1][q], 0x114, 0xf, 0xa, false);   // odd quads: from four lanes below
        o[1][q] = (uint32_t)__builtin_amdgcn_update_dpp((int)quad[1][q], (int)quad[0][q], 0x104, 0xf, 0x5, false);   // even quads: from four lanes above
    }
#pragma unroll
    for (int h = 0; h < 2; ++h) {
        const int at = (c & ~7) * 2 + h * 8 + (c & 7);
        if (at < n) put_out<HOW>(row + at, o[h]);
    }
}

// Combine: every thread owns a 16-byte chunk of y's rows, pulls that chunk of the token's k rows and accumulates in fp32
// with one fused multiply-add per term in ascending j.
struct CombineArgs {
    const u32x4 *y;
    const float *w;
    void *out;
    const int32_t *pair_slot;
    int32_t k;
    int32_t C;   // 16-byte chunks per y row
    int32_t first;   // row handled by workgroup 0; the walk goes upwards from there and wraps around
    int32_t n_rows;  // rows of the walk (tokens, or send rows in the per-send-row mode)
    int32_t segs;    // workgroups per row: the columns of a row longer than one workgroup covers
    // per-send-row mode (level 2 reversed): one workgroup per send row, only the token's entries on that row
    const int32_t *pair_send_row, *send_src, *n_rows_dev;
};

// acc += w * v, one fused multiply-add per element
template <bool Y_BF16, int EPC>
__device__ __forceinline__ void add_row(float (&acc)[EPC], u32x4 v, float w)
{
    if constexpr (Y_BF16) {
#pragma unroll
        for (int q = 0; q < 4; ++q) {
            acc[2 * q] = __builtin_fmaf(w, bf16_lo(v[q]), acc[2 * q]);
            acc[2 * q + 1] = __builtin_fmaf(w, bf16_hi(v[q]), acc[2 * q + 1]);
        }
    } else {
#pragma unroll
        for (int q = 0; q < 4; ++q) acc[q] = __builtin_fmaf(w, __uint_as_float(v[q]), acc[q]);
    }
}

// The next JU entries of `left`: all their loads without a branch or a wait between them, then the sums.
template <bool Y_BF16, int JU, int EPC, typename PART>
__device__ __forceinline__ void combine_rows(const CombineArgs &a, uint64_t &left, int my_slot, float my_w, const PART &part, float (&acc)[EPC])
{
    u32x4 v[JU];
    float wj[JU];
    const u32x4 *row[JU];
#pragma unroll
    for (int jj = 0; jj < JU; ++jj) {
        const int j = __builtin_ctzll(left);
        left &= left - 1;
        row[jj] = a.y + (size_t)__builtin_amdgcn_readlane(my_slot, j) * a.C;
        wj[jj] = __uint_as_float(__builtin_amdgcn_readlane(__float_as_uint(my_w), j));
    }
    if (part.in[0]) {
#pragma unroll
        for (int jj = 0; jj < JU; ++jj) v[jj] = part.load(row[jj]);
    }
#pragma unroll
    for (int jj = 0; jj < JU; ++jj) add_row<Y_BF16>(acc, v[jj], wj[jj]);
}

// JU: rows of a token that a thread has in flight.
// 4 or 8 (inputs bound by latency): slots and weights come into the lanes of a wave with one load each, and the rows are requested
// back to back.  Behind a branch per entry the compiler waited for each row before it requested the next (with those waits / without, us:
// 64 tokens x 8 x 14 KiB 6.0 / 3.1, 128 x 8 6.6 / 4.3, 1537 x 6 x 5760 B to fp32 15.5 / 13.9).
// 1 or 2 (inputs bound by memory, which is faster the fewer rows are being read at a time): slots and weights are scalar
// loads, which do not queue behind the rows, one step ahead of their use.  Rows in flight 1 / 2 / 4 / 8, us: 8192 x 8 x 14 KiB
// 173 / 180 / 184 / 181, 16384 x 8 x 8 KiB 203 / 210 / 211 / 212, 32768 x 8 x 14 KiB 700 / 750 / 754 / 744; two entries per
// token 20000 x 14 KiB 144 / 139 (slots in lanes instead: 155 with 1).
// kSpacedRows: eight rows, each slot looked up when the row before it has been requested.  The requests lie a scalar load apart, which is what
// inputs of fp32 rows between the two prefer (one after the other / in lanes, back to back / so, us: 5298 tokens x 5 x 1088 B 9.6 / 7.1 /
// 6.8, 1904 x 8 x 2976 B 9.5 / 9.7 / 9.1, 5151 x 3 x 3488 B 14.1 / 13.6 / 13.0).  Not for bf16 rows, whose sums take twice the registers: the
// compiler waits for a row before it reuses them for the next one's address.
// WIDENED: rows of bf16 to rows of fp32, one at a time or, in inputs bound by memory, the only two: a thread takes 8 bytes in two places
// (exchange / so, us: 23518 x 1 x 8736 B 121 / 103, 2804 x 1 x 2800 B 7.0 / 6.1, 5038 x 8 x 9040 B 84 / 79, 22618 x 2 x 5024 B 87 / 78).  With several in
// flight twice as many loads cost more than the exchange (399 x 8 x 2176 B 3.10 / 3.45, 595 x 12 x 14.2 KiB 24.2 / 26.2, 2469 x 2 x 1536 B 4.3 / 4.5).
constexpr int kSpacedRows = -8;

template <bool Y_BF16, bool OUT_BF16, int JU, OutStores STORES, bool PER_SEND_ROW = false, bool WIDENED = Y_BF16 && !OUT_BF16 && JU == 1>
__global__ __launch_bounds__(1024) void combine_kernel(CombineArgs a)
{
    constexpr int EPC = Y_BF16 ? 8 : 4;   // elements per 16-byte chunk of y
    // The walk starts at row a.first and wraps: when combine follows dispatch, the rows of the last
    // tokens are still in the memory-side cache, and reading them first, oldest first, finds them
    // there before the walk's own traffic pushes them out (see combine_first_row).
    // workgroup = (row, column segment), the segments of one row next to each other in launch order
    const int walk = blockIdx.x / (uint32_t)a.segs, seg = blockIdx.x - (uint32_t)walk * a.segs;
    int r = a.first + walk;   // token, or send row in the per-send-row mode
    if (r >= a.n_rows) r -= a.n_rows;
    int t = r;
    if constexpr (PER_SEND_ROW) {
        if (r >= *a.n_rows_dev) return;
        t = a.send_src[r];
    }
    const int c = seg * blockDim.x + threadIdx.x;
    const Part<WIDENED> part(c, a.C);
    float acc[EPC];
#pragma unroll
    for (int e = 0; e < EPC; ++e) acc[e] = 0.0f;

    if constexpr (JU == kSpacedRows) {
        const int32_t *slots = a.pair_slot + (size_t)t * a.k;
        const float *wt = a.w + (size_t)t * a.k;
        constexpr int ROWS = -kSpacedRows;
        for (int j0 = 0; j0 < a.k; j0 += ROWS) {
            u32x4 v[ROWS];
            float wj[ROWS];
            bool on[ROWS];
#pragma unroll
            for (int jj = 0; jj < ROWS; ++jj) {
                const int j = j0 + jj;
                on[jj] = false;
                if (j >= a.k) continue;
                const int slot = slots[j];
                wj[jj] = wt[j];
                if (slot < 0) continue;
                on[jj] = true;
                if (part.in[0]) v[jj] = part.load(a.y + (size_t)slot * a.C);
            }
#pragma unroll
            for (int jj = 0; jj < ROWS; ++jj)
                if (on[jj]) add_row<Y_BF16>(acc, v[jj], wj[jj]);
        }
    } else if constexpr (JU <= 2) {
        static_assert(!PER_SEND_ROW, "the entries of a send row are picked out in lanes");
        const int32_t *slots = a.pair_slot + (size_t)t * a.k;
        const float *wt = a.w + (size_t)t * a.k;
        int slot[JU], next_slot[JU];
        float wj[JU], next_w[JU];
        const auto look_up = [&](int j0, int (&sl)[JU], float (&w)[JU]) {
#pragma unroll
            for (int jj = 0; jj < JU; ++jj) {
                const int j = min(j0 + jj, a.k - 1);
                sl[jj] = j0 + jj < a.k ? slots[j] : -1;
                w[jj] = wt[j];
            }
        };
        look_up(0, slot, wj);
        for (int j0 = 0; j0 < a.k; j0 += JU) {
            look_up(j0 + JU, next_slot, next_w);
            bool all = true;
#pragma unroll
            for (int jj = 0; jj < JU; ++jj) all = all && slot[jj] >= 0;
            if (part.in[0]) {
                if (all) {
                    u32x4 v[JU];
#pragma unroll
                    for (int jj = 0; jj < JU; ++jj) v[jj] = part.load(a.y + (size_t)slot[jj] * a.C);
#pragma unroll
                    for (int jj = 0; jj < JU; ++jj) add_row<Y_BF16>(acc, v[jj], wj[jj]);
                } else if (JU > 1) {
#pragma unroll
                    for (int jj = 0; jj < JU; ++jj)
                        if (slot[jj] >= 0) add_row<Y_BF16>(acc, part.load(a.y + (size_t)slot[jj] * a.C), wj[jj]);
                }
            }
#pragma unroll
            for (int jj = 0; jj < JU; ++jj) {
                slot[jj] = next_slot[jj];
                wj[jj] = next_w[jj];
            }
        }
    } else {
        // entry j's slot and weight in lane j; -1: nothing to add
        const int lane = threadIdx.x & (kWave - 1);
        int my_slot = -1;
        float my_w = 0.0f;
        if (lane < a.k) {
            const size_t p = (size_t)t * a.k + lane;
            my_slot = a.pair_slot[p];
            my_w = a.w[p];
            if constexpr (PER_SEND_ROW) my_slot = a.pair_send_row[p] == r ? my_slot : -1;
        }
        uint64_t left = __builtin_amdgcn_ballot_w64(my_slot >= 0);   // entries still to be added, in ascending order
        int n = __builtin_popcountll(left);
        for (; n >= JU; n -= JU) combine_rows<Y_BF16, JU>(a, left, my_slot, my_w, part, acc);
        // the entries left over are requested at once too: 1153 tokens x 7 x 736 B 3.7 us by fours, twos and ones, 3.2 so; 675 x 3 x
        // 1888 B of fp32 2.7 / 2.5
        switch (n) {
        case 1: combine_rows<Y_BF16, 1>(a, left, my_slot, my_w, part, acc); break;
        case 2: combine_rows<Y_BF16, 2>(a, left, my_slot, my_w, part, acc); break;
        case 3: combine_rows<Y_BF16, 3>(a, left, my_slot, my_w, part, acc); break;
        case 4: combine_rows<Y_BF16, 4>(a, left, my_slot, my_w, part, acc); break;
        case 5: combine_rows<Y_BF16, 5>(a, left, my_slot, my_w, part, acc); break;
        case 6: combine_rows<Y_BF16, 6>(a, left, my_slot, my_w, part, acc); break;
        case 7: combine_rows<Y_BF16, 7>(a, left, my_slot, my_w, part, acc); break;
        }
    }

    if constexpr (WIDENED) {
        part.template store_f32<STORES>((u32x4 *)a.out + (size_t)r * a.C * 2, acc);
        return;
    } else if constexpr (Y_BF16 && !OUT_BF16) {
        put_floats<STORES>((u32x4 *)a.out + (size_t)r * a.C * 2, c, a.C * 2, acc);
        return;
    }
    if (c >= a.C) return;
    const size_t e0 = ((size_t)r * a.C + c) * EPC;   // first output element of this chunk
    if constexpr (OUT_BF16) {
        uint32_t pk[EPC / 2];
#pragma unroll
        for (int q = 0; q < EPC / 2; ++q) pk[q] = to_bf16(acc[2 * q]) | (to_bf16(acc[2 * q + 1]) << 16);
        if constexpr (Y_BF16) {
            const u32x4 o = {pk[0], pk[1], pk[2], pk[3]};
            put_out<STORES>((u32x4 *)((uint16_t *)a.out + e0), o);
        } else {
            const u32x2 o = {pk[0], pk[1]};
            put_out<STORES>((u32x2 *)((uint16_t *)a.out + e0), o);
        }
    } else {
        const u32x4 o = {__float_as_uint(acc[0]), __float_as_uint(acc[1]), __float_as_uint(acc[2]), __float_as_uint(acc[3])};
        put_out<STORES>((u32x4 *)((float *)a.out + e0), o);
    }
}

// Two-hop combine for k <= 8 in one pass: the token's k source chunks are loaded once, the partial
// sum of every destination device is formed (same operation order as the two-kernel path: fused
// multiply-adds in ascending j inside a device, then plain additions of the partial sums in order
// of first appearance), stored to the device's partial row, and added to the token's output.
struct TwoHopArgs {
    const u32x4 *y;
    const float *w;
    float *partial;
    void *out;
    const int32_t *pair_slot, *pair_send_row;
    const uint8_t *pair_first;
    int32_t k;
    int32_t C;   // 16-byte chunks per y row
};

// How a token's rows are requested (launch_two_hop): all at once; each when the one before has arrived; or in turn, an entry being looked
// up only when the row before it has arrived.
enum TwoHopRows : int32_t { kRowsAtOnce, kRowsOneByOne, kRowsInTurn };

template <bool Y_BF16, bool OUT_BF16, OutStores STORES, TwoHopRows ROWS, OutStores PARTIAL>
__global__ __launch_bounds__(1024) void combine_two_hop_kernel(TwoHopArgs a)
{
    constexpr int EPC = Y_BF16 ? 8 : 4;
    constexpr int KMAX = 8;
    const int t = gridDim.x - 1 - blockIdx.x;
    constexpr bool WIDENED = Y_BF16 && ROWS != kRowsInTurn;   // in turn the loads are what counts (6851 x 8 x 1040 B 32.1, 33.9 us in two places)
    const int c = blockIdx.y * blockDim.x + threadIdx.x;
    const bool in = c < a.C;
    const Part<WIDENED> part(c, a.C);
    u32x4 v[KMAX];
    int row[KMAX];
    float wj[KMAX];
    bool on[KMAX], lead[KMAX];
    int n;   // entries held in v; absent ones among them are not on
    if constexpr (ROWS == kRowsInTurn) {
        const int32_t *slots = a.pair_slot + (size_t)t * a.k, *rows = a.pair_send_row + (size_t)t * a.k;
        const uint8_t *first = a.pair_first + (size_t)t * a.k;
        const float *wt = a.w + (size_t)t * a.k;
        n = KMAX;
#pragma unroll
        for (int j = 0; j < KMAX; ++j) {
            on[j] = lead[j] = false;
            row[j] = -1;
            if (j >= a.k) continue;   // uniform
            const int slot = slots[j];
            row[j] = rows[j];
            wj[j] = wt[j];
            lead[j] = first[j];   // a byte: a vector load, behind the request before it and waited for ahead of the next
            if (slot < 0) continue;
            on[j] = true;
            if (in) v[j] = part.load(a.y + (size_t)slot * a.C);
        }
    } else {
        // entry j's slot, send row and weight in lane j; the entries with a slot are taken in ascending order
        const int lane = threadIdx.x & (kWave - 1);
        int my_slot = -1, my_row = -1;
        float my_w = 0.0f;
        bool my_first = false;
        if (lane < a.k) {
            const size_t p = (size_t)t * a.k + lane;
            my_slot = a.pair_slot[p];
            my_row = a.pair_send_row[p];
            my_w = a.w[p];
            my_first = a.pair_first[p];
        }
        uint64_t left = __builtin_amdgcn_ballot_w64(my_slot >= 0);
        const uint64_t firsts = __builtin_amdgcn_ballot_w64(my_first);
        n = __builtin_popcountll(left);
#pragma unroll
        for (int j = 0; j < KMAX; ++j) {
            if (j >= n) break;   // uniform
            const int at = __builtin_ctzll(left);
            left &= left - 1;
            on[j] = true;
            row[j] = __builtin_amdgcn_readlane(my_row, at);
            wj[j] = __uint_as_float(__builtin_amdgcn_readlane(__float_as_uint(my_w), at));
            lead[j] = firsts >> at & 1;
            const u32x4 *src = a.y + (size_t)__builtin_amdgcn_readlane(my_slot, at) * a.C;
            if constexpr (WIDENED) v[j] = part.load(src);
            else v[j] = load16_stream(src + (in ? c : 0));   // lanes past the row read its first chunk
            if constexpr (ROWS == kRowsOneByOne) __builtin_amdgcn_s_waitcnt(0x0f70);   // vmcnt(0)
        }
    }
    // All rows are there before the first sum: waited for one by one behind the stores of the sums, they would wait for those too (128 tokens x 8 x 14
    // KiB 8.5 us, 7.4 so; both with partial rows written through).
    if constexpr (ROWS == kRowsAtOnce) __builtin_amdgcn_s_waitcnt(0x0f70);   // vmcnt(0)
    float total[EPC];
#pragma unroll
    for (int e = 0; e < EPC; ++e) total[e] = 0.0f;
#pragma unroll
    for (int f = 0; f < KMAX; ++f) {
        if (f >= n) break;
        if (!lead[f]) continue;
        float acc[EPC];
#pragma unroll
        for (int e = 0; e < EPC; ++e) acc[e] = 0.0f;
#pragma unroll
        for (int j = f; j < KMAX; ++j) {
            if (j >= n) break;
            if (!on[j] || row[j] != row[f]) continue;
            add_row<Y_BF16>(acc, v[j], wj[j]);
        }
        u32x4 *prow = (u32x4 *)a.partial + (size_t)row[f] * a.C * (EPC / 4);
        if constexpr (WIDENED) {
            part.template store_f32<PARTIAL>(prow, acc);
        } else if constexpr (Y_BF16) {
            put_floats<PARTIAL>(prow, c, a.C * 2, acc);
        } else if (in) {
            const u32x4 o = {__float_as_uint(acc[0]), __float_as_uint(acc[1]), __float_as_uint(acc[2]), __float_as_uint(acc[3])};
            put_out<PARTIAL>(prow + c, o);
        }
#pragma unroll
        for (int e = 0; e < EPC; ++e) total[e] = total[e] + acc[e];
    }
    if constexpr (WIDENED) {
        if constexpr (OUT_BF16) part.template store_bf16<STORES>((u32x2 *)a.out + (size_t)t * a.C * 2, total);
        else part.template store_f32<STORES>((u32x4 *)a.out + (size_t)t * a.C * 2, total);
        return;
    } else if constexpr (Y_BF16 && !OUT_BF16) {
        put_floats<STORES>((u32x4 *)a.out + (size_t)t * a.C * 2, c, a.C * 2, total);
        return;
    }
    if (!in) return;
    const size_t e0 = ((size_t)t * a.C + c) * EPC;
    if constexpr (OUT_BF16) {
        uint32_t pk[EPC / 2];
#pragma unroll
        for (int q = 0; q < EPC / 2; ++q) pk[q] = to_bf16(total[2 * q]) | (to_bf16(total[2 * q + 1]) << 16);
        if constexpr (Y_BF16) {
            const u32x4 o = {pk[0], pk[1], pk[2], pk[3]};
            put_out<STORES>((u32x4 *)((uint16_t *)a.out + e0), o);
        } else {
            const u32x2 o = {pk[0], pk[1]};
            put_out<STORES>((u32x2 *)((uint16_t *)a.out + e0), o);
        }
    } else {
        const u32x4 o = {__float_as_uint(total[0]), __float_as_uint(total[1]), __float_as_uint(total[2]), __float_as_uint(total[3])};
        put_out<STORES>((u32x4 *)((float *)a.out + e0), o);
    }
}

// Level 1 reversed: out[t] = sum of the token's partial rows (fp32, one per destination device),
// plain additions from +0 in the order in which the devices first appear among the token's entries.
struct SumPartialsArgs {
    const u32x4 *partial;   // [send rows, C] chunks of 4 floats
    void *out;
    const int32_t *pair_send_row;
    const uint8_t *pair_first;
    int32_t k;
    int32_t C;              // 16-byte chunks (4 floats) per partial row
};

template <bool OUT_BF16>
__global__ __launch_bounds__(1024) void sum_partials_kernel(SumPartialsArgs a)
{
    const int t = gridDim.x - 1 - blockIdx.x;
    const int c = blockIdx.y * blockDim.x + threadIdx.x;
    const bool in = c < a.C;   // lanes past the row hold entries too
    const int lane = threadIdx.x & (kWave - 1);
    int my_row = -1;   // entry j's partial row in lane j, where it is the first of its device
    if (lane < a.k) {
        const size_t p = (size_t)t * a.k + lane;
        my_row = a.pair_first[p] ? a.pair_send_row[p] : -1;
    }
    float acc[4] = {0.0f, 0.0f, 0.0f, 0.0f};
    uint64_t left = __builtin_amdgcn_ballot_w64(my_row >= 0);
    while (left) {
        u32x4 v[4];
        const int n = __builtin_popcountll(left);
#pragma unroll
        for (int jj = 0; jj < 4; ++jj) {
            if (jj >= n) break;   // uniform
            v[jj] = load16_stream(a.partial + (size_t)__builtin_amdgcn_readlane(my_row, __builtin_ctzll(left)) * a.C + (in ? c : 0));
            left &= left - 1;
        }
#pragma unroll
        for (int jj = 0; jj < 4; ++jj) {
            if (jj >= n) break;
#pragma unroll
            for (int q = 0; q < 4; ++q) acc[q] = acc[q] + __uint_as_float(v[jj][q]);
        }
    }
    if (!in) return;
    const size_t e0 = ((size_t)t * a.C + c) * 4;
    if constexpr (OUT_BF16) {
        u32x2 o = {to_bf16(acc[0]) | (to_bf16(acc[1]) << 16), to_bf16(acc[2]) | (to_bf16(acc[3]) << 16)};
        store8_through((u32x2 *)((uint16_t *)a.out + e0), o);
    } else {
        u32x4 o = {__float_as_uint(acc[0]), __float_as_uint(acc[1]), __float_as_uint(acc[2]), __float_as_uint(acc[3])};
        store16_through((u32x4 *)((float *)a.out + e0), o);
    }
}

// Row gather in destination order: dst[r] = src[idx2 ? idx2[idx1[r]] : idx1[r]] for r < n_rows, one
// workgroup column per destination row.  n_rows_dev, when set, is a device-resident row count that
// caps n_rows (data-dependent lengths such as U).  Used by the two-hop dispatch (second hop) and by
// the disaggregated baseline, whose every stage is such a pass over the whole buffer.
struct GatherArgs {
    const u32x4 *src;
    u32x4 *dst;
    const int32_t *idx1, *idx2;
    const int32_t *n_rows_dev;
    int32_t C;   // 16-byte chunks per row
};

template <int CPT, bool STREAM_LOAD>
__global__ __launch_bounds__(256) void gather_rows_kernel(GatherArgs a)
{
    const int r = blockIdx.x;
    if (a.n_rows_dev && r >= *a.n_rows_dev) return;
    int q = a.idx1[r];
    if (q >= 0 && a.idx2) q = a.idx2[q];
    if (q < 0) return;
    const int c0 = blockIdx.y * (blockDim.x * CPT) + threadIdx.x;
    u32x4 v[CPT];
#pragma unroll
    for (int i = 0; i < CPT; ++i) {
        const int c = min(c0 + i * (int)blockDim.x, a.C - 1);   // no branch between the loads
        v[i] = STREAM_LOAD ? load16_stream(a.src + (size_t)q * a.C + c) : a.src[(size_t)q * a.C + c];
    }
#pragma unroll
    for (int i = 0; i < CPT; ++i) {
        const int c = c0 + i * blockDim.x;
        if (c < a.C) a.dst[(size_t)r * a.C + c] = v[i];
    }
}

// dev[p] = device of expert A[p] (or -1 for an id outside [0, E)): the key of the rank-major order
__global__ __launch_bounds__(256) void expert_to_device_kernel(int32_t *dev, const int32_t *A, int64_t n, int E, int Eloc)
{
    const int64_t p = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (p >= n) return;
    const int e = A[p];
    dev[p] = (unsigned)e < (unsigned)E ? e / Eloc : -1;
}

}   // namespace

#endif
