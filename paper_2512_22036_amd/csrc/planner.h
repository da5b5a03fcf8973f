// Planner kernels: token-expert matrix -> two-level layout descriptor (paper section 3.3).
#ifndef FUSCO_CSRC_PLANNER_H
#define FUSCO_CSRC_PLANNER_H

#include "common.h"

namespace {

// ------------------------------------------------------------------------------------------
// Planner
// ------------------------------------------------------------------------------------------
struct PlanArgs {
    const int32_t *A;
    int32_t N, k, E, D, Eloc;
    uint32_t k_magic, eloc_magic;   // ceil(2^20 / k), ceil(2^20 / Eloc): see div20
    int32_t eloc_shift;             // log2 of Eloc, -1 where it is no power of two
    int32_t ebits, dbits;           // bits of an expert's and of a device's number
    int32_t tpt;      // tokens per tile
    int32_t rank_rounds;   // rounds of 16 waves x (64 / k) tokens of a workgroup of pass 1
    int32_t n_tiles;
    int32_t small_groups;   // single-tile planner: workgroups that write descriptors
    int32_t stride;   // words per tile in tile_hist: E expert counts, D device counts, 1 invalid count; 16 bits for each half of the tile
    int32_t *tile_hist;
    int32_t chunk_tiles, n_chunks;   // 0, 0: no chunk level
    int32_t *chunk_hist;             // [n_chunks][stride]: tile_hist summed over the tiles of a chunk
    int32_t *exp_count, *exp_off, *send_count, *send_off;
    int32_t *pair_slot, *slot_pair, *slot_token, *send_src, *pair_send_row, *slot_send_row;
    int32_t *tile_slots;   // [n_tiles][tpt * k]: the slots of a tile's pairs in ascending order, then -1
    uint8_t *pair_first;
    int32_t *status;
};

__host__ __device__ __forceinline__ int bits_for(int nb)
{
    int n = 0;
    while ((1 << n) < nb) ++n;
    return n;
}

// Narrows a set of lanes (lo, hi) to those whose keys agree with the calling lane's in bits [from, to), STEP bits between
// two branches; a bit that is the same in all keys changes nothing, so bits above a key's may be compared too.
template <int STEP>
__device__ __forceinline__ void match_bits(int key, int from, int to, uint32_t &lo, uint32_t &hi)
{
    for (int b0 = from; b0 < to; b0 += STEP) {
#pragma unroll
        for (int b = b0; b < b0 + STEP; ++b) {
            const int bit = __builtin_amdgcn_sbfe(key, b, 1);   // all ones where the lane's bit is set
            const uint64_t set = __builtin_amdgcn_ballot_w64(bit != 0);
            lo = __builtin_amdgcn_bitop3_b32(lo, (uint32_t)set, bit, 0x90);           // lo & ~(set ^ bit)
            hi = __builtin_amdgcn_bitop3_b32(hi, (uint32_t)(set >> 32), bit, 0x90);
        }
    }
}

// Lanes of this wave that take part and hold the same key as the calling lane.
template <int STEP = 2>
__device__ __forceinline__ uint64_t same_key_lanes(int key, bool part, int nbits)
{
    const uint64_t all = __builtin_amdgcn_ballot_w64(part);
    uint32_t lo = (uint32_t)all, hi = (uint32_t)(all >> 32);
    match_bits<STEP>(key, 0, nbits, lo, hi);
    return (uint64_t)hi << 32 | lo;
}

// Element i of an array, counted from a place that is the same for all lanes; i is small, so that a 32-bit offset does.
template <typename T>
__device__ __forceinline__ T &at(T *base, int i) { return *(T *)((char *)const_cast<std::remove_const_t<T> *>(base) + (uint32_t)i * (uint32_t)sizeof(T)); }

// Stores v there, for runs of lanes next to each other.  THROUGH: through the L2 at once.  What plans of many tiles leave dirty there is only
// written back when their kernels end (us, plain / through, over the same buffers and over more than the memory-side cache holds: 65536 tokens x 8 16.2 / 16.2,
// 17.3 / 17.1, 131072 x 8 21.4 / 21.2, 22.5 / 22.2, 200000 x 4 18.5 / 18.1, 19.6 / 19.3, 262144 x 8, 1024 tiles, 35.5 / 35.2, 37.8 / 37.9; fewer tiles 30000 x
// 10, 148 tiles, 15.4 / 16.1, 8192 x 8, 32, 9.7 / 10.2).  Not
// - more than kPlanThroughMost tiles: 350000 x 8, 1368 tiles, 47.8 / 47.9, 50.1 / 50.3 (three sets of buffers 48.3 / 49.1), 524288 x 8 60.8 / 62.1, 67.0 / 68.1,
//   1048576 x 8 123.6 / 131.3, 130.0 / 137.5;
// - tiles whose pairs are no whole 64-byte units, whose stores go to memory as partial writes: 100000 x 6 19.7 / 20.0, 21.0 / 23.2, 136694 x 10 25.8 / 26.1, 27.3 /
//   33.0, 60000 x 7 15.6 / 16.0, 16.8 / 17.1;
// - the arrays indexed by slot, whose runs are shorter than a line (131072 x 8 25.6).
// A relaxed store at agent scope is that store (global_store_dword ... sc1) in a form that the compiler knows: what it must wait for between writing the
// base's scalar registers and reading them here it sees for itself, which it would not for an asm statement.
constexpr int kPlanThroughTiles = 200, kPlanThroughMost = 1024;
inline bool plan_through(int n_tiles, int tile_pairs) { return n_tiles >= kPlanThroughTiles && n_tiles <= kPlanThroughMost && tile_pairs % 16 == 0; }
template <bool THROUGH>
__device__ __forceinline__ void put(int32_t *base, int i, int v)
{
    if constexpr (THROUGH) __hip_atomic_store(&at(base, i), v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    else at(base, i) = v;
}

// Lanes of a set that come before the calling lane
__device__ __forceinline__ int lanes_before(uint32_t lo, uint32_t hi) { return (int)__builtin_amdgcn_mbcnt_hi(hi, __builtin_amdgcn_mbcnt_lo(lo, 0)); }

// n / d for the small operands of the planner through magic = ceil(2^20 / d): a pair's index in a tile (below 2048; up to
// 63 more in lanes whose result is not used) over k <= 64, an expert id below 1024 over E / D <= 1024.  The result is
// exact while n * (magic * d - 2^20), which is below n * d, stays below 2^20, and n * magic below 2^32.
// Both factors have fewer than 24 bits.
__device__ __forceinline__ int div20(int n, uint32_t magic) { return (int)(__umul24((uint32_t)n, magic) >> 20); }

// device of a valid expert id (any value for another)
__device__ __forceinline__ int device(const PlanArgs &a, int e) { return a.eloc_shift >= 0 ? e >> a.eloc_shift : div20(e, a.eloc_magic); }

// Orders LDS traffic between the lanes of one wave (no instruction is emitted: LDS serves the
// accesses of a wave in program order, the fences only stop the compiler from moving them).
__device__ __forceinline__ void wave_lds_order()
{
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}

// Inclusive prefix sum over the 64 lanes of a wave, without LDS: within each row of 16 lanes by row shifts, then the
// last lane of row 0 and 2 to rows 1 and 3, and of the lower half to the upper half.
__device__ __forceinline__ int wave_inclusive_sum(int x)
{
    x += __builtin_amdgcn_update_dpp(0, x, 0x111, 0xf, 0xf, false);   // row_shr:1 (lanes without a source add 0)
    x += __builtin_amdgcn_update_dpp(0, x, 0x112, 0xf, 0xf, false);
    x += __builtin_amdgcn_update_dpp(0, x, 0x114, 0xf, 0xf, false);
    x += __builtin_amdgcn_update_dpp(0, x, 0x118, 0xf, 0xf, false);
    x += __builtin_amdgcn_update_dpp(0, x, 0x142, 0xa, 0xf, false);   // row_bcast:15 into rows 1 and 3
    x += __builtin_amdgcn_update_dpp(0, x, 0x143, 0xc, 0xf, false);   // row_bcast:31 into rows 2 and 3
    return x;
}

// Pass 1 of the multi-tile planner: per tile, the counts of pairs per expert and of first (token, device) appearances
// per device, and for every pair its rank among the tile's pairs of the same expert and its send row's rank among the
// tile's rows of the same device.  The ranks are left, packed, in the pair's own places of pair_slot and
// pair_send_row, where pass 2 reads them; the second kernel then only adds what lies before the tile.
//
// Ranks are stable and do not depend on atomics: lanes of a wave that hold the same key are found with ballots, and a
// wave keeps its running count of every key in a byte of LDS; the 16 waves' bytes of a key lie next to each other, so
// that one 16-byte read and four byte sums give the pairs in earlier waves.  A wave takes whole tokens (64 / k of them
// per round), so that a device's first appearance in a token is settled among its lanes.
//
// HALVED: a tile is shared by two workgroups, the first one taking half of its tokens (rounded
// up): the ranking is bound by the instructions of its waves, and a compute unit ranks 1024 pairs in half the time of
// 2048.  Their counts are the halves of the tile's 32-bit words (at most 1024 + 63 pairs each), and ranks are within the
// half.  Chosen where there is no chunk level; with more tiles the chip is full and the halves only cost pass 2 (plan
// alone, k = 8, one / two workgroups per tile, us: 5000 tokens 11.2 / 9.9, 16384 12.0 / 10.9, 24000 14.8 / 13.8; 40000 17.6 / 18.0, and 15.4 with
// one and the chunk level).
constexpr int kRankRounds = 4, kHalfRounds = 2;   // rounds of 16 waves x (64 / k) tokens that cover a tile of 2048 / k tokens, half of it

__host__ __device__ __forceinline__ int first_half_tokens(int tile_tokens) { return (tile_tokens + 1) / 2; }
__device__ __forceinline__ int both_halves(int counts) { return (int)(((uint32_t)counts & 0xFFFFu) + ((uint32_t)counts >> 16)); }

__device__ __forceinline__ int sum_bytes(u32x4 v)
{
    return (int)__builtin_amdgcn_sad_u8(v[3], 0, __builtin_amdgcn_sad_u8(v[2], 0, __builtin_amdgcn_sad_u8(v[1], 0, __builtin_amdgcn_sad_u8(v[0], 0, 0))));
}

// packed ranks: experts in pair_slot, devices in pair_send_row; -1 for an invalid pair
__device__ __forceinline__ int pack_rank(int rank, int key, bool first) { return rank | key << 11 | (int)first << 21; }
__device__ __forceinline__ int packed_rank(int v) { return v & 2047; }
__device__ __forceinline__ int packed_key(int v) { return v >> 11 & 1023; }
__device__ __forceinline__ bool packed_first(int v) { return v >> 21 & 1; }

// Which of n units (tiles, or halves of tiles, in token order) workgroup b of n takes.  Workgroup b runs on XCD b mod 8, and an
// XCD takes a run of neighbouring units: what neighbouring tiles write next to each other in the arrays indexed by slot (a
// tile has a few pairs of an expert, a part of a 64-byte unit) then meets in one L2 and leaves it as whole lines, and pass 2 reads
// ranks that its own XCD has written.  Plan alone, k = 8, units dealt out in turn / in runs, us: 8192 tokens 11.15 / 10.93, 24000 tokens
// 15.3 / 14.5, 131072 tokens 27.4 / 25.3, 524288 tokens 89.8 / 75.3; pass 2 alone with runs, 131072 tokens 26.3.
__device__ __forceinline__ int unit_of_workgroup(uint32_t b, uint32_t n)
{
    const uint32_t x = b % kXcds, each = n / kXcds, more = n % kXcds;   // the first `more` XCDs have one unit more than the others
    return (int)(x * each + min(x, more) + b / kXcds);
}

// The ranking of one workgroup's tokens [tok0, tok0 + ntok).  A wave's rounds follow one another in token order; each thread
// has one pair of every round in which held() is true.
template <int ROUNDS>   // at most
struct Ranking {
    int lane, wave, per_wave, tok, rounds, ntok;
    int raw[ROUNDS];     // expert id as given
    int erank[ROUNDS];   // rank among the wave's pairs of the expert
    int drank[ROUNDS];   // rank of the token's row among the wave's rows of the device
    bool first[ROUNDS];
    __device__ __forceinline__ Ranking(const PlanArgs &a, int rounds_, int ntok_)
        : lane(threadIdx.x & (kWave - 1)), wave(__builtin_amdgcn_readfirstlane(threadIdx.x / kWave)),
          per_wave(div20(kWave, a.k_magic)), tok(div20(lane, a.k_magic)), rounds(rounds_), ntok(ntok_) {}
    __device__ __forceinline__ int first_token(int r) const { return (wave * rounds + r) * per_wave; }
    __device__ __forceinline__ bool done(int r) const { return r >= rounds || first_token(r) >= ntok; }   // uniform over the wave
    __device__ __forceinline__ bool held(int r) const { return tok < per_wave && first_token(r) + tok < ntok; }
    __device__ __forceinline__ int pair(const PlanArgs &a, int r) const { return first_token(r) * a.k + lane; }   // from tok0 on
    __device__ __forceinline__ void load(const PlanArgs &a, int64_t pair0)
    {
#pragma unroll
        for (int r = 0; r < ROUNDS; ++r) raw[r] = r < rounds && held(r) ? at(a.A + pair0, pair(a, r)) : -1;
    }
    // byte[key * kPlanWaves + wave]: the wave's running counts, all zero at the start; returns the number of invalid ids
    __device__ __forceinline__ int rank(const PlanArgs &a, uint8_t *byte)
    {
        const uint64_t not_before_token = ~(((uint64_t)1 << (tok * a.k)) - 1);
        int bad = 0;
#pragma unroll
        for (int r = 0; r < ROUNDS; ++r) {
            if (done(r)) break;
            const int e = raw[r];
            const bool ok = (unsigned)e < (unsigned)a.E;
            const uint64_t part = __builtin_amdgcn_ballot_w64(ok);
            bad += __builtin_popcountll(__builtin_amdgcn_ballot_w64(held(r)) & ~part);
            // lanes of the same device, and of the same expert: where a device has a power of two of experts its number is the
            // upper bits of theirs
            const int d = device(a, e);
            uint32_t dlo = (uint32_t)part, dhi = (uint32_t)(part >> 32), elo, ehi;
            if (a.eloc_shift >= 0) {
                match_bits<2>(e, a.eloc_shift, a.ebits, dlo, dhi);
                elo = dlo;
                ehi = dhi;
                match_bits<4>(e, 0, a.eloc_shift, elo, ehi);
            } else {
                elo = dlo;
                ehi = dhi;
                match_bits<4>(e, 0, a.ebits, elo, ehi);
                match_bits<2>(d, 0, a.dbits, dlo, dhi);
            }
            uint8_t *const ebyte = byte + (ok ? e : 0) * kPlanWaves + wave, *const dbyte = byte + (a.E + (ok ? d : 0)) * kPlanWaves + wave;
            const int ebefore = *ebyte, dbefore = *dbyte;
            const uint32_t tlo = dlo & (uint32_t)not_before_token, thi = dhi & (uint32_t)(not_before_token >> 32);   // from the token's first entry on the device
            first[r] = ok && lanes_before(tlo, thi) == 0;
            const uint64_t firsts = __builtin_amdgcn_ballot_w64(first[r]);
            dlo &= (uint32_t)firsts;
            dhi &= (uint32_t)(firsts >> 32);
            const int ein = lanes_before(elo, ehi), din = lanes_before(dlo, dhi);
            erank[r] = ebefore + ein;
            wave_lds_order();
            if (ok && ein == 0) *ebyte = (uint8_t)(ebefore + __builtin_popcount(elo) + __builtin_popcount(ehi));
            if (first[r] && din == 0) *dbyte = (uint8_t)(dbefore + __builtin_popcount(dlo) + __builtin_popcount(dhi));
            wave_lds_order();
            // the token's row on the device
            drank[r] = __shfl(dbefore + din, ok ? (tlo ? __builtin_ctz(tlo) : 32 + __builtin_ctz(thi)) : lane, kWave);
        }
        return bad;
    }
    // mask of the bytes of the waves before this one
    __device__ __forceinline__ u32x4 earlier_waves() const
    {
        u32x4 earlier;
#pragma unroll
        for (int q = 0; q < 4; ++q) earlier[q] = wave >= 4 * q + 4 ? ~0u : wave <= 4 * q ? 0u : (1u << 8 * (wave - 4 * q)) - 1;
        return earlier;
    }
};

template <bool HALVED, bool THROUGH>
__global__ __launch_bounds__(kPlanThreads) void plan_rank_kernel(PlanArgs a)
{
    __shared__ u32x4 cnt[2 * kMaxBins];   // [key]: a byte per wave, experts then devices
    __shared__ int invalid;
    uint8_t *byte = (uint8_t *)cnt;
    const int tid = threadIdx.x;
    // tokens from tile * tpt + half * split on; there may be none for the second half
    const int unit = unit_of_workgroup(blockIdx.x, gridDim.x), tile = HALVED ? unit >> 1 : unit, half = HALVED ? unit & 1 : 0;
    const int split = HALVED ? first_half_tokens(a.tpt) : a.tpt;
    const int tok0 = tile * a.tpt + half * split;
    const int64_t pair0 = (int64_t)tok0 * a.k;
    const int nb = a.E + a.D;
    constexpr int kRounds = HALVED ? kHalfRounds : kRankRounds;
    Ranking<kRounds> k(a, a.rank_rounds, min(half ? a.tpt - split : split, a.N - tok0));
    k.load(a, pair0);
    for (int b = tid; b < nb; b += kPlanThreads) cnt[b] = u32x4{0, 0, 0, 0};
    if (tid == 0) invalid = 0;
    __syncthreads();

    const int bad = k.rank(a, byte);
    if (bad && k.lane == 0) atomicAdd(&invalid, bad);
    __syncthreads();

    int32_t *out = a.tile_hist + (int64_t)tile * a.stride;
    for (int b = tid; b <= nb; b += kPlanThreads) {
        const int c = b < nb ? sum_bytes(cnt[b]) : invalid;
        if constexpr (HALVED) ((uint16_t *)(out + b))[half] = (uint16_t)c;
        else out[b] = c;
    }
    const u32x4 earlier = k.earlier_waves();
#pragma unroll
    for (int r = 0; r < kRounds; ++r) {
        if (k.done(r)) break;
        if (!k.held(r)) continue;
        const int e = k.raw[r];
        int ew = -1, dw = -1;
        if ((unsigned)e < (unsigned)a.E) {
            const int d = device(a, e);
            ew = pack_rank(k.erank[r] + sum_bytes(cnt[e] & earlier), e, false);
            dw = pack_rank(k.drank[r] + sum_bytes(cnt[a.E + d] & earlier), d, k.first[r]);
        }
        put<THROUGH>(a.pair_slot + pair0, k.pair(a, r), ew);
        put<THROUGH>(a.pair_send_row + pair0, k.pair(a, r), dw);
    }
}

// Optional pass between counting and placing: sums the per-tile counts over chunks of consecutive tiles, and leaves in a tile's row
// the sums of the chunk's earlier tiles, so that a workgroup of pass 2 reads one row of its chunk.  A workgroup takes kChunkColumns
// columns of a chunk, its rows split over kChunkParts groups of threads.  Plan, k = 8, 256 experts on 8 devices, us, a workgroup per chunk that left
// the sums alone (pass 2 added up the chunk's earlier tiles) / so: 65536 tokens 16.6 / 16.1, 131072 24.1 / 21.7; in columns of 64 / 128 100000 x 3 with 60
// experts on 4 devices 13.9 / 13.2, 131072 x 8 21.1 / 21.0.
constexpr int kChunkColumns = 2 * kWave, kChunkParts = kPlanThreads / kChunkColumns, kChunkRows = 4;   // kChunkRows: a thread's rows in registers
__global__ __launch_bounds__(kPlanThreads) void plan_chunk_kernel(PlanArgs a)
{
    __shared__ int sum[kChunkParts][kChunkColumns];
    const int lane = threadIdx.x % kChunkColumns, part = threadIdx.x / kChunkColumns, chunk = blockIdx.x;
    const int col = blockIdx.y * kChunkColumns + lane;
    const int each = (a.chunk_tiles + kChunkParts - 1) / kChunkParts;
    const int end = min((chunk + 1) * a.chunk_tiles, a.n_tiles), t0 = min(chunk * a.chunk_tiles + part * each, end), t1 = min(t0 + each, end);
    const bool in = col < a.stride;
    int32_t *const h = a.tile_hist + col;
    int v[kChunkRows], mine = 0;
#pragma unroll
    for (int i = 0; i < kChunkRows; ++i) v[i] = in && t0 + i < t1 ? h[(int64_t)(t0 + i) * a.stride] : 0;
#pragma unroll
    for (int i = 0; i < kChunkRows; ++i) mine += v[i];
    for (int t = t0 + kChunkRows; t < t1; ++t) mine += in ? h[(int64_t)t * a.stride] : 0;
    sum[part][lane] = mine;
    __syncthreads();
    int run = 0, total = 0;
#pragma unroll
    for (int q = 0; q < kChunkParts; ++q) {
        const int n = sum[q][lane];
        total += n;
        run += q < part ? n : 0;
    }
    if (!in) return;
    if (part == 0) a.chunk_hist[(int64_t)chunk * a.stride + col] = total;
#pragma unroll
    for (int i = 0; i < kChunkRows; ++i) {
        if (t0 + i < t1) h[(int64_t)(t0 + i) * a.stride] = run;
        run += v[i];
    }
    for (int t = t0 + kChunkRows; t < t1; ++t) {
        const int n = h[(int64_t)t * a.stride];
        h[(int64_t)t * a.stride] = run;
        run += n;
    }
}

// Pass 2: every pair's slot and send row, from its rank in the tile (pass 1) and the counts of the other tiles; all
// descriptor arrays.  One workgroup per tile.  The arrays indexed by slot, and tile_slots, are written in the tile's
// transfer order (its slots ascending: expert by expert, tokens ascending): neighbouring threads then write
// neighbouring slots of one expert, a few cache lines per wave instead of 64; the pairs meet their place in that
// order through LDS.  Bound by latency: three barriers between the loads and the stores.  Kernel times of pass 1 + pass 2
// (and the chunk pass between them), k = 8, us: 8192 tokens 3.8 + 6.4, 131072 tokens 7.7 + 3.1 + 12.6 (8.6 + 3.6 + 13.9 with plain stores and a chunk's
// earlier tiles added up here); with a pass 1 that only counted and a pass 2 that ranked all pairs: 5.2 + 11.8, 7.0 + 4.2 + 29.9.  With many
// tiles also bound by instructions: 330 vector instructions a wave, eight waves on a SIMD.
constexpr int kTilePairs = kMaxRounds * kRoundPairs;
constexpr int kCross = 12;           // rows of counts that a thread requests before anything else: 36 rows of 256 experts + 8 devices
constexpr int kMaxChunks = 2 * (kMaxBins / kWave);   // groups of 64 experts, then groups of 64 devices

// Sums of one column over the rows part, part + parts, ... of a list of n rows; rows below `limit` also count towards
// `before`.  Loads are issued back to back: beyond the list they read its last row, and their values are left out.
template <bool HALVED>
struct RowSums {
    const char *rows;
    int n, part, parts, limit;
    uint32_t at, step, last;   // byte offsets: the thread's first row, from one of its rows to the next, the list's last row
    int total, before;
    __device__ __forceinline__ RowSums(const int32_t *r, int count, int part_, int parts_, int limit_, int stride, int column)
        : rows((const char *)r), n(count), part(part_), parts(parts_), limit(limit_), at((uint32_t)(part_ * stride + column) * 4),
          step((uint32_t)(parts_ * stride) * 4), last((uint32_t)(max(count - 1, 0) * stride + column) * 4), total(0), before(0) {}
    template <int NV>
    __device__ __forceinline__ void load(int (&v)[NV], int i0) const   // the thread's rows i0, i0 + 1, ...
    {
#pragma unroll
        for (int i = 0; i < NV; ++i) {
            if ((i0 + i) * parts >= n) break;   // uniform: nobody has a row left
            v[i] = *(const int32_t *)(rows + min(at + (uint32_t)(i0 + i) * step, last));
        }
    }
    template <int NV>
    __device__ __forceinline__ void add(const int (&v)[NV], int i0)
    {
#pragma unroll
        for (int i = 0; i < NV; ++i) {
            const int first = (i0 + i) * parts;
            if (first >= n) break;
            const int c = HALVED ? both_halves(v[i]) : v[i];
            total += part < n - first ? c : 0;
            before += part < limit - first ? c : 0;
        }
    }
    __device__ __forceinline__ void walk(int i0)   // eight loads in flight
    {
        for (; i0 * parts < n; i0 += 8) {
            int v[8];
            load(v, i0);
            add(v, i0);
        }
    }
};

// HALVED as in pass 1 (there is no chunk level then).
// 80 scalar registers: with more than 96 a compute unit holds one workgroup of 16 waves at a time instead of two; with up to
// 96 (fewer spills) plans of few tiles take the same time (8192 tokens 10.6 us, 10.7 with 80), those of several tiles per
// compute unit longer (k = 8, 98304 tokens 26.9 us, 23.9 with 80; 131072 tokens 29.0 and 27.1).
template <bool HALVED, bool THROUGH>
__global__ __launch_bounds__(kPlanThreads) __attribute__((amdgpu_num_sgpr(80))) void plan_place_kernel(PlanArgs a)
{
    // per group of threads and column: total over all tiles, and over the earlier ones (`before` again holds the place
    // where the tile's run of the key starts, without its group's offset)
    __shared__ int total[2 * kMaxBins], before[2 * kMaxBins];
    __shared__ int tile_at[kMaxBins];                          // start of the expert's run in the tile, within its group
    __shared__ uint16_t half_cnt[HALVED ? 2 * kMaxBins : 1];   // the key's pairs in the first half of the tile
    __shared__ int group_total[kMaxChunks], group_tile[kMaxChunks];   // sums over 64 experts or devices
    __shared__ int slot_of[kTilePairs], row_of[kTilePairs];
    __shared__ uint16_t sorted[kTilePairs];
    const int tid = threadIdx.x;
    const int lane = tid & (kWave - 1), wave = __builtin_amdgcn_readfirstlane(tid / kWave);
    const int tile = unit_of_workgroup(blockIdx.x, gridDim.x), tok0 = tile * a.tpt, npairs = min(a.tpt, a.N - tok0) * a.k;
    const int64_t pair0 = (int64_t)tok0 * a.k;
    const int nb = a.E + a.D;
    const int egroups = (a.E + kWave - 1) / kWave, groups = egroups + (a.D + kWave - 1) / kWave;

    int ew[kMaxRounds], dw[kMaxRounds];
#pragma unroll
    for (int r = 0; r < kMaxRounds; ++r) {
        const int p = r * kPlanThreads + tid;
        ew[r] = dw[r] = -1;
        if (p < npairs) {
            ew[r] = at(a.pair_slot + pair0, p);
            dw[r] = at(a.pair_send_row + pair0, p);
        }
    }
    // Rows to add up: all tiles; with a chunk level (not HALVED) all chunks, and the tile's row, which then holds what its chunk's earlier
    // tiles count.  Thread (part, c) takes rows part, part + parts, ... of column c (parts: groups of columns that fit the workgroup)
    const int chunk = HALVED ? 0 : tile / a.chunk_tiles;
    const int32_t *rows1 = HALVED ? a.tile_hist : a.chunk_hist;
    const int n1 = HALVED ? a.n_tiles : a.n_chunks, limit1 = HALVED ? tile : chunk;
    const int cols = min(nb, kPlanThreads), pad = (cols + kWave - 1) / kWave * kWave, parts = kPlanThreads / pad;
    const int part = tid / pad, c = tid - part * pad;
    // this tile's own counts: its row, or what the next row of the chunk, or the chunk's, has more than its row
    const int32_t *own_row = a.tile_hist + (int64_t)tile * a.stride;
    const int32_t *next_row = HALVED ? nullptr : (tile + 1 < min((chunk + 1) * a.chunk_tiles, a.n_tiles) ? own_row + a.stride : a.chunk_hist + (int64_t)chunk * a.stride);
    const auto own_count = [&](int column) { return HALVED ? own_row[column] : next_row[column] - own_row[column]; };
    // of the column that the thread has in the first round of groups below
    const int col0 = wave < egroups ? tid : a.E + (wave - egroups) * kWave + lane;
    const int own0 = col0 < (wave < egroups ? a.E : HALVED ? nb : 0) ? own_count(col0) : 0;
    if (part < parts && c < cols) {
        RowSums<HALVED> s(rows1, n1, part, parts, limit1, a.stride, c);
        int v[kCross];
        s.load(v, 0);
        const int in_chunk = !HALVED && part == 0 ? own_row[c] : 0;
        s.add(v, 0);
        s.walk(kCross);
        total[part * pad + c] = s.total;   // parts * pad <= 1024
        before[part * pad + c] = s.before + in_chunk;
    }
    // the columns beyond the workgroup's kPlanThreads (more than 1024 experts and devices, parts is 1): one thread each
    for (int e = kPlanThreads + tid; e < nb; e += kPlanThreads) {
        RowSums<HALVED> s(rows1, n1, 0, 1, limit1, a.stride, e);
        s.walk(0);
        total[e] = s.total;
        before[e] = s.before + (HALVED ? 0 : own_row[e]);
    }
    __syncthreads();
    // Per group of 64 experts or devices, one wave: exclusive sums inside the group
    for (int g = wave; g < groups; g += kPlanWaves) {
        const bool expert = g < egroups;
        const int e = expert ? g * kWave + lane : a.E + (g - egroups) * kWave + lane;   // column
        const bool in = expert ? e < a.E : e < nb;
        int tot = 0, pre = 0, own = 0;
        if (in) {
            if (HALVED || expert) own = g == wave ? own0 : own_count(e);
            if constexpr (HALVED) {
                half_cnt[e] = (uint16_t)own;
                own = expert ? both_halves(own) : 0;
            }
            for (int q = 0; q < parts; ++q) {
                tot += total[q * pad + e];
                pre += before[q * pad + e];
            }
        }
        const int incl = wave_inclusive_sum(tot), own_incl = wave_inclusive_sum(own);
        if (tile == 0 && in) (expert ? a.exp_count + e : a.send_count + (e - a.E))[0] = tot;
        wave_lds_order();
        if (in) {
            total[e] = incl - tot;   // offset inside the group (only this wave reads or writes column e from here to the barrier)
            before[e] = incl - tot + pre;
            if (expert) tile_at[e] = own_incl - own;
        }
        if (lane == kWave - 1) {
            group_total[g] = incl;
            group_tile[g] = own_incl;
        }
    }
    __syncthreads();
    // offsets of the groups, one per lane
    const int of_group = lane < groups ? group_total[lane] : 0, of_tile = lane < groups ? group_tile[lane] : 0;
    const int incl = wave_inclusive_sum(of_group), tile_incl = wave_inclusive_sum(of_tile);
    const int group_off = incl - of_group, tile_group_off = tile_incl - of_tile;
    const int experts_total = __builtin_amdgcn_readlane(incl, egroups - 1);
    const int half_pairs = first_half_tokens(a.tpt) * a.k;
    const int tile_pairs = __builtin_amdgcn_readlane(tile_incl, egroups - 1);   // pairs of this tile with a valid expert id
#pragma unroll
    for (int r = 0; r < kMaxRounds; ++r) {
        const int p = r * kPlanThreads + tid;
        if (r * kPlanThreads >= npairs) break;   // uniform
        const int e = packed_key(ew[r]), d = packed_key(dw[r]), rank = packed_rank(ew[r]);
        const int eoff = __shfl(group_off, e / kWave, kWave), toff = __shfl(tile_group_off, e / kWave, kWave);
        const int doff = __shfl(group_off, egroups + d / kWave, kWave) - experts_total;
        if (p >= npairs) continue;
        int slot = -1, row = -1;
        bool first = false;
        if (ew[r] >= 0) {
            const bool second = HALVED && p >= half_pairs;
            const int in_tile = rank + (second ? half_cnt[e] : 0);
            slot = before[e] + eoff + in_tile;
            row = before[a.E + d] + doff + packed_rank(dw[r]) + (second ? half_cnt[a.E + d] : 0);
            first = packed_first(dw[r]);
            sorted[tile_at[e] + toff + in_tile] = (uint16_t)p;
        }
        slot_of[p] = slot;
        row_of[p] = row;
        put<THROUGH>(a.pair_slot + pair0, p, slot);
        put<THROUGH>(a.pair_send_row + pair0, p, row);
        at(a.pair_first + pair0, p) = first ? 1 : 0;
        if (first) a.send_src[row] = tok0 + div20(p, a.k_magic);
    }
    __syncthreads();
    const int cap = a.tpt * a.k;
    int32_t *order = a.tile_slots + (int64_t)tile * cap;
    for (int q = tid; q < cap; q += kPlanThreads) {
        int sl = -1;
        if (q < tile_pairs) {
            const int p = sorted[q];
            sl = slot_of[p];
            a.slot_pair[sl] = (int32_t)(pair0 + p);
            a.slot_token[sl] = tok0 + div20(p, a.k_magic);
            a.slot_send_row[sl] = row_of[p];
        }
        put<THROUGH>(order, q, sl);
    }

    if (tile == 0) {
        for (int g = wave; g < groups; g += kPlanWaves) {
            const int off = __builtin_amdgcn_readlane(group_off, g);
            const int i = (g < egroups ? g : g - egroups) * kWave + lane;
            if (g < egroups && i < a.E) a.exp_off[i] = total[i] + off;
            if (g >= egroups && i < a.D) a.send_off[i] = total[a.E + i] + off - experts_total;
        }
        if (tid == 0) {
            a.exp_off[a.E] = experts_total;
            a.send_off[a.D] = __builtin_amdgcn_readlane(incl, kWave - 1) - experts_total;
        }
        if (wave == kPlanWaves - 1) {
            // the last column of the counts holds the invalid ids of a tile (or of a chunk of tiles)
            int bad = 0;
            for (int r = lane; r < n1; r += kWave) {
                const int c = rows1[(int64_t)r * a.stride + nb];
                bad += HALVED ? both_halves(c) : c;
            }
            bad = wave_inclusive_sum(bad);
            if (lane == kWave - 1) *a.status = bad;
        }
    }
}

// Planner for inputs of a few tiles, in one launch: every workgroup counts the whole routing for itself instead of
// reading counts that an earlier launch has left.  A workgroup ranks an eighth of a tile's tokens in one round (as pass 1
// does) and adds the other tokens to counters in LDS, a token per thread; a token's devices are bits in two registers, and an
// entry whose bit is set already adds no row.  Four counters per expert (and eight per device), taken by lane, keep popular
// keys from serialising a wave's additions.  Bound by latency (routing, counters, scan, places: four barriers) and, from
// about 8192 pairs on, by the additions, 0.14 us per 1024 pairs.  Kernel of one launch / the two launches it replaces, us:
// 300 tokens x 8 5.1 / 8.6, 4096 x 2 5.3 / 8.5, 1537 x 6 5.7 / 9.5, 2000 x 10 7.5 / 10.2.  An eighth and
// not half a tile per workgroup because its own pairs are a chain of their own: 1537 x 6 7.1 with halves, 6.3 with quarters.
// VEC: ids that are read at once (a token's ids start on multiples of it); IDS: ids of a token that a thread requests at a
// time, of 16 / IDS tokens (k <= 4: 4; 8000 x 1 6.3, 7.5 us with 8).
constexpr int kDirectParts = 8;      // workgroups per tile
constexpr int kDirectMaxD = 64;      // bits of the mask
constexpr int kDirectMaxK = 16;      // a thread takes all of a token's ids: 600 tokens x 33 10.5 us, 9.9 with two launches
constexpr int kDirectMaxTokens = 8192;
// Sizes up to which the one launch is the faster one or even, whatever a router gives.  Popular experts cost it additions to one address, and
// the two launches are faster with them, so the line lies lower than for scores without a trend (a routing that names one expert in
// every entry, which no router gives, is left behind from about 20000 pairs on).  One launch / two, us; scores
// without a trend, popular experts (by rank^-1.2), expert 0 in every token, all entries the same expert:
// 3072 x 8, 256 experts on 8 devices 7.5 / 9.2, 8.3 / 8.5, 7.9 / 9.1, 9.6 / 8.4; 4096 x 8 8.5 / 9.2, 9.8 / 8.7, 9.0 / 9.3, 11.5 / 8.5.
// 3072 x 8, 1024 experts on 64 devices 8.2 / 11.1, 9.0 / 10.2, 8.6 / 11.0, 10.2 / 10.1.
// 4096 x 6, 160 experts 7.8 / 9.3, 8.6 / 9.0, 8.3 / 9.3, 9.8 / 8.9; 5461 x 6 9.3 / 9.5, 10.5 / 9.1, 9.8 / 9.5, 12.4 / 9.0.
// 5120 x 4, 60 experts on 4 devices 7.4 / 8.1, 8.1 / 8.0, 8.0 / 8.1, 9.0 / 7.9; 6144 x 4 8.0 / 8.1, 8.8 / 8.0, 8.7 / 8.1, 10.0 / 7.9.
// 8192 x 2, 16 experts on 4 devices 7.0 / 7.8, 7.8 / 7.7, 7.9 / 7.7, 8.2 / 7.7.
inline int direct_max_pairs(int k) { return k <= 4 ? 20480 : 24576; }
inline bool planned_directly(int N, int k, int D)
{
    return k <= kDirectMaxK && D <= kDirectMaxD && N <= kDirectMaxTokens && N * k <= direct_max_pairs(k);
}
constexpr int kEcopies = 4, kDcopies = 8;
// where a token counts for a workgroup's experts: in an earlier tile, in the tile before the workgroup's own, in the tile after them, in a
// later tile
constexpr int kPlaces = 4;

__host__ __device__ __forceinline__ int direct_part_tokens(int tile_tokens) { return (tile_tokens + kDirectParts - 1) / kDirectParts; }

struct DirectLds {
    u32x4 rank[kMaxBins + kDirectMaxD];            // as in pass 1: a byte per wave and key
    u32x4 ecount[kPlaces * kMaxBins];              // the other tokens' pairs by place and expert
    int dcount[2 * kDirectMaxD * kDcopies];        // the other tokens' rows by device: before and after the workgroup's tokens
    int slot_at[kMaxBins], tile_at[kMaxBins], own_at[kMaxBins], row_at[kDirectMaxD];
    int group[3][kMaxBins / kWave];                // sums over 64 experts: all pairs, the tile's, the workgroup's
    u32x4 sorted[kTilePairs / kDirectParts + kWave];   // the workgroup's pairs in the order of their slots: slot, pair, row, place in the tile
};

__device__ __forceinline__ int sum4(u32x4 v) { return (int)(v[0] + v[1] + v[2] + v[3]); }

template <int VEC, int IDS>
__global__ __launch_bounds__(kPlanThreads) void plan_direct_kernel(PlanArgs a)
{
    constexpr int TOKENS = 16 / IDS;
    __shared__ DirectLds s;
    const int tid = threadIdx.x;
    const int unit = unit_of_workgroup(blockIdx.x, gridDim.x), tile = unit / kDirectParts, part = unit % kDirectParts;
    const int each = direct_part_tokens(a.tpt), tile0 = tile * a.tpt, tile1 = min(tile0 + a.tpt, a.N);
    const int tok0 = min(tile0 + part * each, tile1), tok1 = min(tok0 + each, tile1), ntok = tok1 - tok0;
    const int pair0 = tok0 * a.k;
    Ranking<1> k(a, 1, ntok);
    k.load(a, pair0);
    for (int b = tid; b < a.E + a.D; b += kPlanThreads) s.rank[b] = u32x4{0, 0, 0, 0};
    for (int b = tid; b < kPlaces * a.E; b += kPlanThreads) s.ecount[b] = u32x4{0, 0, 0, 0};
    for (int b = tid; b < 2 * kDirectMaxD * kDcopies; b += kPlanThreads) s.dcount[b] = 0;
    __syncthreads();

    // the other tokens: numbered without the workgroup's own
    const int others = a.N - ntok;
    for (int w0 = k.wave * kWave; w0 < others; w0 += kPlanThreads * TOKENS) {   // uniform over the wave
        uint32_t lo[TOKENS], hi[TOKENS];
        int t[TOKENS], *ec[TOKENS], *dc[TOKENS];
        bool in[TOKENS];
#pragma unroll
        for (int u = 0; u < TOKENS; ++u) {
            const int i = w0 + k.lane + u * kPlanThreads;
            in[u] = i < others;
            t[u] = i < tok0 ? i : i + ntok;
            lo[u] = hi[u] = 0;
            const int place = t[u] < tile0 ? 0 : t[u] < tok0 ? 1 : t[u] < tile1 ? 2 : 3;
            ec[u] = (int *)(s.ecount + place * a.E) + (k.lane & (kEcopies - 1));
            dc[u] = s.dcount + (i < tok0 ? 0 : kDirectMaxD * kDcopies) + (k.lane & (kDcopies - 1));
        }
        for (int j0 = 0; j0 < a.k; j0 += IDS) {
            uint32_t e[TOKENS][IDS];
#pragma unroll
            for (int u = 0; u < TOKENS; ++u) {
                const int32_t *ids = a.A + (int64_t)t[u] * a.k + j0;
#pragma unroll
                for (int j = 0; j < IDS; j += VEC) {
                    typedef uint32_t vec __attribute__((ext_vector_type(VEC)));
                    vec v = ~(vec)0;
                    if (in[u] && j0 + j < a.k) v = *(const vec *)(ids + j);
#pragma unroll
                    for (int q = 0; q < VEC; ++q) e[u][j + q] = v[q];
                }
            }
#pragma unroll
            for (int u = 0; u < TOKENS; ++u) {
                if (w0 + u * kPlanThreads >= others) break;   // uniform
#pragma unroll
                for (int j = 0; j < IDS; ++j) {
                    if (j0 + j >= a.k) break;   // uniform
                    const uint32_t id = e[u][j];
                    if (id >= (uint32_t)a.E) continue;
                    atomicAdd(ec[u] + id * kEcopies, 1);
                    const int d = div20((int)id, a.eloc_magic);
                    const uint32_t bit = 1u << (d & 31);
                    if (bit & ~(d < 32 ? lo[u] : hi[u])) atomicAdd(dc[u] + d * kDcopies, 1);
                    lo[u] |= d < 32 ? bit : 0u;
                    hi[u] |= d < 32 ? 0u : bit;
                }
            }
        }
    }
    k.rank(a, (uint8_t *)s.rank);
    __syncthreads();

    // a wave per 64 experts, and one for the devices: sums before the key, over all pairs, the tile's and the workgroup's
    const int egroups = (a.E + kWave - 1) / kWave;
    for (int g = k.wave; g <= egroups; g += kPlanWaves) {
        if (g < egroups) {
            const int e = g * kWave + k.lane;
            int own = 0, in_tile = 0, total = 0, earlier = 0, in_tile_earlier = 0;
            if (e < a.E) {
                own = sum_bytes(s.rank[e]);
                earlier = sum4(s.ecount[e]);
                in_tile_earlier = sum4(s.ecount[a.E + e]);
                in_tile = in_tile_earlier + own + sum4(s.ecount[2 * a.E + e]);
                total = earlier + in_tile + sum4(s.ecount[3 * a.E + e]);
                if (unit == 0) a.exp_count[e] = total;
            }
            const int total_incl = wave_inclusive_sum(total), tile_incl = wave_inclusive_sum(in_tile), own_incl = wave_inclusive_sum(own);
            if (e < a.E) {
                s.slot_at[e] = total_incl - total + earlier + in_tile_earlier;
                s.tile_at[e] = tile_incl - in_tile + in_tile_earlier;
                s.own_at[e] = own_incl - own;
            }
            if (k.lane == kWave - 1) {
                s.group[0][g] = total_incl;
                s.group[1][g] = tile_incl;
                s.group[2][g] = own_incl;
            }
        } else {
            const int d = k.lane;
            int earlier = 0, total = 0;
            if (d < a.D) {
                const u32x4 *c = (const u32x4 *)(s.dcount + d * kDcopies), *later = c + kDirectMaxD * kDcopies / 4;
                earlier = sum4(c[0]) + sum4(c[1]);
                total = earlier + sum_bytes(s.rank[a.E + d]) + sum4(later[0]) + sum4(later[1]);
            }
            const int incl = wave_inclusive_sum(total);
            s.row_at[d] = incl - total + earlier;
            if (unit == 0 && d < a.D) {
                a.send_count[d] = total;
                a.send_off[d] = incl - total;
            }
            if (unit == 0 && d == kWave - 1) a.send_off[a.D] = incl;
        }
    }
    __syncthreads();

    int off[3], sum[3];   // offsets of the groups, one per lane, and the sums over all of them
#pragma unroll
    for (int q = 0; q < 3; ++q) {
        const int v = k.lane < egroups ? s.group[q][k.lane] : 0, incl = wave_inclusive_sum(v);
        off[q] = incl - v;
        sum[q] = __builtin_amdgcn_readlane(incl, kWave - 1);
    }
    if (!k.done(0)) {
        const int e = k.raw[0];
        const bool ok = (unsigned)e < (unsigned)a.E;
        const int g = ok ? e / kWave : 0;
        const int slot_off = __shfl(off[0], g, kWave), tile_off = __shfl(off[1], g, kWave), own_off = __shfl(off[2], g, kWave);
        if (k.held(0)) {
            const int p = pair0 + k.pair(a, 0);
            int slot = -1, row = -1;
            if (ok) {
                const u32x4 earlier = k.earlier_waves();
                const int d = device(a, e), rank = k.erank[0] + sum_bytes(s.rank[e] & earlier);
                slot = s.slot_at[e] + slot_off + rank;
                row = s.row_at[d] + k.drank[0] + sum_bytes(s.rank[a.E + d] & earlier);
                s.sorted[s.own_at[e] + own_off + rank] = u32x4{(uint32_t)slot, (uint32_t)p, (uint32_t)row, (uint32_t)(s.tile_at[e] + tile_off + rank)};
                if (k.first[0]) a.send_src[row] = tok0 + k.first_token(0) + k.tok;
            }
            a.pair_slot[p] = slot;
            a.pair_send_row[p] = row;
            a.pair_first[p] = ok && k.first[0] ? 1 : 0;
        }
    }
    __syncthreads();
    const int cap = a.tpt * a.k;
    int32_t *order = a.tile_slots + (int64_t)tile * cap;
    for (int q = tid; q < sum[2]; q += kPlanThreads) {
        const u32x4 v = s.sorted[q];
        const int slot = (int)v[0], p = (int)v[1];
        a.slot_pair[slot] = p;
        a.slot_token[slot] = tok0 + div20(p - pair0, a.k_magic);
        a.slot_send_row[slot] = (int)v[2];
        order[v[3]] = slot;
    }
    if (part == kDirectParts - 1)
        for (int q = sum[1] + tid; q < cap; q += kPlanThreads) order[q] = -1;
    if (unit == 0) {
        for (int g = k.wave; g < egroups; g += kPlanWaves) {
            const int at = __builtin_amdgcn_readlane(off[0], g), e = g * kWave + k.lane;
            if (e < a.E) a.exp_off[e] = s.slot_at[e] + at;   // the first workgroup has no pairs before its own
        }
        if (tid == 0) {
            a.exp_off[a.E] = sum[0];
            *a.status = a.N * a.k - sum[0];
        }
    }
}

// Planner for inputs of a single tile (at most 2048 pairs), in one launch and without counters or scans over keys: a
// pair's slot is the number of pairs that come before it in (expert, pair) order, and the workgroup that owns the
// pair counts them by comparing its key with everybody's - the keys of all pairs fit the registers of one
// workgroup, one comparison of a wave settles 64 of them.  Likewise the send row of a (token, device) is the number
// of first appearances before it in (device, token) order.  Every workgroup reads the whole (tiny) routing; one
// barrier stands between the loads and the slots.
constexpr int kSmallThreads = 512;
constexpr int kSmallWaves = kSmallThreads / kWave;
// rounds of kSmallWaves x (64 / k) whole tokens that cover 2048 / k tokens, for every k <= 64
constexpr int kSmallRounds = 64 / kSmallWaves;
// pairs that one workgroup writes the descriptors of (256 tokens x 8 with 8 / 16 / 32: 7.4 / 8.2 / 10.8 us)
constexpr int kSmallPairs = 8;

struct SmallLds {
    int before[2][kSmallWaves][kWave];   // per wave and query: pairs, first appearances
    int count[2 * kMaxBins];             // counting workgroup: pairs per expert, then first appearances per device
    int valid, invalid;
    uint8_t first[kSmallPairs];          // placing workgroup: its pairs that are first appearances
};

// This thread's pairs of a round: whole tokens per wave, one pair per lane.
struct SmallLane {
    int lane, wave, per_wave, tok;   // tok: token of the lane among the wave's per_wave tokens
    __device__ __forceinline__ SmallLane(const PlanArgs &a)
        : lane(threadIdx.x & (kWave - 1)), wave(__builtin_amdgcn_readfirstlane(threadIdx.x / kWave)),
          per_wave(div20(kWave, a.k_magic)), tok(div20(lane, a.k_magic)) {}
    __device__ __forceinline__ int first_token(int r) const { return (r * kSmallWaves + wave) * per_wave; }
    __device__ __forceinline__ bool part(const PlanArgs &a, int r) const { return tok < per_wave && first_token(r) + tok < a.N; }
};

__device__ __forceinline__ void small_load(const PlanArgs &a, const SmallLane &l, int (&raw)[kSmallRounds])
{
#pragma unroll
    for (int r = 0; r < kSmallRounds; ++r) raw[r] = l.part(a, r) ? a.A[l.first_token(r) * a.k + l.lane] : -1;
}

// First appearance of its device in its token, for a pair of device d (-1: no valid pair) held by every lane; `same`:
// the lanes with the same device.
__device__ __forceinline__ bool small_first(const PlanArgs &a, const SmallLane &l, int d, int dbits, uint64_t &same)
{
    same = same_key_lanes(d, d >= 0, dbits);
    const uint64_t earlier = (((uint64_t)1 << l.lane) - 1) & ~(((uint64_t)1 << (l.tok * a.k)) - 1);   // of the token
    return d >= 0 && !(same & earlier);
}

// Number of this wave's keys (one per lane and round, ~0: none) below each of the n (<= 64) query keys that the lanes
// hold; the count for the j-th query is returned in lane j.
__device__ __forceinline__ int small_count_below(const SmallLane &l, const PlanArgs &a, const uint32_t (&key)[kSmallRounds],
                                                 uint32_t query, int n)
{
    // eight queries at a time: their comparisons are independent, and a round costs one branch for all of them
    int mine = 0;
    for (int j0 = 0; j0 < n; j0 += 8) {
        uint32_t q[8];
        int c[8];
#pragma unroll
        for (int j = 0; j < 8; ++j) {
            q[j] = __builtin_amdgcn_readlane(query, j0 + j);   // the lanes past n hold some value, counted for nobody
            c[j] = 0;
        }
#pragma unroll
        for (int r = 0; r < kSmallRounds; ++r) {
            if (l.first_token(r) >= a.N) break;   // uniform over the wave
#pragma unroll
            for (int j = 0; j < 8; ++j) c[j] += __builtin_popcountll(__builtin_amdgcn_ballot_w64(key[r] < q[j]));
        }
#pragma unroll
        for (int j = 0; j < 8; ++j) mine = l.lane == j0 + j ? c[j] : mine;
    }
    return mine;
}

__device__ __forceinline__ int small_sum(const int (*before)[kWave], const SmallLane &l)
{
    int sum = 0;
#pragma unroll
    for (int w = 0; w < kSmallWaves; ++w) sum += before[w][l.lane];
    return sum;
}

// Exclusive prefix of count[0 .. nb) written out together with the counts, by the calling wave
__device__ __forceinline__ void small_offsets(const int *count, int nb, int32_t *out_count, int32_t *out_off)
{
    const int lane = threadIdx.x & (kWave - 1);
    int base = 0;
    for (int b0 = 0; b0 < nb; b0 += kWave) {
        const int b = b0 + lane, c = b < nb ? count[b] : 0;
        const int incl = wave_inclusive_sum(c);
        if (b < nb) {
            out_count[b] = c;
            out_off[b] = base + incl - c;
        }
        base += __builtin_amdgcn_readlane(incl, kWave - 1);
    }
    if (lane == 0) out_off[nb] = base;
}

// One workgroup: counts and offsets per expert and per device, the transfer order (a single tile's slots in
// ascending order are 0, 1, 2, ...) and the number of invalid ids.
__device__ __forceinline__ void small_counts(SmallLds &s, const PlanArgs &a)
{
    const int tid = threadIdx.x;
    const SmallLane l(a);
    int raw[kSmallRounds];
    small_load(a, l, raw);
    for (int b = tid; b < a.E + a.D; b += kSmallThreads) s.count[b] = 0;
    if (tid == 0) s.valid = s.invalid = 0;
    __syncthreads();
    const int dbits = bits_for(a.D);
    int good = 0, bad = 0;
#pragma unroll
    for (int r = 0; r < kSmallRounds; ++r) {
        if (l.first_token(r) >= a.N) break;   // uniform over the wave
        const bool ok = (unsigned)raw[r] < (unsigned)a.E;
        const int d = ok ? div20(raw[r], a.eloc_magic) : -1;
        uint64_t same;
        const bool first = small_first(a, l, d, dbits, same);
        same &= __builtin_amdgcn_ballot_w64(first);
        if (ok) atomicAdd(&s.count[raw[r]], 1);
        if (first && !(same & (((uint64_t)1 << l.lane) - 1))) atomicAdd(&s.count[a.E + d], __builtin_popcountll(same));
        good += __builtin_popcountll(__builtin_amdgcn_ballot_w64(ok));
        bad += __builtin_popcountll(__builtin_amdgcn_ballot_w64(l.part(a, r) && !ok));
    }
    if (l.lane == 0) {
        atomicAdd(&s.valid, good);
        atomicAdd(&s.invalid, bad);
    }
    __syncthreads();
    if (l.wave == 0) small_offsets(s.count, a.E, a.exp_count, a.exp_off);
    if (l.wave == 1) small_offsets(s.count + a.E, a.D, a.send_count, a.send_off);
    const int cap = a.tpt * a.k, valid = s.valid;
    for (int q = tid; q < cap; q += kSmallThreads) a.tile_slots[q] = q < valid ? q : -1;
    if (tid == 0) *a.status = s.invalid;
}

__device__ __forceinline__ void small_expert_keys(const PlanArgs &a, const SmallLane &l, const int (&raw)[kSmallRounds],
                                                  uint32_t (&key)[kSmallRounds])
{
#pragma unroll
    for (int r = 0; r < kSmallRounds; ++r)
        key[r] = (unsigned)raw[r] < (unsigned)a.E ? (uint32_t)raw[r] << 12 | (uint32_t)(l.first_token(r) * a.k + l.lane) : ~0u;
}

// Slots of the n (<= 64) pairs from p0 on: the j-th one's in lane j of every wave, -1 for a pair without a valid expert.
__device__ __forceinline__ int small_slots(SmallLds &s, const PlanArgs &a, int p0, int n)
{
    const SmallLane l(a);
    const int own = l.lane < n ? a.A[p0 + l.lane] : -1;
    int raw[kSmallRounds];
    uint32_t key[kSmallRounds];
    small_load(a, l, raw);
    small_expert_keys(a, l, raw, key);
    s.before[0][l.wave][l.lane] = small_count_below(l, a, key, (uint32_t)own << 12 | (uint32_t)(p0 + l.lane), n);
    __syncthreads();
    const int slot = small_sum(s.before[0], l);
    return (unsigned)own < (unsigned)a.E ? slot : -1;
}

// All descriptors of the n (<= kSmallPairs) pairs from p0 on.
__device__ __forceinline__ void small_place(SmallLds &s, const PlanArgs &a, int p0, int n)
{
    const SmallLane l(a);
    const int p = p0 + l.lane, t = div20(p, a.k_magic);   // this lane's query, in the first n lanes
    const int own = l.lane < n ? a.A[p] : -1;
    int raw[kSmallRounds];
    uint32_t key[kSmallRounds];
    small_load(a, l, raw);
    small_expert_keys(a, l, raw, key);
    s.before[0][l.wave][l.lane] = small_count_below(l, a, key, (uint32_t)own << 12 | (uint32_t)p, n);
    const bool ok = (unsigned)own < (unsigned)a.E;
    const int dbits = bits_for(a.D), d = ok ? div20(own, a.eloc_magic) : 0;
#pragma unroll
    for (int r = 0; r < kSmallRounds; ++r) {
        if (l.first_token(r) >= a.N) break;   // uniform over the wave; no key there
        const int dr = key[r] != ~0u ? div20(raw[r], a.eloc_magic) : -1;
        const uint32_t pr = (uint32_t)(l.first_token(r) * a.k + l.lane);
        uint64_t same;
        const bool f = small_first(a, l, dr, dbits, same);
        if (l.part(a, r) && pr - (uint32_t)p0 < (uint32_t)n) s.first[pr - (uint32_t)p0] = f;
        key[r] = f ? (uint32_t)dr << 12 | pr : ~0u;
    }
    // a token's own entries do not come before its row
    s.before[1][l.wave][l.lane] = small_count_below(l, a, key, (uint32_t)d << 12 | (uint32_t)(t * a.k), n);
    __syncthreads();
    if (threadIdx.x >= n) return;
    const int slot = ok ? small_sum(s.before[0], l) : -1, row = ok ? small_sum(s.before[1], l) : -1;
    const bool first = s.first[l.lane];
    a.pair_slot[p] = slot;
    a.pair_send_row[p] = row;
    a.pair_first[p] = first ? 1 : 0;
    if (ok) {
        a.slot_pair[slot] = p;
        a.slot_token[slot] = t;
        a.slot_send_row[slot] = row;
    }
    if (first) a.send_src[row] = t;
}

// fusco_plan for a single tile: workgroup 0 counts, the others place kSmallPairs pairs each.  200 tokens x 10 of 384
// experts: 5.4 us, against 10.1 us with one workgroup that counts, scans and ranks.
__global__ __launch_bounds__(kSmallThreads) void plan_small_kernel(PlanArgs a)
{
    __shared__ SmallLds s;
    if (blockIdx.x == 0) {
        small_counts(s, a);
        return;
    }
    const int p0 = (int)(blockIdx.x - 1) * kSmallPairs;
    small_place(s, a, p0, min(kSmallPairs, a.N * a.k - p0));
}

// Cross-node traffic load of the GPU that owns this plan (section 3.4): bytes of the send rows whose
// destination device lies on another node than `home_node`.  One wave.
__global__ __launch_bounds__(kWave) void cross_node_load_kernel(const int32_t *send_count, int D, int devices_per_node,
                                                               int home_node, uint64_t row_bytes, int64_t *load)
{
    int64_t rows = 0;
    for (int d = threadIdx.x; d < D; d += kWave)
        if (d / devices_per_node != home_node) rows += send_count[d];
    for (int s = kWave / 2; s > 0; s >>= 1) rows += __shfl_down(rows, s, kWave);
    if (threadIdx.x == 0) *load = rows * (int64_t)row_bytes;
}

}   // namespace

#endif
