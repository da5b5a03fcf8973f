// Types, limits and small host helpers shared by every part of the library (one translation unit).
#ifndef FUSCO_CSRC_COMMON_H
#define FUSCO_CSRC_COMMON_H

#include <hip/hip_runtime.h>
#include <hip/hip_ext.h>
#include <stdint.h>
#include <stdlib.h>
#include <type_traits>
#include "fusco.h"
#include "fusco_probe.h"

namespace {

typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));
typedef uint32_t u32x2 __attribute__((ext_vector_type(2)));

constexpr int kWave = 64;
constexpr int kXcds = 8;                                  // accelerator complexes of an MI355X
constexpr int kPlanThreads = 1024;                      // 16 waves per planner workgroup
constexpr int kPlanWaves = kPlanThreads / kWave;
// A planner tile holds R * 1024 (token, expert) pairs, R rounds of 64 pairs per wave: one round for inputs of
// up to 1024 pairs, two otherwise.
constexpr int kMaxRounds = 2;
constexpr int kRoundPairs = kPlanThreads;               // pairs of one round of the whole workgroup
constexpr int kMaxBins = FUSCO_MAX_E;
constexpr size_t kMaxRowChunks = FUSCO_MAX_ROW_BYTES / 16;

static_assert(kRoundPairs >= FUSCO_MAX_K, "a tile must hold at least one token");
static_assert(kMaxBins <= kPlanThreads, "the planner gives every bin a thread");

inline size_t align_up(size_t v, size_t a) { return (v + a - 1) / a * a; }

bool sizes_ok(int32_t N, int32_t k, int32_t E, int32_t D)
{
    if (N < 0 || k < 1 || k > FUSCO_MAX_K || E < 1 || E > FUSCO_MAX_E || D < 1 || D > E) return false;
    if (E % D != 0) return false;
    if ((int64_t)N * k >= ((int64_t)1 << 31)) return false;
    return true;
}

// From this many tiles on, per-tile counts are first summed over chunks of tiles (one more small launch),
// so that a placement workgroup reads about 2 * sqrt(tiles) rows of counts instead of one per tile.
// Measured, k = 8, 256 experts and 8 devices, plan alone with / without the chunks, us: 49 tiles 13.9 / 11.6, 80 tiles 14.3 / 13.1, 94 tiles
// 14.5 / 13.8, 98 tiles 14.7 / 13.9, 128 tiles 14.7 / 15.1, 157 tiles 15.4 / 18.0, 256 tiles 17.8 / 24.0; 1024 experts and 1024 devices, 128 tiles 23.6 /
// 38.3.  (Fewer columns cross later: 64 experts and 8 devices, 128 tiles 13.4 / 11.6.)
constexpr int kChunkMinTiles = 96;

inline int tokens_per_tile(int k, int rounds) { return rounds * kRoundPairs / k; }
inline int num_tiles(int N, int k, int rounds)
{
    const int tpt = tokens_per_tile(k, rounds);
    const int n = (N + tpt - 1) / tpt;
    return n < 1 ? 1 : n;
}

// Rounds with which the whole input is one tile (single-launch planner, fused plan + dispatch), or 0.
inline int single_tile_rounds(int N, int k)
{
    for (int r = 1; r <= kMaxRounds; r *= 2)
        if (N <= tokens_per_tile(k, r)) return r;
    return 0;
}

// Rounds per tile of the planner for these sizes.  A tile is also the unit in which dispatch moves rows
// (expert by expert inside a tile): two rounds give every expert twice as many neighbouring rows per tile,
// which is worth 5 us to dispatch at 8192 tokens x 8 rows of 14 KiB, half of what the whole plan takes there.
inline int plan_rounds(int N, int k)
{
    const int single = single_tile_rounds(N, k);
    return single ? single : kMaxRounds;
}

// tiles per chunk (a power of two near sqrt(n_tiles)), or 0 when the tiles are few enough to be read one by one
inline int chunk_tiles_for(int n_tiles)
{
    if (n_tiles < kChunkMinTiles) return 0;
    int c = 8;
    while (c * c < n_tiles) c *= 2;
    return c;
}
inline int num_chunks(int n_tiles)
{
    const int c = chunk_tiles_for(n_tiles);
    return c ? (n_tiles + c - 1) / c : 0;
}

}   // namespace

#endif
