// skim_tail.h -- how one level of the discrepancy tail's tree is dealt to
// workgroups (the host sizes the launch by it, the kernel finds its work by it).
//
// A level adds the rows of survival functions two by two.  The sum of a pair is
// made in tiles of kTailTile cells, tile t from 16 t + 16 steps (see
// k_tail_pair).  With many tiles a workgroup takes whole tiles, a long one with a
// short one; with fewer than kTailSplit every tile is cut into parts of `part`
// steps, a workgroup each.
#pragma once

#include <hip/hip_runtime.h>

#include <cstdint>

namespace skim {

constexpr int kTailTile = 256, kTailChunk = 32;
constexpr uint32_t kTailCounters = 1024;        // arrival counters, cleared at the start of a tail
constexpr uint64_t kTailSplit = kTailCounters;  // fewer tiles than this: split their steps
constexpr uint64_t kTailPartials = 2 * kTailSplit;  // parts of a level at most

struct TailLevel {
    uint32_t tiles;     // of a row
    uint32_t part;      // steps of a workgroup (whole tiles: as many as the longest has)
    uint64_t pairs, per_pair, items;  // workgroups of a pair, of the level
    bool whole;
};

// A workgroup's work: part `part` of `nparts` of a tile of a pair, then tile
// `more` if that is not negative; or (pair = pairs) `tile` of the odd last row.
struct TailItem {
    uint64_t pair;
    uint32_t tile, part, nparts;
    int more;
};

__host__ __device__ inline uint32_t tail_tiles(uint64_t cells) {
    return (uint32_t)((cells + kTailTile - 1) / kTailTile);
}
__host__ __device__ inline uint32_t tail_parts(uint32_t tile, uint32_t part) {
    return (16 * tile + 16 + part - 1) / part;
}

inline TailLevel tail_level(uint32_t rows, uint64_t cells) {
    TailLevel L{};
    L.tiles = tail_tiles(cells);
    L.pairs = rows / 2;
    L.whole = L.pairs * L.tiles >= kTailSplit;
    if (L.whole) {
        L.part = 16 * L.tiles;
        L.per_pair = (L.tiles + 1) / 2;
    } else {
        // about kTailSplit parts in all, none below one chunk of steps: a tile
        // adds at most one more than its share, so there are at most
        // kTailPartials of them
        const uint64_t steps = L.pairs * 8 * L.tiles * (L.tiles + 1);
        const uint64_t share = (steps + kTailSplit - 1) / kTailSplit;
        L.part = (uint32_t)(share > (uint64_t)kTailChunk ? share : kTailChunk);
        for (uint32_t t = 0; t < L.tiles; ++t) L.per_pair += tail_parts(t, L.part);
    }
    L.items = L.pairs * L.per_pair + (rows % 2 ? L.tiles : 0);
    return L;
}

__host__ __device__ inline TailItem tail_item(const TailLevel &L, uint64_t item) {
    TailItem w{L.per_pair ? item / L.per_pair : 0, 0, 0, 1, -1};
    if (w.pair >= L.pairs) {
        w.pair = L.pairs;
        w.tile = (uint32_t)(item - L.pairs * L.per_pair);
        return w;
    }
    uint64_t rest = item - w.pair * L.per_pair;
    w.tile = L.tiles - 1;  // the longest first
    if (L.whole) {
        w.more = (int)rest < (int)w.tile - (int)rest ? (int)rest : -1;
        w.tile -= (uint32_t)rest;
        return w;
    }
    while (rest >= tail_parts(w.tile, L.part)) rest -= tail_parts(w.tile--, L.part);
    w.part = (uint32_t)rest;
    w.nparts = tail_parts(w.tile, L.part);
    return w;
}

}  // namespace skim
