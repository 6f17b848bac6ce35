// Pieces shared by the grouped-FFN kernels: the work items of a launch, bf16 packing.
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

#include "device_utils.h"
#include "mfma_common.h"

namespace metro {
namespace {

constexpr int kMaxSpr = 64;

constexpr int kNarrowMost = 64;             // rows of a narrow tile at most

struct Tile {
    int slot, row0, rows, col;              // rows [row0, row0 + rows) of a slot x column tile `col`
};

// Upper bound of the tile count: cap / tile_rows full tiles, and per slot one remainder -- or two tiles where one-tile
// slots are cut finer (each at least half a tile).
inline int max_tiles(int cap, int spr, int tile_rows, bool finer_singles) {
    return (finer_singles ? 2 : 1) * spr + cap / tile_rows;
}

// ------------------------------------------------------------------------------------------ work items
// A slot of m rows gives m / tile_rows full tiles and one tile for the remainder; a remainder is tall if it has more
// than `narrow_rows` rows, wide if it has more than `stream_rows` (>= narrow_rows).  Tile order: full tiles, then the
// remainders, larger classes of rows first (ties: lower slot first); so wide tiles come first, then the other tall
// ones, then the narrow ones.  Work item = (tile, column tile), tile-major.
// Every workgroup derives its own items from group_offsets (65 integers, one memory round trip, some
// hundred scalar-ish instructions): no planning kernel, no list in memory.  Each wave computes the
// same result with lane = local slot.
// The slots' tiles in the registers of a wave (lane = local slot), from which any item can be picked.
struct WorkList {
    int begin, th, full, part, incl, rank;      // per lane
    int n_full, n_wide, n_tall, n_tiles;        // uniform

    __device__ __forceinline__ void read(const int32_t* __restrict__ group_offsets, int spr, int cap, int tile_rows,
                                         int single_rows, int stream_rows, int narrow_rows) {
        const int l = lane_id();
        int m = 0;
        begin = 0;
        if (l < spr) {                          // offsets that are not a partition of [0, cap] are clamped
            begin = min(max(group_offsets[l], 0), cap);
            m = min(max(group_offsets[l + 1], begin), cap) - begin;
        }
        // one-tile slots may be cut finer than the slots that re-read their weights once per tile
        th = (single_rows > 0 && m <= tile_rows) ? single_rows : tile_rows;
        full = m / th;
        part = m % th;
        incl = wave_inclusive_sum(full);
        n_full = __builtin_amdgcn_readlane(incl, kWave - 1);
        // remainders: in classes of rows, larger ones first, inside a class by slot
        const uint64_t below = lanes_below();
        rank = 0;
        uint64_t larger = 0;
        constexpr int kEdges[] = {96, 64, 32, 16, 0};
#pragma unroll
        for (int c = 0; c < 5; ++c) {
            const uint64_t in = __ballot(part > kEdges[c]) & ~larger;
            if (part > kEdges[c] && !((larger >> l) & 1)) rank = __popcll(larger) + __popcll(in & below);
            larger |= in;
        }
        // stream_rows >= tile_rows: no wide class at all, full tiles take the stream path too
        n_wide = stream_rows >= tile_rows ? 0 : n_full + __popcll(__ballot(part > stream_rows));
        // full tiles run as tall ones unless no tile is tall (those of slots cut finer too, to keep the order simple)
        n_tall = (tile_rows > narrow_rows ? n_full : 0) + __popcll(__ballot(part > narrow_rows));
        n_tiles = n_full + __popcll(__ballot(part > 0));
    }

    __device__ __forceinline__ Tile tile(int ti, int col) const {
        Tile t;
        t.col = col;
        if (ti < n_full) {
            const uint64_t owner = __ballot(incl - full <= ti && ti < incl);      // exactly one lane
            const int o = __ffsll((unsigned long long)owner) - 1;
            const int first = __builtin_amdgcn_readlane(incl - full, o);
            t.slot = o;
            t.rows = __builtin_amdgcn_readlane(th, o);
            t.row0 = __builtin_amdgcn_readlane(begin, o) + (ti - first) * t.rows;
        } else {
            const uint64_t owner = __ballot(part > 0 && n_full + rank == ti);     // exactly one lane
            const int o = __ffsll((unsigned long long)owner) - 1;
            t.slot = o;
            t.row0 = __builtin_amdgcn_readlane(begin + full * th, o);
            t.rows = __builtin_amdgcn_readlane(part, o);
        }
        return t;
    }
};

struct Item {
    Tile tile;
    bool valid;
};

// Without classes: tiles of at most `tile_rows` rows, slot by slot, `n_cols` column tiles each.
__device__ __forceinline__ Item locate_in_order(const int32_t* __restrict__ group_offsets, int spr, int cap,
                                                int tile_rows, int n_cols, int64_t id) {
    const int l = lane_id();
    int begin = 0, m = 0;
    if (l < spr) {                              // offsets that are not a partition of [0, cap] are clamped
        begin = min(max(group_offsets[l], 0), cap);
        m = min(max(group_offsets[l + 1], begin), cap) - begin;
    }
    const int tiles = (m + tile_rows - 1) / tile_rows;
    const int incl = wave_inclusive_sum(tiles);
    const int ti = (int)(id >> 32 ? id / n_cols : (int64_t)((uint32_t)id / (uint32_t)n_cols));  // < 2^24 / tile_rows + 64
    Item it;
    it.tile = Tile{0, 0, 0, 0};
    const uint64_t owner = __ballot(incl - tiles <= ti && ti < incl);          // exactly one lane, or none past the end
    it.valid = owner != 0;
    if (!it.valid) return it;
    const int o = __ffsll((unsigned long long)owner) - 1;
    const int first = (ti - __builtin_amdgcn_readlane(incl - tiles, o)) * tile_rows;
    it.tile.slot = o;
    it.tile.row0 = __builtin_amdgcn_readlane(begin, o) + first;
    it.tile.rows = min(tile_rows, __builtin_amdgcn_readlane(m, o) - first);
    it.tile.col = (int)(id - (int64_t)ti * n_cols);
    return it;
}

__device__ __forceinline__ uint32_t pack_bf16x2(float a, float b) {
    uint32_t ua = __float_as_uint(a), ub = __float_as_uint(b);
    const uint32_t ra = ua + 0x7fffu + ((ua >> 16) & 1u);       // round to nearest even
    const uint32_t rb = ub + 0x7fffu + ((ub >> 16) & 1u);
    // NaN stays a (quiet) NaN: the rounding add could carry its mantissa into Inf or -0
    ua = (a != a) ? (ua | 0x00400000u) : ra;
    ub = (b != b) ? (ub | 0x00400000u) : rb;
    return (ua >> 16) | (ub & 0xffff0000u);
}

}  // namespace
}  // namespace metro
