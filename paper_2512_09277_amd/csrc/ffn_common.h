// Pieces shared by the grouped-FFN kernels: operand types, the work items of a launch, bf16 packing.
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

#include <type_traits>
#include <utility>

#include "device_utils.h"

namespace metro {
namespace {

typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef float floatx4 __attribute__((ext_vector_type(4)));
typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));
typedef uint32_t u32x2 __attribute__((ext_vector_type(2)));
typedef int i32x4 __attribute__((ext_vector_type(4)));

constexpr int kMaxSpr = 64;

struct Tile {
    int slot, row0, rows, col;              // rows [row0, row0 + rows) of a slot x column tile `col`
};

// Upper bound of the tile count (the launch grid; workgroups past the real count exit after locating
// nothing): cap / tile_rows full tiles, and per slot one remainder -- or two tiles where one-tile slots
// are cut finer (each at least half a tile).
inline int max_tiles(int cap, int spr, int tile_rows, bool finer_singles) {
    return (finer_singles ? 2 : 1) * spr + cap / tile_rows;
}

// ------------------------------------------------------------------------------------------ work items
// A slot of m rows gives m / tile_rows full tiles and one tile for the remainder; a tile is wide if it has
// more than `stream_rows` rows.  Tile order: full tiles, then the remainders by rows descending
// (ties: lower slot first); the first n_wide of them are the wide ones.  Work item = (tile, column
// tile), tile-major, wide items first, `ntw` column tiles per wide tile and `nts` per stream tile.
// Every workgroup derives its own item from group_offsets (65 integers, one memory round trip, a few
// hundred scalar-ish instructions): no planning kernel, no list in memory.  Each wave computes the
// same result with lane = local slot; everything returned is uniform.
struct Item {
    Tile tile;
    bool valid, wide;
};

__device__ __forceinline__ Item locate_item(const int32_t* __restrict__ group_offsets, int spr, int cap,
                                            int tile_rows, int single_rows, int stream_rows, int ntw, int nts,
                                            int id) {
    const int l = lane_id();
    int begin = 0, m = 0;
    if (l < spr) {                              // offsets that are not a partition of [0, cap] are clamped
        begin = min(max(group_offsets[l], 0), cap);
        m = min(max(group_offsets[l + 1], begin), cap) - begin;
    }
    // one-tile slots may be cut finer than the slots that re-read their weights once per tile
    const int th = (single_rows > 0 && m <= tile_rows) ? single_rows : tile_rows;
    const int full = m / th, part = m % th;
    const int incl = wave_inclusive_sum(full);
    const int n_full = __builtin_amdgcn_readlane(incl, kWave - 1);
    int rank = 0;                               // remainders: more rows first, then lower slot
#pragma unroll
    for (int j = 0; j < kWave; ++j) {
        const int pj = __builtin_amdgcn_readlane(part, j);
        rank += (pj > part || (pj == part && j < l)) ? 1 : 0;
    }
    const int n_part_wide = __popcll(__ballot(part > stream_rows));
    const int n_part = __popcll(__ballot(part > 0));
    // stream_rows >= 128: no wide class at all, full tiles take the stream path too
    const int n_wide = stream_rows >= tile_rows ? 0 : n_full + n_part_wide;
    const int n_stream = n_full + n_part - n_wide;
    const int wide_items = n_wide * ntw, n_items = wide_items + n_stream * nts;

    Item it;
    it.valid = id < n_items;
    it.wide = id < wide_items;
    it.tile = Tile{0, 0, 0, 0};
    if (!it.valid) return it;
    const int nt = it.wide ? ntw : nts, r = it.wide ? id : id - wide_items;
    const int tl = r / nt;
    const int ti = it.wide ? tl : n_wide + tl;
    it.tile.col = r - tl * nt;
    if (ti < n_full) {
        const uint64_t owner = __ballot(incl - full <= ti && ti < incl);      // exactly one lane
        const int o = __ffsll((unsigned long long)owner) - 1;
        const int first = __builtin_amdgcn_readlane(incl - full, o);
        it.tile.slot = o;
        const int th_o = __builtin_amdgcn_readlane(th, o);
        it.tile.row0 = __builtin_amdgcn_readlane(begin, o) + (ti - first) * th_o;
        it.tile.rows = th_o;
    } else {
        const uint64_t owner = __ballot(part > 0 && n_full + rank == ti);     // exactly one lane
        const int o = __ffsll((unsigned long long)owner) - 1;
        it.tile.slot = o;
        it.tile.row0 = __builtin_amdgcn_readlane(begin + full * th, o);
        it.tile.rows = __builtin_amdgcn_readlane(part, o);
    }
    it.valid = it.tile.rows > 0;                // always true here; keeps a broken invariant from indexing row -1
    return it;
}

// The same without classes: tiles of at most `tile_rows` rows, slot by slot, `n_cols` column tiles each.
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
    it.wide = false;
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

// do_step(U, s) for U = 0..n-1 with compile-time U (buffer indices), s = s0 + U.
template <int... Us, typename F>
__device__ __forceinline__ void run_steps(std::integer_sequence<int, Us...>, F&& f, int s0) {
    (f(std::integral_constant<int, Us>{}, s0 + Us), ...);
}
template <int... Us, typename F>
__device__ __forceinline__ void run_steps_tail(std::integer_sequence<int, Us...>, F&& f, int s0, int n_steps) {
    // short-circuit: once a step is past the end nothing after it is tested, the paths join only at the end
    (void)((s0 + Us < n_steps && (f(std::integral_constant<int, Us>{}, s0 + Us), true)) && ...);
}

}  // namespace
}  // namespace metro
