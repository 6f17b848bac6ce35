// Pieces shared by the grouped-FFN kernels: the work items of a launch, bf16 packing.
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

#include "device_utils.h"
#include "mfma_common.h"

namespace metro {
namespace {

constexpr int kMaxSpr = 64;

// From 17 rows on a tile is better tall: a narrow one reads its rows once per 64 weight rows.  Measured, a layer, us, narrow up to
// 16 / 32 / 48 / 64 rows: 1024 tokens at 7168 x 2048 (METRO rank) 606 / 607 / 611 / 615, 97 tokens of it 443.3 / 445.0 / 444.8 / 445.4,
// 512 tokens at 4096 x 1536 150.7 / 151.7 / 152.9 / 151.6.  Where a long launch has only a few such tiles, they would start first
// and stand alone: a layer at 4096 x 1536 of 128 / 256 / 384 tokens, narrow up to 32 / 16 rows, METRO 122.6 / 134.9 / 144.4 against
// 124.5 / 139.4 / 145.9, token-balanced 132.0 / 138.3 / 141.0 against 134.6 / 138.0 / 142.7.
constexpr int kTallRows = 128;              // rows of a full tall tile
constexpr int kNarrowRows = 16;             // tiles of at most this many rows are narrow,
constexpr int kNarrowIfFew = 32;            // or of this many in launches past kFewItems of which few would be tall (kTallItems),
constexpr int kCutRows = 64;                // or of this many where a launch is cut into narrow tiles only

struct Tile {
    int slot, row0, rows, col;              // rows [row0, row0 + rows) of a slot x column tile `col`
};

// Upper bound of the tile count: cap / tile_rows full tiles, and per slot one remainder.
inline int max_tiles(int cap, int spr, int tile_rows) { return spr + cap / tile_rows; }

// ------------------------------------------------------------------------------------------ work items
// A slot of m rows gives m / th full tiles of th rows and one tile for the remainder.  Launches of few work items cut all
// slots into narrow tiles (th = 64); the others cut 128-row tiles, of which the full ones and the remainders above 16 rows
// are tall.  Tall ones come first, slot by slot; of the narrow ones full tiles, then the remainders, larger classes of rows
// first (ties: lower slot first).  Work item = (tile, column tile), for narrow ones tile-major.
// Every workgroup derives its own items from group_offsets (65 integers, one memory round trip, some
// hundred scalar-ish instructions): no planning kernel, no list in memory.  Each wave computes the
// same result with lane = local slot.

// Narrow tiles only, where that gives at most
//   kOneRound items: each has a CU for itself and ends earlier than the longer K loop of a tall tile; a second workgroup on a
//     CU may cost more than that.  Measured, gate/up + down, us, weights from HBM, narrow only / with tall tiles: one slot of 128 rows at
//     2048 x 768 (48 items) 17.7 / 28.7, one of 256 rows at 7168 x 2048 (256 items) 58 / 93.  Past it items alone do not tell: 288 of
//     them are 59 / 52 and 71 / 59 as 6 slots of 32 and 64 rows at 4096 x 1536 and 35 / 30 as 12 slots of 32 rows at 2048 x 768, but 43 / 60
//     as 3 slots of 96 rows at 4096 x 1536 and 28 / 36 as 6 of them at 2048 x 768; 18 slots of 64 rows at 2048 x 768 (432) 51 / 47, 6 of
//     96 rows at 7168 x 2048 (768) 188 / 129;
//   kFewItems items, if the tall tiles would be few (below kTallItems items) and not nearly alone (3 in 4): few long workgroups
//     beside many short ones leave CUs idle at the end.  A whole layer of 2048 x 768 at 256, 320, 384 and 512 tokens (skewed
//     popularity, 480 to 768 items, 60 to 170 of them would be tall), METRO 52 / 58, 53 / 61, 55 / 64 and 59 / 65, token-balanced 50 / 54,
//     52 / 56, 53 / 57 and 55 / 58; from 768 tokens on narrow tiles only lose (68.6 / 66.2 and 64.9 / 62.0).
constexpr int kOneRound = 256, kFewItems = 768, kTallItems = 170;

struct CutRule {
    int one_round, few, tall;               // the limits in tiles: of 64 rows, of 64 rows, tall
    CutRule() = default;
    CutRule(int narrow_cols, int tall_cols)
        : one_round(kOneRound / narrow_cols), few(kFewItems / narrow_cols), tall((kTallItems + tall_cols - 1) / tall_cols) {}
};

// The slots' tiles in the registers of a wave (lane = local slot), from which any item can be picked.
struct WorkList {
    int begin, rows;                            // per lane: the slot's rows
    int tall_tiles;                             // tall tiles of the slot
    int tall_first, tall_mine, tall_incl;       // in the XCD's list: first column, items of the slot, of the slots up to it
    int full, part, incl, rank, narrow_begin;   // full narrow tiles, rows of the remainder; narrow rows start here
    int n_full, n_narrow, tall_stride;          // uniform

    __device__ __forceinline__ void read(const int32_t* __restrict__ group_offsets, int spr, int cap, const CutRule& rule) {
        const int l = lane_id();
        int m = 0;
        begin = 0;
        if (l < spr) {                          // offsets that are not a partition of [0, cap] are clamped
            begin = min(max(group_offsets[l], 0), cap);
            m = min(max(group_offsets[l + 1], begin), cap) - begin;
        }
        // narrow and tall tiles in one scan; a clamped slot is past every limit by itself
        constexpr uint32_t kClamp = 1023 * kCutRows;
        static_assert(kFewItems < 1023 && 64 * 1023 < 65536, "the packed sums");
        const uint32_t u = min((uint32_t)m, kClamp);
        const uint32_t counts = __builtin_amdgcn_readlane(wave_inclusive_sum((int)((u + kCutRows - 1) / kCutRows |
                                    (u + kTallRows - 1 - kNarrowRows) / kTallRows << 16)), kWave - 1);
        const int cut = (int)(counts & 0xffff), tall = (int)(counts >> 16), rest = m & (kTallRows - 1);
        const int small = __popcll(__ballot(rest > 0 && rest <= kNarrowRows));
        const bool narrow_only = cut <= rule.one_round || (cut <= rule.few && tall < rule.tall && 3 * small > tall);
        const int limit = cut > rule.few && tall < rule.tall ? kNarrowIfFew : kNarrowRows;
        rows = m;
        full = narrow_only ? (uint32_t)m / kCutRows : (uint32_t)m / kTallRows;
        part = narrow_only ? m & (kCutRows - 1) : rest;
        tall_tiles = narrow_only ? 0 : full + (part > limit);
        narrow_begin = begin;
        if (!narrow_only) {                     // what the tall tiles leave: remainders up to the limit
            narrow_begin += full * kTallRows;
            full = 0;
            if (part > limit) part = 0;
        }
        incl = wave_inclusive_sum(full);
        n_full = __builtin_amdgcn_readlane(incl, kWave - 1);
        // remainders: in classes of rows, larger ones first, inside a class by slot
        const uint64_t below = lanes_below();
        rank = 0;
        uint64_t larger = 0;
        constexpr int kEdges[] = {48, 32, 16, 0};
#pragma unroll
        for (int c = 0; c < 4; ++c) {
            const uint64_t in = __ballot(part > kEdges[c]) & ~larger;
            if (part > kEdges[c] && !((larger >> l) & 1)) rank = __popcll(larger) + __popcll(in & below);
            larger |= in;
        }
        n_narrow = n_full + __popcll(larger);
    }

    // The tall items of an XCD; returns their number.  Workgroup i runs on XCD i mod 8, each with an L2 of its own.  The tiles of a
    // column of one slot read the same weights: they are neighbours in the list of one XCD.  The columns of a slot go round the XCDs, so
    // that each has the same share of every slot.  Measured, gate/up + down, us, against items by tile, columns inside: 4096 tokens
    // at 2048 x 768 47.6 + 31.9 / 54.1 + 34.3, 512 tokens at 4096 x 1536 107.9 + 53.0 / 108.6 + 53.4, 1024 tokens at 7168 x 2048 376.9 +
    // 201.1 / 375.0 + 202.4.  Columns round 4 or 2 XCDs, whose L2s then take fewer rows, but unequal shares of the slots, are slower
    // (by 4 to 7 and 15 to 23 %), and so is an eighth of the items in one piece (4096 x 1536: 112.8 + 59.4).
    // With fewer columns than XCDs the items themselves go round: the host cannot know the longest list, and a grid for 8 columns
    // would be mostly empty workgroups (4096 tokens at 128 x 128 36 us a layer, 30 without).
    __device__ __forceinline__ int list_tall(int xcd, int n_cols) {
        tall_stride = n_cols < 8 ? 1 : 8;
        tall_first = n_cols < 8 ? 0 : (xcd - lane_id() * n_cols) & 7;
        tall_mine = tall_tiles * (n_cols < 8 ? n_cols : (n_cols - tall_first + 7) >> 3);
        tall_incl = wave_inclusive_sum(tall_mine);
        const int n = __builtin_amdgcn_readlane(tall_incl, kWave - 1);
        return n_cols < 8 ? (n - xcd + 7) >> 3 : n;
    }
    __device__ __forceinline__ Tile tall(int nth, int xcd) const {
        const int i = tall_stride == 1 ? nth * 8 + xcd : nth;
        const uint64_t owner = __ballot(tall_incl - tall_mine <= i && i < tall_incl);      // exactly one lane
        const int o = __ffsll((unsigned long long)owner) - 1;
        const int tiles = __builtin_amdgcn_readlane(tall_tiles, o), at = i - __builtin_amdgcn_readlane(tall_incl - tall_mine, o);
        const int c = (uint32_t)at / (uint32_t)tiles, row = (at - c * tiles) * kTallRows;
        Tile t;
        t.slot = o;
        t.col = __builtin_amdgcn_readlane(tall_first, o) + c * tall_stride;
        t.row0 = __builtin_amdgcn_readlane(begin, o) + row;
        t.rows = min(kTallRows, __builtin_amdgcn_readlane(rows, o) - row);
        return t;
    }

    __device__ __forceinline__ Tile narrow(int ti, int col) const {
        Tile t;
        t.col = col;
        if (ti < n_full) {
            const uint64_t owner = __ballot(incl - full <= ti && ti < incl);      // exactly one lane
            const int o = __ffsll((unsigned long long)owner) - 1;
            t.slot = o;
            t.rows = kCutRows;
            t.row0 = __builtin_amdgcn_readlane(narrow_begin, o) + (ti - __builtin_amdgcn_readlane(incl - full, o)) * kCutRows;
        } else {
            const uint64_t owner = __ballot(part > 0 && n_full + rank == ti);     // exactly one lane
            const int o = __ffsll((unsigned long long)owner) - 1;
            t.slot = o;
            t.row0 = __builtin_amdgcn_readlane(narrow_begin + full * kCutRows, o);
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
