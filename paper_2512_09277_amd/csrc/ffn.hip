// moe_grouped_ffn for gfx950: SwiGLU expert FFN over one rank's per-slot token lists.
//
// Decode is HBM-bound: runtime follows the bytes of the activated experts' weights (Sec. 3.2 of
// arxiv 2512.09277).  Every activated weight row is streamed from HBM once per tile, with 128-bit loads that
// land directly in the matrix-core operand layout (16 rows x 64 contiguous bytes per instruction).
// Work is cut into tiles of one slot's rows (at most 128; 64 on the smallest shapes):
//   narrow tiles (<= 64 rows, 32 at large shapes; the bulk of the bytes): ffn_split.h -- K split over the four waves, 64 weight rows per
//       workgroup, activations straight into registers, no barrier in the K loop;
//   tall tiles (up to 128 rows, the popular experts), activations staged through LDS: wide ones (large shapes) with 4 x 16
//       weight rows per wave and K steps of 64, so that each activation fragment read from LDS feeds four MFMAs;
//       stream ones (mid shapes) with 2 x 16 weight rows per wave.  They are listed first so that they spread over
//       the chip early.
//   gate/up: a wave owns gate rows and the matching up rows, so silu(gate)*up is formed in
//            registers and written once as bf16;   down: same structure over K = I.
// A slot with no rows produces no tile and its weights are never touched.  There is no planning pass:
// every workgroup finds its (tile, column tile) from group_offsets itself.
#include <hip/hip_runtime.h>
#include <stdint.h>

#include <algorithm>
#include <type_traits>
#include <utility>

#include "ffn_common.h"
#include "ffn_split.h"
#include "host_utils.h"
#include "metro.h"

namespace metro {
namespace {

constexpr int kThreads = 256;
constexpr int kWideRows = 128;              // rows of a full wide tile

// ------------------------------------------------------------------------------------------ MFMA path
struct FfnArgs {
    const __bf16* src;        // gate/up: x[T,H]; down: act[cap,I]
    const int32_t* perm_pair; // gate/up only
    const __bf16* w;          // gate/up: w13[spr,2I,H]; down: w2[spr,H,I]
    __bf16* dst;              // gate/up: act[cap,I]; down: y_perm[cap,H]
    const int32_t* group_offsets;
    int T, k, spr, H, I;
    int ldw;                  // elements between consecutive weight rows (>= K)
    int tile_rows;            // rows of a full tile (<= 128)
    int single_rows;          // > 0: slots of at most tile_rows rows are cut into tiles of this many rows
    int stream_rows;          // tiles with more rows are wide
    int ntw, nts;             // column tiles per wide / stream tile
    int narrow_rows;          // tiles of at most this many rows are narrow (<= 64)
    int ntn;                  // column tiles per narrow tile
};

__device__ __forceinline__ float silu(float g) { return g / (1.0f + __expf(-g)); }

// D[i][j] of block b, sub-tile mt: i = output column 4*q + v of the block, j = tile row r16.
template <bool kGateUp, int NB, int MT>
__device__ __forceinline__ void store_tile(const FfnArgs& a, const Tile& t, const floatx4 (&acc)[NB][MT], int col0,
                                           int n_out, int mt_count, int r16, int q) {
    const int H = a.H, I = a.I;
#pragma unroll
    for (int mt = 0; mt < MT; ++mt) {
        const int row = mt * 16 + r16;
        if (mt < mt_count && row < t.rows) {
            if (kGateUp) {
#pragma unroll
                for (int b = 0; b < NB / 2; ++b) {
                    const int col = col0 + b * 16;
                    if (col < n_out) {
                        const floatx4 g = acc[b][mt], u = acc[b + NB / 2][mt];
                        u32x2 o;
                        o.x = pack_bf16x2(silu(g[0]) * u[0], silu(g[1]) * u[1]);
                        o.y = pack_bf16x2(silu(g[2]) * u[2], silu(g[3]) * u[3]);
                        *reinterpret_cast<u32x2*>(a.dst + (size_t)(t.row0 + row) * I + col + q * 4) = o;
                    }
                }
            } else {
#pragma unroll
                for (int b = 0; b < NB; ++b) {
                    const int col = col0 + b * 16;
                    if (col < n_out) {
                        u32x2 o;
                        o.x = pack_bf16x2(acc[b][mt][0], acc[b][mt][1]);
                        o.y = pack_bf16x2(acc[b][mt][2], acc[b][mt][3]);
                        *reinterpret_cast<u32x2*>(a.dst + (size_t)(t.row0 + row) * H + col + q * 4) = o;
                    }
                }
            }
        }
    }
}

// One tile x one column tile.
//   NB    16-row weight blocks per wave (gate/up: NB/2 gate blocks + the matching up blocks)
//   MT    16-row activation sub-tiles (tile rows <= 16*MT)
//   BK    K elements per step;  DEPTH  steps the loads run ahead
// Lane (r16, q) of a wave supplies, for MFMA j of a step, the 8 elements k = j*32 + q*8 .. +8 of
// weight row r16 (A operand) and of tile row r16 (B operand): one load instruction reads 64
// contiguous bytes of each of 16 rows.  D[i][j]: i = weight row 4*q + v, j = tile row r16.
template <bool kGateUp, int NB, int MT, int BK, int DEPTH>
__device__ __forceinline__ void ffn_tile(const FfnArgs& a, const Tile t, const int nt, char* lds) {
    constexpr int NJ = BK / 32;                 // MFMAs per block per step
    constexpr int NW = DEPTH + 1;               // weight register buffers
    constexpr int kLdsRow = BK * 2 + 16;        // bytes per staged row (+16 spreads the banks)
    constexpr int kChunks = BK * 2 / 16;        // 16-byte chunks per staged row
    constexpr int kRowsPerPass = kThreads / kChunks;
    constexpr int NP = (MT * 16 + kRowsPerPass - 1) / kRowsPerPass;   // staging loads per thread
    constexpr int kPeriod = (DEPTH == 1) ? 2 : (DEPTH == 2) ? 6 : 12; // lcm(NW, DEPTH, 2)
    static_assert(DEPTH >= 1 && DEPTH <= 3, "prefetch distance");

    const int tid = threadIdx.x, lane = tid & 63;
    const int wv = __builtin_amdgcn_readfirstlane(tid >> 6);        // wave index, kept in a scalar register
    const int r16 = lane & 15, q = lane >> 4;
    const int H = a.H, I = a.I;
    const int K = kGateUp ? H : I;
    const int n_steps = K / BK;
    const int mt_count = (t.rows + 15) >> 4;
    const int n_out = kGateUp ? I : H;          // output columns of this stage
    const int cols_per_wave = kGateUp ? NB * 8 : NB * 16;
    const int col0 = nt * 4 * cols_per_wave + wv * cols_per_wave;     // first output column of the wave

    // Addresses are a uniform base (scalar registers) plus a 32-bit per-lane offset, which keeps the
    // vector registers for data in flight.  Weight row of block b: gate/up pairs block b (gate) with
    // block b + NB/2 (up).
    const char* wslot = reinterpret_cast<const char*>(a.w) + (size_t)t.slot * (kGateUp ? 2 * I : H) * a.ldw * 2;
    const uint32_t w_lane = (uint32_t)(r16 * a.ldw + q * 8) * 2u;
    const char* pw[NB];                                               // uniform: first row of block b
#pragma unroll
    for (int b = 0; b < NB; ++b) {
        int col = kGateUp ? col0 + (b % (NB / 2)) * 16 : col0 + b * 16;
        col = col < n_out ? col : n_out - 16;   // a block past the last column repeats the last block
        const int row = (kGateUp && b >= NB / 2) ? I + col : col;
        pw[b] = wslot + (size_t)row * a.ldw * 2;
    }

    // activation staging: thread (frow, fchunk) copies 16 bytes of rows frow, frow + kRowsPerPass, ...
    // (the host only takes this path while every activation byte offset fits 32 bits)
    const int frow = tid / kChunks, fchunk = tid % kChunks;
    const char* xbase = reinterpret_cast<const char*>(a.src);
    uint32_t x_lane[NP];
#pragma unroll
    for (int pz = 0; pz < NP; ++pz) {
        int row = pz * kRowsPerPass + frow;
        row = row < t.rows ? row : t.rows - 1;  // rows past the tile repeat its last row
        const uint32_t src_row = kGateUp ? (uint32_t)min(max(a.perm_pair[t.row0 + row] / a.k, 0), a.T - 1)
                                         : (uint32_t)(t.row0 + row);
        x_lane[pz] = src_row * (uint32_t)(K * 2) + fchunk * 16;
    }
    const int wr_off = frow * kLdsRow + fchunk * 16;
    const int rd_off = r16 * kLdsRow + q * 16;
    constexpr int kLdsBuf = NP * kRowsPerPass * kLdsRow;   // staged rows past 16*MT are never read

    floatx4 acc[NB][MT];
#pragma unroll
    for (int b = 0; b < NB; ++b)
#pragma unroll
        for (int mt = 0; mt < MT; ++mt) acc[b][mt] = floatx4{0.f, 0.f, 0.f, 0.f};

    u32x4 w[NW][NB * NJ];
    u32x4 xr[DEPTH][NP];

    auto load_w = [&](int buf, int step) {
#pragma unroll
        for (int b = 0; b < NB; ++b)
#pragma unroll
            for (int j = 0; j < NJ; ++j)
                w[buf][b * NJ + j] = *reinterpret_cast<const u32x4*>(pw[b] + (size_t)step * (BK * 2) + w_lane + j * 64);
    };
    auto load_x = [&](int set, int step) {
#pragma unroll
        for (int pz = 0; pz < NP; ++pz)
            xr[set][pz] = *reinterpret_cast<const u32x4*>(xbase + (size_t)step * (BK * 2) + x_lane[pz]);
    };
    auto park_x = [&](int set, int buf) {
#pragma unroll
        for (int pz = 0; pz < NP; ++pz)
            *reinterpret_cast<u32x4*>(lds + buf * kLdsBuf + wr_off + pz * kRowsPerPass * kLdsRow) = xr[set][pz];
    };

    // Every load below is unconditional (past the last step the index is clamped, which re-reads
    // the last step): the compiler can then count outstanding loads exactly and waits only for
    // the ones a step consumes, instead of draining the queue at every branch join.
    const int last = n_steps - 1;
    // (the weight addresses need only the tile, the activation addresses also need perm_pair: the
    // weight loads go out first so that they overlap that extra round trip)
#pragma unroll
    for (int d = 0; d < DEPTH; ++d) load_w(d, min(d, last));
    load_x(0, 0);
#pragma unroll
    for (int d = 1; d < DEPTH; ++d) load_x(d % DEPTH, min(d, last));
    park_x(0, 0);
    __syncthreads();

    // One K step with compile-time buffer indices u (= step s mod kPeriod).
    auto do_step = [&](auto U, const int s) {
        constexpr int u = decltype(U)::value;
        // Loads retire in issue order: the activations go first so that waiting for them (to park
        // them one step later) never waits for the younger weight loads.
        const int ps = min(s + DEPTH, last);                          // past the end: re-read the last step
        load_x(u % DEPTH, ps);
        load_w((u + DEPTH) % NW, ps);
        const char* cur = lds + (u % 2) * kLdsBuf + rd_off;
#pragma unroll
        for (int mt = 0; mt < MT; ++mt) {
            if (mt < mt_count) {
#pragma unroll
                for (int j = 0; j < NJ; ++j) {
                    const bf16x8 xb = *reinterpret_cast<const bf16x8*>(cur + mt * 16 * kLdsRow + j * 64);
#pragma unroll
                    for (int b = 0; b < NB; ++b)
                        acc[b][mt] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(
                            __builtin_bit_cast(bf16x8, w[u % NW][b * NJ + j]), xb, acc[b][mt], 0, 0, 0);
                }
            }
        }
        // activations of the next step were loaded DEPTH-1 steps ago (set (u+1) % DEPTH)
        park_x((u + 1) % DEPTH, (u + 1) % 2);
        __syncthreads();
    };

    int s0 = 0;
    for (; s0 + kPeriod <= n_steps; s0 += kPeriod) run_steps(std::make_integer_sequence<int, kPeriod>{}, do_step, s0);
    run_steps_tail(std::make_integer_sequence<int, kPeriod - 1>{}, do_step, s0, n_steps);
    store_tile<kGateUp, NB, MT>(a, t, acc, col0, n_out, mt_count, r16, q);
}

constexpr int kLdsSplit = 4 * 4 * (kNarrowMost / 16) * 64 * (int)sizeof(floatx4);      // partial sums of four waves
constexpr int kLdsStream = 2 * 64 * (128 * 2 + 16);
constexpr int kLdsWide = 2 * 128 * (64 * 2 + 16);
constexpr int kLdsBytes = std::max(kLdsSplit, std::max(kLdsWide, kLdsStream));

// Narrow tiles.  Measured against tiles staged through LDS with a barrier per K step (gate/up + down, us): 8 tokens of the
// 2048 x 768 shape 21 + 10 -> 13 + 6.5 (twice the workgroups for the same bytes, nobody waits for a sibling wave's loads);
// 256 tokens of it 38 + 18 -> 30 + 16; 97 tokens of the 7168 x 2048 shape (token-balanced) 288 + 152 -> 268 + 138; 1024
// tokens of it (METRO, whose time is in the tall tiles) 384 + 205 -> 383 + 201.
//   Blocks: 2 instead of 4 weight blocks per workgroup re-read the activations twice as often and lose everywhere (97 tokens:
//   276 + 177).
//   Depth: what 256 registers hold.
constexpr int kNarrowBlocks = 4;
// Workgroups of the narrow tiles at most; a workgroup past the last item costs about 2 ns, so the grid is not sized for
// the most tiles a rank could have, and the rest is taken in turns.  Three times the 512 resident ones: with fewer, who
// gets one item more is decided at launch and not by who is free (512: 287 us, 1024: 269, 1536 and more: 268; 97
// tokens, gate/up).
constexpr int kNarrowGrid = 1536;

template <bool kGateUp>
__global__ __launch_bounds__(kThreads, 2) void ffn_mfma_kernel(FfnArgs a) {
    extern __shared__ __attribute__((aligned(16))) char lds[];
    // Work items = (tile, column tile), wide items first: a wide workgroup lives several times longer
    // than a stream one, so it has to start early for the other items to fill in around it.
    // (Measured alternatives that lost: spreading the wide items through the launch order,
    // alternating wide and stream items, and per-XCD work queues.)  Everything here is uniform per
    // workgroup.
    WorkList wl;
    wl.read(a.group_offsets, a.spr, a.T * a.k, a.tile_rows, a.single_rows, a.stream_rows, a.narrow_rows);
    const int wide_items = wl.n_wide * a.ntw, tall_items = wide_items + (wl.n_tall - wl.n_wide) * a.nts;
    if ((int)blockIdx.x >= tall_items) {
        const SplitArgs sa{a.src, a.perm_pair, a.w, a.dst, a.T, a.k, a.H, a.I, a.ldw};
        const int n = (wl.n_tiles - wl.n_tall) * a.ntn, stride = gridDim.x - tall_items;
        for (int id = blockIdx.x - tall_items; id < n; id += stride) {
            const int ti = id / a.ntn;
            const Tile t = wl.tile(wl.n_tall + ti, id - ti * a.ntn);
            if (t.rows <= 16) split_tile<kGateUp, __bf16, __bf16, __bf16, kNarrowBlocks, 1, 4, KRows::kWhole>(sa, t, lds);
            else if (t.rows <= 32) split_tile<kGateUp, __bf16, __bf16, __bf16, kNarrowBlocks, 2, 3, KRows::kWhole>(sa, t, lds);
            else if (t.rows <= 48) split_tile<kGateUp, __bf16, __bf16, __bf16, kNarrowBlocks, 3, 2, KRows::kWhole>(sa, t, lds);
            else split_tile<kGateUp, __bf16, __bf16, __bf16, kNarrowBlocks, 4, 2, KRows::kWhole>(sa, t, lds);
            __syncthreads();                                             // the next item's sums reuse the LDS
        }
        return;
    }
    const int id = blockIdx.x;
    const bool wide = id < wide_items;
    const int nt = wide ? a.ntw : a.nts, r = wide ? id : id - wide_items, tl = r / nt;
    const Tile t = wl.tile(wide ? tl : wl.n_wide + tl, r - tl * nt);
    // partial wide tiles stage only the rows they have; with half the accumulators the 64-row variant
    // also affords a second K step of weights in flight (token-balanced rank: gate/up 401 -> 390 us)
    if (wide && t.rows <= 64) ffn_tile<kGateUp, 4, 4, 64, 2>(a, t, t.col, lds);
    else if (wide && t.rows <= 96) ffn_tile<kGateUp, 4, 6, 64, 1>(a, t, t.col, lds);
    else if (wide) ffn_tile<kGateUp, 4, 8, 64, 1>(a, t, t.col, lds);
    else if (t.rows <= 64) ffn_tile<kGateUp, 2, 4, 128, 2>(a, t, t.col, lds);
    else ffn_tile<kGateUp, 2, 8, 64, 3>(a, t, t.col, lds);
}

// Tall workgroups for the most tall tiles `cap` rows can make, and the narrow ones.
inline int mfma_grid(const FfnArgs& a, int cap, int spr) {
    const int tall = a.tile_rows > a.narrow_rows ? std::min(cap / a.narrow_rows, max_tiles(cap, spr, a.tile_rows, a.single_rows > 0)) : 0;
    const int narrow = std::min(a.ntn * (std::min(spr, cap) + cap / a.narrow_rows), kNarrowGrid);
    return tall * std::max(a.ntw, a.nts) + narrow;
}

// ------------------------------------------------------------------------------------------ general path
// fp32 storage, and 16-bit shapes whose H or I is no multiple of 128 (activations between the stages in fp32): K-split
// tiles (ffn_split.h) of at most 32 rows x 16 gate/up columns or 32 down columns.  What bounds it is HBM latency times
// occupancy (fp32 matrix instructions take about a third of the time at 32 rows), so the tiles are small -- many
// workgroups -- and registers are kept low enough for three workgroups per CU.  Measured on the 17-slot, 362-row
// fp32 rank of the 2048 x 768 shape, gate/up + down: 94 + 42 us with 64 rows x 32/64 columns at two workgroups per CU,
// 71 + 39 us with 32 rows x 16/32 columns, 73 + 35 us with three per CU (this one); on 2000 x 712 in bf16
// 30 + 21 us against 33 + 28 us.  (The vector-ALU kernels these replaced: 328 + 119 and 440 + 137 us.)
constexpr int kGenRows = 32;
constexpr int kGenBlocks = 2;               // 16-row weight blocks of a workgroup
constexpr int kGenGateUpCols = kGenBlocks * 8, kGenDownCols = kGenBlocks * 16;
constexpr int kGenLds = 4 * kGenBlocks * (kGenRows / 16) * 64 * (int)sizeof(floatx4);
// Two rounds of the 768 resident workgroups; more items loop.  (The grid can only be sized for a rank that gets every
// pair of the batch; a workgroup that finds no item costs about 2 ns.)
constexpr int kGenGrid = 1536;

template <bool kGateUp, typename WT, KRows kRows>
__global__ __launch_bounds__(kThreads, 3) void general_ffn_kernel(SplitArgs a, const int32_t* __restrict__ group_offsets,
                                                                  int spr, int n_cols, int64_t n_items) {
    __shared__ __attribute__((aligned(16))) char lds[kGenLds];
    using XT = std::conditional_t<kGateUp, WT, float>;
    using OT = std::conditional_t<kGateUp, float, WT>;
    for (int64_t id = blockIdx.x; id < n_items; id += gridDim.x) {
        const Item it = locate_in_order(group_offsets, spr, a.T * a.k, kGenRows, n_cols, id);
        if (!it.valid) return;                                       // uniform; items are consecutive
        if constexpr (kRows == KRows::kTiny) split_tile<kGateUp, WT, XT, OT, kGenBlocks, 2, 1, kRows>(a, it.tile, lds);
        else if (it.tile.rows <= 16) split_tile<kGateUp, WT, XT, OT, kGenBlocks, 1, 3, kRows>(a, it.tile, lds);
        else split_tile<kGateUp, WT, XT, OT, kGenBlocks, 2, 2, kRows>(a, it.tile, lds);
        __syncthreads();                                             // the next item's sums reuse the LDS
    }
}

template <bool kGateUp>
int launch_general(const SplitArgs& a, const int32_t* group_offsets, int spr, int dtype, hipStream_t st) {
    const int n_out = kGateUp ? a.I : a.H, K = kGateUp ? a.H : a.I;
    const int cols = kGateUp ? kGenGateUpCols : kGenDownCols, n_cols = (n_out + cols - 1) / cols;
    const int64_t n_items = (int64_t)max_tiles(a.T * a.k, spr, kGenRows, false) * n_cols;
    const uint32_t grid = (uint32_t)(n_items < kGenGrid ? n_items : kGenGrid);
    auto go = [&](auto kernel) {
        hipLaunchKernelGGL(kernel, dim3(grid), dim3(kThreads), 0, st, a, group_offsets, spr, n_cols, n_items);
    };
    // vectors of 16 bytes need a row of at least one
    if (dtype == METRO_DTYPE_F32) {
        if (K < 4) go(general_ffn_kernel<kGateUp, float, KRows::kTiny>);
        else go(general_ffn_kernel<kGateUp, float, KRows::kRagged>);
    } else {
        if (K < 8) go(general_ffn_kernel<kGateUp, __bf16, KRows::kTiny>);
        else go(general_ffn_kernel<kGateUp, __bf16, KRows::kRagged>);
    }
    return hipGetLastError() == hipSuccess ? METRO_OK : METRO_ERR_HIP;
}

inline bool mfma_shape(int H, int I, int dtype) {
    return dtype == METRO_DTYPE_BF16 && H % 128 == 0 && I % 128 == 0;
}

inline bool mfma_fits(int T, int k, int H, int I);
inline bool use_mfma(int T, int k, int H, int I, int dtype) { return mfma_shape(H, I, dtype) && mfma_fits(T, k, H, I); }

// The MFMA kernels address activations with 32-bit byte offsets.
inline bool mfma_fits(int T, int k, int H, int I) {
    return (uint64_t)T * H * 2 < (1ull << 32) && (uint64_t)T * k * I * 2 < (1ull << 32);
}

inline size_t align256(size_t v) { return (v + 255) & ~(size_t)255; }

// Workspace: the activations between the two stages, act[cap, I] (bf16 on the MFMA path, else f32).
inline char* act_of(void* ws) { return (char*)ws; }

int check_common(const int32_t* group_offsets, int T, int k, int spr, int H, int I, int dtype, const void* ws,
                 size_t ws_bytes) {
    if (!group_offsets || !ws) return METRO_ERR_INVALID_ARG;
    if (T < 0 || k < 1 || spr < 1 || H < 1 || I < 1) return METRO_ERR_INVALID_ARG;
    if (dtype != METRO_DTYPE_BF16 && dtype != METRO_DTYPE_F32) return METRO_ERR_UNSUPPORTED;
    if (spr > kMaxSpr || (int64_t)T * k >= (1 << 24)) return METRO_ERR_UNSUPPORTED;
    if (((uintptr_t)ws & 255) != 0) return METRO_ERR_INVALID_ARG;
    if (ws_bytes < moe_grouped_ffn_workspace_bytes(T, k, spr, H, I, dtype)) return METRO_ERR_WORKSPACE;
    return METRO_OK;
}

int enable_large_lds() {                            // opt in to > 64 KB of dynamic LDS, once per device
    static PerDeviceOnce once;
    return once.run([] {
        hipError_t e = hipFuncSetAttribute((const void*)ffn_mfma_kernel<true>,
                                           hipFuncAttributeMaxDynamicSharedMemorySize, kLdsBytes);
        if (e == hipSuccess)
            e = hipFuncSetAttribute((const void*)ffn_mfma_kernel<false>, hipFuncAttributeMaxDynamicSharedMemorySize,
                                    kLdsBytes);
        return e;
    });
}

// Tall remainders of at most this many rows become stream tiles.  A wide workgroup prefetches one step
// ahead, so its K loop runs at about one memory latency per step: at large shapes that hides behind
// the narrow items, at mid ones (short launches, HBM not saturated) it is the critical path, and they keep tall tiles on
// the deep-prefetch stream path, whose narrower column tile costs more activation re-reads.
inline bool large_shape(int H, int I) { return (size_t)H * I >= (size_t)4096 * 2048; }
inline int stream_rows_for(int H, int I) { return large_shape(H, I) ? 32 : kWideRows; }

// Tiles above this many rows stage their activations through LDS.  A narrow tile reads each activation once per 64 weight
// rows, which at 33..64 rows is as much L2 traffic as the weights themselves: large shapes, at the fabric's rate
// already, lose by it (7168 x 2048, 1024 tokens, METRO rank: 399 + 205 us with 64, 383 + 201 with 32); shorter launches
// gain from the smaller work items (4096 x 1536: 103 + 57 with 64, 107 + 57 with 32; 2048 x 768 has only these tiles).
inline int narrow_rows_for(int H, int I) { return large_shape(H, I) ? 32 : kNarrowMost; }

// Rows of a full tile.  128 amortises a slot's weights over the most rows (one HBM pass per 128 rows; all
// tiles narrow at 4096 x 1536: 116 + 59 instead of 103 + 57 us).
// The smallest FFNs finish in a few tens of microseconds and are bound by their longest workgroup, not
// by bytes: a 128-row tile spends longer in its matrix instructions than the whole launch should take,
// while re-reading a small slot's weights from L2 is cheap, so they cut groups into narrow tiles (2048 x 768: 256 tokens
// 30 + 16 us with 64 rows, 35 + 16 with 32; 4096 tokens 110 + 63 with 64, 159 + 83 with 32).
inline int tile_rows_for(int H, int I) { return (size_t)H * I < (size_t)2048 * 1024 ? kNarrowMost : kWideRows; }

inline int launched() { return hipGetLastError() == hipSuccess ? METRO_OK : METRO_ERR_HIP; }

// Built-in workspace of moe_grouped_ffn_static_ws: one array per GPU, held from the moment the library is
// loaded on that GPU until the process ends.  In host code this name is only a handle for
// hipGetSymbolAddress; the device address it yields (one per device) is what kernels and copies get.
constexpr size_t kStaticWsBytes = METRO_STATIC_WS_BYTES;
static __device__ __align__(256) unsigned char scratch[kStaticWsBytes];

// Device address of `scratch` on the current device, looked up once per device.
int static_ws(void** out) {
    constexpr int kMaxDevices = 64;
    static std::atomic<void*> table[kMaxDevices] = {};
    int dev = 0;
    if (hipGetDevice(&dev) != hipSuccess || dev < 0 || dev >= kMaxDevices) return METRO_ERR_HIP;
    void* p = table[dev].load(std::memory_order_acquire);
    if (!p) {
        if (hipGetSymbolAddress(&p, HIP_SYMBOL(scratch)) != hipSuccess || !p) return METRO_ERR_HIP;
        table[dev].store(p, std::memory_order_release);      // a racing first call stores the same address
    }
    *out = p;
    return METRO_OK;
}

}  // namespace
}  // namespace metro

extern "C" size_t moe_grouped_ffn_workspace_bytes(int T, int k, int spr, int H, int I, int dtype) {
    using namespace metro;
    if (T < 0 || k < 1 || spr < 1 || H < 1 || I < 1) return 0;
    const size_t cap = (size_t)T * k;
    const size_t act = align256(cap * I * (use_mfma(T, k, H, I, dtype) ? 2 : 4));
    return act + 256;
}

extern "C" int moe_grouped_ffn_gate_up(const void* x, const int32_t* perm_pair, const int32_t* group_offsets, int T,
                                       int k, int spr, int H, int I, int dtype, const void* w13, int ldw13,
                                       void* ws, size_t ws_bytes, void* stream) {
    using namespace metro;
    const int rc = check_common(group_offsets, T, k, spr, H, I, dtype, ws, ws_bytes);
    if (rc != METRO_OK) return rc;
    if (!x || !perm_pair || !w13 || (((uintptr_t)x | (uintptr_t)w13) & 15) != 0) return METRO_ERR_INVALID_ARG;
    if (ldw13 < H || ldw13 % 8 != 0) return METRO_ERR_INVALID_ARG;
    const int cap = T * k;
    if (cap == 0) return METRO_OK;
    hipStream_t st = (hipStream_t)stream;
    char* act = act_of(ws);
    if (!use_mfma(T, k, H, I, dtype)) {
        const SplitArgs g{x, perm_pair, w13, act, T, k, H, I, ldw13};
        return launch_general<true>(g, group_offsets, spr, dtype, st);
    }
    if (enable_large_lds() != METRO_OK) return METRO_ERR_HIP;
    FfnArgs a;
    a.src = (const __bf16*)x;
    a.perm_pair = perm_pair;
    a.w = (const __bf16*)w13;
    a.ldw = ldw13;
    a.dst = (__bf16*)act;
    a.group_offsets = group_offsets;
    a.T = T; a.k = k; a.spr = spr; a.H = H; a.I = I;
    a.stream_rows = stream_rows_for(H, I);
    a.tile_rows = tile_rows_for(H, I);
    a.narrow_rows = narrow_rows_for(H, I);
    // mid shapes (every tile on the stream path, 128-row tiles): a one-tile slot of 65..128 rows is the
    // longest workgroup of a launch that has fewer workgroups than the chip has slots; two 64-row tiles
    // balance it (token-balanced rank of the 4096 x 1536 shape: gate/up 109 -> 101 us; no gain for down)
    a.single_rows = (a.stream_rows >= kWideRows && a.tile_rows == kWideRows) ? 64 : 0;
    a.ntw = I / 128;
    a.nts = I / 64;
    a.ntn = I / (kNarrowBlocks * 8);
    hipLaunchKernelGGL(ffn_mfma_kernel<true>, dim3(mfma_grid(a, cap, spr)), dim3(kThreads), kLdsBytes, st, a);
    return launched();
}

extern "C" int moe_grouped_ffn_down(const int32_t* group_offsets, int T, int k, int spr, int H, int I, int dtype,
                                    const void* w2, int ldw2, void* y_perm, void* ws, size_t ws_bytes,
                                    void* stream) {
    using namespace metro;
    const int rc = check_common(group_offsets, T, k, spr, H, I, dtype, ws, ws_bytes);
    if (rc != METRO_OK) return rc;
    if (!w2 || !y_perm || (((uintptr_t)w2 | (uintptr_t)y_perm) & 15) != 0) return METRO_ERR_INVALID_ARG;
    if (ldw2 < I || ldw2 % 8 != 0) return METRO_ERR_INVALID_ARG;
    const int cap = T * k;
    if (cap == 0) return METRO_OK;
    hipStream_t st = (hipStream_t)stream;
    char* act = act_of(ws);
    if (!use_mfma(T, k, H, I, dtype)) {
        const SplitArgs g{act, nullptr, w2, y_perm, T, k, H, I, ldw2};
        return launch_general<false>(g, group_offsets, spr, dtype, st);
    }
    if (enable_large_lds() != METRO_OK) return METRO_ERR_HIP;
    FfnArgs a;
    a.src = (const __bf16*)act;
    a.perm_pair = nullptr;
    a.w = (const __bf16*)w2;
    a.ldw = ldw2;
    a.dst = (__bf16*)y_perm;
    a.group_offsets = group_offsets;
    a.T = T; a.k = k; a.spr = spr; a.H = H; a.I = I;
    a.stream_rows = stream_rows_for(H, I);
    a.tile_rows = tile_rows_for(H, I);
    a.narrow_rows = narrow_rows_for(H, I);
    a.single_rows = 0;
    // mid shapes: the full 128-row tiles of a several-tile slot take the wide path in this stage (half
    // the column tiles, each activation fragment feeding four matrix instructions); smaller tiles stay
    // on the stream path (METRO rank of the 4096 x 1536 shape: down 71 -> 60 us; a 113-row one-tile
    // slot on the wide path costs the token-balanced rank 8 us, hence "full tiles only")
    if (a.stream_rows >= kWideRows && a.tile_rows == kWideRows) a.stream_rows = kWideRows - 1;
    a.ntw = (H + 255) / 256;
    a.nts = H / 128;
    a.ntn = H / (kNarrowBlocks * 16);
    hipLaunchKernelGGL(ffn_mfma_kernel<false>, dim3(mfma_grid(a, cap, spr)), dim3(kThreads), kLdsBytes, st, a);
    return launched();
}

extern "C" int moe_grouped_ffn(const void* x, const int32_t* perm_pair, const int32_t* group_offsets, int T, int k,
                               int spr, int H, int I, int dtype, const void* w13, int ldw13, const void* w2,
                               int ldw2, void* y_perm, void* ws, size_t ws_bytes, void* stream) {
    // all arguments are checked before the first launch
    if (!x || !perm_pair || !w13 || !w2 || !y_perm) return METRO_ERR_INVALID_ARG;
    if ((((uintptr_t)x | (uintptr_t)w13 | (uintptr_t)w2 | (uintptr_t)y_perm) & 15) != 0) return METRO_ERR_INVALID_ARG;
    if (ldw13 < H || ldw2 < I || ldw13 % 8 != 0 || ldw2 % 8 != 0) return METRO_ERR_INVALID_ARG;
    int rc = moe_grouped_ffn_gate_up(x, perm_pair, group_offsets, T, k, spr, H, I, dtype, w13, ldw13, ws, ws_bytes,
                                     stream);
    if (rc == METRO_OK)
        rc = moe_grouped_ffn_down(group_offsets, T, k, spr, H, I, dtype, w2, ldw2, y_perm, ws, ws_bytes, stream);
    return rc;
}

extern "C" size_t moe_grouped_ffn_static_ws_bytes(void) { return metro::kStaticWsBytes; }

extern "C" int moe_grouped_ffn_static_ws(const void* x, const int32_t* perm_pair, const int32_t* group_offsets, int T,
                                         int k, int spr, int H, int I, int dtype, const void* w13, int ldw13,
                                         const void* w2, int ldw2, void* y_perm, void* stream) {
    using namespace metro;
    if (T < 0 || k < 1 || spr < 1 || H < 1 || I < 1) return METRO_ERR_INVALID_ARG;
    if (dtype != METRO_DTYPE_BF16 && dtype != METRO_DTYPE_F32) return METRO_ERR_UNSUPPORTED;
    if (spr > kMaxSpr || (int64_t)T * k >= (1 << 24)) return METRO_ERR_UNSUPPORTED;
    if (moe_grouped_ffn_workspace_bytes(T, k, spr, H, I, dtype) > kStaticWsBytes) return METRO_ERR_TOO_LARGE;
    void* ws = nullptr;
    const int rc = static_ws(&ws);
    if (rc != METRO_OK) return rc;
    // the intermediate activations of rows < n_pairs are written by the first stage before the second reads
    // them, so nothing in the array has to start at zero
    return moe_grouped_ffn(x, perm_pair, group_offsets, T, k, spr, H, I, dtype, w13, ldw13, w2, ldw2, y_perm, ws,
                           kStaticWsBytes, stream);
}
