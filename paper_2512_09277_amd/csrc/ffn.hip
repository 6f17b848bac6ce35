// moe_grouped_ffn for gfx950: SwiGLU expert FFN over one rank's per-slot token lists.
//
// Decode is HBM-bound: runtime follows the bytes of the activated experts' weights (Sec. 3.2 of
// arxiv 2512.09277).  Every activated weight row is streamed from HBM once per tile, with loads of whole lines that get their
// matrix-core operand layout in LDS.
// Work is cut into tiles of one slot's rows:
//   narrow tiles (at most 16 rows, 64 where the launch is short; the bulk of the bytes): ffn_split.h -- K split over the
//       four waves, 64 weight rows per workgroup, each wave's operands through its own LDS, no barrier in the K loop;
//   tall tiles (up to 128 rows, the popular experts and large batches): ring_k.h -- both operands through LDS, 128 weight
//       rows per workgroup.  They are listed first.
//   gate/up: a wave owns gate rows and the matching up rows, so silu(gate)*up is formed in
//            registers and written once as bf16;   down: same structure over K = I.
// A slot with no rows produces no tile and its weights are never touched.  There is no planning pass:
// every workgroup finds its (tile, column tile) from group_offsets itself.
#include <hip/hip_runtime.h>
#include <stdint.h>

#include <algorithm>
#include <atomic>
#include <type_traits>
#include <utility>

#include "ffn_common.h"
#include "ffn_split.h"
#include "metro.h"
#include "ring_k.h"

namespace metro {
namespace {

constexpr int kThreads = 256;

// ------------------------------------------------------------------------------------------ MFMA path
struct FfnArgs {
    const __bf16* src;        // gate/up: x[T,H]; down: act[cap,I]
    const int32_t* perm_pair; // gate/up only
    const __bf16* w;          // gate/up: w13[spr,2I,H]; down: w2[spr,H,I]
    __bf16* dst;              // gate/up: act[cap,I]; down: y_perm[cap,H]
    const int32_t* group_offsets;
    int T, k, spr, H, I;
    int ldw;                  // elements between consecutive weight rows (>= K)
    int ntt;                  // column tiles per tall tile
    int ntn;                  // column tiles per narrow tile
    CutRule rule;
};

__device__ __forceinline__ float silu(float g) { return g / (1.0f + __expf(-g)); }

// Tall tile: 16 MT rows x 64 gate/up columns or 128 down columns, both operands through LDS (ring_k.h).  Bound, in launches of many
// rows, by the work of a step inside a CU (with operands that cost no memory traffic 33 instead of 44 us for 4096 tokens at
// 2048 x 768, of which the matrix instructions need 14), elsewhere by what the fabric delivers.  It replaced tiles with both operands
// through registers, three steps deep, two LDS buffers with padded rows and the loads of a step behind its products.  Measured with
// weights from HBM, gate/up + down, us: 4096 tokens at 2048 x 768 57 + 38.5 -> 51.3 + 35.2, 512 tokens at 4096 x 1536 108.7 + 56.7 ->
// 108.4 + 53.6, 1024 tokens at 7168 x 2048 (METRO rank) 388.5 + 209 -> 388.3 + 205.1.  Weights straight to registers in operand layout:
// slower than either (weights in the Infinity Cache, 50 + 34 against 44 + 31; 130 + 63; 425 + 218), see ring_k.h.
template <bool kGateUp, int MT>
__device__ __forceinline__ void ring_tile(const FfnArgs& a, const Tile t) {
    const int tid = threadIdx.x, lane = tid & 63, wv = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int r16 = lane & 15, q = lane >> 4, srow = tid >> 3;
    const int K = kGateUp ? a.H : a.I, n_out = kGateUp ? a.I : a.H;
    const int col0 = t.col * (kGateUp ? 64 : 128);
    uint32_t x_lane[MT / 2];                // every activation byte offset fits 32 bits on this path
#pragma unroll
    for (int p = 0; p < MT / 2; ++p) {
        const int at = p * 32 + srow, row = t.row0 + min(at, t.rows - 1);          // rows past the tile repeat its last row
        const int src = kGateUp ? min(max(a.perm_pair[row] / a.k, 0), a.T - 1) : row;
        x_lane[p] = (uint32_t)src * (uint32_t)(K * 2) + ring_piece(at);
    }
    const __bf16* wslot = a.w + (size_t)t.slot * (kGateUp ? 2 * a.I : a.H) * a.ldw;
    const char* wb[4];
#pragma unroll
    for (int p = 0; p < 4; ++p) {
        const int row = kGateUp ? (p >> 1) * a.I + col0 + (p & 1) * 32 : col0 + p * 32;
        wb[p] = reinterpret_cast<const char*>(wslot + (size_t)row * a.ldw);
    }
    floatx4 acc[4][MT / 2];
    ring_dot<MT>(reinterpret_cast<const char*>(a.src), x_lane, wb, (size_t)srow * a.ldw * 2 + (tid & 7) * 16, 0, K / kRingStep, acc);
    const int ty = wv >> 1, tx = wv & 1;
#pragma unroll
    for (int mt = 0; mt < MT / 2; ++mt) {
        const int row = (mt * 2 + ty) * 16 + r16;
        if (row >= t.rows) continue;
        __bf16* out = a.dst + (size_t)(t.row0 + row) * n_out + col0 + tx * 32 + q * 4;
        if (kGateUp) {
#pragma unroll
            for (int b = 0; b < 2; ++b) {
                const floatx4 g = acc[b][mt], u = acc[b + 2][mt];
                *reinterpret_cast<u32x2*>(out + b * 16) =
                    u32x2{pack_bf16x2(silu(g[0]) * u[0], silu(g[1]) * u[1]), pack_bf16x2(silu(g[2]) * u[2], silu(g[3]) * u[3])};
            }
        } else {
#pragma unroll
            for (int b = 0; b < 4; ++b)
                *reinterpret_cast<u32x2*>(out + (b >> 1) * 64 + (b & 1) * 16) =
                    u32x2{pack_bf16x2(acc[b][mt][0], acc[b][mt][1]), pack_bf16x2(acc[b][mt][2], acc[b][mt][3])};
        }
    }
}

// Narrow tiles: K split over the waves, whole lines loaded, operand layout through the wave's LDS (split_k.h).  Measured against
// loads in operand layout, which left a CU at 38 GB/s for both operands together (gate/up + down, us, weights from HBM): 256 tokens of
// the 2048 x 768 shape 29.2 + 16.0 -> 24.9 + 14.7, 512 tokens at 4096 x 1536 (about half of the time narrow tiles) 108.5 + 53.6 ->
// 94.9 + 48.6, 1024 tokens at 7168 x 2048 (METRO rank) 388 + 205 -> 378 + 201, 97 tokens of it 291 + 145.5 -> 288 + 145.
//   Blocks: 2 instead of 4 weight blocks per workgroup re-read the activations twice as often and lose everywhere (97 tokens:
//   276 + 177).
//   Depth: what 256 registers hold.
constexpr int kNarrowBlocks = 4;
// Workgroups of the narrow tiles at most; a workgroup past the last item costs about 2 ns, so the grid is not sized for
// the most tiles a rank could have, and the rest is taken in turns.  Three times the 512 resident ones: with fewer, who
// gets one item more is decided at launch and not by who is free (512: 287 us, 1024: 269, 1536 and more: 268; 97
// tokens, gate/up).
constexpr int kNarrowGrid = 1536;

// The ring's LDS as split_tile uses it: per wave a step of weights and of activations, then the partial sums.
struct NarrowLds {
    __device__ __forceinline__ char* wave_w(int wave) const { return ring_buf_at(2 * wave); }
    __device__ __forceinline__ char* wave_x(int wave) const { return ring_buf_at(2 * wave + 1); }
    __device__ __forceinline__ floatx4* part(int u) const { return reinterpret_cast<floatx4*>(ring_buf_at(u >> 1) + (u & 1) * (kRingBuf / 2)); }
};

template <bool kGateUp>
__global__ __launch_bounds__(kThreads, 2) void ffn_mfma_kernel(FfnArgs a) {
    // Work items = (tile, column tile).  Every XCD has a list of them, tall tiles first: their workgroups live longest, so they
    // start early for the narrow ones to fill in around them.  Everything here is uniform per workgroup.
    WorkList wl;
    wl.read(a.group_offsets, a.spr, a.T * a.k, a.rule);
    const int xcd = blockIdx.x & 7, tall = wl.list_tall(xcd, a.ntt);
    int id = blockIdx.x >> 3;
    if (id < tall) {
        const Tile t = wl.tall(id, xcd);
        if (t.rows <= 32) ring_tile<kGateUp, 2>(a, t);
        else if (t.rows <= 64) ring_tile<kGateUp, 4>(a, t);
        else if (t.rows <= 96) ring_tile<kGateUp, 6>(a, t);
        else ring_tile<kGateUp, 8>(a, t);
        return;
    }
    const NarrowLds lds;
    const SplitArgs sa{a.src, a.perm_pair, a.w, a.dst, a.T, a.k, a.H, a.I, a.ldw};
    const int n = wl.n_narrow * a.ntn, stride = gridDim.x - tall * 8;
    for (id = (id - tall) * 8 + xcd; id < n; id += stride) {
        const int ti = id / a.ntn;
        const Tile t = wl.narrow(ti, id - ti * a.ntn);
        if (t.rows <= 16) split_tile<kGateUp, __bf16, __bf16, __bf16, kNarrowBlocks, 1, 3, KRows::kWhole>(sa, t, lds);
        else if (t.rows <= 32) split_tile<kGateUp, __bf16, __bf16, __bf16, kNarrowBlocks, 2, 2, KRows::kWhole>(sa, t, lds);
        else if (t.rows <= 48) split_tile<kGateUp, __bf16, __bf16, __bf16, kNarrowBlocks, 3, 1, KRows::kWhole>(sa, t, lds);
        else split_tile<kGateUp, __bf16, __bf16, __bf16, kNarrowBlocks, 4, 1, KRows::kWhole>(sa, t, lds);
        __syncthreads();                                                 // the next item's sums reuse the LDS
    }
}

// Workgroups, a multiple of 8: per XCD one for each of the most tall items that `cap` rows can make, and the narrow ones.
inline int mfma_grid(const FfnArgs& a, int cap, int spr) {
    const int tall = std::min(cap / (kNarrowRows + 1), max_tiles(cap, spr, kTallRows));
    const int narrow = std::min(a.ntn * (std::min(spr, cap) + cap / kNarrowRows), kNarrowGrid);
    return ((tall * (a.ntt < 8 ? a.ntt : (a.ntt + 7) & ~7) + 7) & ~7) + ((narrow + 7) & ~7);
}

// ------------------------------------------------------------------------------------------ general path
// fp32 storage, and 16-bit shapes whose H or I is no multiple of 128 (activations between the stages in fp32): K-split
// tiles (ffn_split.h) of at most 32 rows x 16 gate/up columns or 32 down columns, of 16 rows where 16-bit weights meet fp32
// activations.  What bounds it is latency and, in fp32, the matrix instructions (46 % of the time at 362 rows over 17 slots), so
// registers are kept low enough for four workgroups per CU, a single step of loads in flight per wave (three and two steps at three
// workgroups per CU: 57.5 + 30.3 us against 54.0 + 30.2; 64 rows or four weight blocks a tile lose 5 %).  Measured, gate/up + down, us,
// weights from HBM: 362 rows of the 2048 x 768 shape in fp32 72.6 + 36.5 -> 54.0 + 30.2, 2000 x 712 in bf16 27.0 + 22.6 -> 24.4 + 20.9,
// with operands loaded in operand layout (both stages then took what a CU gets of such loads, see ring_k.h).
constexpr int kGenRows = 32, kGenWideRows = 16;
constexpr int kGenBlocks = 2;               // 16-row weight blocks of a workgroup
constexpr int kGenGateUpCols = kGenBlocks * 8, kGenDownCols = kGenBlocks * 16;
// One and a half rounds of the 1024 resident workgroups; more items loop.  (The grid can only be sized for a rank that gets every
// pair of the batch; a workgroup that finds no item costs about 2 ns.)
constexpr int kGenGrid = 1536;

template <bool kGateUp, typename WT>
constexpr int gen_rows() { return !kGateUp && sizeof(WT) == 2 ? kGenWideRows : kGenRows; }

template <bool kGateUp, typename WT, KRows kRows>
__global__ __launch_bounds__(kThreads, kRows == KRows::kTiny ? 3 : 4) void general_ffn_kernel(SplitArgs a, const int32_t* __restrict__ group_offsets,
                                                                  int spr, int n_cols, int64_t n_items) {
    using XT = std::conditional_t<kGateUp, WT, float>;
    using OT = std::conditional_t<kGateUp, float, WT>;
    constexpr int kRowsMax = gen_rows<kGateUp, WT>(), MT = kRowsMax / 16;
    constexpr int kW = split_w_bytes<WT, XT, kGenBlocks, MT>(), kWave = kW + split_x_bytes<WT, XT, kGenBlocks, MT>();
    __shared__ __attribute__((aligned(16))) char mem[4 * kWave];
    static_assert(sizeof(mem) >= 4 * kGenBlocks * MT * 64 * sizeof(floatx4), "the partial sums");
    struct Lds {
        char* mem;
        __device__ __forceinline__ char* wave_w(int wave) const { return mem + wave * kWave; }
        __device__ __forceinline__ char* wave_x(int wave) const { return mem + wave * kWave + kW; }
        __device__ __forceinline__ floatx4* part(int u) const { return reinterpret_cast<floatx4*>(mem) + u * 4 * 64; }
    };
    const Lds lds{mem};
    for (int64_t id = blockIdx.x; id < n_items; id += gridDim.x) {
        const Item it = locate_in_order(group_offsets, spr, a.T * a.k, kRowsMax, n_cols, id);
        if (!it.valid) return;                                       // uniform; items are consecutive
        if (kRows != KRows::kTiny && it.tile.rows <= 16) split_tile<kGateUp, WT, XT, OT, kGenBlocks, 1, 1, kRows>(a, it.tile, lds);
        else split_tile<kGateUp, WT, XT, OT, kGenBlocks, MT, 1, kRows>(a, it.tile, lds);
        __syncthreads();                                             // the next item's sums reuse the LDS
    }
}

template <bool kGateUp>
int launch_general(const SplitArgs& a, const int32_t* group_offsets, int spr, int dtype, hipStream_t st) {
    const int n_out = kGateUp ? a.I : a.H, K = kGateUp ? a.H : a.I;
    const int cols = kGateUp ? kGenGateUpCols : kGenDownCols, n_cols = (n_out + cols - 1) / cols;
    const int rows = dtype == METRO_DTYPE_F32 ? gen_rows<kGateUp, float>() : gen_rows<kGateUp, __bf16>();
    const int64_t n_items = (int64_t)max_tiles(a.T * a.k, spr, rows) * n_cols;
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
    FfnArgs a;
    a.src = (const __bf16*)x;
    a.perm_pair = perm_pair;
    a.w = (const __bf16*)w13;
    a.ldw = ldw13;
    a.dst = (__bf16*)act;
    a.group_offsets = group_offsets;
    a.T = T; a.k = k; a.spr = spr; a.H = H; a.I = I;
    a.ntt = I / 64;
    a.ntn = I / (kNarrowBlocks * 8);
    a.rule = CutRule(a.ntn, a.ntt);
    hipLaunchKernelGGL(ffn_mfma_kernel<true>, dim3(mfma_grid(a, cap, spr)), dim3(kThreads), 0, st, a);
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
    FfnArgs a;
    a.src = (const __bf16*)act;
    a.perm_pair = nullptr;
    a.w = (const __bf16*)w2;
    a.ldw = ldw2;
    a.dst = (__bf16*)y_perm;
    a.group_offsets = group_offsets;
    a.T = T; a.k = k; a.spr = spr; a.H = H; a.I = I;
    a.ntt = H / 128;
    a.ntn = H / (kNarrowBlocks * 16);
    a.rule = CutRule(a.ntn, a.ntt);
    hipLaunchKernelGGL(ffn_mfma_kernel<false>, dim3(mfma_grid(a, cap, spr)), dim3(kThreads), 0, st, a);
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
