// One tile of the grouped FFN with K split over the four waves of a workgroup (split_k.h).  No wave needs another wave's
// activations, so nothing waits for the slowest of four waves until the partial sums meet in LDS after the last step.
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

#include <type_traits>
#include <utility>

#include "ffn_common.h"
#include "split_k.h"

namespace metro {
namespace {

template <typename T>
__device__ __forceinline__ T from_f32(float v);
template <>
__device__ __forceinline__ float from_f32<float>(float v) { return v; }
template <>
__device__ __forceinline__ __bf16 from_f32<__bf16>(float v) {
    const uint16_t bits = (uint16_t)(pack_bf16x2(v, 0.f) & 0xffffu);
    return __builtin_bit_cast(__bf16, bits);
}

struct SplitArgs {
    const void* src;          // gate/up: x[T,H]; down: act[cap,I]
    const int32_t* perm_pair; // gate/up only
    const void* w;
    void* dst;                // gate/up: act[cap,I]; down: y_perm[cap,H]
    int T, k, H, I, ldw;
};

// WT weights, XT activations, OT output.
template <bool kGateUp, typename WT, typename XT, typename OT, int NB, int MT, int DEPTH, KRows kRows, typename Lds>
__device__ __forceinline__ void split_tile(const SplitArgs& a, const Tile t, Lds lds) {
    constexpr int kVec = 16 / (int)sizeof(WT);              // k per lane and load
    constexpr int kStep = 8 * kVec;                         // k per step
    constexpr int kUnits = kGateUp ? NB / 2 : NB;           // 16-column blocks of the output

    const int tid = threadIdx.x, lane = tid & 63;
    const int wv = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int r16 = lane & 15, q = lane >> 4;
    const int K = kGateUp ? a.H : a.I, n_out = kGateUp ? a.I : a.H;
    const int n_steps = (K + kStep - 1) / kStep;            // the last one may be partial
    const int mine = (n_steps - wv + 3) >> 2;               // steps wv, wv + 4, ...
    const int mt_count = (t.rows + 15) >> 4;
    const int col0 = t.col * kUnits * 16;

    auto w_block = [&](int b) { return (kGateUp && b >= kUnits ? a.I : 0) + col0 + (b % kUnits) * 16; };
    auto w_row = [&](int b, int r) { return w_block(b) + min(r, n_out - 1 - (col0 + (b % kUnits) * 16)); };  // past the last column: that one
    auto x_row = [&](int mt, int r) {
        const int row = t.row0 + min(mt * 16 + r, t.rows - 1);      // past the tile: its last row
        return kGateUp ? min(max(a.perm_pair[row] / a.k, 0), a.T - 1) : row;
    };
    struct Rows {
        const WT* w_base;
        const XT* x_base;
        int w_pitch, x_pitch;
        decltype(w_block) w_block;
        decltype(w_row) w_row;
        decltype(x_row) x_row;
    };
    const WT* wslot = reinterpret_cast<const WT*>(a.w) + (size_t)t.slot * (kGateUp ? 2 * a.I : a.H) * a.ldw;
    floatx4 acc[NB][MT];
    split_dot<WT, XT, NB, MT, DEPTH, kRows>(Rows{wslot, reinterpret_cast<const XT*>(a.src), a.ldw, K, w_block, w_row, x_row}, K, wv, 4,
                                            mine, lds.wave_w(wv), lds.wave_x(wv), acc);
    __syncthreads();                                        // the partial sums take the LDS of all waves

    // partial sums of the four waves, [block][row sub-tile][wave][lane]; a sum is formed in wave order.  lds.part(u): the LDS of
    // (block, sub-tile) u.
#pragma unroll
    for (int b = 0; b < NB; ++b)
#pragma unroll
        for (int mt = 0; mt < MT; ++mt)
            if (mt < mt_count) lds.part(b * MT + mt)[wv * 64 + lane] = acc[b][mt];
    __syncthreads();
    auto total = [&](int u) {
        const floatx4* p = lds.part(u) + lane;
        floatx4 s = p[0];
#pragma unroll
        for (int o = 1; o < 4; ++o) s += p[o * 64];
        return s;
    };
#pragma unroll
    for (int u0 = 0; u0 < kUnits * MT; u0 += 4) {
        const int u = u0 + wv, b = u / MT, mt = u % MT;     // (output block, row sub-tile) of this wave
        if (u >= kUnits * MT || mt >= mt_count) continue;
        const int row = mt * 16 + r16, col = col0 + b * 16 + q * 4;
        float o[4];
        const floatx4 g = total(u);
        if (kGateUp) {
            const floatx4 h = total(u + kUnits * MT);
#pragma unroll
            for (int v = 0; v < 4; ++v) o[v] = g[v] / (1.0f + (sizeof(OT) == 4 ? expf(-g[v]) : __expf(-g[v]))) * h[v];
        } else {
#pragma unroll
            for (int v = 0; v < 4; ++v) o[v] = g[v];
        }
        if (row < t.rows) {
            OT* out = reinterpret_cast<OT*>(a.dst) + (size_t)(t.row0 + row) * n_out + col;
            if (n_out % 4 == 0) {                           // uniform; dst and its rows are then 4-element aligned
                if (col < n_out) {
                    if constexpr (sizeof(OT) == 4) *reinterpret_cast<floatx4*>(out) = floatx4{o[0], o[1], o[2], o[3]};
                    else *reinterpret_cast<u32x2*>(out) = u32x2{pack_bf16x2(o[0], o[1]), pack_bf16x2(o[2], o[3])};
                }
            } else {
#pragma unroll
                for (int v = 0; v < 4; ++v)
                    if (col + v < n_out) out[v] = from_f32<OT>(o[v]);
            }
        }
    }
}

}  // namespace
}  // namespace metro
