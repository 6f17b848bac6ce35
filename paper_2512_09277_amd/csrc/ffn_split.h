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
template <bool kGateUp, typename WT, typename XT, typename OT, int NB, int MT, int DEPTH, KRows kRows>
__device__ __forceinline__ void split_tile(const SplitArgs& a, const Tile t, char* lds) {
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

    // Whole rows (the host checks that activation offsets fit): a uniform base per block and 32-bit lane offsets, which
    // leaves the vector registers to the data in flight.  Otherwise a pointer per lane, rows past the last column
    // repeating it.
    constexpr bool kWhole = kRows == KRows::kWhole;
    const WT* wslot = reinterpret_cast<const WT*>(a.w) + (size_t)t.slot * (kGateUp ? 2 * a.I : a.H) * a.ldw;
    const WT* pw[NB];
#pragma unroll
    for (int b = 0; b < NB; ++b) {
        const int at = col0 + (b % kUnits) * 16, col = kWhole ? at : min(at + r16, n_out - 1);
        pw[b] = wslot + (size_t)((kGateUp && b >= kUnits) ? a.I + col : col) * a.ldw;
    }
    const uint32_t w_lane = (uint32_t)(r16 * a.ldw + q * kVec);
    int token[MT];
#pragma unroll
    for (int mt = 0; mt < MT; ++mt) {
        const int row = t.row0 + min(mt * 16 + r16, t.rows - 1);    // rows past the tile repeat its last row
        token[mt] = kGateUp ? a.perm_pair[row] : row;
    }
    auto x_rows = [&](const XT* (&px)[MT], uint32_t (&x_lane)[MT]) {
#pragma unroll
        for (int mt = 0; mt < MT; ++mt) {
            const int src = kGateUp ? min(max(token[mt] / a.k, 0), a.T - 1) : token[mt];
            px[mt] = reinterpret_cast<const XT*>(a.src) + (kWhole ? 0 : (size_t)src * K);
            x_lane[mt] = (uint32_t)src * (uint32_t)K + q * kVec;
        }
    };

    floatx4 acc[NB][MT];
    split_dot<WT, XT, NB, MT, DEPTH, kRows>(pw, w_lane, x_rows, K, wv, 4, mine, acc);

    // partial sums of the four waves, [wave][b][mt][lane]; the sums of a block are formed in wave order
    floatx4* part = reinterpret_cast<floatx4*>(lds);
#pragma unroll
    for (int b = 0; b < NB; ++b)
#pragma unroll
        for (int mt = 0; mt < MT; ++mt)
            if (mt < mt_count) part[((wv * NB + b) * MT + mt) * 64 + lane] = acc[b][mt];
    __syncthreads();
    auto total = [&](int b, int mt) {
        floatx4 s = part[(b * MT + mt) * 64 + lane];
#pragma unroll
        for (int o = 1; o < 4; ++o) s += part[((o * NB + b) * MT + mt) * 64 + lane];
        return s;
    };
#pragma unroll
    for (int u0 = 0; u0 < kUnits * MT; u0 += 4) {
        const int u = u0 + wv, b = u / MT, mt = u % MT;     // (output block, row sub-tile) of this wave
        if (u >= kUnits * MT || mt >= mt_count) continue;
        const int row = mt * 16 + r16, col = col0 + b * 16 + q * 4;
        float o[4];
        const floatx4 g = total(b, mt);
        if (kGateUp) {
            const floatx4 up = total(b + kUnits, mt);
#pragma unroll
            for (int v = 0; v < 4; ++v) o[v] = g[v] / (1.0f + (sizeof(OT) == 4 ? expf(-g[v]) : __expf(-g[v]))) * up[v];
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
