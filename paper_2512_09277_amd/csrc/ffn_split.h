// One tile of the grouped FFN with K split over the four waves of a workgroup: no LDS and no barrier in the K loop.
//
// All four waves work on the same NB x 16 weight rows; wave w takes the K steps w, w + 4, ... .  A step is 128 bytes
// of every weight row (one cache line: two load instructions of 16 rows x 64 contiguous bytes), so the workgroup
// reads 512 contiguous bytes of a row at about the same time.  No wave needs another wave's activations, so both
// operands go from memory into registers in matrix-operand layout and every wave runs ahead on its own: DEPTH
// steps of loads are in flight per wave and nothing waits for the slowest of four waves until the partial sums meet
// in LDS after the last step (in a fixed order, so results are deterministic).
//
// Lane (r16, q) supplies kVec consecutive k of weight row r16 (A operand) and the same k of tile row r16 (B
// operand).  The sum over k does not care which k sits in which operand slot as long as both sides agree.
//   bf16 x bf16   v_mfma_f32_16x16x32_bf16: one per 16-byte load
//   f32 x f32     v_mfma_f32_16x16x4_f32: four per 16-byte load, fp32 products and sums
//   bf16 x f32    (fp32 activations kept between the stages of ragged 16-bit shapes) weights widened, eight of the
//                 fp32 instruction per 16-byte load
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

#include <type_traits>
#include <utility>

#include "ffn_common.h"

namespace metro {
namespace {

// Memory at any element alignment (rows of an odd length); the hardware takes unaligned 128-bit global loads.
typedef u32x4 u32x4_any __attribute__((aligned(2)));

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

// Mask of word `e` of a vector of T whose first `drop` elements are to be zeroed.
template <typename T>
__device__ __forceinline__ uint32_t keep_mask(int drop, int e) {
    if (sizeof(T) == 4) return drop <= e ? 0xffffffffu : 0u;
    return drop <= 2 * e ? 0xffffffffu : drop == 2 * e + 1 ? 0xffff0000u : 0u;
}

enum class KRows { kWhole, kRagged, kTiny };  // K a multiple of a step; any K >= kVec; K < kVec (element-wise loads)

// WT weights, XT activations, OT output.
template <bool kGateUp, typename WT, typename XT, typename OT, int NB, int MT, int DEPTH, KRows kRows>
__device__ __forceinline__ void split_tile(const SplitArgs& a, const Tile t, char* lds) {
    constexpr int kVec = 16 / (int)sizeof(WT);              // k per lane and load
    constexpr int kStep = 8 * kVec;                         // k per step
    constexpr int XV = kVec * (int)sizeof(XT) / 16;         // 16-byte loads of activations per weight load
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
    const XT* px[MT];
    uint32_t x_lane[MT];
#pragma unroll
    for (int mt = 0; mt < MT; ++mt) {
        const int row = t.row0 + min(mt * 16 + r16, t.rows - 1);    // rows past the tile repeat its last row
        const int src = kGateUp ? min(max(a.perm_pair[row] / a.k, 0), a.T - 1) : row;
        px[mt] = reinterpret_cast<const XT*>(a.src) + (kWhole ? 0 : (size_t)src * K);
        x_lane[mt] = (uint32_t)src * (uint32_t)K + q * kVec;
    }

    floatx4 acc[NB][MT];
#pragma unroll
    for (int b = 0; b < NB; ++b)
#pragma unroll
        for (int mt = 0; mt < MT; ++mt) acc[b][mt] = floatx4{0.f, 0.f, 0.f, 0.f};

    u32x4 w[DEPTH][2][NB], x[DEPTH][2][MT][XV];
    auto guarded = [&](const auto* p, int k) {              // K < kVec: element by element
        using T = std::remove_cv_t<std::remove_pointer_t<decltype(p)>>;
        constexpr int n = 16 / (int)sizeof(T);
        typedef T vec __attribute__((ext_vector_type(n)));
        vec v;
#pragma unroll
        for (int e = 0; e < n; ++e) v[e] = k + e < K ? p[k + e] : (T)0.f;
        return __builtin_bit_cast(u32x4, v);
    };
    // Every lane's vector stays inside its row: one that would pass the end is moved back to end with the row, and
    // the elements it then repeats are zeroed (in both operands) when the partial step is consumed.
    auto load = [&](auto B, int s) {
        constexpr int buf = decltype(B)::value;
        const int step = wv + 4 * min(s, mine - 1);
        // past the wave's last step: every lane the same 16 bytes of a line that is there already
        const uint32_t w_off = s < mine ? w_lane : 0u;
        uint32_t x_off[MT];
#pragma unroll
        for (int mt = 0; mt < MT; ++mt) x_off[mt] = s < mine ? x_lane[mt] : 0u;
#pragma unroll
        for (int j = 0; j < 2; ++j) {
            const int k = step * kStep + j * 4 * kVec + q * kVec;
            const int at = min(k, K - kVec);
            const size_t whole_at = (size_t)step * kStep + j * 4 * kVec;      // uniform
#pragma unroll
            for (int mt = 0; mt < MT; ++mt)
#pragma unroll
                for (int v = 0; v < XV; ++v) {
                    constexpr int n = 16 / (int)sizeof(XT);
                    if constexpr (kRows == KRows::kTiny) x[buf][j][mt][v] = guarded(px[mt], k + v * n);
                    else if constexpr (kWhole) x[buf][j][mt][v] = *reinterpret_cast<const u32x4*>(px[mt] + whole_at + x_off[mt] + v * n);
                    else x[buf][j][mt][v] = *reinterpret_cast<const u32x4_any*>(px[mt] + at + v * n);
                }
#pragma unroll
            for (int b = 0; b < NB; ++b) {
                if constexpr (kRows == KRows::kTiny) w[buf][j][b] = guarded(pw[b], k);
                else if constexpr (kWhole) w[buf][j][b] = *reinterpret_cast<const u32x4*>(pw[b] + whole_at + w_off);
                else w[buf][j][b] = *reinterpret_cast<const u32x4_any*>(pw[b] + at);
            }
        }
    };
    auto consume = [&](auto B, int step, auto Masked) {
        constexpr int buf = decltype(B)::value;
        constexpr bool masked = decltype(Masked)::value && kRows == KRows::kRagged;
#pragma unroll
        for (int j = 0; j < 2; ++j) {
            u32x4 xv[MT][XV], wm = {}, xm[XV] = {};
            if constexpr (masked) {                         // zeroes the elements that a moved vector repeats, in both
                const int k = step * kStep + j * 4 * kVec + q * kVec, drop = max(k - (K - kVec), 0);    // operands (0 x inf
#pragma unroll                                              // would be NaN)
                for (int e = 0; e < 4; ++e) {
                    wm[e] = keep_mask<WT>(drop, e);
#pragma unroll
                    for (int v = 0; v < XV; ++v) xm[v][e] = keep_mask<XT>(drop - v * (16 / (int)sizeof(XT)), e);
                }
            }
#pragma unroll
            for (int mt = 0; mt < MT; ++mt)
#pragma unroll
                for (int v = 0; v < XV; ++v) xv[mt][v] = masked ? x[buf][j][mt][v] & xm[v] : x[buf][j][mt][v];
#pragma unroll
            for (int b = 0; b < NB; ++b) {
                const u32x4 wr = masked ? w[buf][j][b] & wm : w[buf][j][b];
                if constexpr (sizeof(XT) == 2) {
#pragma unroll
                    for (int mt = 0; mt < MT; ++mt)
                        acc[b][mt] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8, wr),
                                                                             __builtin_bit_cast(bf16x8, xv[mt][0]),
                                                                             acc[b][mt], 0, 0, 0);
                } else {
#pragma unroll
                    for (int c = 0; c < kVec; ++c) {
                        const float wf = sizeof(WT) == 4 ? __uint_as_float(wr[c & 3])
                                                         : __uint_as_float((c & 1) ? wr[c >> 1] & 0xffff0000u : wr[c >> 1] << 16);
#pragma unroll
                        for (int mt = 0; mt < MT; ++mt)
                            acc[b][mt] = __builtin_amdgcn_mfma_f32_16x16x4f32(wf, __uint_as_float(xv[mt][c >> 2][c & 3]),
                                                                              acc[b][mt], 0, 0, 0);
                    }
                }
            }
        }
    };

    if (mine > 0) {
        // Buffer s % DEPTH holds the wave's step s.  Loads are unconditional (past the end: the last step again) so
        // that the compiler counts what is outstanding exactly and waits for the consumed step only; the last
        // DEPTH steps load nothing.
        run_steps(std::make_integer_sequence<int, DEPTH>{}, [&](auto U, int s) { load(U, s); }, 0);
        auto step = [&](auto U, int s) {
            consume(U, wv + 4 * s, std::false_type{});
            __builtin_amdgcn_sched_barrier(0);              // the loads refill the registers just read, none earlier
            load(U, s + DEPTH);
            __builtin_amdgcn_sched_barrier(0);
        };
        auto final_step = [&](auto U, int s) { consume(U, wv + 4 * s, std::true_type{}); };
        int s = 0;
        for (; s + DEPTH < mine; s += DEPTH) run_steps(std::make_integer_sequence<int, DEPTH>{}, step, s);
        run_steps_tail(std::make_integer_sequence<int, DEPTH>{}, final_step, s, mine);
    }

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
