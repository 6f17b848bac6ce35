// Dot products of NB x 16 weight rows with MT x 16 activation rows over the K steps of one wave: no barrier, no wave needs another
// one's operands.
//
// A step is 128 bytes of every weight row, a cache line.  A load instruction takes whole lines (8 rows x 128 bytes; 16 rows x 64 bytes,
// which is matrix-operand layout, take a CU four times as long, see ring_k.h), DEPTH steps of loads in registers per wave.  A step
// then passes through the wave's own LDS, which turns it into operand layout: 128 bytes per row, its 16-byte piece p at place
// p ^ (row & 7), so that the 16 rows of a fragment read spread over the banks.  LDS accesses of a wave are done in order, so the next
// step can be stored as soon as the reads of the last are issued; a fence of wave scope, which is no instruction, keeps the compiler
// from moving a lane's reads of other lanes' data over the stores.  The waves of a workgroup share K (wave w takes steps w, w + waves,
// ..., so that together they read contiguous bytes of a row) and add their partial sums up through LDS afterwards, in a fixed
// order, so results are deterministic.
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

#include "mfma_common.h"

namespace metro {
namespace {

// Memory at any element alignment (rows of an odd length); the hardware takes unaligned 128-bit global loads.
typedef u32x4 u32x4_any __attribute__((aligned(2)));

// Mask of word `e` of a vector of T whose first `drop` elements are to be zeroed.
template <typename T>
__device__ __forceinline__ uint32_t keep_mask(int drop, int e) {
    if (sizeof(T) == 4) return drop <= e ? 0xffffffffu : 0u;
    return drop <= 2 * e ? 0xffffffffu : drop == 2 * e + 1 ? 0xffff0000u : 0u;
}

enum class KRows { kWhole, kRagged, kTiny };  // K a multiple of a step; any K >= kVec; K < kVec (element-wise loads)


// LDS of a wave: bytes for the weights of a step, for the activations.
template <typename WT, typename XT, int NB, int MT>
constexpr int split_w_bytes() { return NB * 2048; }
template <typename WT, typename XT, int NB, int MT>
constexpr int split_x_bytes() { return MT * 2048 * (int)sizeof(XT) / (int)sizeof(WT); }

// rows: w_base, w_pitch, x_base, x_pitch (elements, uniform), and the rows behind them, any per lane:
//   x_row(mt, r)  row r (0..15) of sub-tile mt; may hang on a load of its own
//   w_row(b, r)   row r of weight block b; kWhole: w_block(b), row 0 of it, uniform, the others follow
// kWhole: offsets of activations fit 32 bits.  Rows are kept, not addresses, which leaves the vector registers to data in flight.
// The wave's steps are s0, s0 + stride, ... (`mine` of them).  lds_w / lds_x: the wave's own.  WT weights, XT activations.  kChains
// accumulators per block shorten the chains of additions.
template <typename WT, typename XT, int NB, int MT, int DEPTH, KRows kRows, int kChains = 1, typename Rows>
__device__ __forceinline__ void split_dot(Rows rows, int K, int s0, int stride, int mine, char* lds_w, char* lds_x, floatx4 (&sum)[NB][MT]) {
    constexpr int kVec = 16 / (int)sizeof(WT);              // k per lane and load
    constexpr int kStep = 8 * kVec;                         // k per step
    constexpr int XV = (int)sizeof(XT) / (int)sizeof(WT);   // 128-byte lines per activation row and step
    constexpr int XR = 8 / XV;                              // activation rows per load instruction
    constexpr int kXLoads = MT * 16 / XR;
    constexpr int kXVec = 16 / (int)sizeof(XT);
    constexpr bool kWhole = kRows == KRows::kWhole;
    const int lane = threadIdx.x & 63, r16 = lane & 15, q = lane >> 4;
    floatx4 acc[kChains][NB][MT];
#pragma unroll
    for (int h = 0; h < kChains; ++h)
#pragma unroll
        for (int b = 0; b < NB; ++b)
#pragma unroll
            for (int mt = 0; mt < MT; ++mt) acc[h][b][mt] = floatx4{0.f, 0.f, 0.f, 0.f};

    u32x4 w[DEPTH][NB][2], x[DEPTH][kXLoads];
    auto guarded = [&](const auto* p, int k) {              // K < kVec: element by element
        using T = std::remove_cv_t<std::remove_pointer_t<decltype(p)>>;
        constexpr int n = 16 / (int)sizeof(T);
        typedef T vec __attribute__((ext_vector_type(n)));
        vec v;
#pragma unroll
        for (int e = 0; e < n; ++e) v[e] = k + e < K ? p[k + e] : (T)0.f;
        return __builtin_bit_cast(u32x4, v);
    };
    // This lane's rows and, inside a step, its k: of the weights 8 rows x 8 pieces per instruction, of the activations XR x 8 XV.
    const int w_r = lane >> 3, w_k = (lane & 7) * kVec;
    const int x_r = lane / (8 * XV), x_p = lane & (8 * XV - 1), x_k = x_p / XV * kVec, x_v = x_p % XV * kXVec;
    int wr[kWhole ? 1 : NB][2];
    uint32_t xr[kXLoads];                                   // kWhole: the element offset
    const uint32_t w_lane = kWhole ? (uint32_t)(w_r * rows.w_pitch + w_k) : 0u;
    if constexpr (!kWhole) {
#pragma unroll
        for (int b = 0; b < NB; ++b)
#pragma unroll
            for (int h = 0; h < 2; ++h) wr[b][h] = rows.w_row(b, h * 8 + w_r);
    }
    auto x_rows = [&]() {
#pragma unroll
        for (int i = 0; i < kXLoads; ++i) {
            const uint32_t row = (uint32_t)rows.x_row(i * XR / 16, i * XR % 16 + x_r);
            xr[i] = kWhole ? row * (uint32_t)rows.x_pitch + (uint32_t)(x_k + x_v) : row;
        }
    };
    // Every lane's vector stays inside its row: one that would pass the end is moved back to end with the row, and
    // the elements it then repeats are zeroed (in both operands) when the partial step is consumed.
    // Past the wave's last step (kWhole) every lane reads the same 16 bytes of a line that is there already.
    auto load_w = [&](auto B, int s) {
        constexpr int buf = decltype(B)::value;
        const int step = s0 + stride * min(s, mine - 1);
        const uint32_t off = s < mine ? w_lane : 0u;
        const int k = step * kStep + w_k, at = min(k, K - kVec);
#pragma unroll
        for (int b = 0; b < NB; ++b)
#pragma unroll
            for (int h = 0; h < 2; ++h) {
                if constexpr (kWhole) {
                    w[buf][b][h] = *reinterpret_cast<const u32x4*>(rows.w_base + (size_t)(rows.w_block(b) + h * 8) * rows.w_pitch + (size_t)step * kStep + off);
                } else {
                    const WT* p = rows.w_base + (size_t)(uint32_t)wr[b][h] * (uint32_t)rows.w_pitch;
                    if constexpr (kRows == KRows::kTiny) w[buf][b][h] = guarded(p, k);
                    else w[buf][b][h] = *reinterpret_cast<const u32x4_any*>(p + at);
                }
            }
    };
    auto load_x = [&](auto B, int s) {
        constexpr int buf = decltype(B)::value;
        const int step = s0 + stride * min(s, mine - 1);
        const int k = step * kStep + x_k, at = min(k, K - kVec);
#pragma unroll
        for (int i = 0; i < kXLoads; ++i) {
            if constexpr (kWhole) {
                x[buf][i] = *reinterpret_cast<const u32x4*>(rows.x_base + (size_t)step * kStep + (s < mine ? xr[i] : 0u));
            } else {
                const XT* p = rows.x_base + (size_t)xr[i] * (uint32_t)rows.x_pitch;
                if constexpr (kRows == KRows::kTiny) x[buf][i] = guarded(p, k + x_v);
                else x[buf][i] = *reinterpret_cast<const u32x4_any*>(p + at + x_v);
            }
        }
    };
    // line `l` of 128 bytes (16 to a block or sub-tile and line of it), piece p
    auto place = [](int l, int p) { return l * 128 + ((p ^ (l & 7)) * 16); };
    auto store = [&](auto B) {
        constexpr int buf = decltype(B)::value;
#pragma unroll
        for (int b = 0; b < NB; ++b)
#pragma unroll
            for (int h = 0; h < 2; ++h) *reinterpret_cast<u32x4*>(lds_w + b * 2048 + h * 1024 + place(w_r, lane & 7)) = w[buf][b][h];
#pragma unroll
        for (int i = 0; i < kXLoads; ++i) {
            const int mt = i * XR / 16, r = i * XR % 16 + x_r;
            *reinterpret_cast<u32x4*>(lds_x + mt * (2048 * XV) + (x_p >> 3) * 2048 + place(r, x_p & 7)) = x[buf][i];
        }
    };
    auto wave_fence = [] { __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront"); };
    auto consume = [&](int step, auto Masked) {
        constexpr bool masked = decltype(Masked)::value && kRows == KRows::kRagged;
#pragma unroll
        for (int j = 0; j < 2; ++j) {
            u32x4 wf[NB], xf[MT][XV];
#pragma unroll
            for (int b = 0; b < NB; ++b) wf[b] = *reinterpret_cast<const u32x4*>(lds_w + b * 2048 + place(r16, j * 4 + q));
#pragma unroll
            for (int mt = 0; mt < MT; ++mt)
#pragma unroll
                for (int v = 0; v < XV; ++v) {
                    const int p = (j * 4 + q) * XV + v;
                    xf[mt][v] = *reinterpret_cast<const u32x4*>(lds_x + mt * (2048 * XV) + (p >> 3) * 2048 + place(r16, p & 7));
                }
            u32x4 xv[MT][XV], wm = {}, xm[XV] = {};
            if constexpr (masked) {                         // zeroes the elements that a moved vector repeats, in both
                const int k = step * kStep + j * 4 * kVec + q * kVec, drop = max(k - (K - kVec), 0);    // operands (0 x inf
#pragma unroll                                              // would be NaN)
                for (int e = 0; e < 4; ++e) {
                    wm[e] = keep_mask<WT>(drop, e);
#pragma unroll
                    for (int v = 0; v < XV; ++v) xm[v][e] = keep_mask<XT>(drop - v * kXVec, e);
                }
            }
#pragma unroll
            for (int mt = 0; mt < MT; ++mt)
#pragma unroll
                for (int v = 0; v < XV; ++v) xv[mt][v] = masked ? xf[mt][v] & xm[v] : xf[mt][v];
#pragma unroll
            for (int b = 0; b < NB; ++b) {
                const u32x4 wr = masked ? wf[b] & wm : wf[b];
                if constexpr (sizeof(XT) == 2) {
#pragma unroll
                    for (int mt = 0; mt < MT; ++mt)
                        acc[j % kChains][b][mt] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(
                            __builtin_bit_cast(bf16x8, wr), __builtin_bit_cast(bf16x8, xv[mt][0]),
                            acc[j % kChains][b][mt], 0, 0, 0);
                } else {
#pragma unroll
                    for (int c = 0; c < kVec; ++c) {
                        const float wf1 = sizeof(WT) == 4 ? __uint_as_float(wr[c & 3])
                                                          : __uint_as_float((c & 1) ? wr[c >> 1] & 0xffff0000u : wr[c >> 1] << 16);
#pragma unroll
                        for (int mt = 0; mt < MT; ++mt)
                            acc[(j * kVec + c) % kChains][b][mt] = __builtin_amdgcn_mfma_f32_16x16x4f32(
                                wf1, __uint_as_float(xv[mt][c >> 2][c & 3]), acc[(j * kVec + c) % kChains][b][mt], 0, 0, 0);
                    }
                }
            }
        }
    };

    if (mine > 0) {
        // Buffer s % DEPTH holds the wave's step s.  Loads are unconditional (past the end: the last step again) so
        // that the compiler counts what is outstanding exactly and waits for the consumed step only; the last
        // DEPTH steps load nothing.
        // The rows of activations may hang on a load of their own: weights that need not wait for it go out first (the
        // kernels of the general path; in the 16-bit ones, with more bytes in flight, it makes no difference).
        if constexpr (kWhole) {
            x_rows();
            run_steps(std::make_integer_sequence<int, DEPTH>{}, [&](auto U, int s) { load_x(U, s); load_w(U, s); }, 0);
        } else {
            run_steps(std::make_integer_sequence<int, DEPTH>{}, load_w, 0);
            __builtin_amdgcn_sched_barrier(0);
            x_rows();
            run_steps(std::make_integer_sequence<int, DEPTH>{}, load_x, 0);
        }
        auto step = [&](auto U, int s) {
            wave_fence();
            store(U);
            wave_fence();
            __builtin_amdgcn_sched_barrier(0);              // the loads refill the registers just stored, none earlier
            load_x(U, s + DEPTH);
            load_w(U, s + DEPTH);
            __builtin_amdgcn_sched_barrier(0);
            consume(s0 + stride * s, std::false_type{});
        };
        auto final_step = [&](auto U, int s) {
            wave_fence();
            store(U);
            wave_fence();
            consume(s0 + stride * s, std::true_type{});
        };
        int s = 0;
        for (; s + DEPTH < mine; s += DEPTH) run_steps(std::make_integer_sequence<int, DEPTH>{}, step, s);
        run_steps_tail(std::make_integer_sequence<int, DEPTH>{}, final_step, s, mine);
    }
#pragma unroll
    for (int h = 1; h < kChains; h *= 2)                    // pairwise
#pragma unroll
        for (int i = 0; i + h < kChains; i += 2 * h)
#pragma unroll
            for (int b = 0; b < NB; ++b)
#pragma unroll
                for (int mt = 0; mt < MT; ++mt) acc[i][b][mt] += acc[i + h][b][mt];
#pragma unroll
    for (int b = 0; b < NB; ++b)
#pragma unroll
        for (int mt = 0; mt < MT; ++mt) sum[b][mt] = acc[0][b][mt];
}

}  // namespace
}  // namespace metro
