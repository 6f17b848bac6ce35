// Dot products of NB x 16 weight rows with MT x 16 activation rows over the K steps of one wave, operands straight from
// memory: no LDS and no barrier.
//
// A step is 128 bytes of every weight row (one cache line: two load instructions of 16 rows x 64 contiguous bytes).  Both
// operands go into registers in matrix-operand layout, DEPTH steps of loads in flight per wave.  The waves of a
// workgroup share K (wave w takes steps w, w + waves, ..., so that together they read contiguous bytes of a row) and add
// their partial sums up through LDS afterwards, in a fixed order, so results are deterministic.
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


// pw / px: first element of this lane's row of every block (kWhole: of the block, uniform, and w_lane / x_lane the lane's
// offset in elements, which keeps the vector registers for data in flight).  The wave's steps are s0, s0 + stride, ...
// (`mine` of them).  x_rows(px, x_lane) fills the last two.  WT weights, XT activations.  kChains accumulators per block shorten the chains of additions.
template <typename WT, typename XT, int NB, int MT, int DEPTH, KRows kRows, int kChains = 1, typename XRows>
__device__ __forceinline__ void split_dot(const WT* const (&pw)[NB], uint32_t w_lane, XRows x_rows, int K, int s0, int stride,
                                          int mine, floatx4 (&sum)[NB][MT]) {
    constexpr int kVec = 16 / (int)sizeof(WT);              // k per lane and load
    constexpr int kStep = 8 * kVec;                         // k per step
    constexpr int XV = kVec * (int)sizeof(XT) / 16;         // 16-byte loads of activations per weight load
    constexpr bool kWhole = kRows == KRows::kWhole;
    const int q = (threadIdx.x & 63) >> 4;
    floatx4 acc[kChains][NB][MT];
#pragma unroll
    for (int h = 0; h < kChains; ++h)
#pragma unroll
        for (int b = 0; b < NB; ++b)
#pragma unroll
            for (int mt = 0; mt < MT; ++mt) acc[h][b][mt] = floatx4{0.f, 0.f, 0.f, 0.f};

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
    const XT* px[MT];
    uint32_t x_lane[MT];
    // Past the wave's last step every lane reads the same 16 bytes of a line that is there already.
    auto load_w = [&](auto B, int s) {
        constexpr int buf = decltype(B)::value;
        const int step = s0 + stride * min(s, mine - 1);
        const uint32_t off = s < mine ? w_lane : 0u;
#pragma unroll
        for (int j = 0; j < 2; ++j) {
            const int k = step * kStep + j * 4 * kVec + q * kVec, at = min(k, K - kVec);
            const size_t whole_at = (size_t)step * kStep + j * 4 * kVec;      // uniform
#pragma unroll
            for (int b = 0; b < NB; ++b) {
                if constexpr (kRows == KRows::kTiny) w[buf][j][b] = guarded(pw[b], k);
                else if constexpr (kWhole) w[buf][j][b] = *reinterpret_cast<const u32x4*>(pw[b] + whole_at + off);
                else w[buf][j][b] = *reinterpret_cast<const u32x4_any*>(pw[b] + at);
            }
        }
    };
    auto load_x = [&](auto B, int s) {
        constexpr int buf = decltype(B)::value;
        const int step = s0 + stride * min(s, mine - 1);
        uint32_t off[MT];
#pragma unroll
        for (int mt = 0; mt < MT; ++mt) off[mt] = s < mine ? x_lane[mt] : 0u;
#pragma unroll
        for (int j = 0; j < 2; ++j) {
            const int k = step * kStep + j * 4 * kVec + q * kVec, at = min(k, K - kVec);
            const size_t whole_at = (size_t)step * kStep + j * 4 * kVec;      // uniform
#pragma unroll
            for (int mt = 0; mt < MT; ++mt)
#pragma unroll
                for (int v = 0; v < XV; ++v) {
                    constexpr int n = 16 / (int)sizeof(XT);
                    if constexpr (kRows == KRows::kTiny) x[buf][j][mt][v] = guarded(px[mt], k + v * n);
                    else if constexpr (kWhole) x[buf][j][mt][v] = *reinterpret_cast<const u32x4*>(px[mt] + whole_at + off[mt] + v * n);
                    else x[buf][j][mt][v] = *reinterpret_cast<const u32x4_any*>(px[mt] + at + v * n);
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
                        acc[j % kChains][b][mt] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(
                            __builtin_bit_cast(bf16x8, wr), __builtin_bit_cast(bf16x8, xv[mt][0]),
                            acc[j % kChains][b][mt], 0, 0, 0);
                } else {
#pragma unroll
                    for (int c = 0; c < kVec; ++c) {
                        const float wf = sizeof(WT) == 4 ? __uint_as_float(wr[c & 3])
                                                         : __uint_as_float((c & 1) ? wr[c >> 1] & 0xffff0000u : wr[c >> 1] << 16);
#pragma unroll
                        for (int mt = 0; mt < MT; ++mt)
                            acc[(j * kVec + c) % kChains][b][mt] = __builtin_amdgcn_mfma_f32_16x16x4f32(
                                wf, __uint_as_float(xv[mt][c >> 2][c & 3]), acc[(j * kVec + c) % kChains][b][mt], 0, 0, 0);
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
            x_rows(px, x_lane);
            run_steps(std::make_integer_sequence<int, DEPTH>{}, [&](auto U, int s) { load_x(U, s); load_w(U, s); }, 0);
        } else {
            run_steps(std::make_integer_sequence<int, DEPTH>{}, load_w, 0);
            __builtin_amdgcn_sched_barrier(0);
            x_rows(px, x_lane);
            run_steps(std::make_integer_sequence<int, DEPTH>{}, load_x, 0);
        }
        auto step = [&](auto U, int s) {
            consume(U, s0 + stride * s, std::false_type{});
            __builtin_amdgcn_sched_barrier(0);              // the loads refill the registers just read, none earlier
            load_x(U, s + DEPTH);
            load_w(U, s + DEPTH);
            __builtin_amdgcn_sched_barrier(0);
        };
        auto final_step = [&](auto U, int s) { consume(U, s0 + stride * s, std::true_type{}); };
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
