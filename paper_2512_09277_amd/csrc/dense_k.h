// Dense tile: 32 MT activation rows x 128 weight rows x a range of K, both operands staged through LDS, by one workgroup of
// four waves (2 x 2, each 16 MT x 64).
//
// Global loads are fully coalesced (8 lanes read the 128 contiguous bytes a row contributes to a K step of 64: a wave
// instruction covers 8 whole cache lines instead of 16 half lines), each operand byte enters the CU once per
// workgroup, and the waves read their fragments from LDS in operand layout.  Three register sets: the loads of steps
// s + 1 .. s + 3 are in flight while step s is multiplied.  Loads are unconditional -- past the range they re-read its
// last step -- so that the compiler counts outstanding loads exactly.
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

#include <type_traits>

#include "mfma_common.h"

namespace metro {
namespace {

constexpr int kDenseBK = 64;
constexpr int kDenseRow = kDenseBK * 2 + 16;                     // LDS bytes per staged row (+16 spreads the banks)
constexpr int kDenseRows = 128;                                  // weight rows, and activation rows at most
constexpr int kDenseBuf = 2 * kDenseRows * kDenseRow;            // x tile + w tile of one step
constexpr int kDenseLds = 2 * kDenseBuf;

// x + x_lane[p] / w[p] + w_lane: this thread's 16 bytes (piece tid & 7) of activation / weight row p * 32 + (tid >> 3) at
// k = 0 (x, w[p] uniform).  wave_x: first staged activation row of the wave; wave_w[b]: staged weight row of
// block b.  kHalves: the two halves of a K step have accumulators of their own (chains of additions half as long), added at the
// end.  sum[b][mt]: lane (r16, q) holds weight rows 4 q + v of block b, activation row r16 of sub-tile mt.
template <int MT, bool kHalves = false>
__device__ __forceinline__ void dense_dot(const char* x, const uint32_t (&x_lane)[MT], const char* const (&w)[4],
                                          size_t w_lane, int wave_x,
                                          const int (&wave_w)[4], int s_begin, int s_end, char* lds,
                                          floatx4 (&sum)[4][MT]) {
    floatx4 acc[kHalves ? 2 : 1][4][MT];
    const int tid = threadIdx.x, lane = tid & 63;
    const int r16 = lane & 15, q = lane >> 4;
    const int last = s_end - 1;
    const int st_off = (tid >> 3) * kDenseRow + (tid & 7) * 16;
    u32x4 xr[3][MT], wr[3][4];
    auto load = [&](int set, int s) {
#pragma unroll
        for (int p = 0; p < MT; ++p) xr[set][p] = *reinterpret_cast<const u32x4*>(x + (size_t)s * (kDenseBK * 2) + x_lane[p]);
#pragma unroll
        for (int p = 0; p < 4; ++p) wr[set][p] = *reinterpret_cast<const u32x4*>(w[p] + (size_t)s * (kDenseBK * 2) + w_lane);
    };
    auto park = [&](int set, int buf) {
        char* base = lds + buf * kDenseBuf + st_off;
#pragma unroll
        for (int p = 0; p < MT; ++p) *reinterpret_cast<u32x4*>(base + p * 32 * kDenseRow) = xr[set][p];
#pragma unroll
        for (int p = 0; p < 4; ++p) *reinterpret_cast<u32x4*>(base + (kDenseRows + p * 32) * kDenseRow) = wr[set][p];
    };
    const int rd = r16 * kDenseRow + q * 16;
    const int x_off = wave_x * kDenseRow + rd;
    int w_off[4];
#pragma unroll
    for (int b = 0; b < 4; ++b) w_off[b] = (kDenseRows + wave_w[b]) * kDenseRow + rd;
#pragma unroll
    for (int h = 0; h < (kHalves ? 2 : 1); ++h)
#pragma unroll
        for (int b = 0; b < 4; ++b)
#pragma unroll
            for (int mt = 0; mt < MT; ++mt) acc[h][b][mt] = floatx4{0.f, 0.f, 0.f, 0.f};

    // step U of a period of 6 (register set U % 3, LDS buffer U % 2 known at compile time)
    auto step = [&](auto Uc, int s) {
        constexpr int U = decltype(Uc)::value;
        load(U % 3, min(s + 3, last));                            // set U % 3 was parked one step ago
        const char* base = lds + (U % 2) * kDenseBuf;
#pragma unroll
        for (int j = 0; j < kDenseBK / 32; ++j) {
            bf16x8 xb[MT], wa[4];
#pragma unroll
            for (int mt = 0; mt < MT; ++mt) xb[mt] = *reinterpret_cast<const bf16x8*>(base + x_off + mt * 16 * kDenseRow + j * 64);
#pragma unroll
            for (int b = 0; b < 4; ++b) wa[b] = *reinterpret_cast<const bf16x8*>(base + w_off[b] + j * 64);
#pragma unroll
            for (int b = 0; b < 4; ++b)
#pragma unroll
                for (int mt = 0; mt < MT; ++mt)
                    acc[kHalves ? j : 0][b][mt] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(wa[b], xb[mt], acc[kHalves ? j : 0][b][mt], 0, 0, 0);
        }
        park((U + 1) % 3, (U + 1) % 2);                           // step s + 1, loaded two steps ago
        __syncthreads();
    };
    load(0, min(s_begin, last));
    load(1, min(s_begin + 1, last));
    load(2, min(s_begin + 2, last));
    park(0, 0);
    __syncthreads();
    int s = s_begin;
    for (; s + 6 <= s_end; s += 6) run_steps(std::make_integer_sequence<int, 6>{}, step, s);
    run_steps_tail(std::make_integer_sequence<int, 5>{}, step, s, s_end);
#pragma unroll
    for (int b = 0; b < 4; ++b)
#pragma unroll
        for (int mt = 0; mt < MT; ++mt) sum[b][mt] = kHalves ? acc[0][b][mt] + acc[kHalves ? 1 : 0][b][mt] : acc[0][b][mt];
}

}  // namespace
}  // namespace metro
