// Dense tile: 16 MT activation rows x 128 weight rows x a range of K, both operands staged through LDS, by one workgroup of
// four waves (2 x 2).
//
// What bounds it is how operands enter a CU: a load instruction whose 4 neighbouring lanes read 4 different lines (matrix-operand
// layout straight from memory) takes 64 cycles, 38 GB/s per CU wherever the data is, one that covers whole lines 16 (146 GB/s from
// L2).  So all global loads here are coalesced (8 lanes read the 128 bytes a row contributes to a step) and the operand layout comes from
// LDS.  Activations go from memory to LDS without passing registers, into a ring of D stages; weights through registers, D steps of
// them in flight, into two LDS buffers, so that the LDS of two workgroups per CU holds it all.
//
// One barrier per step, in its middle: the first half step's fragments are in registers when a step begins, the second half's are
// read while those are multiplied, and behind the barrier -- every wave has read all of step s, and step s + 1 has arrived -- the
// next step's first half is read while the second half is multiplied.  The stage of step s then takes step s + D.
// A wait that lets newer loads stay in flight is a count of these, so what is counted must really be issued.  Loads are unconditional
// (past the end every lane takes the same 16 bytes), but the compiler drops a load to registers that no path uses: in the steps
// behind the unrolled loop, weights that no later step of them stores.  Those are not loaded there, and not counted.
//
// LDS: 128 bytes per staged row, its 16-byte piece p at place p ^ (row & 7), so that the 16 rows of a fragment read spread over the
// banks.  A direct load puts lane i's 16 bytes at place i behind a common base, so the lane that fills place i reads piece
// i ^ (row & 7) of the row: still whole lines.  Every half stage is an LDS variable of its own: that is how the compiler knows that a
// fragment read does not depend on the loads in flight to other stages.
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

#include <type_traits>
#include <utility>

#include "mfma_common.h"

namespace metro {
namespace {

constexpr int kRingStep = 64;                                    // bf16 values of K per step
constexpr int kRingRows = 128;                                   // weight rows, and activation rows at most
constexpr int kRingBuf = 64 * kRingStep * 2;                     // a half stage: 64 rows
constexpr int kRingBufs = 10;                                    // 80 KB: two workgroups per CU

template <int I>
__device__ __forceinline__ char* ring_buf() {
    __shared__ __attribute__((aligned(1024))) char buf[kRingBuf];
    return buf;
}

// The same memory by a run-time index (past the K loop).
template <int I = 0>
__device__ __forceinline__ char* ring_buf_at(int i) {
    if constexpr (I == kRingBufs - 1) return ring_buf<I>();
    else return i == I ? ring_buf<I>() : ring_buf_at<I + 1>(i);
}

// Outstanding vector loads at most `n`, no LDS access outstanding.
template <int n>
__device__ __forceinline__ void wait_loads() {
    static_assert(n < 64, "");
    __builtin_amdgcn_s_waitcnt((n & 15) | (7 << 4) | ((n >> 4) << 14));
}

// Kinds of instructions for __builtin_amdgcn_sched_group_barrier.
constexpr int kMatrix = 0x8, kVectorLoad = 0x10, kDsRead = 0x100, kDsWrite = 0x200;

// Byte offset, inside the 128 bytes of a step, of the 16 bytes that this lane stages of `row` of the activations.
__device__ __forceinline__ uint32_t ring_piece(int row) { return (uint32_t)(((threadIdx.x & 7) ^ (row & 7)) * 16); }

// x + x_lane[p]: the 16 bytes that this lane stages of activation row p * 32 + tid / 8 (ring_piece); w[p] + w_lane: those of weight row
// p * 32 + tid / 8 (piece tid & 7).  x, w[p] uniform.  acc[b][mt]: lane (r16, q) of wave (ty, tx) holds weight rows
// (b >> 1) * 64 + tx * 32 + (b & 1) * 16 + 4 q + v, activation row (2 mt + ty) * 16 + r16.  kChains = 2: the two halves of a step have
// accumulators of their own (chains of additions half as long), added at the end; 4: even and odd steps too.
template <int MT, int kChains = 1>
__device__ __forceinline__ void ring_dot(const char* x, const uint32_t (&x_lane)[MT / 2], const char* const (&w)[4],
                                         size_t w_lane, int s_begin, int s_end, floatx4 (&sum)[4][MT / 2]) {
    constexpr int D = MT <= 4 ? 4 : 3, kHalf = MT <= 4 ? 1 : 2, kWBuf = D * kHalf;
    static_assert(MT % 2 == 0 && kWBuf + 4 <= kRingBufs && (kChains < 4 || D % 2 == 0), "");
    constexpr int M2 = MT / 2, kX = MT / 2, kW = 4;              // loads of a step
    const int tid = threadIdx.x, lane = tid & 63, wv = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int r16 = lane & 15, q = lane >> 4, ty = wv >> 1, tx = wv & 1;
    const int rd = r16 * 128 + ((q ^ (r16 & 7)) * 16);
    const int x_rd[2] = {ty * 2048 + rd, ty * 2048 + (rd ^ 64)}, w_rd[2] = {tx * 4096 + rd, tx * 4096 + (rd ^ 64)};
    const int st = (tid >> 3) * 128 + (((tid & 7) ^ ((tid >> 3) & 7)) * 16);
    u32x4 wr[D][4];
    auto load_w = [&](auto U, int s) {
        constexpr int set = decltype(U)::value % D;
        const size_t off = s < s_end ? w_lane : 0u, at = (size_t)min(s, s_end - 1) * 128;
#pragma unroll
        for (int p = 0; p < 4; ++p) wr[set][p] = *reinterpret_cast<const u32x4*>(w[p] + at + off);
    };
    auto park_w = [&](auto U) {
        constexpr int set = decltype(U)::value % D, buf = kWBuf + decltype(U)::value % 2 * 2;
#pragma unroll
        for (int p = 0; p < 4; ++p)
            *reinterpret_cast<u32x4*>((p < 2 ? ring_buf<buf>() : ring_buf<buf + 1>()) + (p & 1) * 4096 + st) = wr[set][p];
    };
    const __amdgpu_buffer_rsrc_t x_rsrc = __builtin_amdgcn_make_buffer_rsrc((void*)x, 0, -1, 0x00027000);
    auto load_x = [&](auto U, int s) {
        constexpr int set = decltype(U)::value % D;
        const int at = min(s, s_end - 1) * 128;
        auto piece = [&](auto P, int) {
            constexpr int p = decltype(P)::value;
            const uint32_t off = s < s_end ? x_lane[p] : 0u;
            __builtin_amdgcn_raw_ptr_buffer_load_lds(
                x_rsrc, (__attribute__((address_space(3))) void*)(ring_buf<set * kHalf + p / 2>() + ((p & 1) * 4 + wv) * 1024), 16, (int)off, at, 0, 0);
        };
        run_steps(std::make_integer_sequence<int, kX>{}, piece, 0);
    };
    floatx4 acc[kChains][4][M2];

    struct Fragments { bf16x8 x[M2], w[4]; } f[2];
    auto read = [&](auto U, auto J) {
        constexpr int set = decltype(U)::value % D, j = decltype(J)::value, buf = kWBuf + decltype(U)::value % 2 * 2;
#pragma unroll
        for (int b = 0; b < 4; ++b)
            f[j].w[b] = *reinterpret_cast<const bf16x8*>((b < 2 ? ring_buf<buf>() : ring_buf<buf + 1>()) + (b & 1) * 2048 + w_rd[j]);
#pragma unroll
        for (int mt = 0; mt < M2; ++mt)
            f[j].x[mt] = *reinterpret_cast<const bf16x8*>((mt < 2 ? ring_buf<set * kHalf>() : ring_buf<set * kHalf + kHalf - 1>()) + (mt & 1) * 4096 + x_rd[j]);
    };
    auto multiply = [&](auto U, auto J) {
        constexpr int j = decltype(J)::value, h = (decltype(U)::value % 2 * 2 + j) % kChains;
#pragma unroll
        for (int b = 0; b < 4; ++b)
#pragma unroll
            for (int mt = 0; mt < M2; ++mt)
                acc[h][b][mt] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(f[j].w[b], f[j].x[mt], acc[h][b][mt], 0, 0, 0);
    };
    constexpr std::integral_constant<int, 0> j0{};
    constexpr std::integral_constant<int, 1> j1{};
    auto arrive = [&](auto Left) {                                // at most `Left` loads outstanding, in every wave
        __builtin_amdgcn_sched_barrier(0);
        wait_loads<decltype(Left)::value>();
        __builtin_amdgcn_s_barrier();
        asm volatile("" ::: "memory");
        __builtin_amdgcn_sched_barrier(0);
    };
    // Last: the last step, counted like U, whose weights are loaded, or stored by a step that follows in the code.
    auto step = [&](auto U, int s, auto Last) {
        constexpr int u = decltype(U)::value, newer = decltype(Last)::value - (u + 1);
        constexpr std::integral_constant<int, u + 1> next{};
        // Fragment reads first, then stores and loads between the products: a wave issues in order, and a burst of loads from four
        // waves holds the products behind it back for some 500 cycles (4096 tokens at 2048 x 768 53.2 + 38.3 -> 51.3 + 35.2 us).
        read(U, j1);
        multiply(U, j0);
        park_w(next);
        __builtin_amdgcn_sched_group_barrier(kDsRead, 4 + M2, 0);
        __builtin_amdgcn_sched_group_barrier(kMatrix, M2, 0);
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            __builtin_amdgcn_sched_group_barrier(kDsWrite, 1, 0);
            __builtin_amdgcn_sched_group_barrier(kMatrix, M2 > 1 ? M2 - 1 : 1, 0);
        }
        // behind the activations of s + 1: those of s + 2 .. s + D - 1 and the weights of s + 2 .. s + D, as far as there are any
        arrive(std::integral_constant<int, kW * (newer <= 0 ? 0 : newer < D - 1 ? newer : D - 1) + kX * (D - 2)>{});
        read(next, j0);
        load_x(U, s + D);
        if constexpr (newer >= D) load_w(next, s + 1 + D);
        multiply(U, j1);
        __builtin_amdgcn_sched_group_barrier(kDsRead, 4 + M2, 0);
#pragma unroll
        for (int i = 0; i < kX + kW; ++i) {
            __builtin_amdgcn_sched_group_barrier(kVectorLoad, 1, 0);
            __builtin_amdgcn_sched_group_barrier(kMatrix, 4 * M2 / (kX + kW), 0);
        }
        __builtin_amdgcn_sched_barrier(0);
    };
    asm volatile("; ring of %0 stages, %1 loads each" ::"i"(D), "i"(kX));          // a comment in the assembly, no instruction
    run_steps(std::make_integer_sequence<int, D>{}, [&](auto U, int s) {
        load_w(U, s);
        load_x(U, s);
        __builtin_amdgcn_sched_barrier(0);                       // the waits count on this order
    }, s_begin);
    // up to 128 registers to clear, while the first loads are on their way
#pragma unroll
    for (int h = 0; h < kChains; ++h)
#pragma unroll
        for (int b = 0; b < 4; ++b)
#pragma unroll
            for (int mt = 0; mt < M2; ++mt) acc[h][b][mt] = floatx4{0.f, 0.f, 0.f, 0.f};
    park_w(j0);
    load_w(j0, s_begin + D);
    arrive(std::integral_constant<int, (D - 1) * (kW + kX) + kW>{});
    read(j0, j0);
    constexpr int kPeriod = D % 2 ? 2 * D : D;
    int s = s_begin;
    for (; s + kPeriod <= s_end; s += kPeriod)
        run_steps(std::make_integer_sequence<int, kPeriod>{}, [&](auto U, int at) { step(U, at, std::integral_constant<int, 2 * kPeriod>{}); }, s);
    run_steps_tail(std::make_integer_sequence<int, kPeriod - 1>{}, [&](auto U, int at) { step(U, at, std::integral_constant<int, kPeriod - 1>{}); },
                   s, s_end);
    wait_loads<0>();                                             // nothing is on its way to LDS when the workgroup ends or goes on
    asm volatile("; ring done");
#pragma unroll
    for (int b = 0; b < 4; ++b)
#pragma unroll
        for (int mt = 0; mt < M2; ++mt) {
            sum[b][mt] = acc[0][b][mt];
            if constexpr (kChains > 1) sum[b][mt] += acc[1][b][mt];
            if constexpr (kChains > 2) sum[b][mt] += acc[2][b][mt] + acc[3][b][mt];
        }
}

}  // namespace
}  // namespace metro
