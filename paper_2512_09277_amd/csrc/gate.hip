// moe_gate_topk for gfx950: router logits + top-k + gating weights on the full (gathered) token set,
// the step that produces the global top-k ids the routing solve consumes (Sec. 4.3 of arxiv
// 2512.09277: every rank runs top-k over all tokens).
//
//   logit[t][e] = x[t] . w_gate[e]        ids[t] = k largest logits (descending, ties to the lower id)
//   w[t][j]     = softmax over the k selected logits          cnt[e] = pairs that selected expert e
//
// The logits are a small dense contraction ([T,H] x [H,N], 3.8 GFLOP at T=1024, H=7168, N=256) whose
// operands total 18 MB: neither the matrix cores nor HBM is the limit, launch latency and the number
// of busy CUs are.  Launches:
//   1. gate_logits_mfma_kernel: 64 tokens x 64 experts x one K chunk per workgroup (split-K so that
//      ~512 workgroups exist at any batch size); both operands go straight from global memory into
//      the MFMA operand layout; large batches: gate_logits_lds_kernel, both operands staged through LDS;
//      fp32 partial sums land in the workspace, part[chunk][t][e];
//   2. gate_topk_kernel: one wave per token sums the chunks in a fixed order (deterministic), picks the
//      top-k by k rounds of a wave-wide arg-max over (logit, -id) and forms the softmax weights;
//   3. (only when the caller wants expert_count) gate_count_kernel: pairs per expert, one workgroup.
// Shapes these kernels do not take (fp32, N not a multiple of 64, H not a multiple of 32, misaligned operands) use
// gate_logits_split_kernel instead, K split over the waves of a workgroup, or, for few fp32 logits of long rows,
// gate_logits_wave_kernel.
#include <hip/hip_runtime.h>
#include <float.h>
#include <stdint.h>

#include <algorithm>
#include <type_traits>

#include "device_utils.h"
#include "metro.h"
#include "ring_k.h"
#include "split_k.h"

namespace metro {
namespace {

constexpr int kThreads = 256;
constexpr int kMaxN = 512;
constexpr int kTokTile = 16;              // tokens of one matrix-instruction sub-tile
constexpr int kMinChunkSteps = 2;           // K steps of 32 a wave gets at least

struct GateArgs {
    const void* x;
    const void* w_gate;
    float* part;              // [n_chunks][T][N]
    int T, H, N, ldw;
    int steps_per_chunk;      // K steps of 32 per chunk
};

// One workgroup: 16*MT tokens x 64 experts x one K chunk; its four waves split the chunk's K steps and
// meet through LDS, so one partial tile leaves the workgroup.  (Splitting K over workgroups only would
// need four times the chunks for the same number of waves, and the partial sums -- written here, read
// by the top-k kernel -- would outweigh the operands.)
// Lane (r16, q) supplies the 8 elements k = kk + q*8 .. +8 of expert row r16 of a block (A operand) and of
// token row r16 of a sub-tile (B operand); D[i][j]: i = expert 4*q + v of the block, j = token r16.
constexpr int kExpTile = 64, kNB = kExpTile / 16;

template <int MT>
__global__ __launch_bounds__(kThreads, 2) void gate_logits_mfma_kernel(GateArgs a) {
    __shared__ floatx4 xch[3][kNB * MT][kWave];                   // sums of waves 1..3
    const int lane = threadIdx.x & 63, wv = threadIdx.x >> 6;
    const int r16 = lane & 15, q = lane >> 4;
    // K chunk fastest in launch order: workgroup i runs on XCD i mod 8, so with a multiple of 8 chunks
    // every XCD (own L2) streams its own K range of x and w_gate instead of all eight fetching everything.
    const int chunk = blockIdx.x, t0 = blockIdx.y * (16 * MT), e0 = blockIdx.z * kExpTile;
    const int n_steps = a.H / 32;
    const int c_begin = chunk * a.steps_per_chunk, c_end = min(c_begin + a.steps_per_chunk, n_steps);
    const int per_wave = (c_end - c_begin + 3) / 4;
    const int s_begin = min(c_begin + wv * per_wave, c_end), s_end = min(s_begin + per_wave, c_end);
    const char* xp[MT];
#pragma unroll
    for (int mt = 0; mt < MT; ++mt) {
        const int tok = min(t0 + mt * 16 + r16, a.T - 1);         // rows past the batch repeat the last token
        xp[mt] = reinterpret_cast<const char*>(a.x) + ((size_t)tok * a.H + q * 8) * 2;
    }
    const char* wp = reinterpret_cast<const char*>(a.w_gate) + ((size_t)(e0 + r16) * a.ldw + q * 8) * 2;
    const size_t blk = (size_t)16 * a.ldw * 2;                    // bytes between 16-row blocks

    floatx4 acc[kNB][MT];
#pragma unroll
    for (int b = 0; b < kNB; ++b)
#pragma unroll
        for (int mt = 0; mt < MT; ++mt) acc[b][mt] = floatx4{0.f, 0.f, 0.f, 0.f};
    // U steps at a time: all their loads are issued before the first matrix instruction (the scheduling
    // barrier keeps the compiler from sinking each load next to its use, which would leave one or two
    // loads in flight per wave).
    auto steps = [&](auto U, int s) {
        constexpr int n = decltype(U)::value;
        bf16x8 xb[n][MT], wa[n][kNB];
#pragma unroll
        for (int u = 0; u < n; ++u) {
#pragma unroll
            for (int mt = 0; mt < MT; ++mt) xb[u][mt] = *reinterpret_cast<const bf16x8*>(xp[mt] + (size_t)(s + u) * 64);
#pragma unroll
            for (int b = 0; b < kNB; ++b) wa[u][b] = *reinterpret_cast<const bf16x8*>(wp + b * blk + (size_t)(s + u) * 64);
        }
        __builtin_amdgcn_sched_barrier(0);
#pragma unroll
        for (int u = 0; u < n; ++u)
#pragma unroll
            for (int b = 0; b < kNB; ++b)
#pragma unroll
                for (int mt = 0; mt < MT; ++mt)
                    acc[b][mt] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(wa[u][b], xb[u][mt], acc[b][mt], 0, 0, 0);
    };
    int s = s_begin;
    for (; s + 3 <= s_end; s += 3) steps(std::integral_constant<int, 3>{}, s);
    for (; s < s_end; ++s) steps(std::integral_constant<int, 1>{}, s);

    if (wv > 0) {
#pragma unroll
        for (int b = 0; b < kNB; ++b)
#pragma unroll
            for (int mt = 0; mt < MT; ++mt) xch[wv - 1][b * MT + mt][lane] = acc[b][mt];
    }
    __syncthreads();
    if (wv == 0) {
#pragma unroll
        for (int mt = 0; mt < MT; ++mt) {
            const int t = t0 + mt * 16 + r16;
            float* out = a.part + ((size_t)chunk * a.T + min(t, a.T - 1)) * a.N + e0 + q * 4;
#pragma unroll
            for (int b = 0; b < kNB; ++b) {
                floatx4 sum = acc[b][mt];
#pragma unroll
                for (int o = 0; o < 3; ++o) sum += xch[o][b * MT + mt][lane];     // waves in a fixed order
                if (t < a.T) *reinterpret_cast<floatx4*>(out + b * 16) = sum;
            }
        }
    }
}

// Large batches: one workgroup = 16 MT tokens x 128 experts x one K chunk, both operands staged through LDS (ring_k.h).
constexpr int kBigTile = kRingRows;                              // experts of a workgroup

// kChains: accumulators per block, which keep the chains of additions short.  Tiles of 128 tokens: 1, at 8 chunks; of 64: 2 from 1024
// tokens on, whose chunks are as many and as long, and 4 below, see gate_big.
template <int MT, int kChains>
__global__ __launch_bounds__(kThreads, 2) void gate_logits_lds_kernel(GateArgs a) {
    const int tid = threadIdx.x, lane = tid & 63, wv = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int r16 = lane & 15, q = lane >> 4, srow = tid >> 3;
    const int chunk = blockIdx.x, t0 = blockIdx.y * (16 * MT), e0 = blockIdx.z * kBigTile;
    const int n_steps = a.H / kRingStep;                          // the host takes this path only if H % 64 == 0
    const int s_begin = chunk * a.steps_per_chunk, s_end = min(s_begin + a.steps_per_chunk, n_steps);
    uint32_t x_lane[MT / 2];                                      // from the tile's first token
#pragma unroll
    for (int p = 0; p < MT / 2; ++p)                              // rows past the batch repeat the last token
        x_lane[p] = (uint32_t)(min(t0 + p * 32 + srow, a.T - 1) - t0) * (uint32_t)(a.H * 2) + ring_piece(p * 32 + srow);
    const char* w[4];
#pragma unroll
    for (int p = 0; p < 4; ++p) w[p] = reinterpret_cast<const char*>(a.w_gate) + (size_t)(e0 + p * 32) * a.ldw * 2;
    floatx4 acc[4][MT / 2];
    ring_dot<MT, kChains>(
        reinterpret_cast<const char*>(a.x) + (size_t)t0 * a.H * 2, x_lane, w, (size_t)srow * a.ldw * 2 + (tid & 7) * 16, s_begin, s_end, acc);
    const int ty = wv >> 1, tx = wv & 1;
#pragma unroll
    for (int mt = 0; mt < MT / 2; ++mt) {
        const int t = t0 + (mt * 2 + ty) * 16 + r16;
        if (t < a.T) {
            float* out = a.part + ((size_t)chunk * a.T + t) * a.N + e0 + tx * 32 + q * 4;
#pragma unroll
            for (int b = 0; b < 4; ++b) *reinterpret_cast<floatx4*>(out + (b >> 1) * 64 + (b & 1) * 16) = acc[b][mt];
        }
    }
}

// Any shape and alignment, fp32 storage among them: a tile of 16 MT tokens x 16 NB experts per workgroup, K split over its
// waves (split_k.h; fp32 operands in fp32 matrix instructions), a single chunk.  What bounds it is latency and the number
// of busy CUs; which tile when: launch_general_logits.
template <typename T, int NB, int MT, int kSplit, int DEPTH, KRows kRows>
__global__ __launch_bounds__(kSplit * kWave) void gate_logits_split_kernel(GateArgs a) {
    constexpr int kLdsW = split_w_bytes<T, T, NB, MT>(), kLds = kLdsW + split_x_bytes<T, T, NB, MT>();   // of a wave
    __shared__ __attribute__((aligned(16))) char lds[kSplit * kLds];
    static_assert(kLds >= NB * MT * kWave * (int)sizeof(floatx4), "the partial sums");
    floatx4 (*part)[NB * MT][kWave] = reinterpret_cast<floatx4 (*)[NB * MT][kWave]>(lds);
    const int lane = lane_id(), wv = __builtin_amdgcn_readfirstlane(wave_id());
    const int r16 = lane & 15, q = lane >> 4;
    const int t0 = blockIdx.x * (16 * MT), e0 = blockIdx.y * (16 * NB);
    constexpr int kStep = 8 * (16 / (int)sizeof(T));
    const int n_steps = (a.H + kStep - 1) / kStep;
    auto w_block = [&](int b) { return e0 + b * 16; };
    auto w_row = [&](int b, int r) { return min(e0 + b * 16 + r, a.N - 1); };
    auto x_row = [&](int mt, int r) { return min(t0 + mt * 16 + r, a.T - 1); };
    struct Rows {
        const T *w_base, *x_base;
        int w_pitch, x_pitch;
        decltype(w_block) w_block;
        decltype(w_row) w_row;
        decltype(x_row) x_row;
    };
    floatx4 acc[NB][MT];
    // fp32 logits decide the top-k: chains of additions about as short as those of one product per lane and a tree
    constexpr int kChains = sizeof(T) == 2 ? 2 : NB * MT > 4 ? 2 : 8;
    split_dot<T, T, NB, MT, DEPTH, kRows, kChains>(Rows{(const T*)a.w_gate, (const T*)a.x, a.ldw, a.H, w_block, w_row, x_row}, a.H, wv, kSplit,
                                                   max(n_steps - wv + kSplit - 1, 0) / kSplit, lds + wv * kLds, lds + wv * kLds + kLdsW, acc);
    __syncthreads();                                        // the partial sums take the LDS of all waves
#pragma unroll
    for (int b = 0; b < NB; ++b)
#pragma unroll
        for (int mt = 0; mt < MT; ++mt) part[wv][b * MT + mt][lane] = acc[b][mt];
    __syncthreads();
    for (int u = wv; u < NB * MT; u += kSplit) {
        floatx4 p[kSplit];
#pragma unroll
        for (int o = 0; o < kSplit; ++o) p[o] = part[o][u][lane];
#pragma unroll
        for (int h = 1; h < kSplit; h *= 2)                                // pairwise, in a fixed order
#pragma unroll
            for (int o = 0; o + h < kSplit; o += 2 * h) p[o] += p[o + h];
        const floatx4 sum = p[0];
        const int t = t0 + (u % MT) * 16 + r16, e = e0 + (u / MT) * 16 + q * 4;
        if (t >= a.T) continue;
        float* out = a.part + (size_t)t * a.N + e;
#pragma unroll
        for (int v = 0; v < 4; ++v)
            if (e + v < a.N) out[v] = sum[v];
    }
}

// fp32, few logits of long rows: one wave per logit (long_rows says when).
__global__ __launch_bounds__(kThreads) void gate_logits_wave_kernel(GateArgs a) {
    const int t = blockIdx.x, e = blockIdx.y * (kThreads / kWave) + wave_id();
    if (e >= a.N) return;
    const float *x = (const float*)a.x + (size_t)t * a.H, *w = (const float*)a.w_gate + (size_t)e * a.ldw;
    float acc = 0.f;
    for (int h = lane_id(); h < a.H; h += kWave) acc = fmaf(x[h], w[h], acc);
#pragma unroll
    for (int d = kWave / 2; d > 0; d >>= 1) acc += __shfl_xor(acc, d);
    if (lane_id() == 0) a.part[(size_t)t * a.N + e] = acc;
}

// Position of a float (no NaN) in an order of unsigned integers; 0 comes before all of them.  -0 and +0 are one value.
__device__ __forceinline__ uint32_t order_of(float v) {
    const uint32_t u = __float_as_uint(v + 0.0f);
    return u ^ ((u >> 31) ? 0xffffffffu : 0x80000000u);
}
// Maximum over the wave, in registers (a shuffle through LDS per step costs several times as much).
__device__ __forceinline__ uint32_t wave_max(uint32_t v) {
    v = max(v, (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0x111, 0xf, 0xf, false));          // row_shr:1
    v = max(v, (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0x112, 0xf, 0xf, false));
    v = max(v, (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0x114, 0xf, 0xf, false));
    v = max(v, (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0x118, 0xf, 0xf, false));
    v = max(v, (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0x142, 0xa, 0xf, false));          // row_bcast:15
    v = max(v, (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0x143, 0xc, 0xf, false));          // row_bcast:31
    return __builtin_amdgcn_readlane(v, kWave - 1);
}

// (k rounds of shuffles through LDS took most of this kernel: 1024 tokens x 256 experts 11.2 -> 6.6 us, 256 x 128 7.6 -> 4.0.)
// One wave per token.  Lane l holds the logits of experts l, l + 64, ... (kPerLane = ceil(N / 64) of them).
// Tokens at or past *n_valid (a padded batch) get ids -1 and weights 0.
template <int kPerLane>
__global__ __launch_bounds__(kThreads) void gate_topk_kernel(const float* __restrict__ part, int n_chunks, int T, int N,
                                                              int k, const int32_t* __restrict__ n_valid,
                                                              int32_t* __restrict__ ids, float* __restrict__ w) {
    const int t = blockIdx.x * (kThreads / kWave) + wave_id();
    if (t >= T) return;                                          // uniform per wave
    const int l = lane_id();
    if (n_valid && t >= min(max(*n_valid, 0), T)) {              // padded token (uniform per wave)
        if (l < k) {
            ids[(size_t)t * k + l] = -1;
            w[(size_t)t * k + l] = 0.f;
        }
        return;
    }
    // Chunk sums in ascending chunk order (fixed, so the result is deterministic); the loads of a batch
    // of chunks x all of the lane's experts are issued together, only the additions are sequential.
    float v[kPerLane];
#pragma unroll
    for (int j = 0; j < kPerLane; ++j) v[j] = 0.f;
    const float* row = part + (size_t)t * N + l;
    const size_t chunk_stride = (size_t)T * N;
    constexpr int kBatch = kPerLane <= 4 ? 8 : 4;
    for (int c0 = 0; c0 < n_chunks; c0 += kBatch) {
        float p[kBatch][kPerLane];
#pragma unroll
        for (int u = 0; u < kBatch; ++u) {
            const int c = min(c0 + u, n_chunks - 1);             // past the end: re-read, not added
#pragma unroll
            for (int j = 0; j < kPerLane; ++j)
                p[u][j] = (j * kWave + l < N) ? row[c * chunk_stride + j * kWave] : 0.f;
        }
#pragma unroll
        for (int u = 0; u < kBatch; ++u)
            if (c0 + u < n_chunks) {
#pragma unroll
                for (int j = 0; j < kPerLane; ++j) v[j] += p[u][j];
            }
    }
    uint32_t ord[kPerLane];                                      // 0: no expert, or already selected
#pragma unroll
    for (int j = 0; j < kPerLane; ++j) {
        if (v[j] != v[j]) v[j] = -FLT_MAX;                       // NaN counts as the lowest finite number
        ord[j] = j * kWave + l < N ? order_of(v[j]) : 0u;
    }
    float my_v = 0.f;
    int my_id = 0;
    for (int r = 0; r < k; ++r) {
        uint32_t best = 0;
        int at = 0;
        float best_v = 0.f;
#pragma unroll
        for (int j = 0; j < kPerLane; ++j)
            if (ord[j] > best) {                                 // equal logits of a lane: the lower id stays
                best = ord[j];
                at = j;
                best_v = v[j];
            }
        const uint32_t top = wave_max(best);                     // > 0: k <= N
        uint64_t who = __ballot(best == top);
        if (who & (who - 1)) {                                   // the same logit in several lanes (uniform): the lowest id
            const uint32_t first = ~wave_max(best == top ? ~(uint32_t)(at * kWave + l) : 0u);
            who = __ballot(best == top && (uint32_t)(at * kWave + l) == first);
        }
        const int lane = __ffsll((unsigned long long)who) - 1;
        const float val = __uint_as_float(__builtin_amdgcn_readlane(__float_as_uint(best_v), lane));
        const int id = __builtin_amdgcn_readlane(at, lane) * kWave + lane;
#pragma unroll
        for (int j = 0; j < kPerLane; ++j)
            if (l == lane && at == j) ord[j] = 0u;
        if (l == r) {
            my_v = val;
            my_id = id;
        }
    }
    // lanes 0..k-1 hold the selection in descending order; softmax over it
    const float top = __shfl(my_v, 0);
    const float ex = l < k ? expf(my_v - top) : 0.f;
    float sum = ex;
#pragma unroll
    for (int d = kWave / 2; d > 0; d >>= 1) sum += __shfl_xor(sum, d);
    if (l < k) {
        ids[(size_t)t * k + l] = my_id;
        w[(size_t)t * k + l] = ex / sum;
    }
}

// T[i] of Sec. 4.1: pairs per expert, one workgroup, LDS histogram over the ids just written (padded pairs,
// id -1, count nothing).  A launch of its own because every way of folding it into the top-k kernel measured
// slower at T = 1024: device-scope atomics from every token's wave onto the same few cache lines serialise
// across the eight L2s (~10 us, more than the rest of the top-k kernel), and per-workgroup histograms added up
// by the last workgroup to finish need a device-scope fence in every workgroup, which invalidates that XCD's
// L2 under the workgroups still reading their partial sums (top-k kernel 10.7 -> 33.8 us).
constexpr int kCountThreads = 1024;
__global__ __launch_bounds__(kCountThreads) void gate_count_kernel(const int32_t* __restrict__ ids, int n_pairs, int N,
                                                                   int32_t* __restrict__ cnt) {
    __shared__ int hist[kMaxN];
    for (int e = threadIdx.x; e < N; e += kCountThreads) hist[e] = 0;
    __syncthreads();
    constexpr int kBatch = 8;                                    // independent loads in flight
    for (int p0 = threadIdx.x; p0 < n_pairs; p0 += kBatch * kCountThreads) {
        int e[kBatch];
#pragma unroll
        for (int u = 0; u < kBatch; ++u) e[u] = p0 + u * kCountThreads < n_pairs ? ids[p0 + u * kCountThreads] : -1;
#pragma unroll
        for (int u = 0; u < kBatch; ++u)
            if (e[u] >= 0 && e[u] < N) atomicAdd(&hist[e[u]], 1);
    }
    __syncthreads();
    for (int e = threadIdx.x; e < N; e += kCountThreads) cnt[e] = hist[e];
}

// Whether fp32 logits take one wave each.  The line was drawn for tiles whose rows came into a CU at 45 GB/s, in operand layout, which a
// wave per logit spreads over the chip; that wave costs a longer chain of loads, and all of them read the weights through L2, so
// these have to stay there.  Measured with the tiles as they are, whole call, us, tiles / waves, inside the rule: H = 2048, 16 tokens,
// 16 / 64 / 128 experts 10.1 / 10.3 / 11.3 against 9.9 / 10.0 / 10.8; H = 4096, 64 experts, 4 / 64 tokens 13.5 / 13.9 against 13.3 /
// 13.8, 128 experts, 64 tokens 14.1 / 15.0; H = 7168, 64 experts, 1 / 16 / 128 tokens 17.9 / 17.7 / 18.7 against 18.1 / 18.6 / 20.9, 256
// experts, 2 / 4 tokens 18.9 / 18.8 against 19.2 / 33.5.  So the waves are still ahead, by at most 5 %, with rows up to 4096, and
// behind with longer ones.  Past the rule they lose as before: H = 7168, 256 experts, 8 tokens 18.8 / 41.4; H = 4096, 128 experts,
// 128 tokens 14.3 / 22.8, 256 experts, 8 tokens 14.4 / 26.6.
inline bool long_rows(int T, int H, int N) {
    const int64_t logits = (int64_t)T * N, weights = (int64_t)N * H * (int)sizeof(float);
    if ((int64_t)H * (std::min(T, kTokTile) + std::min(N, kTokTile) - 11) < 32768) return false;
    if (weights > 2 << 20)
        return (T <= 24 && logits <= 24 * 128 && weights <= 15 << 18) || (T <= 4 && logits <= 1024 && weights <= 15 << 19);
    return logits <= std::min<int64_t>(2 * (int64_t)H, 8192);
}

template <typename T>
void launch_general_logits(const GateArgs& a, hipStream_t st) {
    auto tiles = [&](int rows) { return (int64_t)((a.T + rows - 1) / rows) * ((a.N + rows - 1) / rows); };
    auto go = [&](auto kernel, int rows, int waves) {
        hipLaunchKernelGGL(kernel, dim3((a.T + rows - 1) / rows, (a.N + rows - 1) / rows), dim3(waves * kWave), 0, st, a);
    };
    // The largest tile that gives the chip enough workgroups: larger tiles read each operand fewer times, smaller ones put
    // more CUs and waves to work.  Measured, whole call, us, 64 / 32 / 16 wide tiles: bf16, H = 4000, 200 experts, 4096
    // tokens (256 / 896 / 3328 tiles) 35.3 / 44.0 / 61.4, 1024 tokens (64 / 224 / 832) 29.9 / 15.8 / 19.5, 700 tokens (154 of 32) 29.9 /
    // 17.0 / 17.1, 512 tokens (112) 29.5 / 14.8 / 14.2; H = 2048, 40 experts, 1024 tokens (64) 19.7 / 11.9 / 9.9: in bf16 the 32-wide
    // tile pays from about 150 tiles on, the line at 64 is from loads in operand layout.  fp32, H = 2048, 128 experts, 512 / 1024 / 2048
    // tokens (64 / 128 / 256 of 32) 52.7 / 21.1 / 12.2, 53.0 / 21.3 / 15.8, 54.4 / 22.8 / 24.4; H = 7168, 256 experts, 1024 tokens (256)
    // 156 / 49.5 / 53.7: there, its fp32 matrix instructions being the longer part, from 256.  Short loops want little code: 8 waves
    // two steps deep beat 16 waves four deep at 64 tokens, H = 1000, logits kernel 5.1 to 7.6 (loads in operand layout).
    if (std::is_same_v<T, float> && long_rows(a.T, a.H, a.N)) {
        constexpr int per = kThreads / kWave;
        hipLaunchKernelGGL(gate_logits_wave_kernel, dim3(a.T, (a.N + per - 1) / per), dim3(kThreads), 0, st, a);
    } else if (a.H < 16 / (int)sizeof(T)) go(gate_logits_split_kernel<T, 2, 2, 4, 1, KRows::kTiny>, 32, 4);
    else if (tiles(64) >= 256) go(gate_logits_split_kernel<T, 4, 4, 4, 1, KRows::kRagged>, 64, 4);
    else if (tiles(32) >= (sizeof(T) == 2 ? 64 : 256)) go(gate_logits_split_kernel<T, 2, 2, 8, 2, KRows::kRagged>, 32, 8);
    else go(gate_logits_split_kernel<T, 1, 1, 8, 2, KRows::kRagged>, 16, 8);
}

inline bool gate_mfma_shape(int H, int N, int dtype) {
    return dtype == METRO_DTYPE_BF16 && H % 32 == 0 && N % kExpTile == 0 && N <= kMaxN;
}

// The LDS-staged kernel needs N % 128 == 0 and H % 64 == 0.  It takes batches of at least 1024 tokens and smaller ones, from its tile
// of 64 on, of more than 2^28 products, where what the direct kernel reads in operand layout (64 tokens x 64 experts a workgroup, 38 GB/s
// per CU) is more than a launch's latency.  Measured, whole call, us, direct / staged: 256 experts x 7168, 192 / 256 / 512 / 1000 tokens
// 17.4 / 17.9 / 20.4 / 25.9 against 14.3 / 14.7 / 17.0 / 19.4, 512 x 4096, 192 tokens 18.7 / 17.1, 128 x 4096, 768 tokens 15.3 / 13.5,
// 256 x 2048, 768 tokens 16.2 / 14.5; below the line nothing to win (128 x 2048 and 256 x 1024 up to 1000 tokens within 0.2 us, either
// way).  The staged kernel has four accumulators per block there: with two the error of the weights against 64 bits would grow (1000
// tokens x 256 x 7168 1.51e-7 -> 1.72e-7, now 1.51e-7; they cost 0.2 us).  Over 40 inputs, direct / staged, 1e-7: 320 tokens x 256 x
// 4096 1.673 / 1.665, x 7168 1.945 / 1.700, 768 x 128 x 7168 1.570 / 1.561, 512 x 256 x 7168 1.696 / 1.698; larger only where 8 chunks
// replace 4, 1000 x 512 x 4096 1.495 / 1.508.
constexpr int kStagedAlways = 1024, kStagedMin = 64;
constexpr int64_t kStagedProducts = 1 << 28;
inline bool gate_big(int T, int H, int N) {
    return (T >= kStagedAlways || (T >= kStagedMin && (int64_t)T * N * H > kStagedProducts)) && N % kBigTile == 0 && H % kRingStep == 0;
}

// Tokens of its workgroups: 128 where that still makes two workgroups per CU at 8 K chunks, else 64, which takes 8 chunks
// where 128 would need 16 to fill the chip -- half the partial sums to write and for the top-k kernel to read.  Measured,
// whole call, us, 128 / 64: 1024 tokens x 256 experts x 7168 23.6 / 20.0, 1500 x 256 x 4096 26.2 / 22.5, 3000 x 256 x 4096 27.6 / 27.6,
// 3900 x 256 x 4096 31.3 / 34.5, 4096 x 256 x 7168 39.7 / 43.0, 2048 x 512 x 4096 29.6 / 32.2.
inline int gate_big_tokens(int T, int N) { return ((T + 127) / 128) * (N / kBigTile) * 8 >= 512 ? 128 : 64; }

// Tokens per workgroup: 64 (four sub-tiles) unless the batch is a single sub-tile.
inline int gate_tok_tile(int T) { return T > kTokTile ? 4 * kTokTile : kTokTile; }

// K chunks: enough workgroups for two per CU (~512), each chunk at least kMinChunkSteps steps per wave.
inline int gate_steps_per_chunk(int T, int H, int N) {
    if (gate_big(T, H, N)) {                    // steps of 64; ~8 chunks (one K range per XCD), >= 4 steps each
        const int n_steps = H / kRingStep, rows = gate_big_tokens(T, N);
        const int tiles = ((T + rows - 1) / rows) * (N / kBigTile);
        // 16 chunks where 8 are less than one workgroup per CU; below 1024 tokens only as long as 16 are no more than that.  Measured,
        // whole call, us, 16 / 8 chunks: 256 experts x 7168, 576 / 768 / 960 tokens 20.5 / 21.9 / 23.8 against 16.5 / 17.2 / 19.1 (direct
        // kernel 24.0 / 24.5 / 25.8), 512 x 4096, 320 / 448 tokens 21.2 / 23.1 against 16.1 / 17.4 (20.2 / 21.7); error of the weights
        // against 64 bits at 256 x 7168 and 768 tokens 1.67e-7 against 1.50e-7 (1.50e-7).
        const int want = T < kStagedAlways ? (tiles * 16 <= 256 ? 16 : 8) : tiles * 8 >= 256 ? 8 : 16;
        int chunks = n_steps / 4 >= want ? want : n_steps / 4 >= 8 ? 8 : n_steps / 4 > 0 ? n_steps / 4 : 1;
        return (n_steps + chunks - 1) / chunks;
    }
    const int n_steps = H / 32, tile = gate_tok_tile(T);
    const int tiles = ((T + tile - 1) / tile) * (N / kExpTile);
    int chunks = (512 + tiles - 1) / tiles;
    const int max_chunks = n_steps / (4 * kMinChunkSteps) > 0 ? n_steps / (4 * kMinChunkSteps) : 1;
    if (chunks > max_chunks) chunks = max_chunks;
    if (chunks >= 8) chunks = chunks / 8 * 8;                      // one K range (or two, ...) per XCD
    if (chunks < 1) chunks = 1;
    return (n_steps + chunks - 1) / chunks;
}
inline int gate_chunks(int T, int H, int N, int dtype) {
    if (!gate_mfma_shape(H, N, dtype)) return 1;
    const int spc = gate_steps_per_chunk(T, H, N);
    const int n_steps = gate_big(T, H, N) ? H / kRingStep : H / 32;
    return (n_steps + spc - 1) / spc;
}

inline size_t align256(size_t v) { return (v + 255) & ~(size_t)255; }

// What a batch of T tokens itself needs; an empty one has no partial sums.
inline size_t gate_need(int T, int H, int N, int dtype) {
    return T == 0 ? 256 : align256((size_t)gate_chunks(T, H, N, dtype) * T * N * sizeof(float)) + 256;
}

}  // namespace
}  // namespace metro

// The most that any batch of up to T tokens needs.  More tokens make more tiles, which take fewer K chunks, so the most is at T or at
// the last batch before the chunks become fewer: the last of a tile of 64 or 128 tokens, of the tile of 16, or of a kernel.  From
// 32768 tokens on (512 tiles of 64) there is one chunk, or the staged kernel's 8.
extern "C" size_t moe_gate_topk_workspace_bytes(int T, int H, int N, int dtype) {
    using namespace metro;
    if (T < 0 || H < 1 || N < 1) return 0;
    size_t most = gate_need(T, H, N, dtype);
    if (!gate_mfma_shape(H, N, dtype)) return most;               // one chunk, whatever T
    auto with = [&](int64_t t) {
        if (t < T) most = std::max(most, gate_need((int)t, H, N, dtype));
    };
    with(kTokTile);
    with(kStagedMin - 1);
    with(kStagedProducts / ((int64_t)N * H));
    with(kStagedAlways - 1);
    for (int t = 64; t < T && t <= 32768; t += 64) with(t);
    return most;
}

extern "C" int moe_gate_topk(const void* x, const void* w_gate, int ldw, int T, int H, int N, int k, int dtype,
                             const int32_t* n_valid, int32_t* topk_ids, float* topk_w, int32_t* expert_count,
                             void* ws, size_t ws_bytes, void* stream) {
    using namespace metro;
    if (T < 0 || H < 1 || N < 1 || k < 1 || k > N) return METRO_ERR_INVALID_ARG;
    if (dtype != METRO_DTYPE_BF16 && dtype != METRO_DTYPE_F32) return METRO_ERR_UNSUPPORTED;
    if (N > kMaxN || k > kWave || (int64_t)T * k >= (1 << 24)) return METRO_ERR_UNSUPPORTED;
    if (ldw < H) return METRO_ERR_INVALID_ARG;
    if (T == 0) {                                                 // no token: every expert counts zero pairs
        if (expert_count) {
            hipLaunchKernelGGL(gate_count_kernel, dim3(1), dim3(kCountThreads), 0, (hipStream_t)stream,
                               (const int32_t*)nullptr, 0, N, expert_count);
            if (hipGetLastError() != hipSuccess) return METRO_ERR_HIP;
        }
        return METRO_OK;
    }
    if (!x || !w_gate || !topk_ids || !topk_w || !ws) return METRO_ERR_INVALID_ARG;
    if (((uintptr_t)ws & 255) != 0) return METRO_ERR_INVALID_ARG;
    if (ws_bytes < gate_need(T, H, N, dtype)) return METRO_ERR_WORKSPACE;
    const bool mfma = gate_mfma_shape(H, N, dtype) && ldw % 8 == 0 &&
                      (((uintptr_t)x | (uintptr_t)w_gate) & 15) == 0;
    hipStream_t st = (hipStream_t)stream;
    GateArgs a;
    a.x = x;
    a.w_gate = w_gate;
    a.part = (float*)ws;
    a.T = T; a.H = H; a.N = N; a.ldw = ldw;
    int n_chunks = 1;
    if (mfma) {
        a.steps_per_chunk = gate_steps_per_chunk(T, H, N);
        n_chunks = gate_chunks(T, H, N, dtype);
        if (gate_big(T, H, N)) {
            const int rows = gate_big_tokens(T, N);
            const dim3 grid(n_chunks, (T + rows - 1) / rows, N / kBigTile);
            if (rows == 128) hipLaunchKernelGGL((gate_logits_lds_kernel<8, 1>), grid, dim3(kThreads), 0, st, a);
            else if (T >= kStagedAlways) hipLaunchKernelGGL((gate_logits_lds_kernel<4, 2>), grid, dim3(kThreads), 0, st, a);
            else hipLaunchKernelGGL((gate_logits_lds_kernel<4, 4>), grid, dim3(kThreads), 0, st, a);
        } else {
        const int tile = gate_tok_tile(T);
        const dim3 grid(n_chunks, (T + tile - 1) / tile, N / kExpTile);
        if (tile == kTokTile)
            hipLaunchKernelGGL(gate_logits_mfma_kernel<1>, grid, dim3(kThreads), 0, st, a);
        else
            hipLaunchKernelGGL(gate_logits_mfma_kernel<4>, grid, dim3(kThreads), 0, st, a);
        }
    }
    if (!mfma) {
        a.steps_per_chunk = 0;
        n_chunks = 1;
        if (dtype == METRO_DTYPE_F32) launch_general_logits<float>(a, st);
        else launch_general_logits<__bf16>(a, st);
    }
    if (hipGetLastError() != hipSuccess) return METRO_ERR_HIP;
    const int per = kThreads / kWave;
    const dim3 tgrid((T + per - 1) / per);
    const float* part = (const float*)ws;
    auto topk = [&](auto kernel) {
        hipLaunchKernelGGL(kernel, tgrid, dim3(kThreads), 0, st, part, n_chunks, T, N, k, n_valid, topk_ids, topk_w);
    };
    if (N <= 64) topk(gate_topk_kernel<1>);
    else if (N <= 128) topk(gate_topk_kernel<2>);
    else if (N <= 256) topk(gate_topk_kernel<4>);
    else topk(gate_topk_kernel<8>);
    if (expert_count)
        hipLaunchKernelGGL(gate_count_kernel, dim3(1), dim3(kCountThreads), 0, st, (const int32_t*)topk_ids, T * k, N,
                           expert_count);
    return hipGetLastError() == hipSuccess ? METRO_OK : METRO_ERR_HIP;
}
