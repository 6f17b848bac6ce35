// moe_unpermute: one rank's share of the combine step -- a gather of the rows a token owns in
// y_perm, weighted by the gating weights and summed in fp32 in ascending j.
#include <hip/hip_runtime.h>
#include <stdint.h>

#include <algorithm>

#include "metro.h"

namespace metro {
namespace {

constexpr int kThreads = 256;
constexpr int kMaxThreads = 1024;

__device__ __forceinline__ float bf16_bits_to_f32(uint32_t bits16) { return __uint_as_float(bits16 << 16); }
__device__ __forceinline__ uint32_t f32_to_bf16_bits(float v) {
    uint32_t u = __float_as_uint(v);
    if (v != v) return (u >> 16) | 0x0040u;   // NaN stays a (quiet) NaN: the rounding add could carry it into Inf or -0
    u += 0x7fffu + ((u >> 16) & 1u);          // round to nearest even
    return u >> 16;
}

// A 16-byte vector of one row, in fp32 and packed: 8 bf16 or 4 fp32 columns.
template <bool kBf16>
struct Columns {
    static constexpr int kN = kBf16 ? 8 : 4;
    static __device__ __forceinline__ void add(float (&acc)[kN], float w, const uint4& v) {
        const uint32_t u[4] = {v.x, v.y, v.z, v.w};
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            if constexpr (kBf16) {
                acc[2 * i] = fmaf(w, bf16_bits_to_f32(u[i] & 0xffffu), acc[2 * i]);
                acc[2 * i + 1] = fmaf(w, bf16_bits_to_f32(u[i] >> 16), acc[2 * i + 1]);
            } else {
                acc[i] = fmaf(w, __uint_as_float(u[i]), acc[i]);
            }
        }
    }
    static __device__ __forceinline__ uint4 pack(const float (&acc)[kN]) {
        uint32_t o[4];
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            if constexpr (kBf16) o[i] = f32_to_bf16_bits(acc[2 * i]) | (f32_to_bf16_bits(acc[2 * i + 1]) << 16);
            else o[i] = __float_as_uint(acc[i]);
        }
        return make_uint4(o[0], o[1], o[2], o[3]);
    }
};

// Rows of whole 16-byte vectors: every thread owns one vector's columns (one 128-bit load per row).  KMAX > 0:
// k <= KMAX, the token's rows and weights sit in registers and the row loads of a column go out
// together; KMAX == 0: any k.  Bound by HBM (1024 tokens x 7168 in bf16: 45 MB in 10.1 us) and, in small batches, by
// the two dependent loads; fp32 rows took one column per thread and 15 us at 256 tokens x 2048, now 4.8.  How many
// threads a workgroup has: row_threads.
template <bool kBf16, int KMAX>
__global__ __launch_bounds__(kMaxThreads) void unpermute_vec_kernel(const uint4* __restrict__ y,
                                                                 const int32_t* __restrict__ pair_row,
                                                                 const float* __restrict__ topk_w, int k, int HV,
                                                                 uint4* __restrict__ out) {
    using C = Columns<kBf16>;
    const int t = blockIdx.x;
    const int cap = (int)gridDim.x * k;           // rows of y_perm; an entry of pair_row outside [0, cap) is skipped
    if (KMAX > 0) {
        int rows[KMAX > 0 ? KMAX : 1];
        float ws[KMAX > 0 ? KMAX : 1];
#pragma unroll
        for (int j = 0; j < KMAX; ++j) {
            rows[j] = j < k ? pair_row[(size_t)t * k + j] : -1;
            if (rows[j] >= cap) rows[j] = -1;
            ws[j] = j < k ? topk_w[(size_t)t * k + j] : 0.f;
        }
        for (int c = threadIdx.x; c < HV; c += blockDim.x) {
            uint4 v[KMAX > 0 ? KMAX : 1];
#pragma unroll
            for (int j = 0; j < KMAX; ++j)
                if (rows[j] >= 0) v[j] = y[(size_t)rows[j] * HV + c];     // uniform per workgroup
            float acc[C::kN] = {};
#pragma unroll
            for (int j = 0; j < KMAX; ++j)
                if (rows[j] >= 0) C::add(acc, ws[j], v[j]);
            out[(size_t)t * HV + c] = C::pack(acc);
        }
    } else {
        for (int c = threadIdx.x; c < HV; c += blockDim.x) {
            float acc[C::kN] = {};
            for (int j = 0; j < k; ++j) {
                const int r = pair_row[(size_t)t * k + j];
                if (r < 0 || r >= cap) continue;
                C::add(acc, topk_w[(size_t)t * k + j], y[(size_t)r * HV + c]);
            }
            out[(size_t)t * HV + c] = C::pack(acc);
        }
    }
}

template <bool kBf16>
__global__ __launch_bounds__(kThreads) void unpermute_scalar_kernel(const void* __restrict__ y,
                                                                    const int32_t* __restrict__ pair_row,
                                                                    const float* __restrict__ topk_w, int k, int H,
                                                                    void* __restrict__ out) {
    const int t = blockIdx.x;
    const int cap = (int)gridDim.x * k;
    for (int c = threadIdx.x; c < H; c += kThreads) {
        float acc = 0.f;
        for (int j = 0; j < k; ++j) {
            const int r = pair_row[(size_t)t * k + j];
            if (r < 0 || r >= cap) continue;
            const float v = kBf16 ? bf16_bits_to_f32(((const uint16_t*)y)[(size_t)r * H + c])
                                  : ((const float*)y)[(size_t)r * H + c];
            acc = fmaf(topk_w[(size_t)t * k + j], v, acc);
        }
        if (kBf16) ((uint16_t*)out)[(size_t)t * H + c] = (uint16_t)f32_to_bf16_bits(acc);
        else ((float*)out)[(size_t)t * H + c] = acc;
    }
}

// Threads of a workgroup.  Up to 1024 tokens, a thread for every vector of the row, 256 to 1024 (1024 tokens x 896 vectors 10.1 us;
// 12.6 with four turns of 256 threads, a memory round trip each).  More tokens than that come in several rounds of resident
// workgroups, and a workgroup keeps its places until its last wave is done: smaller ones do better, the vectors split evenly
// over their turns.  Measured, an eighth of the pairs here, us, 1024 / 512 / 256 threads: 8192 tokens x 896 vectors (bf16, k = 8)
// 47.9 / 35.7 / 37.0, 4096 x 640 19.7 / 16.5 / 16.7, 2048 x 4096 (fp32, k = 8) 42.6 / 44.9 / 50.3; rows of up to 512 vectors gain 4 to
// 12 % with 256 over 512.  Past k = 8 a vector's rows are loaded one after the other, and more threads hide that until the rounds
// are many: 1500 x 640 (bf16, k = 10, all pairs here) 26.4 with 1024, 30.1 with 512; 8192 x 640, an eighth here, 40.7 and 35.9.  A
// row of 16 vectors took four waves for the work of one (8192 tokens in fp32, k = 8: 7.1 us, now 4.8).  A launch has fewer
// than 2^32 threads.
inline int row_threads(int T, int k, int hv) {
    auto waves = [](int n) { return (n + 63) / 64 * 64; };
    if (T <= 1024) return std::min(std::max(waves(hv), kThreads), kMaxThreads);
    const int most = T >= (1 << 23) ? kThreads : k > 8 ? (T <= 4096 ? kMaxThreads : 512) : hv <= 512 ? kThreads : 512;
    const int turns = (hv + most - 1) / most;
    return waves((hv + turns - 1) / turns);
}

}  // namespace
}  // namespace metro

extern "C" int moe_unpermute(const void* y_perm, const int32_t* pair_row, const float* topk_w, int T, int k, int H,
                             int dtype, void* out, void* stream) {
    using namespace metro;
    if (!y_perm || !pair_row || !topk_w || !out) return METRO_ERR_INVALID_ARG;
    if (T < 0 || k < 1 || H < 1) return METRO_ERR_INVALID_ARG;
    if (dtype != METRO_DTYPE_BF16 && dtype != METRO_DTYPE_F32) return METRO_ERR_UNSUPPORTED;
    if ((int64_t)T * k >= (1 << 24)) return METRO_ERR_UNSUPPORTED;
    if (T == 0) return METRO_OK;
    hipStream_t st = (hipStream_t)stream;
    const bool aligned = (((uintptr_t)y_perm | (uintptr_t)out) & 15) == 0;
    const bool bf16 = dtype == METRO_DTYPE_BF16;
    const int per = bf16 ? 8 : 4;                 // columns of a 16-byte vector
    auto vec = [&](auto kernel) {
        const int hv = H / per;
        hipLaunchKernelGGL(kernel, dim3(T), dim3(row_threads(T, k, hv)), 0, st, (const uint4*)y_perm, pair_row, topk_w, k, hv,
                           (uint4*)out);
    };
    if (H % per == 0 && aligned) {
        if (bf16 && k <= 8) vec(unpermute_vec_kernel<true, 8>);
        else if (bf16) vec(unpermute_vec_kernel<true, 0>);
        else if (k <= 2) vec(unpermute_vec_kernel<false, 2>);          // 8192 tokens x 64, k = 1: 3.8 us, 4.4 with slots for eight
        else if (k <= 8) vec(unpermute_vec_kernel<false, 8>);
        else vec(unpermute_vec_kernel<false, 0>);
    } else if (bf16) {
        hipLaunchKernelGGL(unpermute_scalar_kernel<true>, dim3(T), dim3(kThreads), 0, st, y_perm, pair_row, topk_w,
                           k, H, out);
    } else {
        hipLaunchKernelGGL(unpermute_scalar_kernel<false>, dim3(T), dim3(kThreads), 0, st, y_perm, pair_row, topk_w,
                           k, H, out);
    }
    return hipGetLastError() == hipSuccess ? METRO_OK : METRO_ERR_HIP;
}

extern "C" const char* metro_status_string(int status) {
    switch (status) {
        case METRO_OK: return "ok";
        case METRO_ERR_INVALID_ARG: return "invalid argument";
        case METRO_ERR_UNSUPPORTED: return "size or dtype beyond the supported limits";
        case METRO_ERR_WORKSPACE: return "workspace too small";
        case METRO_ERR_HIP: return "HIP launch failed";
        case METRO_ERR_TOO_LARGE: return "problem larger than the library's built-in scratch buffer";
        default: return "unknown status";
    }
}
