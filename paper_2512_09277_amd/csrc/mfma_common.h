// Operand types of the matrix instructions and compile-time step loops.
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

#include <type_traits>
#include <utility>

namespace metro {
namespace {

typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef float floatx4 __attribute__((ext_vector_type(4)));
typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));
typedef uint32_t u32x2 __attribute__((ext_vector_type(2)));
typedef int i32x4 __attribute__((ext_vector_type(4)));

// do_step(U, s) for U = 0..n-1 with compile-time U (buffer indices), s = s0 + U.
template <int... Us, typename F>
__device__ __forceinline__ void run_steps(std::integer_sequence<int, Us...>, F&& f, int s0) {
    (f(std::integral_constant<int, Us>{}, s0 + Us), ...);
}
template <int... Us, typename F>
__device__ __forceinline__ void run_steps_tail(std::integer_sequence<int, Us...>, F&& f, int s0, int n_steps) {
    // short-circuit: once a step is past the end nothing after it is tested, the paths join only at the end
    (void)((s0 + Us < n_steps && (f(std::integral_constant<int, Us>{}, s0 + Us), true)) && ...);
}

}  // namespace
}  // namespace metro
