// What the matrix-core kernels share (read-out tiles and the products of its gradient): products whose accumulators take all of a
// wavefront's accumulation registers, and loops whose index is a constant.
#pragma once

#include "device_utils.h"

#include <type_traits>
#include <utility>

namespace ais {
namespace tile {

using dev::u32x4;

typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef float f32x4 __attribute__((ext_vector_type(4)));

// The products are written as instructions because the accumulators take all of the accumulation registers: the compiler's own
// form of a product may have its result elsewhere than its addend, and without a register to spare it moved fragments and
// accumulators about in the loop.  It does not know what such a statement is, so what it would wait for is waited for here:
//   fragments come straight from LDS reads, whose arrival it does wait for (an operand that an ordinary instruction has just
//   written would need two wait states; there is none in the loop);
//   settle() stands between the last product and the first look at an accumulator.
__device__ __forceinline__ void multiply(f32x4& c, bf16x8 a, bf16x8 b) {
  asm volatile("v_mfma_f32_16x16x32_bf16 %0, %1, %2, %0" : "+a"(c) : "v"(a), "v"(b));
}
__device__ __forceinline__ void settle() { asm volatile("s_nop 15\n\ts_nop 3"); }
// c = 0, by the matrix pipe, which has nothing else to do between two tiles: beside the soft-max arithmetic of the finished
// one.  Where the accumulators have not held anything before, `first` makes them do so.
struct Clear {
  u32x4 zero;
  __device__ __forceinline__ Clear() {
    zero = u32x4{0u, 0u, 0u, 0u};
    asm volatile("s_nop 3" : "+v"(zero));
  }
  __device__ __forceinline__ void operator()(f32x4& c) const {
    asm volatile("v_mfma_f32_16x16x32_bf16 %0, %1, %1, 0" : "+a"(c) : "v"(zero));
  }
  __device__ __forceinline__ void first(f32x4& c) const {
    asm volatile("v_mfma_f32_16x16x32_bf16 %0, %1, %1, 0" : "=a"(c) : "v"(zero));
  }
};

// f(0), f(1), ... f(N - 1) with the index a constant in each.
template <typename F, int... I>
__device__ __forceinline__ void unrolled_over(F&& f, std::integer_sequence<int, I...>) {
  (f(std::integral_constant<int, I>{}), ...);
}
template <int N, typename F>
__device__ __forceinline__ void unrolled(F&& f) {
  unrolled_over(f, std::make_integer_sequence<int, N>{});
}

}  // namespace tile
}  // namespace ais
