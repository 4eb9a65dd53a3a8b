// Matrix-core and memory primitives shared by the dense scoring kernels.
#pragma once

#include <hip/hip_runtime.h>

#include "oprag_internal.h"

namespace oprag {
namespace dev {

typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef _Float16 f16x8 __attribute__((ext_vector_type(8)));
typedef float f32x4 __attribute__((ext_vector_type(4)));
typedef unsigned int u32x4 __attribute__((ext_vector_type(4)));

template <int DT>
struct Mfma;
template <>
struct Mfma<kDtypeBF16> {
  typedef bf16x8 V;
  typedef __bf16 T;
  static __device__ __forceinline__ f32x4 run(V a, V b, f32x4 c) {
    return __builtin_amdgcn_mfma_f32_16x16x32_bf16(a, b, c, 0, 0, 0);
  }
};
template <>
struct Mfma<kDtypeF16> {
  typedef f16x8 V;
  typedef _Float16 T;
  static __device__ __forceinline__ f32x4 run(V a, V b, f32x4 c) {
    return __builtin_amdgcn_mfma_f32_16x16x32_f16(a, b, c, 0, 0, 0);
  }
};

// fp32: a 16-byte fragment holds four dimensions per lane; element e of every lane forms one
// depth-4 product (the dimensions are permuted alike in both operands).
template <>
struct Mfma<kDtypeF32> {
  typedef f32x4 V;
  typedef float T;
  static __device__ __forceinline__ f32x4 run(V a, V b, f32x4 c) {
#pragma unroll
    for (int e = 0; e < 4; ++e) c = __builtin_amdgcn_mfma_f32_16x16x4f32(a[e], b[e], c, 0, 0, 0);
    return c;
  }
};

// Workgroup barrier after which every wave's LDS traffic so far is complete; global loads stay
// in flight (a __syncthreads() fence would drain them).
__device__ __forceinline__ void lds_barrier() { asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory"); }

constexpr float kNegInf = -__builtin_inff();

// Logical workgroup index with consecutive indices kept on one XCD (the hardware deals
// workgroups round-robin over the 8 XCDs), so the query blocks of one row chunk share an L2:
// XCD x takes the x-th run of G / 8 (the first G % 8 of them one more) consecutive indices.
__device__ __forceinline__ long long logical_block() {
  const unsigned g = blockIdx.x, G = gridDim.x;
  const unsigned x = g % 8, q = G / 8, r = G % 8;
  return (long long)(x * q + min(x, r) + g / 8);
}

}  // namespace dev
}  // namespace oprag
