// What the per-node network's step and its backward pass compute alike: ReLU
// on packed BF16 and the moments of a node.
#pragma once

#include "gnn_common.hpp"
#include "lbm_common.hpp"

namespace gnn {
namespace simple {

typedef short s16x2 __attribute__((ext_vector_type(2)));

// ReLU of eight accumulators, rounded to a BF16 B-operand fragment.  Rounding
// keeps the sign, so ReLU after rounding equals rounding after ReLU; on the
// packed BF16 bits ReLU is a signed 16-bit max with zero (negative values,
// -0 included, have the sign bit set), two values per instruction.
__device__ __forceinline__ uint32_t relu_bf16x2(uint32_t v) {
  s16x2 h = __builtin_bit_cast(s16x2, v);
  h = __builtin_elementwise_max(h, s16x2{0, 0});
  return __builtin_bit_cast(uint32_t, h);
}

__device__ __forceinline__ u32x4 relu_frag(f32x4 lo, f32x4 hi) {
  u32x4 r = frag_from_acc(lo, hi);
  return u32x4{relu_bf16x2(r.x), relu_bf16x2(r.y), relu_bf16x2(r.z), relu_bf16x2(r.w)};
}

// Moments of a node, as lbm::node_moments (same sums, same order) but with
// the hardware reciprocal of rho (about 1 ulp); what only the collision needs
// is left to it.
__device__ __forceinline__ lbm::Moments<float> moments(const float (&g)[9]) {
#pragma clang fp contract(off)
  lbm::Moments<float> M = {};
  M.drho = ((g[0] + (g[1] + g[3])) + (g[2] + g[4])) + ((g[5] + g[7]) + (g[6] + g[8]));
  M.jx = (g[1] - g[3]) + ((g[5] - g[7]) + (g[8] - g[6]));
  M.jy = (g[2] - g[4]) + ((g[5] - g[7]) + (g[6] - g[8]));
  M.rho = 1.0f + M.drho;
  M.inv = __builtin_amdgcn_rcpf(M.rho);
  M.u = M.jx * M.inv;
  M.v = M.jy * M.inv;
  return M;
}

}  // namespace simple
}  // namespace gnn
