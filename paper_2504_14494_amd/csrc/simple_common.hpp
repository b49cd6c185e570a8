// What the kernels of the per-node network compute alike: ReLU on packed BF16,
// the moments of a node, the network over a wave's 64 nodes and the corrected
// collision.
#pragma once

#include "channel_common.hpp"
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

// Eq. 3 with the projected correction at one node, given its moments (with
// Guo's velocity where there is a force).  The sigmoid and the relaxation rate use the
// hardware exp2 and reciprocal (about 1 ulp each); z0 = 0 still gives
// tau_adj = 1 exactly (2^0 = 1, 1/2 = 0.5).  FORCED: under the channel's body
// force rho * gx, f^eq is taken at Guo's velocity and Guo's source is added at
// the effective rate omega = 1 / (tau tau_adj).
template <bool FORCED>
__device__ __forceinline__ void collide(float (&g)[9], const float (&z)[NOUT], float tau,
                                        float sdelta, float gx, lbm::Moments<float> M) {
#pragma clang fp contract(off)
  M.uu = FORCED ? __builtin_fmaf(M.v, M.v, M.u * M.u) : __builtin_fmaf(M.u, M.u, M.v * M.v);
  M.diag = M.u + M.v;
  M.anti = M.v - M.u;
  constexpr float kLog2e = 1.4426950408889634f;
  float sig = __builtin_amdgcn_rcpf(1.0f + __builtin_amdgcn_exp2f(-z[0] * kLog2e));
  float tau_adj = 0.5f + sig;
  float omega = __builtin_amdgcn_rcpf(tau * tau_adj);
  const float fx = M.rho * gx, src_scale = __builtin_fmaf(-0.5f, omega, 1.0f);
  const Projection P(z);
#pragma unroll
  for (int i = 0; i < 9; ++i) {
    float relaxed = lbm::relax(g[i], lbm::geq_of(i, M), omega);
    if constexpr (FORCED)
      relaxed = __builtin_fmaf(src_scale, lbm::guo_source<float>(i, fx, M), relaxed);
    g[i] = __builtin_fmaf(sdelta, P(i, z), relaxed);
  }
}

constexpr int kSlot = 12;   // dwords per node: 8 for the features, then 10 head outputs
constexpr int kStepFrags = 14;   // W1 (4), W2 (8), Wh (2)
constexpr int kStepBias = 9;     // b1 (4), b2 (4), bh (1), per channel group

// Brings the weight and bias fragments of the step to LDS (then a barrier).
__device__ __forceinline__ void load_network(const uint8_t *__restrict__ pack, const FragLayout &F,
                                             u32x4 *w_s, f32x4 *b_s) {
  const u32x4 *frags = (const u32x4 *)(pack + F.frag_off);
  const f32x4 *bias = (const f32x4 *)(pack + F.bias_off);
  for (int k = threadIdx.x; k < kStepFrags * 64; k += blockDim.x) {
    int f = k >> 6, l = k & 63;
    int src_f = f < 4 ? F.W1 + f : (f < 12 ? F.W2 + (f - 4) : F.WH + (f - 12));
    w_s[k] = frags[(size_t)src_f * 64 + l];
  }
  // a bias fragment holds rows 4q..4q+3 for every node column: lane 16 q
  if (threadIdx.x < kStepBias * 4) {
    int b = threadIdx.x >> 2, g = threadIdx.x & 3;
    int src_b = b < 4 ? F.B1 + b : (b < 8 ? F.B2 + (b - 4) : F.BH);
    b_s[threadIdx.x] = bias[(size_t)src_b * 64 + 16 * g];
  }
}

// Normalised features of a node into its slot (16 BF16, the last four zero).
__device__ __forceinline__ void put_features(uint32_t *slot, const float (&g)[9],
                                             const lbm::Moments<float> &M,
                                             const float (&isg)[NFEAT],
                                             const float (&nmi)[NFEAT]) {
  const float raw[NFEAT] = {g[0], g[1], g[2], g[3],   g[4], g[5],
                            g[6], g[7], g[8], M.drho, M.u,  M.v};
  float ft[NFEAT];
#pragma unroll
  for (int k = 0; k < NFEAT; ++k) ft[k] = fmaf(raw[k], isg[k], nmi[k]);
  u32x4 *o = (u32x4 *)slot;
  o[0] = u32x4{pack_bf16(ft[0], ft[1]), pack_bf16(ft[2], ft[3]), pack_bf16(ft[4], ft[5]),
               pack_bf16(ft[6], ft[7])};
  o[1] = u32x4{pack_bf16(ft[8], ft[9]), pack_bf16(ft[10], ft[11]), 0u, 0u};
}

// Head outputs of a node from its slot.
__device__ __forceinline__ void get_head(const uint32_t *slot, float (&z)[NOUT]) {
  const f32x4 *zs = (const f32x4 *)slot;
  const f32x4 z0 = zs[0], z1 = zs[1], z2 = zs[2];
  const float zz[12] = {z0.x, z0.y, z0.z, z0.w, z1.x, z1.y, z1.z, z1.w, z2.x, z2.y, z2.z, z2.w};
#pragma unroll
  for (int k = 0; k < NOUT; ++k) z[k] = zz[k];
}

// The network over the 64 nodes of a wave's slots `sw`: features in, head
// outputs out.
__device__ __forceinline__ void network(const u32x4 *w_s, const f32x4 *b_s, uint32_t *sw,
                                        int lane) {
  const int n = lane & 15, q = lane >> 4;
  // Two column blocks of 16 nodes at a time: each weight and bias fragment
  // read from LDS serves both (half the LDS reads of one block at a time).
#pragma unroll 2
  for (int pair = 0; pair < 2; ++pair) {
    int wo = lane;
    asm volatile("" : "+v"(wo));
    const u32x4 *w = w_s + wo;
    const f32x4 *bs = b_s + q;
    uint32_t *slot[2];
    u32x4 xb[2];
#pragma unroll
    for (int h = 0; h < 2; ++h) {
      slot[h] = sw + (16 * (2 * pair + h) + n) * kSlot;
      xb[h] = q < 2 ? *(const u32x4 *)(slot[h] + 4 * q) : u32x4{0u, 0u, 0u, 0u};
    }
    f32x4 a[2][4];
#pragma unroll
    for (int t = 0; t < 4; ++t) {
      const u32x4 wt = w[t * 64];
      const f32x4 bt = bs[t * 4];
#pragma unroll
      for (int h = 0; h < 2; ++h) a[h][t] = mfma(wt, xb[h], bt);
    }
    u32x4 e1[2][2];
#pragma unroll
    for (int h = 0; h < 2; ++h) {
      e1[h][0] = relu_frag(a[h][0], a[h][1]);
      e1[h][1] = relu_frag(a[h][2], a[h][3]);
    }
#pragma unroll
    for (int t = 0; t < 4; ++t) {
      const u32x4 w0 = w[(4 + 2 * t) * 64], w1 = w[(5 + 2 * t) * 64];
      const f32x4 bt = bs[(4 + t) * 4];
#pragma unroll
      for (int h = 0; h < 2; ++h) a[h][t] = mfma(w1, e1[h][1], mfma(w0, e1[h][0], bt));
    }
    u32x4 hb[2][2];
#pragma unroll
    for (int h = 0; h < 2; ++h) {
      hb[h][0] = relu_frag(a[h][0], a[h][1]);
      hb[h][1] = relu_frag(a[h][2], a[h][3]);
    }
    const u32x4 w12 = w[12 * 64], w13 = w[13 * 64];
    const f32x4 b8 = bs[8 * 4];
#pragma unroll
    for (int h = 0; h < 2; ++h) {
      const f32x4 z = mfma(w13, hb[h][1], mfma(w12, hb[h][0], b8));
      // the features of these 16 nodes are consumed (z depends on them):
      // their slots take the head outputs, rows 4q..4q+3
      if (q < 2) *(f32x4 *)(slot[h] + 4 * q) = z;
      else if (q == 2) *(float2 *)(slot[h] + 8) = float2{z.x, z.y};
    }
  }
}

}  // namespace simple
}  // namespace gnn
