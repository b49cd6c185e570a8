// Backward pass of the per-node network of Fig. 2 (n_rounds = 0) in one
// kernel: with no neighbours in between, a node's gradient goes from the head
// through both layers without leaving the wave.
//
// The activations are recomputed from the populations, with the arithmetic of
// the forward step (so they are the same BF16 values), instead of being
// stored by the forward pass and read back: 314 bytes per node each way against
// 12 MFMAs per 16 nodes.  Only z_0, which the gradient of the rate needs before
// the layers, is kept.  Per node, 76 bytes are read and nothing is written.
//   dz from dL/dg_post, dh = Wh^T dz, dp2 = dh . [p2 > 0],
//   dp1 = (W2^T dp2) . [p1 > 0];  dWh = dz h^T, dW2 = dp2 e^T, dW1 = dp1 x^T
// Per-node work (moments, features, dz) runs one node per lane; the layers run
// on MFMA, 16 nodes at a time.  The weight gradients contract over nodes: the 32
// columns of a chunk (two groups of 16 nodes) are staged transposed in LDS.  A
// wave takes two of its chunks per turn, which fills its lanes, and keeps the
// order of the chunk-by-chunk walk of the message-passing kernels, so each
// wave's partial, and their sum in wave order, is reproducible bit by bit.
//
// 32 lattices of 128^2: head and encoder kernels on stored activations took 141
// us and the storing forward 41; this kernel takes 67 and the plain forward 22.
// One wave per SIMD (the order of the sums fixes 1024 waves): a turn of two
// chunks takes 15,000 cycles for some 1,500 VALU instructions, the rest is the
// latency of its chain of layers and of the transposition.  (Whole-dword staging,
// two nodes per write, changed nothing.)
#include "bwd_common.hpp"
#include "simple_common.hpp"

namespace gnn {
namespace simple {

struct BwdWave {
  uint32_t x[64 * 8];             // normalised features (16 BF16) per node
  uint32_t dz[64 * 8];            // dz (16 BF16) per node
  float dzf[64 * 12];             // dz in FP32, for dbh
  uint16_t d_z[16 * kPitch], d_2[64 * kPitch], d_1[64 * kPitch];  // gradients, channel-major
  uint16_t a_h[64 * kPitch], a_e[64 * kPitch], a_x[16 * kPitch];  // activations
};
// A factor rather than a choice: a gradient that is not finite stays so in the units
// that are off, too.
__device__ __forceinline__ f32x4 relu_grad(f32x4 p) {
  return f32x4{p.x > 0.0f ? 1.0f : 0.0f, p.y > 0.0f ? 1.0f : 0.0f, p.z > 0.0f ? 1.0f : 0.0f,
               p.w > 0.0f ? 1.0f : 0.0f};
}

constexpr int kBwdFrags = 24;     // W1 4, W2 8, W2^T 8, Wh^T 4

__global__ __launch_bounds__(kBT) void simple_backward_kernel(
    const float *__restrict__ G, const float *__restrict__ gpre, const float *__restrict__ tau,
    const float *__restrict__ z0, int batch, int nx, int ny, const float *__restrict__ params, BlobLayout L,
    float *__restrict__ part) {
  __shared__ u32x4 w_s[kBwdFrags * 64];
  __shared__ f32x4 b_s[8 * 4];     // b1 (4), b2 (4) per channel group
  __shared__ __attribute__((aligned(16))) BwdWave waves[4];
  const int lane = threadIdx.x & 63;
  const int wave = __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
  const int n = lane & 15, q = lane >> 4;
  const float *cst = params + L.mu;
  // The fragments straight from the parameters, as gnn_prep_kernel packs them: a
  // launch of its own costs more than its 24 of them here (161.5 -> 158.1 us a
  // training step of 32 lattices of 128^2).  Value k of a row lies at base + stride
  // k; rows of lim values (0: HID, in fragment order) are padded with zeros.
#pragma unroll
  for (int i = 0; i < kBwdFrags / 4; ++i) {
    const int f = 4 * i + wave;
    const int t = f < 4 ? f : f < 12 ? (f - 4) >> 1 : f < 20 ? (f - 12) >> 1 : f - 20;
    const int row = 16 * t + n, s = f & 1;
    const bool transposed = f >= 12;
    const size_t base = f < 4    ? L.W1 + (size_t)row * NFEAT
                        : f < 12 ? L.W2 + (size_t)row * HID
                                 : (f < 20 ? L.W2 : L.Wh) + row;
    const int stride = transposed ? HID : 1, lim = f < 4 ? NFEAT : f < 20 ? 0 : NOUT;
    float x[8];
#pragma unroll
    for (int j = 0; j < 8; ++j) {
      const int k = lim ? 8 * q + j : frag_channel(s, q, j);
      const bool in = !lim || k < lim;
      const float v = params[base + (size_t)(in ? stride * k : 0)];
      x[j] = in ? v : 0.0f;
    }
    w_s[f * 64 + lane] = u32x4{pack_bf16(x[0], x[1]), pack_bf16(x[2], x[3]),
                               pack_bf16(x[4], x[5]), pack_bf16(x[6], x[7])};
  }
  if (threadIdx.x < 8 * 4) {
    const int b = threadIdx.x >> 2;
    const float *src = params + (b < 4 ? L.b1 + 16 * b : L.b2 + 16 * (b - 4)) + 4 * (threadIdx.x & 3);
    b_s[threadIdx.x] = f32x4{src[0], src[1], src[2], src[3]};
  }
  const float sdelta = cst[C_SDELTA];
  float isg[NFEAT], nmi[NFEAT];
#pragma unroll
  for (int k = 0; k < NFEAT; ++k) {
    isg[k] = 1.0f / cst[C_SIGMA + k];
    nmi[k] = -cst[C_MU + k] * isg[k];
  }
  __syncthreads();
  BwdWave &S = waves[wave];

  const int gxn = (nx + 15) / 16, ngroups = batch * ny * gxn, nchunks = (ngroups + 1) / 2;
  const int wv = blockIdx.x * 4 + wave;
  f32x4 acc_h[1][4] = {}, acc_2[4][4] = {}, acc_1[4][1] = {};
  f32x4 s1[4] = {}, s2[4] = {};
  f32x4 bsum = {};                 // lane (n, q): dz[4 q ..] of column n
  float g_nx[9], G_nx[9], t_nx, z_nx;
  // This lane's node of chunks c (lanes 0-31) and c + kBwdWaves (32-63); groups
  // of a row, then rows (fewer than 2^31 nodes keep all of it in 32 bits).
  bool valid_nx = false;
  auto prefetch = [&](int c) {
    const unsigned grp = 2u * (unsigned)(c + (lane >> 5) * kBwdWaves) + ((lane >> 4) & 1);
    const bool in = grp < (unsigned)ngroups;
    const unsigned gi = in ? grp : 0u, row = gi / (unsigned)gxn;
    const unsigned x = (gi - row * (unsigned)gxn) * 16 + n;
    valid_nx = in && x < (unsigned)nx;
    const size_t base = (size_t)row * 9 * nx + (x < (unsigned)nx ? x : nx - 1);
#pragma unroll
    for (int i = 0; i < 9; ++i) {
      g_nx[i] = gpre[base + (size_t)i * nx];
      G_nx[i] = G[base + (size_t)i * nx];
    }
    t_nx = tau[row / (unsigned)ny];
    z_nx = z0[(size_t)row * nx + (x < (unsigned)nx ? x : nx - 1)];
  };
  constexpr int kTurn = 2 * kBwdWaves;
  if (wv < nchunks) prefetch(wv);
  for (int c = wv; c < nchunks; c += kTurn) {
    const bool valid = valid_nx;
    float dz[NOUT];
    const float tb = t_nx, z0c = z_nx;
    {
      float g[9], Gi[9];
#pragma unroll
      for (int i = 0; i < 9; ++i) {
        g[i] = g_nx[i];
        Gi[i] = G_nx[i];
      }
      if (c + kTurn < nchunks) prefetch(c + kTurn);
      put_features(S.x + lane * 8, g, moments(g), isg, nmi);
      head_gradient(g, Gi, sdelta, dz);
    }
    wave_lds_sync();
    // the forward layers of a chunk's two groups of 16 nodes
    int wo = lane;
    asm volatile("" : "+v"(wo));
    const u32x4 *w = w_s + wo;
    const f32x4 *bs = b_s + q;
    auto features = [&](int grp) {
      return q < 2 ? *(const u32x4 *)(S.x + (16 * grp + n) * 8 + 4 * q) : u32x4{0u, 0u, 0u, 0u};
    };
    auto layer1 = [&](const u32x4(&xb)[2], f32x4(&p)[2][4], u32x4(&e)[2][2]) {
#pragma unroll
      for (int t = 0; t < 4; ++t) {
        const u32x4 wt = w[t * 64];
        const f32x4 bt = bs[t * 4];
#pragma unroll
        for (int h = 0; h < 2; ++h) p[h][t] = mfma(wt, xb[h], bt);
      }
#pragma unroll
      for (int h = 0; h < 2; ++h) {
        e[h][0] = relu_frag(p[h][0], p[h][1]);
        e[h][1] = relu_frag(p[h][2], p[h][3]);
      }
    };
    auto layer2 = [&](const u32x4(&e)[2][2], f32x4(&p)[2][4], u32x4(&hf)[2][2]) {
#pragma unroll
      for (int t = 0; t < 4; ++t) {
        const u32x4 w0 = w[(4 + 2 * t) * 64], w1 = w[(5 + 2 * t) * 64];
        const f32x4 bt = bs[(4 + t) * 4];
#pragma unroll
        for (int h = 0; h < 2; ++h) p[h][t] = mfma(w1, e[h][1], mfma(w0, e[h][0], bt));
      }
#pragma unroll
      for (int h = 0; h < 2; ++h) {
        hf[h][0] = relu_frag(p[h][0], p[h][1]);
        hf[h][1] = relu_frag(p[h][2], p[h][3]);
      }
    };
    {
      dz[0] = tau_gradient(dz[0], z0c, tb);
#pragma unroll
      for (int k = 0; k < NOUT; ++k) {
        dz[k] = valid ? dz[k] : 0.0f;
      }
      f32x4 *of = (f32x4 *)(S.dzf + lane * 12);
      of[0] = f32x4{dz[0], dz[1], dz[2], dz[3]};
      of[1] = f32x4{dz[4], dz[5], dz[6], dz[7]};
      of[2] = f32x4{dz[8], dz[9], 0.0f, 0.0f};
      u32x4 *o = (u32x4 *)(S.dz + lane * 8);
      o[0] = u32x4{pack_bf16(dz[0], dz[1]), pack_bf16(dz[2], dz[3]), pack_bf16(dz[4], dz[5]),
                   pack_bf16(dz[6], dz[7])};
      o[1] = u32x4{pack_bf16(dz[8], dz[9]), 0u, 0u, 0u};
    }
    wave_lds_sync();
    const int turns = c + kBwdWaves < nchunks ? 2 : 1;
#pragma unroll 1
    for (int pair = 0; pair < turns; ++pair) {
      const u32x4 xb[2] = {features(2 * pair), features(2 * pair + 1)};
#pragma unroll
      for (int h = 0; h < 2; ++h)
        if (q < 3) bsum += *(const f32x4 *)(S.dzf + (16 * (2 * pair + h) + n) * 12 + 4 * q);
      u32x4 dzb[2];
#pragma unroll
      for (int h = 0; h < 2; ++h)
        dzb[h] = q < 2 ? *(const u32x4 *)(S.dz + (16 * (2 * pair + h) + n) * 8 + 4 * q)
                       : u32x4{0u, 0u, 0u, 0u};
      f32x4 p1[2][4], p2[2][4];
      u32x4 e[2][2], hf[2][2];
      layer1(xb, p1, e);
      layer2(e, p2, hf);
      u32x4 dpb[2][2];
      {
        f32x4 o[2][4];
#pragma unroll
        for (int t = 0; t < 4; ++t) {
          const u32x4 wt = w[(20 + t) * 64];
#pragma unroll
          for (int h = 0; h < 2; ++h) {
            o[h][t] = mfma(wt, dzb[h], f32x4{0.0f, 0.0f, 0.0f, 0.0f});
            o[h][t] *= relu_grad(p2[h][t]);
            s2[t] += o[h][t];
          }
        }
#pragma unroll
        for (int h = 0; h < 2; ++h) {
          dpb[h][0] = frag_from_acc(o[h][0], o[h][1]);
          dpb[h][1] = frag_from_acc(o[h][2], o[h][3]);
        }
      }
      u32x4 dpa[2][2];
      {
        f32x4 o[2][4];
#pragma unroll
        for (int t = 0; t < 4; ++t) {
          const u32x4 w0 = w[(12 + 2 * t) * 64], w1 = w[(13 + 2 * t) * 64];
#pragma unroll
          for (int h = 0; h < 2; ++h) {
            o[h][t] = mfma(w1, dpb[h][1], mfma(w0, dpb[h][0], f32x4{0.0f, 0.0f, 0.0f, 0.0f}));
            o[h][t] *= relu_grad(p1[h][t]);
            s1[t] += o[h][t];
          }
        }
#pragma unroll
        for (int h = 0; h < 2; ++h) {
          dpa[h][0] = frag_from_acc(o[h][0], o[h][1]);
          dpa[h][1] = frag_from_acc(o[h][2], o[h][3]);
        }
      }
#pragma unroll
      for (int h = 0; h < 2; ++h) {
        stage_frag(S.a_h, hf[h], q, 16 * h + n);
        stage_frag(S.d_2, dpb[h], q, 16 * h + n);
        stage_frag(S.a_e, e[h], q, 16 * h + n);
        stage_frag(S.d_1, dpa[h], q, 16 * h + n);
        stage_rows16(S.a_x, xb[h], q, 16 * h + n);
        stage_rows16(S.d_z, dzb[h], q, 16 * h + n);
      }
      wave_lds_sync();
      dw_mma<1, 4>(acc_h, S.d_z, S.a_h, lane);
      dw_mma<4, 4>(acc_2, S.d_2, S.a_e, lane);
      dw_mma<4, 1>(acc_1, S.d_1, S.a_x, lane);
      wave_lds_sync();
    }
  }

  float *pw = part + (size_t)wv * L.nparam;
  float *red = (float *)S.x;  // the per-node buffers are done with
  static_assert(offsetof(BwdWave, d_z) >= 64 * 17 * sizeof(float), "vector sums fit");
  write_dw<1, 4>(pw, L.Wh, HID, 0, NOUT, HID, acc_h, lane);
  write_dw<4, 4>(pw, L.W2, HID, 0, HID, HID, acc_2, lane);
  write_dw<4, 1>(pw, L.W1, NFEAT, 0, HID, NFEAT, acc_1, lane);
  write_vec(pw, L.b2, 1, s2, red, lane);
  write_vec(pw, L.b1, 1, s1, red, lane);
  const float bs4[4] = {bsum.x, bsum.y, bsum.z, bsum.w};
#pragma unroll
  for (int e = 0; e < 4; ++e) red[n * 17 + 4 * q + e] = bs4[e];
  wave_lds_sync();
  if (lane < NOUT) {
    float s = 0.0f;
    for (int m = 0; m < 16; ++m) s += red[m * 17 + lane];
    pw[L.bh + lane] = s;
  }
}

}  // namespace simple

int launch_simple_backward(const float *G, const float *g_pre, const float *tau, const float *z0,
                           int batch, int nx, int ny, const float *params, float *part,
                           hipStream_t s) {
  const BlobLayout L = blob_layout(0);
  hipLaunchKernelGGL(simple::simple_backward_kernel, dim3(kBwdBlocks), dim3(kBT), 0, s, G, g_pre,
                     tau, z0, batch, nx, ny, params, L, part);
  return lbm::launch_check("simple_backward_kernel");
}

}  // namespace gnn
