// Backward pass of the GNN-corrected collision and the pieces of one
// training step (paper: Training Methodology, loss of Eq. 4): gradient of a
// scalar loss with respect to every trainable parameter, the MSE loss and an
// Adam update.  n_rounds >= 1 is the message-passing network (GELU);
// n_rounds = 0 the per-node network of Fig. 2 (ReLU, simple_backward.hip).
//
// The forward saved, per node, the BF16 values the MFMAs consumed: features
// x, first encoder layer e1, node states h_0..h_R and summed messages a_1..a_R,
// plus the FP32 head outputs z.  BF16 rounding is differentiated as the
// identity.  Pre-activations are recomputed from those values.
//
// Per round r (h = h_r, h' = h_{r+1}, a = a_{r+1}), with p = Wn [h; a] + bn,
// q_{n,d} = Wa h_n + Wb h_{n+e_d} + Wc e_d + be and G = dL/dh':
//   dp = G . gelu'(p)                       dWn += dp [h; a]^T, dbn += dp
//   [dh ; da] = Wn^T dp
//   dq_{n,d} = da_n . gelu'(q_{n,d})        T_n = sum_d dq_{n,d}
//   dWa += T_n h_n^T, dbe += T_n, dWc += sum_d dq_{n,d} e_d^T, dh_n += Wa^T T_n
//   S_m = sum_d dq_{m-e_d,d}                dWb += S_m h_m^T,  dh_m += Wb^T S_m
// The sender sum S_m is a gather: dq is stored per edge (BF16) by the
// receiver-side kernel and read back by the sender-side kernel, so no
// gradient is ever scattered.
//
// Weight gradients are MFMA products with the node index as contraction
// dimension.  Each wave stages 32 nodes' gradient rows and activation rows
// transposed (channel-major, BF16) in its own LDS, accumulates dW over all
// the nodes it visits, and writes one FP32 partial per wave; a last kernel
// sums the partials of the fixed grid in a fixed order, so the gradient is
// bitwise reproducible.
#include "bwd_common.hpp"

namespace gnn {

// simple_backward.hip
int launch_simple_backward(const float *G, const float *g_pre, const float *tau, const float *z0,
                           int batch, int nx, int ny, const float *params, float *part,
                           hipStream_t s);

// The kernels below but the head's give two waves, on one SIMD, the chunks of one
// partial, each half of the 64 channels: every sum keeps the order it has with one
// wave, and a SIMD has two waves to issue from (a workgroup holds the four pairs
// of a CU; with one wave each these kernels waited 20 to 40 % of their time).
// What a product over all channels needs of the other half goes through LDS, a
// barrier per group.  A pair past the last chunk spends the turn at the barriers.
//
// 32 lattices of 128^2, one wave per partial and node-by-node buffers -> pairs and
// group planes (bwd_common.hpp): receiver 277 -> 225 us, sender 207 -> 189, node
// 135 -> 114, encoder 88 -> 77, head 76 -> 58 (planes only).  Moving 0.87, 1.0,
// 0.54, 0.22 and 0.24 GB, they take 135, 155, 83, 34 and 37 us at the rate of a
// large copy.
constexpr int kPairT = 2 * kBT;

// ------------------------------------------------------------ the head ---

// dz from dL/dg_post at each node, dh_R = Wh^T dz, dWh, dbh.
__global__ __launch_bounds__(kBT) void bwd_head_kernel(
    const float *__restrict__ G, const float *__restrict__ gpre, const float *__restrict__ tau,
    const float *__restrict__ save_z, const uint16_t *__restrict__ hR, int batch, int nx, int ny,
    const uint8_t *__restrict__ pack, FragLayout F, BlobLayout L, float *__restrict__ dh,
    float *__restrict__ part) {
  __shared__ Stage<16, 64> st[4];
  const int lane = threadIdx.x & 63;
  const unsigned wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int n = lane & 15, q = lane >> 4;
  Stage<16, 64> &S = st[wave];
  const u32x4 *frags = (const u32x4 *)(pack + F.frag_off);
  const float sdelta = ((const float *)(pack + F.const_off))[C_SDELTA];
  u32x4 wht[4];
#pragma unroll
  for (int t = 0; t < 4; ++t) wht[t] = load_frag(frags, F.WHT + t, lane);
  const unsigned gxn = (nx + 15) / 16, ngroups = (unsigned)batch * ny * gxn;
  const unsigned nchunks = (ngroups + 1) / 2;
  const unsigned w = blockIdx.x * 4 + wave;
  f32x4 acc[1][4] = {};
  float bsum[NOUT] = {};
  // One wave per SIMD: the next chunk's inputs (both groups) are loaded while
  // this chunk is computed.
  float g_nx[2][9], G_nx[2][9], z_nx[2], tau_nx[2];
  u32x4 hf_nx[2][2];
  auto prefetch = [&](unsigned cc) {
#pragma unroll
    for (int hh = 0; hh < 2; ++hh) {
      const Pos P = group_pos(2 * cc + hh, ngroups, n, nx, ny, gxn);
      const size_t lat = (size_t)P.b * ny * 9 * nx;
#pragma unroll
      for (int i = 0; i < 9; ++i) {
        g_nx[hh][i] = gpre[lat + lbm::pidx(nx, P.y, i, P.x)];
        G_nx[hh][i] = G[lat + lbm::pidx(nx, P.y, i, P.x)];
      }
      z_nx[hh] = save_z[P.node * 12];
      tau_nx[hh] = tau[P.b];
      load_frags(hR, P.node, q, hf_nx[hh]);
    }
  };
  if (w < nchunks) prefetch(w);
  for (unsigned c = w; c < nchunks; c += kBwdWaves) {
    float gc[2][9], Gc[2][9], zc[2], tauc[2];
    u32x4 hfc[2][2];
#pragma unroll
    for (int hh = 0; hh < 2; ++hh) {
#pragma unroll
      for (int i = 0; i < 9; ++i) {
        gc[hh][i] = g_nx[hh][i];
        Gc[hh][i] = G_nx[hh][i];
      }
      zc[hh] = z_nx[hh];
      tauc[hh] = tau_nx[hh];
      hfc[hh][0] = hf_nx[hh][0];
      hfc[hh][1] = hf_nx[hh][1];
    }
    if (c + kBwdWaves < nchunks) prefetch(c + kBwdWaves);
#pragma unroll
    for (unsigned half = 0; half < 2; ++half) {
      Pos P = group_pos(2 * c + half, ngroups, n, nx, ny, gxn);
      float(&g)[9] = gc[half];
      float(&Gi)[9] = Gc[half];
      float dz[NOUT];
      head_gradient(g, Gi, sdelta, dz);
      dz[0] = tau_gradient(dz[0], zc[half], tauc[half]);
      if (!P.valid)
#pragma unroll
        for (int k = 0; k < NOUT; ++k) dz[k] = 0.0f;
      // B operand: element j of lane group q is head output 8 q + j.
      float e8[8];
#pragma unroll
      for (int j = 0; j < 8; ++j) {
        float a0 = j < NOUT ? dz[j] : 0.0f;
        float a1 = j + 8 < NOUT ? dz[(j + 8) % NOUT] : 0.0f;
        e8[j] = q == 0 ? a0 : (q == 1 ? a1 : 0.0f);
      }
      const u32x4 dzb = {pack_bf16(e8[0], e8[1]), pack_bf16(e8[2], e8[3]),
                         pack_bf16(e8[4], e8[5]), pack_bf16(e8[6], e8[7])};
      f32x4 o[4];
#pragma unroll
      for (int t = 0; t < 4; ++t) o[t] = mfma(wht[t], dzb, f32x4{0.0f, 0.0f, 0.0f, 0.0f});
      store_acc(dh, P, n, q, o);
      const u32x4 hf[2] = {hfc[half][0], hfc[half][1]};
      const int col = 16 * half + n;
#pragma unroll
      for (int k = 0; k < NOUT; ++k)
        if ((k & 3) == q) S.d[k * kPitch + col] = bf16_bits(dz[k]);
      if (q < 2)
#pragma unroll
        for (int k = NOUT; k < 16; ++k)
          if ((k & 1) == q) S.d[k * kPitch + col] = 0;
      stage_frag(S.a, hf, q, col);
      if (q == 0)
#pragma unroll
        for (int k = 0; k < NOUT; ++k) bsum[k] += dz[k];
    }
    wave_lds_sync();
    dw_mma<1, 4>(acc, S.d, S.a, lane);
    wave_lds_sync();
  }
  float *pw = part + (size_t)w * L.nparam;
  write_dw<1, 4>(pw, L.Wh, HID, 0, NOUT, HID, acc, lane);
#pragma unroll
  for (int k = 0; k < NOUT; ++k) S.red[lane * 17 + k] = q == 0 ? bsum[k] : 0.0f;
  wave_lds_sync();
  if (lane < NOUT) {
    float s = 0.0f;
    for (int m = 0; m < 16; ++m) s += S.red[m * 17 + lane];
    pw[L.bh + lane] = s;
  }
}

// ------------------------------------------------------ node update, r ---

// dp, [dh; da] = Wn^T dp, dWn, dbn.  dh_out is overwritten.  Wave 0 of a pair
// forms and stores dh, wave 1 da.
__global__ __launch_bounds__(kPairT, 2) void bwd_node_kernel(
    const float *__restrict__ dh_in, const uint16_t *__restrict__ h, const uint16_t *__restrict__ agg,
    int batch, int nx, int ny, int r, const uint8_t *__restrict__ pack, FragLayout F,
    BlobLayout L, float *__restrict__ dh_out, float *__restrict__ dagg, float *__restrict__ part) {
  __shared__ Stage<64, 128> st[4];
  __shared__ u32x4 wn_s[16 * 64], wnt_s[16 * 64];
  __shared__ u32x4 x_s[4][2][2][64];  // pair, half, channels: dp as an operand
  const int lane = threadIdx.x & 63;
  const int wave = __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
  const int pair = wave & 3, hh = wave >> 2;
  const int n = lane & 15, q = lane >> 4;
  Stage<64, 128> &S = st[pair];
  const u32x4 *frags = (const u32x4 *)(pack + F.frag_off);
  const f32x4 *bias = (const f32x4 *)(pack + F.bias_off);
  for (int k = threadIdx.x; k < 16 * 64; k += kPairT) {
    wn_s[k] = frags[(size_t)F.WN[r] * 64 + k];
    wnt_s[k] = frags[(size_t)F.WNT[r] * 64 + k];
  }
  f32x4 bn[2];
#pragma unroll
  for (int t = 0; t < 2; ++t) bn[t] = load_bias(bias, F.BN[r] + 2 * hh + t, lane);
  __syncthreads();
  const unsigned gxn = (nx + 15) / 16, ngroups = (unsigned)batch * ny * gxn;
  const unsigned nchunks = (ngroups + 1) / 2;
  const unsigned w = blockIdx.x * 4 + pair;
  float *const d_out = hh ? dagg : dh_out;
  f32x4 acc[2][8] = {};
  f32x4 bsum[2] = {};
  // Each group's node state, aggregate and incoming gradient are loaded while
  // the previous group is computed.
  u32x4 hf_nx[2], af_nx[2];
  f32x4 G_nx[2];
  auto prefetch = [&](unsigned grp) {
    const Pos P = group_pos(grp, ngroups, n, nx, ny, gxn);
    load_frags(h, P.node, q, hf_nx);
    load_frags(agg, P.node, q, af_nx);
    load_acc(dh_in, P, n, q, G_nx, 2 * hh);
  };
  if (w < nchunks) prefetch(2 * w);
  for (unsigned c0 = blockIdx.x * 4; c0 < nchunks; c0 += kBwdWaves) {
    const unsigned c = c0 + pair;
    if (c >= nchunks) {
      for (int k = 0; k < 4; ++k) lds_barrier();
      break;
    }
#pragma unroll 1
    for (int half = 0; half < 2; ++half) {
      int wo = lane;
      asm volatile("" : "+v"(wo));
      const u32x4 *wn = wn_s + 8 * hh * 64 + wo, *wnt = wnt_s + 8 * hh * 64 + wo;
      const Pos P = group_pos(2 * c + half, ngroups, n, nx, ny, gxn);
      const u32x4 hf[2] = {hf_nx[0], hf_nx[1]}, af[2] = {af_nx[0], af_nx[1]};
      const f32x4 G[2] = {G_nx[0], G_nx[1]};
      if (half == 0 || c + kBwdWaves < nchunks)
        prefetch(half == 0 ? 2 * c + 1 : 2 * (c + kBwdWaves));
      f32x4 dp[2];
#pragma unroll
      for (int t = 0; t < 2; ++t) {
        f32x4 p = mfma(wn[(4 * t) * 64], hf[0], bn[t]);
        p = mfma(wn[(4 * t + 1) * 64], hf[1], p);
        p = mfma(wn[(4 * t + 2) * 64], af[0], p);
        p = mfma(wn[(4 * t + 3) * 64], af[1], p);
        dp[t] = P.valid ? G[t] * f32x4{gelu_grad(p.x), gelu_grad(p.y), gelu_grad(p.z),
                                       gelu_grad(p.w)}
                        : f32x4{0.0f, 0.0f, 0.0f, 0.0f};
        bsum[t] += dp[t];
      }
      lds_barrier();  // the products with the previous chunk's columns are done
      const int col = 16 * half + n;
      x_s[pair][half][hh][lane] = frag_from_acc(dp[0], dp[1]);
      stage_acc(S.d, dp, q, col, 32 * hh);
      const u32x4 own[2] = {hh ? af[0] : hf[0], hh ? af[1] : hf[1]};
      stage_frag(S.a, own, q, col, HID * hh);
      lds_barrier();
      const u32x4 dpb[2] = {x_s[pair][half][0][lane], x_s[pair][half][1][lane]};
      f32x4 o[4];
#pragma unroll
      for (int t = 0; t < 4; ++t) {
        o[t] = mfma(wnt[(2 * t) * 64], dpb[0], f32x4{0.0f, 0.0f, 0.0f, 0.0f});
        o[t] = mfma(wnt[(2 * t + 1) * 64], dpb[1], o[t]);
      }
      store_acc(d_out, P, n, q, o);
    }
    dw_mma<2, 8>(acc, S.d + 32 * hh * kPitch, S.a, lane);
  }
  lds_barrier();
  float *pw = part + (size_t)w * L.nparam;
  write_dw<2, 8>(pw, L.Wn[r] + (size_t)32 * hh * NODE_IN, NODE_IN, 0, 32, NODE_IN, acc, lane);
  write_vec_half(pw, L.bn[r], 1, hh, bsum, S.red, lane);
}

// --------------------------------------------- edge layer, receiver side ---

// Node states of one 16-receiver group and its ring (3 rows x 18 columns),
// staged in LDS: node ln = 18 hy + hx at byte 144 ln (128 B of state and 16
// B of padding, so that 16 lanes reading one 16-byte chunk of 16 consecutive
// nodes hit 16 disjoint groups of banks).  One direct-to-LDS load of a wave
// fills 64 16-byte slots, node ln's chunk c at slot 9 ln + c.
constexpr int kRingX = 18, kRingY = 3, kRingNodes = kRingX * kRingY;
constexpr int kRingNodeBytes = 144;
constexpr int kRingLoads = (kRingNodes * 9 + 63) / 64;
constexpr int kRingBytes = kRingLoads * 64 * 16;
// slot / 9 and node / 18 by multiply and shift, exact over the whole range
constexpr int kRingDiv9 = 7282, kRingDiv18 = 3641;
constexpr bool ring_divisions_exact() {
  for (int v = 0; v < kRingLoads * 64; ++v)
    if (((v * kRingDiv9) >> 16) != v / 9) return false;
  for (int v = 0; v < kRingNodes; ++v)
    if (((v * kRingDiv18) >> 16) != v / kRingX) return false;
  return true;
}
static_assert(kRingNodeBytes == 9 * 16 && ring_divisions_exact(), "ring staging");

// dq, BF16, lies by group of c columns like the FP32 vectors, in pieces of 64 bytes:
// (direction, half of the channels, column).  The sender side reads it one column
// to the left or right, so the unit it shares with the next group is one 64-byte
// piece, not one of 16 in each of 4 planes (send 194 us instead of 221 for 32
// lattices of 128^2; node by node, 207, and this kernel 15 % slower).
constexpr int kEdgeBytes = 8 * HID * 2;

// dq_{n,d} (stored BF16), T_n, dWa, dbe, dWc; Wa^T T_n over dL/dagg_n.
// 128 GELU derivatives per 16 receivers are 145 us of VALU work for 32 lattices of
// 128^2 (72 % of the cycles issue VALU).  The waves of a pair share the node
// states, each loading half of them, and exchange T, whose product with Wa^T runs
// over all channels.  While a pair works on one group of 16 receivers,
// direct-to-LDS loads bring the next group's node states and ring into its other
// LDS buffer, and the next group's dL/dagg rows come into registers.  A barrier
// per group publishes both; the wait before it leaves the group's stores, issued
// after those loads, in flight.
__global__ __launch_bounds__(kPairT, 2) void bwd_edge_recv_kernel(
    float *__restrict__ dagg_io, const uint16_t *__restrict__ h, int batch, int nx, int ny,
    int r, const uint8_t *__restrict__ pack, FragLayout F, BlobLayout L,
    uint16_t *__restrict__ dq_out, float *__restrict__ part) {
  const float *dagg = dagg_io;
  __shared__ Stage<64, 64> st[4];
  __shared__ u32x4 wa_s[8 * 64], wat_s[8 * 64];
  __shared__ f32x4 be_s[4 * 4];
  __shared__ u32x4 t_s[4][2][2][64];  // pair, half, channels: T as an operand
  __shared__ __attribute__((aligned(16))) uint8_t ring_s[4][2][kRingBytes];
  const int lane = threadIdx.x & 63;
  const int wave = __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
  const int pair = wave & 3, hh = wave >> 2;
  const int n = lane & 15, q = lane >> 4;
  Stage<64, 64> &S = st[pair];
  const u32x4 *frags = (const u32x4 *)(pack + F.frag_off);
  const f32x4 *bias = (const f32x4 *)(pack + F.bias_off);
  wa_s[threadIdx.x] = frags[(size_t)F.WA[r] * 64 + threadIdx.x];
  wat_s[threadIdx.x] = frags[(size_t)F.WAT[r] * 64 + threadIdx.x];
  static_assert(kPairT == 8 * 64, "one fragment entry per thread");
  u32x4 wb[2][2];
  uint32_t wc[2];
  if (threadIdx.x < 4 * 4)  // 16 lanes share a bias
    be_s[threadIdx.x] = bias[(size_t)(F.BE[r] + (threadIdx.x >> 2)) * 64 + 16 * (threadIdx.x & 3)];
#pragma unroll
  for (int t = 0; t < 2; ++t) {
    const int tt = 2 * hh + t;
    wb[t][0] = load_frag(frags, F.WB[r] + 2 * tt, lane);
    wb[t][1] = load_frag(frags, F.WB[r] + 2 * tt + 1, lane);
    wc[t] = load_frag(frags, F.WC[r] + tt, lane).x;
  }
  const unsigned gxn = (nx + 15) / 16, ngroups = (unsigned)batch * ny * gxn;
  const unsigned nchunks = (ngroups + 1) / 2;
  const unsigned w = blockIdx.x * 4 + pair;
  const bool narrow = nx < 16 || ny < 2;  // the ring wraps more than once

  // Issues this wave's loads of group `grp` (clamped as group_pos clamps it):
  // half of its ring into `buf` (direct to LDS, wrapped at the lattice edges;
  // slots past the last node repeat its last chunk) and its channels of the
  // dL/dagg rows into registers.
  auto prefetch = [&](unsigned grp, uint8_t *buf, f32x4(&da)[2]) {
    const Pos P = group_pos(grp, ngroups, n, nx, ny, gxn);
    const size_t lat_nodes = (size_t)P.b * ny * nx;
#pragma unroll
    for (int i = 0; i < kRingLoads / 2; ++i) {
      const int k = 2 * i + hh;
      const unsigned slot = 64 * k + lane;
      unsigned ln = __umul24(slot, kRingDiv9) >> 16;
      unsigned c = slot - 9 * ln;
      if (ln >= (unsigned)kRingNodes) {
        ln = kRingNodes - 1;
        c = 7;
      }
      c = c < 7 ? c : 7;
      const int hy = (int)(__umul24(ln, kRingDiv18) >> 16);
      const int hx = (int)ln - kRingX * hy;
      int gx = P.x0 - 1 + hx, gy = P.y - 1 + hy;
      gx = gx < 0 ? gx + nx : (gx >= nx ? gx - nx : gx);
      gy = gy < 0 ? gy + ny : (gy >= ny ? gy - ny : gy);
      if (narrow) {
        gx %= nx;
        gy %= ny;
      }
      const uint16_t *src = h + (lat_nodes + (size_t)gy * nx + gx) * HID + c * 8;
      __builtin_amdgcn_global_load_lds((const void *)src,
                                       (__attribute__((address_space(3))) void *)(buf + k * 1024),
                                       16, 0, 0);
    }
    __builtin_amdgcn_sched_barrier(0);  // nothing of the group passes its loads
    load_acc(dagg, P, n, q, da, 2 * hh);
  };
  static_assert(kRingLoads % 2 == 0, "each wave of a pair loads half of a ring");

  f32x4 acc[2][4] = {};
  f32x4 tsum[2] = {}, vxs[2] = {}, vys[2] = {};
  f32x4 da_nx[2] = {};
  // One group: half 0 or 1 of chunk c, its ring in `cur`; the next group's
  // loads go to `nxt`.  Leaves T staged.
  auto group = [&](unsigned c, int half, const uint8_t *cur, uint8_t *nxt) {
    int wo = lane;
    asm volatile("" : "+v"(wo));
    const u32x4 *wa = wa_s + 4 * hh * 64 + wo;
    const Pos P = group_pos(2 * c + half, ngroups, n, nx, ny, gxn);
    // (zero on lanes outside the lattice)
    f32x4 da[2];
#pragma unroll
    for (int t = 0; t < 2; ++t) da[t] = P.valid ? da_nx[t] : f32x4{0.0f, 0.0f, 0.0f, 0.0f};
    // chunk q of this receiver's lower-left neighbour; every neighbour's
    // chunk is at a constant offset from it
    const uint8_t *nb = cur + n * kRingNodeBytes + q * 16;
    auto frag_at = [&](int dx, int dy, int sidx) {
      return *(const u32x4 *)(nb + ((dy + 1) * kRingX + dx + 1) * kRingNodeBytes + sidx * 64);
    };
    // all of the group's LDS reads, before the next group's loads: the
    // compiler cannot tell the two buffers apart and would wait for the loads
    // before a read
    const u32x4 hn[2] = {frag_at(0, 0, 0), frag_at(0, 0, 1)};
    u32x4 hj[8][2];
#pragma unroll
    for (int d = 1; d < 9; ++d) {
      hj[d - 1][0] = frag_at(cx(d), cy(d), 0);
      hj[d - 1][1] = frag_at(cx(d), cy(d), 1);
    }
    f32x4 an[2];
#pragma unroll
    for (int t = 0; t < 2; ++t) {
      an[t] = mfma(wa[(2 * t) * 64], hn[0], be_s[4 * (2 * hh + t) + (wo >> 4)]);
      an[t] = mfma(wa[(2 * t + 1) * 64], hn[1], an[t]);
    }
    u32x4 own = hh ? hn[1] : hn[0];
    asm volatile("" : "+v"(own));  // select it once
    // the next group of this wave: the chunk's second half, or the first
    // half of the wave's next chunk
    const unsigned next = half == 0 ? 2 * c + 1 : 2 * (c + kBwdWaves);
    if (half == 0 || c + kBwdWaves < nchunks) prefetch(next, nxt, da_nx);
    const __amdgpu_buffer_rsrc_t dq_rows =
        rows_resource(dq_out, P.node0 * kEdgeBytes, P.cols * kEdgeBytes);
    const int dq_off = P.valid ? n * 64 + q * 16 : 1 << 30;
    f32x4 T[2] = {};
    // The edge loop is unrolled in full, so the direction of each edge (its
    // edge feature, the sign it adds to the Wc gradients with) is a
    // compile-time constant and the loop has no branches to split its
    // schedule.
    const uint32_t q0 = q == 0 ? 0xffffffffu : 0u;
    // pre-activation of the message from direction d (MFMA only)
    auto message = [&](int d, f32x4(&a)[2]) {
      const u32x4 ed = {q0 & (bf16_unit(cx(d)) | (bf16_unit(cy(d)) << 16)), 0u, 0u, 0u};
#pragma unroll
      for (int t = 0; t < 2; ++t) {
        a[t] = mfma(u32x4{wc[t], 0u, 0u, 0u}, ed, an[t]);
        a[t] = mfma(wb[t][0], hj[d - 1][0], a[t]);
        a[t] = mfma(wb[t][1], hj[d - 1][1], a[t]);
      }
    };
    // Software pipeline as in the forward round: the MFMA chains of edge
    // d + 1 are issued among the VALU work of edge d.  The sums run over d in
    // the same order as without the pipeline.
    f32x4 pre[2][2];
    message(1, pre[1]);
    __builtin_amdgcn_sched_barrier(0);
#pragma unroll
    for (int d = 1; d < 9; ++d) {
      if (d < 8) message(d + 1, pre[(d + 1) & 1]);
      f32x4 dq[2];
#pragma unroll
      for (int t = 0; t < 2; ++t) {
        const f32x4 a = pre[d & 1][t];
        dq[t] = da[t] * f32x4{gelu_grad(a.x), gelu_grad(a.y), gelu_grad(a.z), gelu_grad(a.w)};
        {
          // sums of the rounded products, as they are stored
#pragma clang fp contract(off)
          T[t] += dq[t];
          if (cx(d) > 0) vxs[t] += dq[t];
          if (cx(d) < 0) vxs[t] -= dq[t];
          if (cy(d) > 0) vys[t] += dq[t];
          if (cy(d) < 0) vys[t] -= dq[t];
        }
      }
      // non-temporal: 1 KB per node, read back once by the sender side
      // (measured: the sender side then runs 18 % faster, this kernel 4 %
      // slower)
      __builtin_amdgcn_raw_buffer_store_b128(
          __builtin_bit_cast(i32x4_t, frag_from_acc(dq[0], dq[1])), dq_rows,
          dq_off + ((d - 1) * 2 + hh) * 64 * P.cols, 0, kBufferNt);
      if (d < 8) {
        // each of edge d + 1's 6 MFMAs followed by 10 VALU instructions
#pragma unroll
        for (int i = 0; i < 6; ++i) {
          __builtin_amdgcn_sched_group_barrier(0x008, 1, 0);
          __builtin_amdgcn_sched_group_barrier(0x002, 10, 0);
        }
      }
      __builtin_amdgcn_sched_barrier(0);
    }
    // The pair's products with the previous chunk's columns are done.  (Needed
    // in half 0 only, but a branch here makes the compiler put the sums off
    // past it, and spill the products of all edges.)
    lds_barrier();
    const int col = 16 * half + n;
    t_s[pair][half][hh][lane] = frag_from_acc(T[0], T[1]);
    stage_acc(S.d, T, q, col, 32 * hh);
    stage_frag1(S.a, own, hh, q, col);
#pragma unroll
    for (int t = 0; t < 2; ++t) tsum[t] += T[t];
    // the next group's loads, with this group's 8 stores behind them
    __builtin_amdgcn_s_waitcnt(wait_vmcnt(8));
  };
  // After the barrier that follows a group: Wa^T T, both waves' channels.
  auto finish = [&](unsigned c, int half) {
    int wo = lane;
    asm volatile("" : "+v"(wo));
    const u32x4 *wat = wat_s + 4 * hh * 64 + wo;
    const Pos P = group_pos(2 * c + half, ngroups, n, nx, ny, gxn);
    const u32x4 tb[2] = {t_s[pair][half][0][lane], t_s[pair][half][1][lane]};
    f32x4 o[2];
#pragma unroll
    for (int t = 0; t < 2; ++t) {
      o[t] = mfma(wat[(2 * t) * 64], tb[0], f32x4{0.0f, 0.0f, 0.0f, 0.0f});
      o[t] = mfma(wat[(2 * t + 1) * 64], tb[1], o[t]);
    }
    // replaces this group's dL/dagg rows, read by nobody after this group;
    // the sender-side kernel adds it to dh
    store_acc(dagg_io, P, n, q, o, 2 * hh);
  };

  // Group i of a pair works from ring_s[pair][i % 2].  The pairs of a block
  // have the same number of turns but for the last, which those past the end
  // spend at its barriers.
  if (w < nchunks) prefetch(2 * w, ring_s[pair][0], da_nx);
  __builtin_amdgcn_s_waitcnt(wait_vmcnt(0));
  lds_barrier();
  for (unsigned c0 = blockIdx.x * 4; c0 < nchunks; c0 += kBwdWaves) {
    const unsigned c = c0 + pair;
    if (c >= nchunks) {
      for (int k = 0; k < 4; ++k) lds_barrier();
      break;
    }
#pragma unroll 1
    for (int half = 0; half < 2; ++half) {
      group(c, half, ring_s[pair][half], ring_s[pair][half ^ 1]);
      lds_barrier();
      finish(c, half);
    }
    dw_mma<2, 4>(acc, S.d + 32 * hh * kPitch, S.a, lane);
  }
  lds_barrier();
  float *pw = part + (size_t)w * L.nparam;
  write_dw<2, 4>(pw, L.We[r] + (size_t)32 * hh * EDGE_IN, EDGE_IN, 0, 32, HID, acc, lane);
  write_vec_half(pw, L.be[r], 1, hh, tsum, S.red, lane);
  write_vec_half(pw, L.We[r] + 2 * HID, EDGE_IN, hh, vxs, S.red, lane);
  write_vec_half(pw, L.We[r] + 2 * HID + 1, EDGE_IN, hh, vys, S.red, lane);
}

// ----------------------------------------------- edge layer, sender side ---

// S_m = sum_d dq_{m - e_d, d}; dWb; dh_m += Wa^T T_m (left by the receiver
// side in orecv), then dh_m += Wb^T S_m.  Bound by the reads of dq.
__global__ __launch_bounds__(kPairT, 2) void bwd_edge_send_kernel(
    const uint16_t *__restrict__ dq_in, const uint16_t *__restrict__ h, int batch, int nx,
    int ny, int r, const uint8_t *__restrict__ pack, FragLayout F, BlobLayout L,
    const float *__restrict__ orecv, float *__restrict__ dh, float *__restrict__ part) {
  __shared__ Stage<64, 64> st[4];
  __shared__ u32x4 x_s[4][2][2][64];  // pair, half, channels: S as an operand
  const int lane = threadIdx.x & 63;
  const int wave = __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
  const int pair = wave & 3, hh = wave >> 2;
  const int n = lane & 15, q = lane >> 4;
  Stage<64, 64> &S = st[pair];
  const u32x4 *frags = (const u32x4 *)(pack + F.frag_off);
  u32x4 wbt[2][2];
#pragma unroll
  for (int t = 0; t < 2; ++t) {
    wbt[t][0] = load_frag(frags, F.WBT[r] + 2 * (2 * hh + t), lane);
    wbt[t][1] = load_frag(frags, F.WBT[r] + 2 * (2 * hh + t) + 1, lane);
  }
  const unsigned gxn = (nx + 15) / 16, ngroups = (unsigned)batch * ny * gxn;
  const unsigned nchunks = (ngroups + 1) / 2;
  const unsigned w = blockIdx.x * 4 + pair;
  f32x4 acc[2][4] = {};
  // The next group's dq rows (eight directions), node state, dh and the
  // receiver side's term are loaded while this group is computed.
  u32x4 dq_nx[8], hm_nx;
  f32x4 dh_nx[2], or_nx[2];
  auto prefetch = [&](unsigned grp) {
    const Pos P = group_pos(grp, ngroups, n, nx, ny, gxn);
    const size_t lat_nodes = (size_t)P.b * ny * nx;
    // receivers whose edge d points here: columns x - 1, x, x + 1 of three rows
    size_t at[3];
    int wide[3];
#pragma unroll
    for (int k = 0; k < 3; ++k) {
      int xn = P.x + k - 1;
      xn = xn < 0 ? xn + nx : (xn >= nx ? xn - nx : xn);
      const int xg = xn & ~15;
      wide[k] = nx - xg < 16 ? nx - xg : 16;
      at[k] = (size_t)xg * kEdgeBytes + (xn - xg) * 64 + q * 16;
    }
#pragma unroll
    for (int d = 1; d < 9; ++d) {
      int yn = P.y - cy(d);
      yn = yn < 0 ? yn + ny : (yn >= ny ? yn - ny : yn);
      const int k = 1 - cx(d);
      const uint8_t *src = (const uint8_t *)dq_in + (lat_nodes + (size_t)yn * nx) * kEdgeBytes +
                           at[k] + (size_t)(((d - 1) * 2 + hh) * 64 * wide[k]);
      dq_nx[d - 1] = __builtin_nontemporal_load((const u32x4 *)src);  // read once
    }
    hm_nx = ((const u32x4 *)(h + P.node * HID))[4 * hh + q];
    load_acc(dh, P, n, q, dh_nx, 2 * hh);
    load_acc(orecv, P, n, q, or_nx, 2 * hh);
  };
  if (w < nchunks) prefetch(2 * w);
  for (unsigned c0 = blockIdx.x * 4; c0 < nchunks; c0 += kBwdWaves) {
    const unsigned c = c0 + pair;
    if (c >= nchunks) {
      for (int k = 0; k < 4; ++k) lds_barrier();
      break;
    }
#pragma unroll 1
    for (int half = 0; half < 2; ++half) {
      const Pos P = group_pos(2 * c + half, ngroups, n, nx, ny, gxn);
      u32x4 dqc[8];
#pragma unroll
      for (int d = 0; d < 8; ++d) dqc[d] = dq_nx[d];
      const u32x4 hm = hm_nx;
      const f32x4 dhc[2] = {dh_nx[0], dh_nx[1]}, orc[2] = {or_nx[0], or_nx[1]};
      if (half == 0 || c + kBwdWaves < nchunks)
        prefetch(half == 0 ? 2 * c + 1 : 2 * (c + kBwdWaves));
      f32x4 Sm[2] = {};
#pragma unroll
      for (int d = 0; d < 8; ++d) {
        Sm[0] += unpack_lo(dqc[d]);
        Sm[1] += unpack_hi(dqc[d]);
      }
      if (!P.valid)
#pragma unroll
        for (int t = 0; t < 2; ++t) Sm[t] = f32x4{0.0f, 0.0f, 0.0f, 0.0f};
      lds_barrier();  // the products with the previous chunk's columns are done
      const int col = 16 * half + n;
      x_s[pair][half][hh][lane] = frag_from_acc(Sm[0], Sm[1]);
      stage_acc(S.d, Sm, q, col, 32 * hh);
      stage_frag1(S.a, hm, hh, q, col);
      lds_barrier();
      const u32x4 sb[2] = {x_s[pair][half][0][lane], x_s[pair][half][1][lane]};
      f32x4 o[2];
#pragma unroll
      for (int t = 0; t < 2; ++t) {
        o[t] = mfma(wbt[t][0], sb[0], f32x4{0.0f, 0.0f, 0.0f, 0.0f});
        o[t] = mfma(wbt[t][1], sb[1], o[t]);
        o[t] = (dhc[t] + orc[t]) + o[t];
      }
      store_acc(dh, P, n, q, o, 2 * hh);
    }
    dw_mma<2, 4>(acc, S.d + 32 * hh * kPitch, S.a, lane);
  }
  float *pw = part + (size_t)w * L.nparam;
  write_dw<2, 4>(pw, L.We[r] + (size_t)32 * hh * EDGE_IN, EDGE_IN, HID, 32, HID, acc, lane);
}

// ------------------------------------------------------------- encoder ---

__device__ __forceinline__ f32x4 gelu_grad4(f32x4 p) {
  return f32x4{gelu_grad(p.x), gelu_grad(p.y), gelu_grad(p.z), gelu_grad(p.w)};
}

__global__ __launch_bounds__(kPairT, 2) void bwd_encoder_kernel(
    const float *__restrict__ dh0, const uint16_t *__restrict__ sx, const uint16_t *__restrict__ se1,
    int batch, int nx, int ny, const uint8_t *__restrict__ pack, FragLayout F, BlobLayout L,
    float *__restrict__ part) {
  __shared__ Stage<64, 64> st[4];
  __shared__ uint16_t d1s[4][64 * kPitch], x1s[4][16 * kPitch];
  __shared__ u32x4 w2t_s[8 * 64], w1_s[4 * 64];
  __shared__ u32x4 x_s[4][2][2][64];  // pair, half, channels: dp2 as an operand
  const int lane = threadIdx.x & 63;
  const int wave = __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
  const int pair = wave & 3, hh = wave >> 2;
  const int n = lane & 15, q = lane >> 4;
  Stage<64, 64> &S = st[pair];
  uint16_t *D1 = d1s[pair], *X1 = x1s[pair];
  const u32x4 *frags = (const u32x4 *)(pack + F.frag_off);
  const f32x4 *bias = (const f32x4 *)(pack + F.bias_off);
  // W2^T and W1 are read from LDS inside the loop, so that the loop issues
  // no global loads besides its node data
  w2t_s[threadIdx.x] = frags[(size_t)F.W2T * 64 + threadIdx.x];
  if (threadIdx.x < 4 * 64) w1_s[threadIdx.x] = frags[(size_t)F.W1 * 64 + threadIdx.x];
  u32x4 w2[2][2];
  f32x4 b1[2], b2[2];
#pragma unroll
  for (int t = 0; t < 2; ++t) {
    const int tt = 2 * hh + t;
    w2[t][0] = load_frag(frags, F.W2 + 2 * tt, lane);
    w2[t][1] = load_frag(frags, F.W2 + 2 * tt + 1, lane);
    b1[t] = load_bias(bias, F.B1 + tt, lane);
    b2[t] = load_bias(bias, F.B2 + tt, lane);
  }
  const unsigned gxn = (nx + 15) / 16, ngroups = (unsigned)batch * ny * gxn;
  const unsigned nchunks = (ngroups + 1) / 2;
  const unsigned w = blockIdx.x * 4 + pair;
  __syncthreads();
  f32x4 acc2[2][4] = {}, acc1[2][1] = {};
  f32x4 s1[2] = {}, s2[2] = {};
  // The next group's first-layer output, features and incoming gradient are
  // loaded while this group is computed.
  u32x4 e1_nx[2], xb_nx;
  f32x4 G_nx[2];
  auto prefetch = [&](unsigned grp) {
    const Pos P = group_pos(grp, ngroups, n, nx, ny, gxn);
    load_frags(se1, P.node, q, e1_nx);
    xb_nx = q < 2 ? ((const u32x4 *)(sx + P.node * 16))[q] : u32x4{0u, 0u, 0u, 0u};
    load_acc(dh0, P, n, q, G_nx, 2 * hh);
  };
  if (w < nchunks) prefetch(2 * w);
  for (unsigned c0 = blockIdx.x * 4; c0 < nchunks; c0 += kBwdWaves) {
    const unsigned c = c0 + pair;
    if (c >= nchunks) {
      for (int k = 0; k < 5; ++k) lds_barrier();
      break;
    }
#pragma unroll 1
    for (int half = 0; half < 2; ++half) {
      int wo = lane;
      asm volatile("" : "+v"(wo));
      const u32x4 *w2t = w2t_s + 4 * hh * 64 + wo, *w1 = w1_s + 2 * hh * 64 + wo;
      const Pos P = group_pos(2 * c + half, ngroups, n, nx, ny, gxn);
      const u32x4 e1[2] = {e1_nx[0], e1_nx[1]};
      const u32x4 xb = xb_nx;
      const f32x4 G[2] = {G_nx[0], G_nx[1]};
      if (half == 0 || c + kBwdWaves < nchunks)
        prefetch(half == 0 ? 2 * c + 1 : 2 * (c + kBwdWaves));
      f32x4 dp2[2];
#pragma unroll
      for (int t = 0; t < 2; ++t) {
        f32x4 p = mfma(w2[t][0], e1[0], b2[t]);
        p = mfma(w2[t][1], e1[1], p);
        dp2[t] = P.valid ? G[t] * gelu_grad4(p) : f32x4{0.0f, 0.0f, 0.0f, 0.0f};
        s2[t] += dp2[t];
      }
      lds_barrier();  // the products with the previous chunk's columns are done
      const int col = 16 * half + n;
      x_s[pair][half][hh][lane] = frag_from_acc(dp2[0], dp2[1]);
      stage_acc(S.d, dp2, q, col, 32 * hh);
      stage_frag1(S.a, hh ? e1[1] : e1[0], hh, q, col);
      if (hh == 0) stage_rows16(X1, xb, q, col);
      lds_barrier();
      const u32x4 dpb[2] = {x_s[pair][half][0][lane], x_s[pair][half][1][lane]};
      f32x4 dp1[2];
#pragma unroll
      for (int t = 0; t < 2; ++t) {
        f32x4 de1 = mfma(w2t[(2 * t) * 64], dpb[0], f32x4{0.0f, 0.0f, 0.0f, 0.0f});
        de1 = mfma(w2t[(2 * t + 1) * 64], dpb[1], de1);
        f32x4 p1 = mfma(w1[t * 64], xb, b1[t]);
        dp1[t] = de1 * gelu_grad4(p1);
        {
#pragma clang fp contract(off)
          s1[t] += dp1[t];
        }
      }
      stage_acc(D1, dp1, q, col, 32 * hh);
    }
    lds_barrier();
    dw_mma<2, 4>(acc2, S.d + 32 * hh * kPitch, S.a, lane);
    dw_mma<2, 1>(acc1, D1 + 32 * hh * kPitch, X1, lane);
  }
  lds_barrier();
  float *pw = part + (size_t)w * L.nparam;
  write_dw<2, 4>(pw, L.W2 + (size_t)32 * hh * HID, HID, 0, 32, HID, acc2, lane);
  write_dw<2, 1>(pw, L.W1 + (size_t)32 * hh * NFEAT, NFEAT, 0, 32, NFEAT, acc1, lane);
  write_vec_half(pw, L.b2, 1, hh, s2, S.red, lane);
  write_vec_half(pw, L.b1, 1, hh, s1, S.red, lane);
}

// Fixed-order sum of the per-wave partials: one thread per parameter, the
// partials added in wave order.  One-wave blocks spread the ~600 waves over
// every CU, and the unrolled loop keeps 32 independent loads in flight ahead
// of the (sequential) additions.
constexpr int kReduceThreads = 64;
__global__ __launch_bounds__(kReduceThreads) void bwd_reduce_kernel(
    const float *__restrict__ part, size_t nparam, float *__restrict__ grad) {
  size_t p = (size_t)blockIdx.x * kReduceThreads + threadIdx.x;
  if (p >= nparam) return;
  float s = 0.0f;
#pragma unroll 32
  for (int w = 0; w < kBwdWaves; ++w) s += part[(size_t)w * nparam + p];
  grad[p] = s;
}

// The same sum for a network of few parameters, whose 88 waves above wait
// for memory 32 times (22 us for the 5,642 parameters of the per-node network):
// a block takes 32 parameters, brings all of their partials to LDS with 64 loads
// in flight per thread, and 32 lanes add them in wave order (13).  With
// more parameters than CUs x 32 the blocks come in several rounds and the
// kernel above is the better one (38,922: 41 us, 64 and more here).
constexpr int kFewParams = 32;
__global__ __launch_bounds__(kBT) void bwd_reduce_few_kernel(const float *__restrict__ part,
                                                             size_t nparam,
                                                             float *__restrict__ grad) {
  __shared__ float v_s[kBwdWaves * kFewParams];
  const int k = threadIdx.x % kFewParams, w0 = threadIdx.x / kFewParams;
  constexpr int kStride = kBT / kFewParams, kPer = 64;
  const size_t p = (size_t)blockIdx.x * kFewParams + k;
  const size_t pc = p < nparam ? p : nparam - 1;
#pragma unroll 1
  for (int r = w0; r < kBwdWaves; r += kPer * kStride) {
    float v[kPer];
#pragma unroll
    for (int j = 0; j < kPer; ++j) v[j] = part[(size_t)(r + j * kStride) * nparam + pc];
#pragma unroll
    for (int j = 0; j < kPer; ++j) v_s[(r + j * kStride) * kFewParams + k] = v[j];
  }
  static_assert(kBwdWaves % (kPer * kStride) == 0, "whole turns");
  __syncthreads();
  if (threadIdx.x >= kFewParams) return;
  float s = 0.0f;
#pragma unroll 32
  for (int w = 0; w < kBwdWaves; ++w) s += v_s[w * kFewParams + k];
  if (p < nparam) grad[p] = s;
}

// ------------------------------------------------------------ MSE, Adam ---

__global__ __launch_bounds__(kBT) void mse_kernel(const float *__restrict__ a,
                                                  const float *__restrict__ b, size_t n,
                                                  float gscale, float *__restrict__ grad,
                                                  double *__restrict__ partials) {
  __shared__ double sm[kBT];
  double s = 0.0;
  // Reads two arrays, writes one: 9 us at the rate of a copy for 32 lattices of
  // 128^2.  Six elements are loaded ahead of their sums, which keep their order
  // (16.4 us -> 13.1; the launch and the block sums are 4 of it).
  constexpr int kAhead = 6;
  const size_t stride = (size_t)gridDim.x * kBT;
  size_t k = (size_t)blockIdx.x * kBT + threadIdx.x;
  auto add = [&](size_t at, float d) {
    s += (double)d * (double)d;
    if (grad) grad[at] = gscale * d;
  };
  for (; k + (kAhead - 1) * stride < n; k += kAhead * stride) {
    float va[kAhead], vb[kAhead];
#pragma unroll
    for (int j = 0; j < kAhead; ++j) {
      va[j] = a[k + j * stride];
      vb[j] = b[k + j * stride];
    }
#pragma unroll
    for (int j = 0; j < kAhead; ++j) add(k + j * stride, va[j] - vb[j]);
  }
  for (; k < n; k += stride) add(k, a[k] - b[k]);
  sm[threadIdx.x] = s;
  __syncthreads();
  for (int k = kBT / 2; k > 0; k >>= 1) {
    if ((int)threadIdx.x < k) sm[threadIdx.x] += sm[threadIdx.x + k];
    __syncthreads();
  }
  if (threadIdx.x == 0) partials[blockIdx.x] = sm[0];
}

// Eq. 4 with the residual weighted by a symmetric 9 x 9 matrix Q per node:
// sum over nodes of r^T Q r, r = a - b over the nine populations of a node
// (row-interleaved layout [batch][ny][9][nx]); gradient gscale * Q r.  The
// products with Q are taken in FP64.
struct MseWeights {
  double q[81];
};

__global__ __launch_bounds__(kBT) void mse_weighted_kernel(const float *__restrict__ a,
                                                           const float *__restrict__ b,
                                                           int batch, int nx, int ny,
                                                           MseWeights Q, float gscale,
                                                           float *__restrict__ grad,
                                                           double *__restrict__ partials) {
  __shared__ double sm[kBT];
  double s = 0.0;
  const size_t nodes = (size_t)batch * ny * nx;
  for (size_t k = (size_t)blockIdx.x * kBT + threadIdx.x; k < nodes;
       k += (size_t)gridDim.x * kBT) {
    const size_t row = k / (size_t)nx, x = k - row * nx;     // row = b * ny + y
    const size_t base = row * 9 * (size_t)nx + x;
    double r[9];
#pragma unroll
    for (int i = 0; i < 9; ++i) r[i] = (double)a[base + (size_t)i * nx] - (double)b[base + (size_t)i * nx];
#pragma unroll
    for (int i = 0; i < 9; ++i) {
      double t = 0.0;
#pragma unroll
      for (int j = 0; j < 9; ++j) t += Q.q[9 * i + j] * r[j];
      s += r[i] * t;
      if (grad) grad[base + (size_t)i * nx] = gscale * (float)t;
    }
  }
  sm[threadIdx.x] = s;
  __syncthreads();
  for (int k = kBT / 2; k > 0; k >>= 1) {
    if ((int)threadIdx.x < k) sm[threadIdx.x] += sm[threadIdx.x + k];
    __syncthreads();
  }
  if (threadIdx.x == 0) partials[blockIdx.x] = sm[0];
}

__global__ __launch_bounds__(kBT) void mse_finalize(const double *__restrict__ partials, int nb,
                                                    double scale, double *__restrict__ loss) {
  __shared__ double sm[kBT];
  double s = 0.0;
  for (int k = threadIdx.x; k < nb; k += kBT) s += partials[k];
  sm[threadIdx.x] = s;
  __syncthreads();
  for (int k = kBT / 2; k > 0; k >>= 1) {
    if ((int)threadIdx.x < k) sm[threadIdx.x] += sm[threadIdx.x + k];
    __syncthreads();
  }
  if (threadIdx.x == 0) *loss = scale * sm[0];
}

__global__ __launch_bounds__(kBT) void adam_kernel(float *__restrict__ p,
                                                   const float *__restrict__ g,
                                                   float *__restrict__ m, float *__restrict__ v,
                                                   size_t n, float lr, float b1, float b2,
                                                   float eps, float c1, float c2) {
  size_t k = (size_t)blockIdx.x * kBT + threadIdx.x;
  if (k >= n) return;
  float gk = g[k];
  float mk = b1 * m[k] + (1.0f - b1) * gk;
  float vk = b2 * v[k] + (1.0f - b2) * gk * gk;
  m[k] = mk;
  v[k] = vk;
  p[k] -= lr * (mk / c1) / (sqrtf(vk / c2) + eps);
}

}  // namespace gnn

// ------------------------------------------------------------------- ABI ---

using namespace gnn;
using lbm::check_device;
using lbm::fail;
using lbm::launch_check;

static inline void *at(void *base, size_t off) { return (uint8_t *)base + off; }
static inline const void *at(const void *base, size_t off) {
  return (const uint8_t *)base + off;
}

extern "C" int gnn_backward(const float *dL_dgpost, const float *g_pre, const void *saved,
                            int batch, int nx, int ny, const float *tau, const float *params,
                            int n_rounds, float *grad, void *workspace, size_t ws_bytes,
                            void *stream) {
  const int R = n_rounds;
  if (!dL_dgpost || !g_pre || !saved || !tau || !params || !grad)
    return fail(LBM_EINVAL, "gnn_backward: null pointer");
  if (R < 0 || R > MAX_ROUNDS) return fail(LBM_EINVAL, "gnn_backward: bad n_rounds %d", R);
  if (batch < 1 || !lbm::lattice_ok(nx, ny) || (long long)batch * nx * ny >= (1LL << 31))
    return fail(LBM_EINVAL, "gnn_backward: bad sizes");
  const long long nodes = (long long)batch * nx * ny;
  const size_t need = backward_workspace_bytes(batch, nx, ny, R);
  if (!workspace || ws_bytes < need)
    return fail(LBM_EWORKSPACE, "gnn_backward: workspace needs %zu bytes", need);
  if (int rc = check_device()) return rc;
  hipStream_t s = (hipStream_t)stream;
  const BlobLayout L = blob_layout(R);
  const FragLayout F = frag_layout(R);
  const BackwardScratch W = backward_scratch(nodes, R);
  const SavedLayout SL = saved_layout(nodes, R);
  uint8_t *pack = (uint8_t *)at(workspace, W.pack);
  if (R > 0)
    if (int rc = launch_prep(params, R, pack, nullptr, nullptr, s)) return rc;
  float *part = (float *)at(workspace, W.part);
  float *dh[2] = {(float *)at(workspace, W.dhA), (float *)at(workspace, W.dhB)};
  float *dagg = (float *)at(workspace, W.dagg);
  uint16_t *dq = (uint16_t *)at(workspace, W.dq);
  const size_t hstride = align256((size_t)nodes * HID * 2);
  auto hsaved = [&](int r) { return (const uint16_t *)at(saved, SL.h + (size_t)r * hstride); };
  auto asaved = [&](int r) { return (const uint16_t *)at(saved, SL.agg + (size_t)r * hstride); };

  if (R == 0) {  // the per-node network, one kernel
    if (int rc = launch_simple_backward(dL_dgpost, g_pre, tau, (const float *)at(saved, SL.z),
                                        batch, nx, ny, params, part, s))
      return rc;
  } else {
    int cur = 0;
    hipLaunchKernelGGL(bwd_head_kernel, dim3(kBwdBlocks), dim3(kBT), 0, s, dL_dgpost, g_pre, tau,
                       (const float *)at(saved, SL.z), hsaved(R), batch, nx, ny, pack, F, L,
                       dh[cur], part);
    if (int rc = launch_check("bwd_head_kernel")) return rc;
    for (int r = R - 1; r >= 0; --r) {
      float *din = dh[cur], *dout = dh[cur ^ 1];
      hipLaunchKernelGGL(bwd_node_kernel, dim3(kBwdBlocks), dim3(kPairT), 0, s, din, hsaved(r),
                         asaved(r), batch, nx, ny, r, pack, F, L, dout, dagg, part);
      if (int rc = launch_check("bwd_node_kernel")) return rc;
      hipLaunchKernelGGL(bwd_edge_recv_kernel, dim3(kBwdBlocks), dim3(kPairT), 0, s, dagg, hsaved(r),
                         batch, nx, ny, r, pack, F, L, dq, part);
      if (int rc = launch_check("bwd_edge_recv_kernel")) return rc;
      hipLaunchKernelGGL(bwd_edge_send_kernel, dim3(kBwdBlocks), dim3(kPairT), 0, s, dq, hsaved(r),
                         batch, nx, ny, r, pack, F, L, dagg, dout, part);
      if (int rc = launch_check("bwd_edge_send_kernel")) return rc;
      cur ^= 1;
    }
    hipLaunchKernelGGL(bwd_encoder_kernel, dim3(kBwdBlocks), dim3(kPairT), 0, s, dh[cur],
                       (const uint16_t *)at(saved, SL.x), (const uint16_t *)at(saved, SL.e1),
                       batch, nx, ny, pack, F, L, part);
    if (int rc = launch_check("bwd_encoder_kernel")) return rc;
  }
  if (L.nparam <= (size_t)kFewParams * lbm::device_cus())
    hipLaunchKernelGGL(bwd_reduce_few_kernel,
                       dim3((unsigned)((L.nparam + kFewParams - 1) / kFewParams)), dim3(kBT), 0, s,
                       part, L.nparam, grad);
  else
    hipLaunchKernelGGL(bwd_reduce_kernel,
                       dim3((unsigned)((L.nparam + kReduceThreads - 1) / kReduceThreads)),
                       dim3(kReduceThreads), 0, s, part, L.nparam, grad);
  return launch_check("bwd_reduce_kernel");
}

extern "C" int gnn_mse(const float *a, const float *b, int batch, int nx, int ny, double scale,
                       double *loss, float *grad_a, void *workspace, size_t ws_bytes,
                       void *stream) {
  if (!a || !b || !loss) return fail(LBM_EINVAL, "gnn_mse: null pointer");
  if (batch < 1 || !lbm::lattice_ok(nx, ny)) return fail(LBM_EINVAL, "gnn_mse: bad sizes");
  const long long nodes = (long long)batch * nx * ny;
  const int nb = lbm::reduce_blocks(nodes);
  if (!workspace || ws_bytes < (size_t)nb * 8 * sizeof(double))
    return fail(LBM_EWORKSPACE, "gnn_mse: workspace needs %zu bytes",
                (size_t)nb * 8 * sizeof(double));
  if (int rc = check_device()) return rc;
  hipStream_t s = (hipStream_t)stream;
  const size_t n = (size_t)nodes * 9;
  hipLaunchKernelGGL(mse_kernel, dim3(nb), dim3(kBT), 0, s, a, b, n,
                     (float)(2.0 * scale / (double)nodes), grad_a, (double *)workspace);
  if (int rc = launch_check("mse_kernel")) return rc;
  hipLaunchKernelGGL(mse_finalize, dim3(1), dim3(kBT), 0, s, (const double *)workspace, nb,
                     scale / (double)nodes, loss);
  return launch_check("mse_finalize");
}

extern "C" int gnn_mse_weighted(const float *a, const float *b, int batch, int nx, int ny,
                                const double *q, double scale, double *loss, float *grad_a,
                                void *workspace, size_t ws_bytes, void *stream) {
  if (!a || !b || !loss || !q) return fail(LBM_EINVAL, "gnn_mse_weighted: null pointer");
  if (batch < 1 || !lbm::lattice_ok(nx, ny) || (long long)batch * nx * ny >= (1LL << 31))
    return fail(LBM_EINVAL, "gnn_mse_weighted: bad sizes");
  MseWeights Q;
  for (int i = 0; i < 9; ++i)
    for (int j = 0; j < 9; ++j) {
      const double v = q[9 * i + j];
      if (!(fabs(v) < INFINITY) || v != q[9 * j + i])
        return fail(LBM_EINVAL, "gnn_mse_weighted: Q must be finite and symmetric");
      Q.q[9 * i + j] = v;
    }
  const long long nodes = (long long)batch * nx * ny;
  const int nb = lbm::reduce_blocks(nodes);
  if (!workspace || ws_bytes < (size_t)nb * 8 * sizeof(double))
    return fail(LBM_EWORKSPACE, "gnn_mse_weighted: workspace needs %zu bytes",
                (size_t)nb * 8 * sizeof(double));
  if (int rc = check_device()) return rc;
  hipStream_t s = (hipStream_t)stream;
  hipLaunchKernelGGL(mse_weighted_kernel, dim3(nb), dim3(kBT), 0, s, a, b, batch, nx, ny, Q,
                     (float)(2.0 * scale / (double)nodes), grad_a, (double *)workspace);
  if (int rc = launch_check("mse_weighted_kernel")) return rc;
  hipLaunchKernelGGL(mse_finalize, dim3(1), dim3(kBT), 0, s, (const double *)workspace, nb,
                     scale / (double)nodes, loss);
  return launch_check("mse_finalize");
}

extern "C" int gnn_adam(float *params, const float *grad, float *m, float *v, size_t n, float lr,
                        float beta1, float beta2, float eps, int step, void *stream) {
  if (!params || !grad || !m || !v) return fail(LBM_EINVAL, "gnn_adam: null pointer");
  if (step < 1) return fail(LBM_EINVAL, "gnn_adam: step must be >= 1");
  if (n == 0) return LBM_OK;
  if (int rc = check_device()) return rc;
  const double c1 = 1.0 - pow((double)beta1, step), c2 = 1.0 - pow((double)beta2, step);
  hipLaunchKernelGGL(adam_kernel, dim3((unsigned)((n + kBT - 1) / kBT)), dim3(kBT), 0,
                     (hipStream_t)stream, params, grad, m, v, n, lr, beta1, beta2, eps,
                     (float)c1, (float)c2);
  return launch_check("adam_kernel");
}
