// The per-node corrected collision of the paper's Fig. 2 ("SimpleLBMGNN",
// Methodology, "GNN Architecture Details"): the distribution functions,
// density and velocity of one node go through two linear layers with ReLU and
// two heads, tau_adj (sigmoid scaled to [0.5, 1.5]) and the direct correction
// delta f, with no message passing between nodes.  With no neighbour
// dependence the whole network fuses into the pull step: one pass reads the
// nine populations of a node once and writes the corrected post-collision
// populations once, like the plain BGK step, with the network's BF16 MFMA
// work and the correction in registers.
//
// Sizes follow the corrected collision's encoder and head: 12 -> 64 -> 64
// (ReLU) -> 10.  The parameter blob is the zero-round layout:
//   W1[64][12] b1[64] W2[64][64] b2[64] Wh[10][64] bh[10] | mu[12] sigma[12] s_delta
// The weight fragments (gnn_prep_kernel) and the gate kernel are shared with the
// message-passing step; the collision epilogue is this
// file's own, with the same arithmetic except the hardware exp2 and
// reciprocal in the sigmoid and the relaxation rate.
#include "channel_common.hpp"
#include "gnn_common.hpp"
#include "lbm_common.hpp"
#include "simple_common.hpp"

namespace gnn {

namespace simple {

using lbm::cx;
using lbm::cy;

constexpr int kThreads = 256;
constexpr int kWaves = kThreads / 64;

// A wave takes 64 consecutive nodes of one lattice row (ChunkQueue), one
// node per lane for everything that is per node: the coalesced pull of the
// nine populations (kept in registers for the collision), the moments and the
// 12 normalised features (rounded to BF16 into the node's LDS slot), and the
// collision.  The network runs in between on MFMA, four column blocks of 16
// nodes with lane (n, q) = (node, channel group), two blocks at a time; each
// block reads its nodes' features and then writes their head outputs into the
// same slots.  Weight fragments and the (per channel group) bias fragments sit
// in LDS (one 48-byte slot per node keeps the block at 27 KB); each fragment
// read serves two blocks, which needs the registers of four blocks per CU
// instead of five and measured 8 % faster (the LDS reads of one block at a
// time moved ≈ 145 bytes per cycle per CU).
constexpr int kBlocksPerCu = 4;   // resident blocks (LDS 27 KB, <= 128 registers)

// WALLS (with PULL): the channel step, halfway bounce-back at rows 0 and
// ny - 1 and the body force rho * gx along x.
template <bool PULL, bool WALLS>
__global__ __launch_bounds__(kThreads, kBlocksPerCu) void simple_step_kernel(
    const float *__restrict__ src, float *__restrict__ dst, int batch, int nx, int ny,
    const float *__restrict__ tau_arr, float tau_s, float gx, const uint8_t *__restrict__ pack,
    FragLayout F, float *__restrict__ head_out, Q80 *__restrict__ pmass,
    unsigned *__restrict__ pflag, float *__restrict__ save_z0, unsigned *__restrict__ chunkq) {
  __shared__ u32x4 w_s[kStepFrags * 64];
  __shared__ f32x4 b_s[kStepBias * 4];
  __shared__ __attribute__((aligned(16))) uint32_t slot_s[kWaves][64 * kSlot];
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  load_network(pack, F, w_s, b_s);
  const float *cst = (const float *)(pack + F.const_off);
  const float sdelta = cst[C_SDELTA];
  // normalisation (x - mu) / sigma as one FMA per feature: x * isg + nmi
  float isg[NFEAT], nmi[NFEAT];
#pragma unroll
  for (int k = 0; k < NFEAT; ++k) {
    isg[k] = 1.0f / cst[C_SIGMA + k];
    nmi[k] = -cst[C_MU + k] * isg[k];
  }
  __syncthreads();
  uint32_t *sw = slot_s[wave];
  Q80 mass_acc{0ull, 0ll};
  unsigned flag_acc = 0;

  const size_t row = (size_t)9 * nx;
  for (ChunkQueue cw(batch, nx, ny, kWaves, wave, chunkq); cw.more(); cw.next()) {
    const int xc = cw.xc, y = cw.y, b = cw.b;
    const float *lat = src + (size_t)b * ny * row;
    const int x = xc * 64 + lane;
    const bool valid = x < nx;
    const unsigned drawn = cw.draw();
    float gp[9];
    lbm::Moments<float> M;  // kept for the collision
    {
      // rows y - 1, y, y + 1 (uniform) and columns x - 1, x, x + 1 (per lane)
      const int xv = valid ? x : nx - 1;
      const float *r0 = lat + (size_t)(y == 0 ? ny - 1 : y - 1) * row;
      const float *r1 = lat + (size_t)y * row;
      const float *r2 = lat + (size_t)(y == ny - 1 ? 0 : y + 1) * row;
      const int xs0 = xv == 0 ? nx - 1 : xv - 1, xs2 = xv == nx - 1 ? 0 : xv + 1;
#pragma unroll
      for (int i = 0; i < 9; ++i) {
        if constexpr (PULL) {
          // g_i(x, y) = post_i(x - c_ix, y - c_iy)
          const float *r = cy(i) > 0 ? r0 : (cy(i) < 0 ? r2 : r1);
          const int xsrc = cx(i) > 0 ? xs0 : (cx(i) < 0 ? xs2 : xv);
          if constexpr (WALLS) {
            // a population that would come through a wall is the reversed one
            // that left this node (the row is uniform over the wave)
            if ((cy(i) > 0 && y == 0) || (cy(i) < 0 && y == ny - 1))
              gp[i] = r1[(size_t)lbm::opp(i) * nx + xv];
            else
              gp[i] = r[(size_t)i * nx + xsrc];
          } else if (cx(i) == 0) {
            // no other chunk reads these lines (the shifted directions share
            // their edge lines with the neighbouring chunks): non-temporal,
            // -0.5 % (all nine non-temporal: +1.3 %)
            gp[i] = __builtin_nontemporal_load(r + (size_t)i * nx + xsrc);
          } else {
            gp[i] = r[(size_t)i * nx + xsrc];
          }
        } else {
          gp[i] = r1[(size_t)i * nx + xv];
        }
      }
    }
    {
      M = moments(gp);
      cw.take(drawn);
      if (WALLS) M.u = __builtin_fmaf(M.jx, M.inv, 0.5f * gx);  // Guo's velocity
      put_features(sw + lane * kSlot, gp, M, isg, nmi);
    }
    wave_lds_sync();
    network(w_s, b_s, sw, lane);
    wave_lds_sync();
    if (valid) {
      float z[NOUT];
      get_head(sw + lane * kSlot, z);
      const float tau = tau_arr ? tau_arr[b] : tau_s;  // b < batch while cw.more()
      collide<WALLS>(gp, z, tau, sdelta, gx, M);
      float *d = dst + (size_t)b * ny * row + (size_t)y * row + x;
      // node mass in FP32 (rounding ~1e-9 per node, ~1e-13 of the lattice
      // mass), accumulated over the nodes in exact fixed point (a total that
      // does not depend on which wave took which chunk).  A population is negative
      // or not finite exactly when the smallest f_i is below zero or the sum
      // is not finite (an infinity or NaN anywhere reaches the sum; the
      // minimum skips NaN).
      float msum = 0.0f, fmin = INFINITY;
#pragma unroll
      for (int i = 0; i < 9; ++i) {
        __builtin_nontemporal_store(gp[i], d + (size_t)i * nx);
        fmin = fminf(fmin, gp[i] + lbm::wgt<float>(i));
        msum += gp[i];
      }
      const unsigned bad = (fmin >= 0.0f && fabsf(msum) < INFINITY) ? 0u : 1u;
      mass_acc = q80_add_f32(mass_acc, msum);
      flag_acc |= bad;
      // what a training forward keeps for the backward pass
      if (save_z0) save_z0[((size_t)b * ny + y) * nx + x] = z[0];
      if (head_out) {
        const size_t node = ((size_t)b * ny + y) * nx + x;
        for (int k = 0; k < NOUT; ++k) head_out[node * NOUT + k] = z[k];
      }
    }
    wave_lds_sync();
  }

  // every wave is done with its slots: the sum reuses them
  __syncthreads();
  store_partial((PartialSlot *)&slot_s[0][0], mass_acc, flag_acc, pmass, pflag);
}

// nsteps gated (or ungated) steps of a lattice of up to 1024 nodes in one
// workgroup, one node per thread.  The state goes from step to step through LDS
// (the eight directions that move, two buffers), the gate sums its exact mass
// over the waves between the two barriers that a step has anyway, and a step
// that trips is the plain BGK collision of the populations the step pulled,
// which are still in registers.  Same arithmetic as the steps one by one, so
// bitwise the same states and decisions.  Latency bound: a step of 4 x 32 takes
// 2.5 us (channel 2.8), in the kernel of large lattices with packing and gate
// 12.8, its rows filling four lanes of 64; one of 32 x 32 6.0 against 12.3.
constexpr int kResidentNodes = 1024;
constexpr int kResidentSteps = 4096;   // a launch of some 20 ms at most

template <bool WALLS, int THREADS>
__global__ __launch_bounds__(THREADS) void simple_resident_kernel(
    const float *__restrict__ src, float *__restrict__ dst, int nx, int ny, int nsteps, float tau,
    float gx, const uint8_t *__restrict__ pack, FragLayout F, double threshold,
    unsigned *__restrict__ flags, unsigned *__restrict__ n_fallback, double *__restrict__ mass) {
  constexpr int W = THREADS / 64;
  __shared__ u32x4 w_s[kStepFrags * 64];
  __shared__ f32x4 b_s[kStepBias * 4];
  __shared__ __attribute__((aligned(16))) uint32_t slot_s[W][64 * kSlot];
  __shared__ float state_s[2][8 * THREADS];
  __shared__ PartialSlot part_s[2][W];
  __shared__ double sum_s[W];
  const int lane = threadIdx.x & 63;
  const int wave = __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
  load_network(pack, F, w_s, b_s);
  const float *cst = (const float *)(pack + F.const_off);
  const float sdelta = cst[C_SDELTA];
  float isg[NFEAT], nmi[NFEAT];
#pragma unroll
  for (int k = 0; k < NFEAT; ++k) {
    isg[k] = 1.0f / cst[C_SIGMA + k];
    nmi[k] = -cst[C_MU + k] * isg[k];
  }
  const int nodes = nx * ny;
  const bool valid = (int)threadIdx.x < nodes;
  const int k = valid ? (int)threadIdx.x : nodes - 1, y = k / nx, x = k - y * nx;
  const float omega = 1.0f / tau;  // of the fallback
  float g[9];
  if constexpr (WALLS)
    lbm::pull9_walls(src, nx, ny, x, y, g);
  else
    lbm::pull9(src, nx, ny, x, y, g);
  int from[9];  // where population i of the next step comes from
#pragma unroll
  for (int i = 1; i < 9; ++i) {
    int sx = x - cx(i), sy = y - cy(i), d = i;
    sx = sx < 0 ? nx - 1 : (sx == nx ? 0 : sx);
    if (WALLS && (sy < 0 || sy == ny)) {  // back from the wall, reversed
      sx = x;
      sy = y;
      d = lbm::opp(i);
    }
    sy = sy < 0 ? ny - 1 : (sy == ny ? 0 : sy);
    from[i] = (d - 1) * THREADS + sy * nx + sx;
  }
  double m_prev = flags ? *mass : 0.0;
  unsigned seen = 0, fell = 0;
  __syncthreads();

  uint32_t *sw = slot_s[wave];
  for (int s = 0; s < nsteps; ++s) {
    float gn[9];
    {
      lbm::Moments<float> M = moments(g);
      if (WALLS) M.u = __builtin_fmaf(M.jx, M.inv, 0.5f * gx);  // Guo's velocity
      put_features(sw + lane * kSlot, g, M, isg, nmi);
      wave_lds_sync();
      network(w_s, b_s, sw, lane);
      wave_lds_sync();
      float z[NOUT];
      get_head(sw + lane * kSlot, z);
#pragma unroll
      for (int i = 0; i < 9; ++i) gn[i] = g[i];
      collide<WALLS>(gn, z, tau, sdelta, gx, M);
    }
    float *buf = state_s[s & 1];
#pragma unroll
    for (int i = 1; i < 9; ++i) buf[(i - 1) * THREADS + threadIdx.x] = gn[i];
    if (flags) {
      float msum = 0.0f, least = INFINITY;
#pragma unroll
      for (int i = 0; i < 9; ++i) {
        least = fminf(least, gn[i] + lbm::wgt<float>(i));
        msum += gn[i];
      }
      const bool bad = valid && !(least >= 0.0f && fabsf(msum) < INFINITY);
      const Q80 none{0ull, 0ll};
      put_partial(part_s[s & 1], valid ? q80_add_f32(none, msum) : none, bad ? 1u : 0u);
    }
    __syncthreads();
    if (flags) {
      const PartialSlot sum = sum_partials(part_s[s & 1], 0, W);
      const double m_new = (double)nodes + q80_value(sum.mass);
      unsigned fl = sum.flag;
      if (!(fabs(m_new - m_prev) / m_prev <= threshold)) fl |= 2u;
      m_prev = m_new;
      if (fl) {  // the whole workgroup
        seen |= fl;
        ++fell;
#pragma unroll
        for (int i = 0; i < 9; ++i) gn[i] = g[i];
        if constexpr (WALLS)
          lbm::forced_collide(gn, omega, gx);
        else
          lbm::bgk_collide(gn, omega);
#pragma unroll
        for (int i = 1; i < 9; ++i) buf[(i - 1) * THREADS + threadIdx.x] = gn[i];
        double m = 0.0;
#pragma unroll
        for (int i = 0; i < 9; ++i) m += valid ? (double)gn[i] : 0.0;
#pragma unroll
        for (int d = 32; d > 0; d >>= 1) m += __shfl_xor(m, d);
        if (lane == 0) sum_s[wave] = m;
        __syncthreads();
        m = sum_s[0];
        for (int v = 1; v < W; ++v) m += sum_s[v];
        m_prev = (double)nodes + m;
        // (the next step's barrier stands between these reads and new sums)
      }
    }
    g[0] = gn[0];
    if (s + 1 < nsteps) {
#pragma unroll
      for (int i = 1; i < 9; ++i) g[i] = buf[from[i]];
    } else if (valid) {
      float *d = dst + (size_t)y * 9 * nx + x;
#pragma unroll
      for (int i = 0; i < 9; ++i) d[(size_t)i * nx] = gn[i];
    }
  }
  if (flags && threadIdx.x == 0) {
    if (seen) *flags |= seen;
    if (n_fallback) *n_fallback += fell;
    *mass = m_prev;
  }
}

}  // namespace simple

// The gate's fallback kernel, shared with the message-passing step (gnn_kernels.hip).
int launch_gate(const float *g_src, float *g_dst, int nx, int ny, float tau, int walls,
                float gx, const lbm_fallback *fb, const void *pmass, const void *pflag,
                int nparts, void *pmass2, void *ctrl, int turn, bool more, hipStream_t s);

}  // namespace gnn

using namespace gnn;
using lbm::check_device;
using lbm::fail;
using lbm::launch_check;

static inline void *at_(void *base, size_t off) { return (uint8_t *)base + off; }

// pull: the fused step (else the forward of pre-collision states); walls: the
// channel step (with pull), body force rho * gx along x.
static int launch_simple(bool pull, bool walls, float gx, const float *src, float *dst,
                         int batch, int nx, int ny, const float *tau_arr, float tau,
                         const float *params, float *head_out, float *save_z0, void *ws,
                         const lbm_fallback *fb, int *nparts, hipStream_t s,
                         bool packed = false) {
  const FragLayout F = frag_layout(0);
  const SimpleScratch W = simple_scratch();
  uint8_t *pack = (uint8_t *)at_(ws, W.pack);
  unsigned *ctrl = (unsigned *)at_(ws, W.ctrl);
  if (!packed)
    if (int rc = launch_prep(params, 0, pack, ctrl, fb ? fb->mass : nullptr, s)) return rc;
  const long long chunks = (long long)batch * ny * ((nx + 63) / 64);
  long long blocks = (chunks + simple::kWaves - 1) / simple::kWaves;
  // the resident blocks; their waves draw the chunks from a counter
  long long cap = (long long)lbm::device_cus() * simple::kBlocksPerCu;
  if (cap > kMaxGnnBlocks) cap = kMaxGnnBlocks;
  const int nb = (int)(blocks < cap ? blocks : cap);
  *nparts = nb;
  Q80 *pm = (Q80 *)at_(ws, W.pmass);
  unsigned *pf = (unsigned *)at_(ws, W.pflag);
  if (pull && walls)
    hipLaunchKernelGGL((simple::simple_step_kernel<true, true>), dim3(nb),
                       dim3(simple::kThreads), 0, s, src, dst, batch, nx, ny, tau_arr, tau, gx,
                       pack, F, head_out, pm, pf, save_z0, ctrl + kCtrlChunkQueue);
  else if (pull)
    hipLaunchKernelGGL((simple::simple_step_kernel<true, false>), dim3(nb),
                       dim3(simple::kThreads), 0, s, src, dst, batch, nx, ny, tau_arr, tau, 0.0f,
                       pack, F, head_out, pm, pf, save_z0, ctrl + kCtrlChunkQueue);
  else
    hipLaunchKernelGGL((simple::simple_step_kernel<false, false>), dim3(nb),
                       dim3(simple::kThreads), 0, s, src, dst, batch, nx, ny, tau_arr, tau, 0.0f,
                       pack, F, head_out, pm, pf, save_z0, ctrl + kCtrlChunkQueue);
  return launch_check("simple_step_kernel");
}

// nsteps steps of a lattice of up to simple::kResidentNodes nodes.
static int launch_simple_resident(bool walls, float gx, const float *src, float *dst, int nx,
                                  int ny, float tau, const float *params, int nsteps, void *ws,
                                  const lbm_fallback *fb, hipStream_t s) {
  const SimpleScratch W = simple_scratch();
  uint8_t *pack = (uint8_t *)at_(ws, W.pack);
  if (int rc = launch_prep(params, 0, pack, nullptr, nullptr, s)) return rc;
  const FragLayout F = frag_layout(0);
  const double threshold = fb ? fb->drift_threshold : 0.0;
  unsigned *flags = fb ? fb->flags : nullptr, *nf = fb ? fb->n_fallback : nullptr;
  double *mass = fb ? fb->mass : nullptr;
  const int nodes = nx * ny;
  auto launch = [&](auto kernel, int threads) {
    hipLaunchKernelGGL(kernel, dim3(1), dim3(threads), 0, s, src, dst, nx, ny, nsteps, tau, gx,
                       pack, F, threshold, flags, nf, mass);
    return launch_check("simple_resident_kernel");
  };
  // (fewer waves, fewer to wait for at the barrier)
  if (nodes <= 128)
    return walls ? launch(simple::simple_resident_kernel<true, 128>, 128)
                 : launch(simple::simple_resident_kernel<false, 128>, 128);
  if (nodes <= 256)
    return walls ? launch(simple::simple_resident_kernel<true, 256>, 256)
                 : launch(simple::simple_resident_kernel<false, 256>, 256);
  if (nodes <= 512)
    return walls ? launch(simple::simple_resident_kernel<true, 512>, 512)
                 : launch(simple::simple_resident_kernel<false, 512>, 512);
  return walls ? launch(simple::simple_resident_kernel<true, 1024>, 1024)
               : launch(simple::simple_resident_kernel<false, 1024>, 1024);
}

static int check_simple(const char *who, int batch, int nx, int ny, const float *params) {
  if (!params) return fail(LBM_EINVAL, "%s: null parameters", who);
  if (batch < 1 || !lbm::lattice_ok(nx, ny) || (long long)batch * nx * ny >= (1LL << 31))
    return fail(LBM_EINVAL, "%s: bad sizes batch %d, %d x %d", who, batch, nx, ny);
  return LBM_OK;
}

extern "C" int simple_forward(const float *g_pre, float *g_post, int batch, int nx, int ny,
                              const float *tau, const float *params, float *head_out,
                              void *saved, size_t saved_bytes, void *workspace,
                              size_t ws_bytes, void *stream) {
  if (int rc = check_simple("simple_forward", batch, nx, ny, params)) return rc;
  if (!g_pre || !g_post || !tau) return fail(LBM_EINVAL, "simple_forward: null pointer");
  if (lbm::overlap(g_pre, g_post, (size_t)batch * 9 * nx * ny * sizeof(float)))
    return fail(LBM_EINVAL, "simple_forward: g_pre and g_post overlap");
  if (!workspace || ws_bytes < simple_scratch().total)
    return fail(LBM_EWORKSPACE, "simple_forward: workspace needs %zu bytes",
                simple_scratch().total);
  const SavedLayout SL = saved_layout((long long)batch * nx * ny, 0);
  if (saved && saved_bytes < SL.total)
    return fail(LBM_EWORKSPACE, "simple_forward: saved buffer needs %zu bytes", SL.total);
  if (int rc = check_device()) return rc;
  int nparts;
  return launch_simple(false, false, 0.0f, g_pre, g_post, batch, nx, ny, tau, 0.0f, params,
                       head_out, saved ? (float *)at_(saved, SL.z) : nullptr, workspace, nullptr,
                       &nparts, (hipStream_t)stream);
}

// One step and its gate; turn: its number since the weights were packed (0 packs
// them; without a gate, which zeroes the work counters, every step does); more:
// another follows.
static int gated_step(const float *g_src, float *g_dst, int nx, int ny, float tau, bool walls,
                      float gx, const float *params, const lbm_fallback *fb, void *workspace,
                      int turn, bool more, hipStream_t s) {
  int nparts;
  if (int rc = launch_simple(true, walls, gx, g_src, g_dst, 1, nx, ny, nullptr, tau, params,
                             nullptr, nullptr, workspace, fb, &nparts, s, fb && turn > 0))
    return rc;
  if (!fb) return LBM_OK;
  const SimpleScratch W = simple_scratch();
  return launch_gate(g_src, g_dst, nx, ny, tau, walls ? 1 : 0, gx, fb, at_(workspace, W.pmass),
                     at_(workspace, W.pflag), nparts, at_(workspace, W.pmass2),
                     at_(workspace, W.ctrl), turn, more, s);
}

static int check_step_simple(const char *who, const float *g_src, const float *g_dst, int nx,
                             int ny, float tau, bool walls, float gx, const float *params,
                             const lbm_fallback *fb, void *workspace, size_t ws_bytes) {
  if (int rc = check_simple(who, 1, nx, ny, params)) return rc;
  if (!g_src || !g_dst) return fail(LBM_EINVAL, "%s: null pointer", who);
  if (!(tau > 0.0f)) return fail(LBM_EINVAL, "%s: tau must be positive", who);
  if (walls && !(gx == gx && fabsf(gx) < INFINITY))
    return fail(LBM_EINVAL, "%s: force must be finite", who);
  if (lbm::overlap(g_src, g_dst, (size_t)9 * nx * ny * sizeof(float)))
    return fail(LBM_EINVAL, "%s: source and destination overlap", who);
  if (fb && (!fb->flags || !fb->mass))
    return fail(LBM_EINVAL, "%s: fallback needs flags and mass pointers", who);
  if (!workspace || ws_bytes < simple_scratch().total)
    return fail(LBM_EWORKSPACE, "%s: workspace needs %zu bytes", who, simple_scratch().total);
  return LBM_OK;
}

namespace gnn {

int steps_simple_pair(const char *who, float *g_a, float *g_b, int nx, int ny, float tau,
                      const float *params, int nsteps, const lbm_fallback *fb, void *workspace,
                      size_t ws_bytes, hipStream_t s) {
  if (int rc = check_step_simple(who, g_a, g_b, nx, ny, tau, false, 0.0f, params, fb, workspace,
                                 ws_bytes))
    return rc;
  if (int rc = check_device()) return rc;
  const bool resident = (long long)nx * ny <= simple::kResidentNodes;
  for (int k = 0; k < nsteps; ++k) {
    float *src = k & 1 ? g_b : g_a, *dst = k & 1 ? g_a : g_b;
    if (int rc = resident ? launch_simple_resident(false, 0.0f, src, dst, nx, ny, tau, params, 1,
                                                   workspace, fb, s)
                          : gated_step(src, dst, nx, ny, tau, false, 0.0f, params, fb, workspace,
                                       k, k + 1 < nsteps, s))
      return rc;
  }
  return LBM_OK;
}

}  // namespace gnn

// The fused step, periodic (walls = 0) or the channel (walls = 1, force gx).
static int step_simple(const char *who, const float *g_src, float *g_dst, int nx, int ny,
                       float tau, bool walls, float gx, const float *params, int nsteps,
                       const lbm_fallback *fb, void *workspace, size_t ws_bytes, void *stream) {
  if (int rc = check_step_simple(who, g_src, g_dst, nx, ny, tau, walls, gx, params, fb, workspace,
                                 ws_bytes))
    return rc;
  const int most = lbm_steps_simple_max(nx, ny);
  if (nsteps < 1 || nsteps > most)
    return fail(LBM_EINVAL, "%s: %d steps, not 1 to %d", who, nsteps, most);
  if (int rc = check_device()) return rc;
  hipStream_t s = (hipStream_t)stream;
  if ((long long)nx * ny <= simple::kResidentNodes)
    return launch_simple_resident(walls, gx, g_src, g_dst, nx, ny, tau, params, nsteps, workspace,
                                  fb, s);
  return gated_step(g_src, g_dst, nx, ny, tau, walls, gx, params, fb, workspace, 0, false, s);
}

extern "C" int lbm_step_simple(const float *g_src, float *g_dst, int nx, int ny, float tau,
                               const float *params, const lbm_fallback *fb, void *workspace,
                               size_t ws_bytes, void *stream) {
  return step_simple("lbm_step_simple", g_src, g_dst, nx, ny, tau, false, 0.0f, params, 1, fb,
                     workspace, ws_bytes, stream);
}

extern "C" int lbm_step_simple_channel(const float *g_src, float *g_dst, int nx, int ny,
                                       float tau, float gx, const float *params,
                                       const lbm_fallback *fb, void *workspace,
                                       size_t ws_bytes, void *stream) {
  return step_simple("lbm_step_simple_channel", g_src, g_dst, nx, ny, tau, true, gx, params, 1, fb,
                     workspace, ws_bytes, stream);
}

extern "C" int lbm_steps_simple_max(int nx, int ny) {
  return lbm::lattice_ok(nx, ny) && (long long)nx * ny <= simple::kResidentNodes
             ? simple::kResidentSteps
             : 1;
}

extern "C" int lbm_steps_simple(const float *g_src, float *g_dst, int nx, int ny, float tau,
                                const float *params, int nsteps, const lbm_fallback *fb,
                                void *workspace, size_t ws_bytes, void *stream) {
  return step_simple("lbm_steps_simple", g_src, g_dst, nx, ny, tau, false, 0.0f, params, nsteps,
                     fb, workspace, ws_bytes, stream);
}

extern "C" int lbm_steps_simple_channel(const float *g_src, float *g_dst, int nx, int ny,
                                        float tau, float gx, const float *params, int nsteps,
                                        const lbm_fallback *fb, void *workspace, size_t ws_bytes,
                                        void *stream) {
  return step_simple("lbm_steps_simple_channel", g_src, g_dst, nx, ny, tau, true, gx, params,
                     nsteps, fb, workspace, ws_bytes, stream);
}
