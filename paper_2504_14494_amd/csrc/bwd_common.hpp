// Building blocks of the backward kernels: FP32 node vectors in accumulator
// order, transposed staging of node columns for the weight-gradient products,
// and the per-wave partial gradients.
#pragma once

#include "gnn_common.hpp"
#include "lbm_common.hpp"

namespace gnn {

using lbm::cx;
using lbm::cy;

constexpr int kBT = 256;            // threads per block
constexpr int kPitch = 40;          // BF16 per staged row: 32 nodes + padding

// Where a group of 16 nodes of a row lies, and this lane's node of it.  The
// group index is the same in every lane of a wave and fits 32 bits (fewer than
// 2^31 nodes), so the divisions run on scalar values: as 64-bit divisions per
// lane they were a quarter of the instructions of the node kernel's loop.
struct Pos {
  int b, y, x0, x;      // x clamped into the lattice for loads
  bool valid;
  int width;            // columns of the group inside the lattice
  int cols;             // the same, 0 past the last group
  size_t node0, node;   // the group's first node; this lane's (x) node
};

__device__ __forceinline__ Pos group_pos(unsigned grp, unsigned ngroups, int n, int nx, int ny,
                                         unsigned gxn) {
  Pos P;
  const unsigned gu = __builtin_amdgcn_readfirstlane(grp);
  const bool in = gu < ngroups;
  const unsigned g = in ? gu : 0u;
  const unsigned row = g / gxn, b = row / (unsigned)ny;
  P.b = (int)b;
  P.y = (int)(row - b * (unsigned)ny);
  P.x0 = (int)(g - row * gxn) * 16;
  P.width = nx - P.x0 < 16 ? nx - P.x0 : 16;
  P.cols = in ? P.width : 0;
  P.valid = n < P.cols;
  P.x = P.x0 + n;
  if (P.x0 + 16 > nx) P.x = P.x < nx ? P.x : P.x % nx;
  const size_t row0 = (size_t)row * nx;
  P.node0 = row0 + P.x0;
  P.node = row0 + P.x;
  return P;
}

// Node vectors between the backward kernels are kept by group: a group of c
// columns (16, or what is left of the row) holds planes of c 16-byte entries,
// one per 16 bytes of the vector, at its first node's share of the buffer.  Then
// 16 lanes read or write 256 contiguous bytes; node by node, a store instruction
// touched 64 lines with 16 bytes each, or 16 with 64.
//
// Stores go through a raw buffer resource over the group (rows_resource); lanes
// past its last column have an offset past its end and are dropped by the
// hardware, so that the stores are not under a branch, and waits for the loads of
// the next group, issued before them, need not wait for them too (vmcnt counts
// both, in order).  The whole offset is given per lane, never partly as the scalar
// offset: for that form the compiler leaves out the wait state before the store's
// data registers are written again, and the data stored was then, now and then,
// the next value in its first dword.
constexpr int kBufferNt = 2;  // non-temporal
__device__ __forceinline__ int plane_store_offset(const Pos &P, int n, int q) {
  return P.valid ? (q * P.cols + n) * 16 : 1 << 30;
}
// Byte offset of lane (n, q) in plane q of its group; lanes past the last column
// read that column.
__device__ __forceinline__ int plane_load_offset(const Pos &P, int n, int q) {
  return (q * P.width + (n < P.width ? n : P.width - 1)) * 16;
}

// FP32 vectors in accumulator order: lane (n, q) owns row tiles t = 0..3, 4
// values each, plane 4 t + q.  Tiles t0 .. t0 + NT - 1 here.
template <int NT>
__device__ __forceinline__ void load_acc(const float *buf, const Pos &P, int n, int q,
                                         f32x4 (&v)[NT], int t0 = 0) {
  const uint8_t *p = (const uint8_t *)buf + P.node0 * (HID * 4) + plane_load_offset(P, n, q);
#pragma unroll
  for (int t = 0; t < NT; ++t) v[t] = *(const f32x4 *)(p + (size_t)((t0 + t) * 64 * P.width));
}
template <int NT>
__device__ __forceinline__ void store_acc(float *buf, const Pos &P, int n, int q,
                                          const f32x4 (&v)[NT], int t0 = 0) {
  const __amdgpu_buffer_rsrc_t rs = rows_resource(buf, P.node0 * (HID * 4), P.cols * (HID * 4));
  const int off = plane_store_offset(P, n, q);
#pragma unroll
  for (int t = 0; t < NT; ++t)
    __builtin_amdgcn_raw_buffer_store_b128(__builtin_bit_cast(i32x4_t, v[t]), rs,
                                           off + (t0 + t) * 64 * P.cols, 0, 0);
}

// BF16 node state fragments (fragment order, see gnn_common.hpp).
__device__ __forceinline__ void load_frags(const uint16_t *h, size_t node, int q, u32x4 (&f)[2]) {
  const u32x4 *p = (const u32x4 *)(h + node * HID);
  f[0] = p[q];
  f[1] = p[4 + q];
}

__device__ __forceinline__ f32x4 unpack_lo(u32x4 v) {
  return f32x4{bf16_to_f32(v.x & 0xffffu), bf16_to_f32(v.x >> 16), bf16_to_f32(v.y & 0xffffu),
               bf16_to_f32(v.y >> 16)};
}
__device__ __forceinline__ f32x4 unpack_hi(u32x4 v) {
  return f32x4{bf16_to_f32(v.z & 0xffffu), bf16_to_f32(v.z >> 16), bf16_to_f32(v.w & 0xffffu),
               bf16_to_f32(v.w >> 16)};
}

__device__ __forceinline__ uint16_t bf16_bits(float v) {
  __bf16 b = (__bf16)v;
  return __builtin_bit_cast(uint16_t, b);
}

// Staging of one value per (channel row, node column), BF16, channel-major.
// Accumulator-layout vectors: lane (n, q) holds channels 16 t + 4 q + e.
template <int NT>
__device__ __forceinline__ void stage_acc(uint16_t *rows, const f32x4 (&v)[NT], int q, int col,
                                          int row0 = 0) {
#pragma unroll
  for (int t = 0; t < NT; ++t) {
    rows[(row0 + 16 * t + 4 * q + 0) * kPitch + col] = bf16_bits(v[t].x);
    rows[(row0 + 16 * t + 4 * q + 1) * kPitch + col] = bf16_bits(v[t].y);
    rows[(row0 + 16 * t + 4 * q + 2) * kPitch + col] = bf16_bits(v[t].z);
    rows[(row0 + 16 * t + 4 * q + 3) * kPitch + col] = bf16_bits(v[t].w);
  }
}
// Fragment-order vectors: element j of k-step s is channel c(s, q, j).
__device__ __forceinline__ void stage_frag1(uint16_t *rows, u32x4 f, int s, int q, int col) {
  const uint32_t w[4] = {f.x, f.y, f.z, f.w};
#pragma unroll
  for (int j = 0; j < 8; ++j)
    rows[frag_channel(s, q, j) * kPitch + col] =
        (uint16_t)((j & 1) ? (w[j >> 1] >> 16) : (w[j >> 1] & 0xffffu));
}
__device__ __forceinline__ void stage_frag(uint16_t *rows, const u32x4 (&f)[2], int q, int col,
                                           int row0 = 0) {
#pragma unroll
  for (int s = 0; s < 2; ++s) stage_frag1(rows + row0 * kPitch, f[s], s, q, col);
}
// Rows 8 q + j of a 16-row operand (features, head gradients), q < 2.
__device__ __forceinline__ void stage_rows16(uint16_t *rows, u32x4 f, int q, int col) {
  if (q >= 2) return;
  const uint32_t w[4] = {f.x, f.y, f.z, f.w};
#pragma unroll
  for (int j = 0; j < 8; ++j)
    rows[(8 * q + j) * kPitch + col] =
        (uint16_t)((j & 1) ? (w[j >> 1] >> 16) : (w[j >> 1] & 0xffffu));
}

// acc[mt][ct] += D^T-slice x A over the 32 staged nodes: rows of d are the
// output channels (16 mt + ...), rows of a the input channels (16 ct + ...).
template <int MT, int CT>
__device__ __forceinline__ void dw_mma(f32x4 (&acc)[MT][CT], const uint16_t *d,
                                       const uint16_t *a, int lane) {
  const int r = lane & 15, q = lane >> 4;
  u32x4 A[MT];
#pragma unroll
  for (int mt = 0; mt < MT; ++mt) A[mt] = *(const u32x4 *)(d + (16 * mt + r) * kPitch + 8 * q);
#pragma unroll
  for (int ct = 0; ct < CT; ++ct) {
    u32x4 B = *(const u32x4 *)(a + (16 * ct + r) * kPitch + 8 * q);
#pragma unroll
    for (int mt = 0; mt < MT; ++mt) acc[mt][ct] = mfma(A[mt], B, acc[mt][ct]);
  }
}

// Writes a dW accumulator block to this wave's partial: element
// (row 16 mt + 4 q + e, column col0 + 16 ct + (lane & 15)) of a row-major
// [rows][ld] matrix at `base`.
template <int MT, int CT>
__device__ __forceinline__ void write_dw(float *part, size_t base, int ld, int col0, int nrows,
                                         int ncols, const f32x4 (&acc)[MT][CT], int lane) {
  const int c = lane & 15, q = lane >> 4;
#pragma unroll
  for (int mt = 0; mt < MT; ++mt)
#pragma unroll
    for (int ct = 0; ct < CT; ++ct) {
      const float v[4] = {acc[mt][ct].x, acc[mt][ct].y, acc[mt][ct].z, acc[mt][ct].w};
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        int row = 16 * mt + 4 * q + e, col = 16 * ct + c;
        if (row < nrows && col < ncols) part[base + (size_t)row * ld + col0 + col] = v[e];
      }
    }
}

// Sums, over the 16 node lanes, per-lane accumulator-layout vectors (channel
// 16 t + 4 q + e) and writes the 64 channel totals to part[base + stride * ch].
__device__ __forceinline__ void write_vec(float *part, size_t base, int stride,
                                          const f32x4 (&v)[4], float *red, int lane) {
  const int q = lane >> 4;
#pragma unroll
  for (int t = 0; t < 4; ++t) {
    red[lane * 17 + 4 * t + 0] = v[t].x;
    red[lane * 17 + 4 * t + 1] = v[t].y;
    red[lane * 17 + 4 * t + 2] = v[t].z;
    red[lane * 17 + 4 * t + 3] = v[t].w;
  }
  wave_lds_sync();
  const int k = lane & 15;
  float s = 0.0f;
  for (int n = 0; n < 16; ++n) s += red[(16 * q + n) * 17 + k];
  const int ch = 16 * (k >> 2) + 4 * q + (k & 3);
  part[base + (size_t)stride * ch] = s;
  wave_lds_sync();
}

// The same for the half of the channels that wave `hh` of a pair holds; the two
// waves use different columns of `red`.
__device__ __forceinline__ void write_vec_half(float *part, size_t base, int stride, int hh,
                                               const f32x4 (&v)[2], float *red, int lane) {
  const int q = lane >> 4, k = lane & 15;
#pragma unroll
  for (int t = 0; t < 2; ++t) {
    float *o = red + lane * 17 + 8 * hh + 4 * t;
    o[0] = v[t].x;
    o[1] = v[t].y;
    o[2] = v[t].z;
    o[3] = v[t].w;
  }
  wave_lds_sync();
  if ((k >> 3) == hh) {
    float s = 0.0f;
    for (int n = 0; n < 16; ++n) s += red[(16 * q + n) * 17 + k];
    part[base + (size_t)stride * (16 * (k >> 2) + 4 * q + (k & 3))] = s;
  }
  wave_lds_sync();
}

// s_waitcnt vmcnt(n), n < 16, the other counters left at their maximum.
constexpr int wait_vmcnt(int n) { return 0x0F70 | n; }

// dL/dz of one node from dL/dg_post (Gi), its pre-collision populations and
// tau, but for the factor of dz[0] that depends on z_0.
__device__ __forceinline__ void head_gradient(const float (&g)[9], const float (&Gi)[9],
                                              float sdelta, float (&dz)[NOUT]) {
  const lbm::Moments<float> M = lbm::node_moments(g);
  float dta = 0.0f, m0 = 0.0f, mx = 0.0f, my = 0.0f;
#pragma unroll
  for (int i = 0; i < 9; ++i) {
    dta += Gi[i] * (g[i] - lbm::geq_of(i, M));
    m0 += Gi[i];
    mx += float(cx(i)) * Gi[i];
    my += float(cy(i)) * Gi[i];
  }
  dz[0] = dta;
#pragma unroll
  for (int i = 0; i < 9; ++i)
    dz[1 + i] = sdelta * (Gi[i] - m0 * (1.0f / 9.0f) - float(cx(i)) * mx * (1.0f / 6.0f) -
                          float(cy(i)) * my * (1.0f / 6.0f));
}
// dz[0] from what head_gradient left there.
__device__ __forceinline__ float tau_gradient(float dta, float z0, float tb) {
  const float s = 1.0f / (1.0f + expf(-z0));
  const float tadj = 0.5f + s;
  return dta / (tb * tadj * tadj) * s * (1.0f - s);
}

template <int DR, int AR>
struct Stage {
  uint16_t d[DR * kPitch];
  uint16_t a[AR * kPitch];
  float red[64 * 17];
};

}  // namespace gnn
