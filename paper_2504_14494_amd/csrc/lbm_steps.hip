// Several BGK steps in one pass over the lattice: plain and channel, FP32 and
// FP64.  A step alone reads and writes every population once and runs at the
// rate of a copy; a call here reads the state, advances it nsteps times on the
// chip and writes only the last state, with the arithmetic of the single
// step at every node of every step, so the result is bitwise that of nsteps
// single steps.
#include "channel_common.hpp"
#include "lbm_common.hpp"

namespace lbm {

// ------------------------------------------------------------- marching ---

__device__ __forceinline__ double wave_from_left(double v, double) {
  const uint64_t b = __builtin_bit_cast(uint64_t, v);
  const uint32_t lo = __builtin_amdgcn_update_dpp((int)b, (int)b, 0x138, 0xF, 0xF, false);
  const uint32_t hi =
      __builtin_amdgcn_update_dpp((int)(b >> 32), (int)(b >> 32), 0x138, 0xF, 0xF, false);
  return __builtin_bit_cast(double, (uint64_t)hi << 32 | lo);
}
__device__ __forceinline__ double wave_from_right(double v, double) {
  const uint64_t b = __builtin_bit_cast(uint64_t, v);
  const uint32_t lo = __builtin_amdgcn_update_dpp((int)b, (int)b, 0x130, 0xF, 0xF, false);
  const uint32_t hi =
      __builtin_amdgcn_update_dpp((int)(b >> 32), (int)(b >> 32), 0x130, 0xF, 0xF, false);
  return __builtin_bit_cast(double, (uint64_t)hi << 32 | lo);
}

template <typename T, bool WALLS>
__device__ __forceinline__ void collide_at(T (&g)[9], T omega, T gx) {
  if constexpr (WALLS)
    forced_collide(g, omega, gx);
  else
    bgk_collide(g, omega);
}

// What a stage of the march keeps of the rows the stage before it has made:
// of the last row the populations that stay in their row (m) and those that
// move up (up1), of the row below it those that move up, already moved along
// x (up0).
template <typename T>
struct StageRows {
  T m[3];    // 0, 1, 3
  T up1[3];  // 2, 5, 6
  T up0[3];
};

// Stage step: o holds row r of the stage before, in all nine directions; the
// stage forms its own row r - 1 from it and from the rows it has kept, and o
// becomes that row.
template <typename T, bool WALLS>
__device__ __forceinline__ void stage_row(StageRows<T> &S, T (&o)[9], int r, int ny, T omega,
                                          T gx) {
  T g[9];
  g[0] = S.m[0];
  g[1] = wave_from_left(S.m[1], S.m[1]);
  g[3] = wave_from_right(S.m[2], S.m[2]);
  g[2] = S.up0[0];
  g[5] = S.up0[1];
  g[6] = S.up0[2];
  g[4] = o[4];
  g[7] = wave_from_right(o[7], o[7]);
  g[8] = wave_from_left(o[8], o[8]);
  if (WALLS && r == ny) {  // row ny - 1: what went up comes back from the wall
    g[4] = S.up1[0];
    g[7] = S.up1[1];
    g[8] = S.up1[2];
  }
  S.up0[0] = S.up1[0];
  S.up0[1] = wave_from_left(S.up1[1], S.up1[1]);
  S.up0[2] = wave_from_right(S.up1[2], S.up1[2]);
  if (WALLS && r == 0) {  // row 0 next: what went down comes back
    S.up0[0] = o[4];
    S.up0[1] = o[7];
    S.up0[2] = o[8];
  }
  S.up1[0] = o[2];
  S.up1[1] = o[5];
  S.up1[2] = o[6];
  S.m[0] = o[0];
  S.m[1] = o[1];
  S.m[2] = o[3];
  collide_at<T, WALLS>(g, omega, gx);
#pragma unroll
  for (int i = 0; i < 9; ++i) o[i] = g[i];
}

constexpr int kMarchThreads = 256;
constexpr int kMarchWaves = kMarchThreads / 64;

// K steps at once by waves that march up the lattice.  A wave owns `width`
// columns of rows y0 .. y0 + height - 1 and holds 64: one column per lane, K - 1
// more on either side.  At row t its stage 1 pulls row t from memory and
// collides, stage 2 does row t - 1 from stage 1's rows, and so on; stage K
// stores row t - K + 1.  Stages pass rows on in registers: a population that
// moves along x comes from the neighbouring lane (DPP), one that moves along
// y waits a row or two (StageRows), so there is neither LDS nor a barrier.
// Each stage spoils one more lane at either end of the wave, which is
// why only 64 - 2 (K - 1) columns come out, and a segment starts K - 1 rows
// early and ends K - 1 late.
// Workgroup b of a grid of n in the order that keeps neighbours on one XCD:
// consecutive workgroups go to the eight XCDs in turn, so each XCD takes one
// contiguous eighth (any n).
__device__ __forceinline__ int xcd_order(int b, int n) {
  const int x = b & 7, q = n >> 3, r = n & 7;
  return x * q + (x < r ? x : r) + (b >> 3);
}

template <typename T, int K, bool WALLS>
__global__ __launch_bounds__(kMarchThreads) void march_kernel(
    const T *__restrict__ src, T *__restrict__ dst, int nx, int ny, int width, int height,
    int bxn, int cached, T omega, T gx) {
  const int lane = threadIdx.x & 63;
  const int wave = __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
  const int bid = xcd_order(blockIdx.x, gridDim.x);
  const int seg = bid / bxn;
  const int cols = kMarchWaves * width;          // columns of the workgroup
  const int xb = (bid - seg * bxn) * cols;       // its first one
  const int xs = xb + wave * width;
  int xc = (xs - (K - 1) + lane) % nx;
  xc = xc < 0 ? xc + nx : xc;
  const unsigned xm = xc == 0 ? nx - 1 : xc - 1, xp = xc == nx - 1 ? 0 : xc + 1, x0 = xc;
  __shared__ T rows[2][9][kMarchWaves * (64 - 2 * (K - 1))];
  const bool mine = lane >= K - 1 && lane < K - 1 + width;
  const int slot = wave * width + lane - (K - 1);
  const bool out = (int)threadIdx.x < cols && xb + (int)threadIdx.x < nx;
  const int y0 = seg * height, y1 = y0 + height < ny ? y0 + height : ny;
  const size_t row = (size_t)9 * nx;

  // Row pointers of the row to be loaded next and its neighbours, kept along
  // the march; element x of a row is at a 32-bit byte offset from a scalar
  // base (the host keeps nx below 2^28).
  unsigned o0 = x0 * (unsigned)sizeof(T), om = xm * (unsigned)sizeof(T),
           op = xp * (unsigned)sizeof(T);
  // (opaque in each row: hoisted out of the loop, the offsets become 64-bit
  // and every access an address addition of its own)
  auto opaque = [&]() {
    asm volatile("" : "+v"(o0));
    asm volatile("" : "+v"(om));
    asm volatile("" : "+v"(op));
  };
  auto at = [](const T *base, unsigned off) { return *(const T *)((const char *)base + off); };
  const unsigned so = (unsigned)(xb + (int)threadIdx.x) * (unsigned)sizeof(T);
  auto wrap = [&](int t) {
    if (WALLS) return t < 0 ? 0 : (t >= ny ? ny - 1 : t);  // rows off the channel: unused
    t %= ny;
    return t < 0 ? t + ny : t;
  };
  const int t0 = y0 - (K - 1), t1 = y1 + (K - 1);
  int r = wrap(t0);        // row loaded next
  int tl = t0;             // the same before wrapping
  auto load = [&](T(&g)[9]) {
    opaque();
    const T *r0 = src + (size_t)r * row;
    if constexpr (WALLS) {
      pull9_walls(src, nx, ny, xc, r, g);
      ++tl;
      r = tl < 0 ? 0 : (tl >= ny ? ny - 1 : tl);
    } else {
      const T *rm = src + (size_t)(r == 0 ? ny - 1 : r - 1) * row;
      r = r == ny - 1 ? 0 : r + 1;
      const T *rp = src + (size_t)r * row;
      g[0] = at(r0, o0);
      g[1] = at(r0 + nx, om);
      g[2] = at(rm + (size_t)2 * nx, o0);
      g[3] = at(r0 + (size_t)3 * nx, op);
      g[4] = at(rp + (size_t)4 * nx, o0);
      g[5] = at(rm + (size_t)5 * nx, om);
      g[6] = at(rm + (size_t)6 * nx, op);
      g[7] = at(rp + (size_t)7 * nx, op);
      g[8] = at(rp + (size_t)8 * nx, om);
    }
  };

  StageRows<T> S[K - 1] = {};
  auto step = [&](int t, T(&g)[9]) {
    collide_at<T, WALLS>(g, omega, gx);
#pragma unroll
    for (int s = 0; s < K - 1; ++s) stage_row<T, WALLS>(S[s], g, t - s, ny, omega, gx);
    const int y = t - (K - 1);
    if (y >= y0 && y < y1) {
      T(&buf)[9][kMarchWaves * (64 - 2 * (K - 1))] = rows[t & 1];
      if (mine)
#pragma unroll
        for (int i = 0; i < 9; ++i) buf[i][slot] = g[i];
      asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory");
      if (out) {
        unsigned o = so;
        asm volatile("" : "+v"(o));
        T *d = dst + (size_t)y * row;
        if (cached) {
#pragma unroll
          for (int i = 0; i < 9; ++i) *(T *)((char *)(d + (size_t)i * nx) + o) = buf[i][threadIdx.x];
        } else {
#pragma unroll
          for (int i = 0; i < 9; ++i)
            __builtin_nontemporal_store(buf[i][threadIdx.x],
                                        (T *)((char *)(d + (size_t)i * nx) + o));
        }
      }
    }
  };
  // two rows per turn, so that the rows kept and the row loaded ahead change
  // names instead of registers; a last odd row is computed and not stored
  T ga[9], gb[9];
  load(ga);
  for (int t = t0; t < t1; t += 2) {
    load(gb);
    step(t, ga);
    load(ga);
    step(t + 1, gb);
  }
}

// ----------------------------------------------------------------- tiles ---

// nsteps steps of a region of rx x ry nodes, one node per thread, passed from
// step to step through LDS (the eight directions that move, PLANE values each;
// one barrier per step with two buffers in turn, two with one).  The first step pulls
// from memory.  RESIDENT: the region is the whole lattice, whose neighbours
// wrap inside it, and nsteps is any number; else every further step spoils one
// more ring of the region, and the nodes at least nsteps - 1 away from its edge
// are stored.
//
// A step is some 100 VALU instructions and 16 LDS accesses; PLANE is a constant,
// and the steps come in pairs, so that the places in LDS are offsets of the
// accesses instead of 16 additions (1024 steps of 64^2: 851 -> 767 us; 2048 of a
// 4 x 32 channel, resident: 782 -> 629; pairs of one 512^2 FP64 run: -2 %).
template <typename T, bool WALLS, bool RESIDENT, int PLANE>
__global__ __launch_bounds__(PLANE) void tile_kernel(const T *__restrict__ src,
                                                            T *__restrict__ dst, int nx, int ny,
                                                            int rx, int ry, unsigned inv_rx,
                                                            int nsteps, int txn, T omega,
                                                            T gx) {
  // two buffers while two workgroups still fit the LDS of a CU
  constexpr int kBufs = 2 * 8 * PLANE * sizeof(T) <= 65536 ? 2 : 1;
  __shared__ T lds[kBufs * 8 * PLANE];
  const int nodes = rx * ry;
  const int halo = RESIDENT ? 0 : nsteps - 1;
  const int k = threadIdx.x < (unsigned)nodes ? (int)threadIdx.x : nodes - 1;
  // The entry was as many instructions as three steps: no divisions by the region's
  // or the lattice's sides (k < 2^10 and inv_rx = ceil(2^20 / rx) give k / rx
  // exactly), and the neighbours' places are sums.
  const int ty = (int)(__umul24((unsigned)k, inv_rx) >> 20), tx = k - (int)__umul24(ty, rx);
  const int by = blockIdx.x / txn, bx = blockIdx.x - by * txn;
  const int xg = bx * (rx - 2 * halo) + tx - halo, yg = by * (ry - 2 * halo) + ty - halo;
  int x = xg < 0 ? xg + nx : (xg >= nx ? xg - nx : xg);
  int y = yg < 0 ? yg + ny : (yg >= ny ? yg - ny : yg);
  if (nx < rx || ny < ry) {  // lattices narrower than a region
    x = xg % nx;
    y = yg % ny;
    x = x < 0 ? x + nx : x;
    y = y < 0 ? y + ny : y;
  }
  if (WALLS) y = yg < 0 ? 0 : (yg >= ny ? ny - 1 : yg);
  T g[9];
  if constexpr (WALLS)
    pull9_walls(src, nx, ny, x, y, g);
  else
    pull9(src, nx, ny, x, y, g);
  collide_at<T, WALLS>(g, omega, gx);
  // where population i of the next step comes from (the edge of a region
  // reads itself: those nodes are spoilt anyway)
  const int last_x = rx - 1, last_y = (int)__umul24(ry - 1, rx);
  const int left = tx > 0 ? -1 : (RESIDENT ? last_x : 0);
  const int right = tx < last_x ? 1 : (RESIDENT ? -last_x : 0);
  const int down = ty > 0 ? -rx : (RESIDENT && !WALLS ? last_y : 0);
  const int up = ty < ry - 1 ? rx : (RESIDENT && !WALLS ? -last_y : 0);
  int from[9];
#pragma unroll
  for (int i = 1; i < 9; ++i) {
    from[i] = (i - 1) * PLANE + k + (cx(i) > 0 ? left : cx(i) < 0 ? right : 0) +
              (cy(i) > 0 ? down : cy(i) < 0 ? up : 0);
    if (WALLS && ((cy(i) > 0 && yg == 0) || (cy(i) < 0 && yg == ny - 1)))
      from[i] = (opp(i) - 1) * PLANE + k;
    asm volatile("" : "+v"(from[i]));  // not put together again at every step
  }
  auto step = [&](T *buf) {
#pragma unroll
    for (int i = 1; i < 9; ++i) buf[(i - 1) * PLANE + threadIdx.x] = g[i];
    __syncthreads();
#pragma unroll
    for (int i = 1; i < 9; ++i) g[i] = buf[from[i]];
    if (kBufs == 1) __syncthreads();
    collide_at<T, WALLS>(g, omega, gx);
  };
  int s = 1;
  for (; s + 1 < nsteps; s += 2) {
    step(lds + (kBufs - 1) * 8 * PLANE);
    step(lds);
  }
  if (s < nsteps) step(lds + (kBufs - 1) * 8 * PLANE);
  if (threadIdx.x < (unsigned)nodes && tx >= halo && tx < rx - halo && ty >= halo &&
      ty < ry - halo && xg < nx && yg < ny) {
    T *d = dst + (size_t)yg * 9 * nx + xg;
#pragma unroll
    for (int i = 0; i < 9; ++i) d[(size_t)i * nx] = g[i];
  }
}

}  // namespace lbm

// ---------------------------------------------------------------- dispatch ---

namespace lbm {

enum StepsKind { kStepsResident, kStepsTile, kStepsMarch };

// How several steps of an nx x ny lattice are taken together, and at most how
// many.  Where the lines lie (us per step of lattices stepped back and forth
// between two buffers in a captured graph, FP32 unless FP64 is said; the single
// step takes 2.6 at 64^2, 3.4 at 256^2, 5.8 at 512^2, 14.3 at 1024^2):
//  - up to 1024 nodes one workgroup holds the lattice, and a step costs its
//    barrier and its latency: 0.31 at 4 x 32, 0.64 at 32^2, 0.80 in tiles;
//  - then tiles; small regions spread a small lattice over more CUs, large ones
//    recompute less: 64^2: 0.80 with 32 x 16, 1.02 with 32 x 32; 128^2: 1.00 with
//    24 x 24, 1.06 with 32 x 32; 256^2: 1.46 with 32 x 32, 1.86 with 24 x 24.
//    Eight steps while the launch counts, five beyond (512^2: 2.49, six 2.85;
//    FP64 3.61, six 3.99);
//  - from about 700,000 nodes (500,000 in FP64) the march, which recomputes
//    next to nothing but needs many waves: 512^2 3.2, 1024^2 5.8 against 7.7 in
//    tiles; FP64 4.2 and 10.3.  It takes 224 columns at a time, so lattices
//    that would leave most of them idle stay with the tiles.
// March: five steps where the state leaves the Infinity Cache (8192^2: 217 us per
// step; four at a time 14 % slower, six 1 % faster with three waves per SIMD
// left), four where it stays (1501 x 1003: 6.6 against 7.0), and fewer in
// FP64, whose rows take twice the registers.
// Lattices of few rows.  A region of 32 x 32 that steps one row five times makes use
// of 24 of its 1024 nodes: 480,000 x 1 took 42 us per step (single steps 7.3), 240,000 x 2 with
// walls in FP64 60 (15.0).  So a region that has more rows than the lattice and its
// halos takes just those and is wider instead, if the tiles would be more than one per
// CU (below, their latency counts, and they stay ahead whatever they recompute):
// as many steps as leave one per CU (20,000 x 1 with walls in FP64: 2.0 with six, 3.3
// with eight), else ny + 1; more recompute more than they save, and on one row two at
// once are no faster than single steps (240,000 x 1 with walls: 5.0 and 3.6).  In
// the march ny + 1 at most, too (4,000,000 x 1: 44 with two, 53 with four, single 50).
struct StepsPlan {
  StepsKind kind;
  int max_steps;  // that are worth taking at once (1: none)
  int limit;      // that are taken at all
  int rx, ry;     // tile region; ry 0: the lattice's rows (flat_region)
};

constexpr int kResidentNodes = 1024;
constexpr int kResidentSteps = 16384;      // a launch of some 10 ms at most
constexpr size_t kCacheBytes = 128u << 20;  // both buffers well inside the Infinity Cache
constexpr int kRegionNodes = 1024;
constexpr int kTilesAtOnce = 256;  // one per CU

static void flat_region(int ny, int nsteps, int &rx, int &ry) {
  ry = ny + 2 * (nsteps - 1);
  rx = kRegionNodes / ry;
}

static long long tiles_of(int nx, int ny, int rx, int ry, int nsteps) {
  const long long ox = rx - 2 * (nsteps - 1), oy = ry - 2 * (nsteps - 1);
  return ((nx + ox - 1) / ox) * ((ny + oy - 1) / oy);
}

static StepsPlan steps_plan(int nx, int ny, size_t elem, bool walls) {
  const long long nodes = (long long)nx * ny;
  if (nodes <= kResidentNodes) return {kStepsResident, kResidentSteps, kResidentSteps, nx, ny};
  const int block = kMarchWaves * 56;
  const long long covered = (long long)((nx + block - 1) / block) * block;
  const bool wide = 2LL * nx > covered && nx < (1 << 28);
  if (wide && nodes >= (elem == 4 ? 700000 : 500000)) {
    const int k = elem == 8 ? (walls ? 3 : 4)
                            : (walls || 2 * 9 * elem * nodes <= kCacheBytes ? 4 : 5);
    return {kStepsMarch, k < ny + 1 ? k : ny + 1, k, 0, 0};
  }
  const int k = nodes <= 131072 ? 8 : 5;
  const int rx = nodes <= 8192 ? 32 : nodes <= 32768 ? 24 : 32;
  const int ry = nodes <= 8192 ? 16 : nodes <= 32768 ? 24 : 32;
  if (ny + 2 * (k - 1) < ry &&
      tiles_of(nx, ny, rx, ry, k) * rx * ry > kTilesAtOnce * kRegionNodes) {
    int best = k;
    for (; best > 1; --best) {
      int fx, fy;
      flat_region(ny, best, fx, fy);
      if (tiles_of(nx, ny, fx, fy, best) <= kTilesAtOnce) break;
    }
    if (best == 1 && ny > 1) best = k < ny + 1 ? k : ny + 1;
    return {kStepsTile, best, k, 0, 0};
  }
  return {kStepsTile, k, k, rx, ry};
}

template <typename T, int K, bool WALLS>
static int launch_march(const T *src, T *dst, int nx, int ny, T omega, T gx, hipStream_t s) {
  static const int occ = [] {
    int v = 0;
    if (hipOccupancyMaxActiveBlocksPerMultiprocessor(
            &v, reinterpret_cast<const void *>(&march_kernel<T, K, WALLS>), kMarchThreads, 0) !=
            hipSuccess ||
        v < 1)
      v = 2;
    return v;
  }();
  const int width = 64 - 2 * (K - 1) < 56 ? 64 - 2 * (K - 1) : 56;
  const int bxn = (nx + kMarchWaves * width - 1) / (kMarchWaves * width);
  // Rows per segment: a segment costs height + 2 (K - 1) rows, and a row takes
  // about 5 + 3 o units when o workgroups share a CU (0.98, 1.3 and 1.7 us
  // for o = 1, 2, 3, four FP32 steps); beyond the resident workgroups, whole
  // rounds.
  const int cus = device_cus();
  long long best = -1;
  int height = ny;
  for (int n = 1; n <= occ * 64; ++n) {
    const long long segs = (long long)n * cus / bxn;
    if (segs < 1 || (n > occ && n % occ)) continue;
    const int h = (int)((ny + segs - 1) / segs);
    const int o = n < occ ? n : occ;
    const long long cost = (long long)(n / o) * (5 + 3 * o) * (h + 2 * (K - 1));
    if (h <= 128 && (best < 0 || cost < best)) {
      best = cost;
      height = h;
    }
  }
  if (best < 0) height = ny < 64 ? ny : 64;
  const long long blocks = (long long)bxn * ((ny + height - 1) / height);
  if (blocks > 0x7fffffffLL) return fail(LBM_EINVAL, "lbm_steps: lattice too large");
  const int cached = 2 * 9 * sizeof(T) * (size_t)nx * ny <= kCacheBytes;
  hipLaunchKernelGGL((march_kernel<T, K, WALLS>), dim3((unsigned)blocks), dim3(kMarchThreads), 0,
                     s, src, dst, nx, ny, width, height, bxn, cached, omega, gx);
  return launch_check("march_kernel");
}

template <typename T, bool WALLS>
static int launch_tiles(const T *src, T *dst, int nx, int ny, const StepsPlan &P, int nsteps,
                        T omega, T gx, hipStream_t s) {
  int rx = P.rx, ry = P.ry;
  if (!ry) flat_region(ny, nsteps, rx, ry);
  const unsigned inv_rx = ((1u << 20) + rx - 1) / rx;
  if (P.kind == kStepsResident) {
    const int nodes = nx * ny, threads = (nodes + 63) / 64 * 64;
    auto *kernel = threads <= 128   ? tile_kernel<T, WALLS, true, 128>
                   : threads <= 512 ? tile_kernel<T, WALLS, true, 512>
                                    : tile_kernel<T, WALLS, true, 1024>;
    hipLaunchKernelGGL(kernel, dim3(1), dim3(threads), 0, s, src, dst, nx, ny, nx, ny, inv_rx,
                       nsteps, 1, omega, gx);
    return launch_check("tile_kernel");
  }
  const int ox = rx - 2 * (nsteps - 1);
  const int txn = (nx + ox - 1) / ox;
  const long long blocks = tiles_of(nx, ny, rx, ry, nsteps);
  if (blocks > 0x7fffffffLL) return fail(LBM_EINVAL, "lbm_steps: lattice too large");
  const int threads = P.ry ? rx * ry : kRegionNodes;
  auto *kernel = threads == 512   ? tile_kernel<T, WALLS, false, 512>
                 : threads == 576 ? tile_kernel<T, WALLS, false, 576>
                                  : tile_kernel<T, WALLS, false, 1024>;
  hipLaunchKernelGGL(kernel, dim3((unsigned)blocks), dim3(threads), 0, s, src, dst, nx, ny, rx, ry,
                     inv_rx, nsteps, txn, omega, gx);
  return launch_check("tile_kernel");
}

template <typename T, bool WALLS>
static int steps_impl(const T *src, T *dst, int nx, int ny, T tau, T gx, int nsteps,
                      void *stream) {
  const char *who = WALLS ? "lbm_steps_channel" : "lbm_steps_bgk";
  if (!src || !dst) return fail(LBM_EINVAL, "%s: null pointer", who);
  if (!lattice_ok(nx, ny)) return fail(LBM_EINVAL, "%s: bad lattice %d x %d", who, nx, ny);
  if (!(tau > T(WALLS ? 0.5 : 0.0))) return fail(LBM_EINVAL, "%s: tau too small", who);
  if (overlap(src, dst, (size_t)9 * nx * ny * sizeof(T)))
    return fail(LBM_EINVAL, "%s: source and destination overlap", who);
  const StepsPlan P = steps_plan(nx, ny, sizeof(T), WALLS);
  if (nsteps < 2 || nsteps > P.limit)
    return fail(LBM_EINVAL, "%s: %d steps, not 2 to %d", who, nsteps, P.limit);
  if (int rc = check_device()) return rc;
  hipStream_t s = as_stream(stream);
  const T omega = T(1) / tau;
  if (P.kind != kStepsMarch)
    return launch_tiles<T, WALLS>(src, dst, nx, ny, P, nsteps, omega, gx, s);
  switch (nsteps) {
    case 2:
      return launch_march<T, 2, WALLS>(src, dst, nx, ny, omega, gx, s);
    case 3:
      return launch_march<T, 3, WALLS>(src, dst, nx, ny, omega, gx, s);
    case 4:
      if constexpr (!(WALLS && sizeof(T) == 8))
        return launch_march<T, 4, WALLS>(src, dst, nx, ny, omega, gx, s);
      break;
    case 5:
      if constexpr (!WALLS && sizeof(T) == 4)
        return launch_march<T, 5, WALLS>(src, dst, nx, ny, omega, gx, s);
      break;
  }
  return fail(LBM_EINVAL, "%s: %d steps", who, nsteps);
}

}  // namespace lbm

// ------------------------------------------------------------------- ABI ---

extern "C" int lbm_steps_max(int nx, int ny, int f64, int walls) {
  if (!lbm::lattice_ok(nx, ny)) return 1;
  return lbm::steps_plan(nx, ny, f64 ? 8 : 4, walls != 0).max_steps;
}

extern "C" int lbm_steps_bgk(const float *g_src, float *g_dst, int nx, int ny, float tau,
                             int nsteps, void *stream) {
  return lbm::steps_impl<float, false>(g_src, g_dst, nx, ny, tau, 0.0f, nsteps, stream);
}

extern "C" int lbm_steps_bgk_f64(const double *g_src, double *g_dst, int nx, int ny, double tau,
                                 int nsteps, void *stream) {
  return lbm::steps_impl<double, false>(g_src, g_dst, nx, ny, tau, 0.0, nsteps, stream);
}

extern "C" int lbm_steps_channel(const float *g_src, float *g_dst, int nx, int ny, float tau,
                                 float gx, int nsteps, void *stream) {
  return lbm::steps_impl<float, true>(g_src, g_dst, nx, ny, tau, gx, nsteps, stream);
}

extern "C" int lbm_steps_channel_f64(const double *g_src, double *g_dst, int nx, int ny,
                                     double tau, double gx, int nsteps, void *stream) {
  return lbm::steps_impl<double, true>(g_src, g_dst, nx, ny, tau, gx, nsteps, stream);
}
