// Kernels of the single-lattice 2D solver.  One thread owns one lattice node.
#pragma once

#include "lbm_device.hpp"

namespace lbm {

constexpr int kBlock = 256;     // 4 wavefronts of 64 lanes along x
constexpr int kObsQ = 9;        // per-block observable partials

// Map a 2D launch (blocks along x, rows along y) so that the eight XCDs
// (which receive consecutive workgroups round-robin) each get a contiguous
// band of rows: spatial neighbours then share an L2.
__device__ __forceinline__ void xcd_tile(int nbx, int nby, int& bx, int& by) {
  const int flat = blockIdx.y * nbx + blockIdx.x;
  const int total = nbx * nby;
  // XCD j receives flats j, j+8, ...: full + (j < rem) workgroups.  Give it
  // the contiguous logical range starting at j*full + min(j, rem).
  const int xcd = flat & 7;
  const int slot = flat >> 3;
  const int full = total >> 3, rem = total & 7;
  const int logical = xcd * full + (xcd < rem ? xcd : rem) + slot;
  by = logical / nbx;
  bx = logical - by * nbx;
  // Rotate the x-blocks of a row by one every 8 rows.  Without it, the
  // workgroups that share a CU (a fixed stride apart in the XCD's range)
  // tend to sit at the same x position, so the wavefronts holding the inlet
  // or outlet column, whose chains are the longest, pile onto the same
  // SIMDs.  Measured: 1024x256 reverse step 2.6 % and forward 1.2 % faster,
  // 4096x1024 unchanged; each node's arithmetic is unchanged.
  bx = (bx + by / 8) % nbx;
}

// One time step: pull-stream, boundary columns, macros, flow collision,
// reaction, scalar collisions, store.  STREAM: non-temporal loads, each lane
// at its own addresses (see pull), and plain stores, for a state larger than
// the 256 MB last-level cache; smaller ones take cached loads and stores that
// write through to it (aux 16, sc1): the lines are there for the next step,
// and the end of the kernel has no L2 write-back to wait for.  Per step,
// streaming -> cached: 1024x256 FP32 9.8 -> 8.3 us, 2048x512 FP32 31.6 ->
// 25.0, 200x40 FP64 4.92 -> 4.67; 4096x1024 FP32 102.6 -> 120.
template <typename R, int MAT, bool STREAM>
__global__ __launch_bounds__(kBlock) void k_step(const R* __restrict__ src, R* __restrict__ dst,
                                                 const R* __restrict__ phi_f,
                                                 const R* __restrict__ invk_f,
                                                 const R* __restrict__ d_f, Consts<R> k) {
  int bx, by;
  xcd_tile(gridDim.x, gridDim.y, bx, by);
  const int x = bx * kBlock + threadIdx.x;
  const int y = by;
  if (x >= k.nx) return;
  R f[19];
  const Mat<R> mt = pre_collision<R, MAT, STREAM, !STREAM>(src, k, phi_f, invk_f, d_f, x, y, f, y);
  const bool cl = y >= k.y_cl0 && !(k.flags & F_NO_REACTION);
  collide(f, mt, k, cl);
  store_node<STREAM ? 0 : 16>(dst, k, x, y, y, f);
}

// Two time steps in one launch: a workgroup advances a tile of TX x TY
// nodes.  Step one runs over the tile and a halo (two columns on the left,
// where the outlet's feeding column can lie, one elsewhere, and a row above
// and below), one node per thread, from the state in memory, and keeps the
// post-collision populations in LDS, writing the tile's own to `mid` when
// that is given; step two pulls the tile's nodes from LDS and writes `dst`.
// Every node runs the same code as k_step, so the states are the bits of two
// single steps.  Walls and inlet / outlet columns only (the thin-film CL's
// reactive wall included): the host keeps single steps on periodic lattices.
//
// What bounds it depends on the size: the launch and one wavefront's chain
// (the smallest lattices), vector instructions and the overlap of a
// workgroup's load, compute and store phases (the largest: 65 % VALU busy).
// Tiles, per step (FP32 4096x1024, FP64 4096x1024, FP32 1537x431, FP32
// 1024x256; us): 64x12 89.0 / 154 / 15.3 / 8.5, 64x8 86.9 / 172 / 13.9 /
// 7.5, 32x12 86.1 / 147 / 12.4 / 7.9, 48x8 80.8 / 146 / 12.8 / 7.0.  48x8
// with its halo is 510 nodes for 512 threads, and four such workgroups (two
// in FP64) fill a CU's 32 (16) wavefronts with their 39 (78) KB of LDS each,
// so that one's loads run under another's arithmetic.  Lattices of fewer
// than 2^17 nodes, which leave CUs idle, take 16x8: 200x40 FP64 5.7 -> 3.7,
// 300x100 FP32 3.9 -> 3.7, 512x128 FP64 6.4 -> 6.0 (single steps: 4.7, 5.1,
// 7.9).  Loads are cached and stores write through at every size but FP32
// states beyond the last-level cache (4096x1024: 86.1 -> 80.8 without).
template <int TX, int TY>
struct Tile2 {
  static constexpr int W = TX + 3;              // LDS row: x0 - 2 .. x0 + TX
  static constexpr int N = W * (TY + 2);        // LDS rows: y0 - 1 .. y0 + TY
  static constexpr int threads = (N + 63) / 64 * 64;
  static_assert(threads <= 1024 && TX * TY <= threads, "two-step tile");
};
constexpr int kT2X = 48, kT2Y = 8;              // lattices of kT2SmallCells nodes or more
constexpr int kT2SmallX = 16, kT2SmallY = 8;
constexpr int64_t kT2SmallCells = int64_t(1) << 17;

// Pull of node (x, y), LDS node n of rows of W and planes of N nodes, from
// the populations of the step before.
template <int W, int N, typename R>
__device__ __forceinline__ void pull_tile(const R* __restrict__ lds, const Consts<R>& k, int x, int y, int n,
                                          R (&f)[19]) {
  const R* p = lds + n;
  if (__all(x >= 1 && x <= k.nx - 2 && y >= 1 && y <= k.ny - 2)) {  // no wall link: constant offsets
#pragma unroll
    for (int q = 0; q < 19; ++q) f[q] = p[q * N - EY[q] * W - EX[q]];
    return;
  }
#pragma unroll
  for (int q = 0; q < 19; ++q) {
    const int xs = x - EX[q], ys = y - EY[q];
    const bool in = (unsigned)xs < (unsigned)k.nx && (unsigned)ys < (unsigned)k.ny;
    f[q] = p[in ? q * N - EY[q] * W - EX[q] : OPP[q] * N];
  }
}

// The two steps of the tile at (x0, y0), called by every thread of a
// Tile2::threads workgroup (it holds a workgroup barrier).  SAUX: cache
// policy of the final stores.
template <typename R, int MAT, int TX, int TY, int SAUX>
__device__ __forceinline__ void step2_tile(R* __restrict__ lds, const R* __restrict__ src, R* __restrict__ mid,
                                           R* __restrict__ dst, const R* __restrict__ phi_f,
                                           const R* __restrict__ invk_f, const R* __restrict__ d_f,
                                           const Consts<R>& k, int x0, int y0) {
  constexpr int W = Tile2<TX, TY>::W, N = Tile2<TX, TY>::N;
  const bool react = !(k.flags & F_NO_REACTION);
  {
    const int n = threadIdx.x;
    const int i = n % W, j = n / W;
    const int x = x0 - 2 + i, y = y0 - 1 + j;
    if (n < N && (unsigned)x < (unsigned)k.nx && (unsigned)y < (unsigned)k.ny) {
      R f[19];
      const Mat<R> mt =
          pre_collision<R, MAT, false>(src, k, phi_f, invk_f, d_f, x, y, f, y0 > 0 ? y0 - 1 : 0);
      collide(f, mt, k, react && y >= k.y_cl0);
#pragma unroll
      for (int q = 0; q < 19; ++q) lds[q * N + n] = f[q];
      if (mid && i >= 2 && i < TX + 2 && j >= 1 && j <= TY) store_node<16>(mid, k, x, y, y0, f);
    }
  }
  __syncthreads();
  if (threadIdx.x >= TX * TY) return;
  const int x = x0 + int(threadIdx.x) % TX, y = y0 + int(threadIdx.x) / TX;
  if (x >= k.nx || y >= k.ny) return;
  const bool inlet = x == 0 && y < k.ny_ch;
  const bool outlet = x == k.nx - 1;
  const int xp = inlet ? 1 : (outlet ? k.nx - 2 : x);
  R f[19];
  pull_tile<W, N>(lds, k, xp, y, (y - y0 + 1) * W + (xp - x0 + 2), f);
  Mat<R> mt = material<R, MAT>(k, phi_f, invk_f, d_f, xp, y);
  thin_film(f, mt, k, y);
  if (inlet || outlet) {
    Mat<R> mb = material<R, MAT>(k, phi_f, invk_f, d_f, x, y);
    boundary_column(f, k, y, inlet, mt, mb);
    if (outlet) outlet_scalar_material(mb, mt);
    mt = mb;
  }
  collide(f, mt, k, react && y >= k.y_cl0);
  store_node<SAUX>(dst, k, x, y, y0, f);
}

template <typename R, int MAT, int TX, int TY, int SAUX>
__global__ __launch_bounds__((Tile2<TX, TY>::threads)) void k_step2(const R* __restrict__ src, R* __restrict__ mid,
                                                                    R* __restrict__ dst, const R* __restrict__ phi_f,
                                                                    const R* __restrict__ invk_f,
                                                                    const R* __restrict__ d_f, Consts<R> k) {
  __shared__ R lds[19 * Tile2<TX, TY>::N];
  int bx, by;
  xcd_tile(gridDim.x, gridDim.y, bx, by);
  step2_tile<R, MAT, TX, TY, SAUX>(lds, src, mid, dst, phi_f, invk_f, d_f, k, bx * TX, by * TY);
}

// Three time steps in one launch, where no state between them is asked for:
// the state is read and written once for three steps.  Step one runs over
// the tile and a halo of two (three columns on the left, where the outlet's
// feeding columns can lie), one node per thread, as in k_step2; step two
// runs in place over the tile and a halo of one, its nodes held in registers
// until all have been pulled; step three pulls the tile's nodes and writes
// `dst`.  A thread keeps its node throughout, so a node's material is read
// and derived once.  The states are the bits of three single steps.
//
// The halo's extra nodes (512 computed for 27x12 = 324 kept) buy a third of
// the memory traffic and of the launches.  Region rows are 32 nodes, two to
// a wavefront.  Per step with a porosity per cell, k_step2 / 27x12 (us): FP32
// 1024x256 6.9 / 6.7, 1537x431 12.2 / 12.2, 2048x512 16.4 / 17.0, 4096x1024
// 82.4 / 66.5; FP64 1024x256 10.6 / 10.2, 1537x431 20.8 / 19.0, 2048x512 39.0
// / 29.6, 4096x1024 145 / 111.  Lattices of fewer than 2^16 nodes leave CUs
// idle and take 27x4: 200x40 FP64 4.2 / 3.4, FP32 3.8 / 3.0 (27x12 there:
// one workgroup on 32 of 256 CUs).  64 nodes a row (59x12, 1024 threads) is
// slower: 4096x1024 80.7.  Stores write through where the two states fit the
// last-level cache (FP32 1024x256 6.4 against 6.7) and are plain beyond it
// (4096x1024 66.5 against 82, FP64 108 against 143).
template <int TX, int TY>
struct Tile3 {
  static constexpr int W = TX + 5, N = W * (TY + 4);  // LDS: x0 - 3 .. x0 + TX + 1, y0 - 2 .. y0 + TY + 1
  static constexpr int threads = (N + 63) / 64 * 64;
  static_assert(threads <= 1024, "three-step tile: one node per thread");
};
constexpr int kT3X = 27, kT3Y = 12;
constexpr int kT3SmallX = 27, kT3SmallY = 4;
constexpr int64_t kT3SmallCells = int64_t(1) << 16;

// The three steps (or two: what is left of a run on the same tiles) of the
// tile at (x0, y0), called by every thread of a Tile3::threads workgroup (it
// holds workgroup barriers).  SAUX: cache policy of the final stores.
template <typename R, int MAT, int TX, int TY, int SAUX, int STEPS = 3>
__device__ __forceinline__ void step3_tile(R* __restrict__ lds, const R* __restrict__ src, R* __restrict__ dst,
                                           const R* __restrict__ phi_f, const R* __restrict__ invk_f,
                                           const R* __restrict__ d_f, const Consts<R>& k, int x0, int y0) {
  constexpr int W = Tile3<TX, TY>::W, N = Tile3<TX, TY>::N;
  const int yb = y0 > 1 ? y0 - 2 : 0;
  const int n = threadIdx.x, i = n % W, j = n / W;
  const int x = x0 - 3 + i, y = y0 - 2 + j;
  const bool node = n < N && (unsigned)x < (unsigned)k.nx && (unsigned)y < (unsigned)k.ny;
  // the nodes each of the last two steps runs over: the tile and a ring, the tile
  const bool ring = node && i >= 1 && i <= TX + 3 && j >= 1 && j <= TY + 2;
  const bool own = node && i >= 3 && i < TX + 3 && j >= 2 && j < TY + 2;
  const bool inlet = x == 0 && y < k.ny_ch, outlet = x == k.nx - 1;
  const int xp = inlet ? 1 : (outlet ? k.nx - 2 : x);
  const bool cl = y >= k.y_cl0 && !(k.flags & F_NO_REACTION);
  Mat<R> m;  // of the column whose populations the node pulls
  R f[19];
  auto finish = [&] {
    thin_film(f, m, k, y);
    Mat<R> mt = m;
    if (inlet || outlet) {
      mt = material<R, MAT>(k, phi_f, invk_f, d_f, x, y);
      boundary_column(f, k, y, inlet, m, mt);
      if (outlet) outlet_scalar_material(mt, m);
    }
    collide(f, mt, k, cl);
  };
  static_assert(STEPS == 2 || STEPS == 3, "steps of a launch");
  if (STEPS == 3 ? node : ring) {
    pull<R, false>(src, k, xp, y, f, yb);
    m = material<R, MAT>(k, phi_f, invk_f, d_f, xp, y);
    finish();
#pragma unroll
    for (int q = 0; q < 19; ++q) lds[q * N + n] = f[q];
  }
  if constexpr (STEPS == 3) {
    __syncthreads();
    if (ring) {
      pull_tile<W, N>(lds, k, xp, y, n + xp - x, f);
      finish();
    }
    __syncthreads();
    if (ring) {
#pragma unroll
      for (int q = 0; q < 19; ++q) lds[q * N + n] = f[q];
    }
  }
  __syncthreads();
  if (own) {
    pull_tile<W, N>(lds, k, xp, y, n + xp - x, f);
    finish();
    store_node<SAUX>(dst, k, x, y, yb, f);
  }
}

template <typename R, int MAT, int TX, int TY, int SAUX>
__global__ __launch_bounds__((Tile3<TX, TY>::threads)) void k_step3(const R* __restrict__ src, R* __restrict__ dst,
                                                                    const R* __restrict__ phi_f,
                                                                    const R* __restrict__ invk_f,
                                                                    const R* __restrict__ d_f, Consts<R> k) {
  __shared__ R lds[19 * Tile3<TX, TY>::N];
  int bx, by;
  xcd_tile(gridDim.x, gridDim.y, bx, by);
  step3_tile<R, MAT, TX, TY, SAUX>(lds, src, dst, phi_f, invk_f, d_f, k, bx * TX, by * TY);
}

// Equilibrium initial state: rest fluid at zero pressure (shifted f = 0),
// theta = 0, O2 at c_in.
template <typename R, int MAT>
__device__ __forceinline__ void init_node(R* __restrict__ dst, const R* __restrict__ phi_f,
                                          const R* __restrict__ invk_f, const R* __restrict__ d_f,
                                          const Consts<R>& k, int x, int y) {
  if (x >= k.nx) return;
  const Mat<R> mt = material<R, MAT>(k, phi_f, invk_f, d_f, x, y);
  R g[5] = {R(0), R(0), R(0), R(0), R(0)};
  add_geq(k.c_in, R(0), R(0), mt.bC, R(1), g);
  const int o = y * k.pitch + x;
#pragma unroll
  for (int q = 0; q < 14; ++q) dst[q * k.plane + o] = R(0);
#pragma unroll
  for (int q = 0; q < 5; ++q) dst[(14 + q) * k.plane + o] = g[q];
}
template <typename R, int MAT>
__global__ __launch_bounds__(kBlock) void k_init(R* __restrict__ dst, const R* __restrict__ phi_f,
                                                 const R* __restrict__ invk_f,
                                                 const R* __restrict__ d_f, Consts<R> k) {
  init_node<R, MAT>(dst, phi_f, invk_f, d_f, k, blockIdx.x * kBlock + threadIdx.x, blockIdx.y);
}

__device__ __forceinline__ double wave_sum(double v) {
#pragma unroll
  for (int off = 32; off > 0; off >>= 1) v += __shfl_down(v, off, 64);
  return v;
}
__device__ __forceinline__ double wave_max(double v) {
#pragma unroll
  for (int off = 32; off > 0; off >>= 1) v = fmax(v, __shfl_down(v, off, 64));
  return v;
}

// Observable partial sums over the pre-collision state, one row of partials
// per workgroup: sum f (shifted), sum theta, sum c, sum s_c, sum S_T,
// sum s_c (eta + T dU0/dT), max theta, count of non-finite values, sum of
// u_x over the inlet nodes.
// The thin-film CL's reaction at the bottom node of column x, as the last
// streaming applied it: from the populations of the pulled column (column
// nx - 2 for the outlet, whose scalars are that column's) that crossed the
// wall, with the scalar material the node collides with.
template <typename R>
__device__ __forceinline__ React<R> film(const R* __restrict__ src, const Consts<R>& k, int x, const Mat<R>& mt) {
  const int xp = (!(k.flags & F_PERIODIC_X) && x == k.nx - 1) ? k.nx - 2 : x;
  const int o = (k.ny - 1) * k.pitch + xp;
  return surface_reaction(src[11 * k.plane + o], src[16 * k.plane + o], mt, k);
}

template <typename R, int MAT>
__device__ __forceinline__ void obs_cells(const R* __restrict__ src, const R* __restrict__ phi_f,
                                          const R* __restrict__ invk_f, const R* __restrict__ d_f,
                                          const Consts<R>& k, int bx, int y, double* __restrict__ partial) {
  const int x = bx * kBlock + threadIdx.x;
  double v[kObsQ] = {0, 0, 0, 0, 0, 0, -1e300, 0, 0};
  if (x < k.nx) {
    R f[19];
    const Mat<R> mt = pre_collision<R, MAT, true>(src, k, phi_f, invk_f, d_f, x, y, f, y);
    if (x == 0 && y < k.ny_ch && !(k.flags & F_PERIODIC_X)) v[8] = double(flow_macros(f, mt, k).ux);
    double sf = 0, th = 0, c = 0;
#pragma unroll
    for (int q = 0; q < 9; ++q) sf += double(f[q]);
#pragma unroll
    for (int q = 9; q < 14; ++q) th += double(f[q]);
    if (k.flags & F_SIGMA_ENERGY) th /= double(mt.sig);
#pragma unroll
    for (int q = 14; q < 19; ++q) c += double(f[q]);
    v[0] = sf;
    v[1] = th;
    v[2] = c;
    if (y >= k.y_cl0 && !(k.flags & F_NO_REACTION)) {
      const React<R> r = reaction(R(th), R(c), mt.rhocp, k);
      v[3] = double(r.s_c);
      v[4] = double(r.S_T);
      v[5] = double(r.s_c) * double(r.ehs);
    } else if ((k.flags & F_THIN_CL) && !(k.flags & F_NO_REACTION) && y == k.ny - 1) {
      const React<R> r = film(src, k, x, mt);
      v[3] = double(r.s_c);
      v[4] = double(r.S_T);
      v[5] = double(r.s_c) * double(r.ehs);
    }
    v[6] = th;
    bool bad = false;
#pragma unroll
    for (int q = 0; q < 19; ++q) bad |= !isfinite(f[q]);
    v[7] = bad ? 1.0 : 0.0;
  }
  __shared__ double red[kObsQ][kBlock / 64];
  const int lane = threadIdx.x & 63, wid = threadIdx.x >> 6;
#pragma unroll
  for (int i = 0; i < kObsQ; ++i) {
    const double s = i == 6 ? wave_max(v[i]) : wave_sum(v[i]);
    if (lane == 0) red[i][wid] = s;
  }
  __syncthreads();
  if (threadIdx.x < kObsQ) {
    const int i = threadIdx.x;
    double s = red[i][0];
    for (int w = 1; w < kBlock / 64; ++w) s = i == 6 ? fmax(s, red[i][w]) : s + red[i][w];
    partial[i] = s;
  }
}

template <typename R, int MAT>
__global__ __launch_bounds__(kBlock) void k_obs_cells(const R* __restrict__ src, const R* __restrict__ phi_f,
                                                      const R* __restrict__ invk_f, const R* __restrict__ d_f,
                                                      Consts<R> k, double* __restrict__ partial) {
  obs_cells<R, MAT>(src, phi_f, invk_f, d_f, k, blockIdx.x, blockIdx.y,
                    partial + size_t(blockIdx.y * gridDim.x + blockIdx.x) * kObsQ);
}

// Sum quantity i of the per-workgroup partials in a fixed order: thread t
// takes every kFinal-th from t on, then a fixed tree combines the threads.
// (With 256 threads that each walked a contiguous chunk, the 16384 partials
// of a 4096x1024 lattice took 24 us: one chain of dependent, uncoalesced
// loads per thread.)
constexpr int kFinal = 1024;
template <int Q>
__device__ __forceinline__ void obs_final(const double* __restrict__ partial, int nblocks, int i,
                                          double* __restrict__ out) {
  const bool is_max = i == 6;
  double s = is_max ? -1e300 : 0.0;
#pragma unroll 4
  for (int b = threadIdx.x; b < nblocks; b += kFinal) {
    const double v = partial[(size_t)b * Q + i];
    s = is_max ? fmax(s, v) : s + v;
  }
  s = is_max ? wave_max(s) : wave_sum(s);
  __shared__ double red[kFinal / 64];
  if ((threadIdx.x & 63) == 0) red[threadIdx.x >> 6] = s;
  __syncthreads();
  if (threadIdx.x == 0) {
    for (int w = 1; w < kFinal / 64; ++w) s = is_max ? fmax(s, red[w]) : s + red[w];
    out[i] = s;
  }
}

template <int Q = kObsQ>  // a template so that every translation unit may instantiate it
__global__ __launch_bounds__(kFinal) void k_obs_final(const double* __restrict__ partial, int nblocks,
                                                      double* __restrict__ out) {
  obs_final<Q>(partial, nblocks, blockIdx.x, out);
}

// Per-column CL profiles: i(x) = sum over CL rows of 4 F C_ref s_c / dt * dx,
// and c, T on the CL row next to the GDL.  A workgroup takes 64 columns, a
// wavefront one CL row at a time; the rows' reactions meet in LDS and are
// added in the order of the rows.  (One thread per column walked the 51 rows
// of a 4096x1024 lattice one after the other, 16 workgroups in all: 150 us in
// FP32, now 16.)  Eight wavefronts in FP64, whose 1024-thread form spills.
template <typename R>
constexpr int kProfRows = sizeof(R) == 8 ? 8 : 16;
template <typename R, int MAT>
__global__ __launch_bounds__(64 * kProfRows<R>) void k_obs_profiles(const R* __restrict__ src,
                                                                 const R* __restrict__ phi_f,
                                                                 const R* __restrict__ invk_f,
                                                                 const R* __restrict__ d_f, Consts<R> k,
                                                                 double i_scale, double* __restrict__ prof) {
  const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
  const int x = blockIdx.x * 64 + lane;
  const bool react = !(k.flags & F_NO_REACTION);
  constexpr int rows = kProfRows<R>;
  __shared__ double part[rows][64];
  double isum = 0, c0 = 0, t0 = 0;
  if ((k.flags & F_THIN_CL) && w == 0 && x < k.nx) {  // the film's current, the profiles of the row above it
    R f[19];
    const Mat<R> mt = pre_collision<R, MAT, true>(src, k, phi_f, invk_f, d_f, x, k.ny - 1, f, k.ny - 1);
    c0 = double(f[14] + f[15] + f[16] + f[17] + f[18]);
    t0 = double(k.T_in) + double(theta_of(f + 9, mt.sig, k));
    if (react) isum = double(film(src, k, x, mt).s_c);
  }
  for (int y0 = k.y_cl0; y0 < k.ny; y0 += rows) {
    const int y = y0 + w;
    if (y < k.ny && x < k.nx) {
      R f[19];
      const Mat<R> mt = pre_collision<R, MAT, true>(src, k, phi_f, invk_f, d_f, x, y, f, y);
      const R th = theta_of(f + 9, mt.sig, k);
      const R c = f[14] + f[15] + f[16] + f[17] + f[18];
      part[w][lane] = react ? double(reaction(th, c, mt.rhocp, k).s_c) : 0.0;
      if (y == k.y_cl0) {  // wavefront 0
        c0 = double(c);
        t0 = double(k.T_in) + double(th);
      }
    }
    __syncthreads();
    if (w == 0)
      for (int r = 0; r < rows && y0 + r < k.ny; ++r) isum += part[r][lane];
    __syncthreads();
  }
  if (w != 0 || x >= k.nx) return;
  prof[x] = isum * i_scale;
  prof[k.nx + x] = c0;
  prof[2 * k.nx + x] = t0;
}

// Macroscopic fields of the pre-collision state into dense [ny][nx] arrays.
template <typename R, int MAT>
__global__ __launch_bounds__(kBlock) void k_fields(const R* __restrict__ src,
                                                   const R* __restrict__ phi_f,
                                                   const R* __restrict__ invk_f,
                                                   const R* __restrict__ d_f, Consts<R> k,
                                                   R* ux, R* uy, R* p, R* T, R* theta, R* c) {
  const int x = blockIdx.x * kBlock + threadIdx.x;
  const int y = blockIdx.y;
  if (x >= k.nx) return;
  R f[19];
  const Mat<R> mt = pre_collision<R, MAT, true, false>(src, k, phi_f, invk_f, d_f, x, y, f, y);
  const Macro<R> a = flow_macros(f, mt, k);
  const int o = y * k.nx + x;
  if (ux) ux[o] = a.ux;
  if (uy) uy[o] = a.uy;
  if (p) p[o] = a.p;
  const R th = theta_of(f + 9, mt.sig, k);
  if (T) T[o] = k.T_in + th;
  if (theta) theta[o] = th;
  if (c) c[o] = f[14] + f[15] + f[16] + f[17] + f[18];
}

// Internal (pitched, shifted rest population) <-> canonical dense populations.
template <typename R>
__global__ __launch_bounds__(kBlock) void k_export(const R* __restrict__ src, R* __restrict__ dst,
                                                   Consts<R> k) {
  const int x = blockIdx.x * kBlock + threadIdx.x;
  const int y = blockIdx.y;
  if (x >= k.nx) return;
  const size_t dense = (size_t)k.nx * k.ny;
  for (int q = 0; q < 19; ++q) {
    R v = src[q * k.plane + y * k.pitch + x];
    if (q == 0) v += R(1);
    dst[q * dense + (size_t)y * k.nx + x] = v;
  }
}

template <typename R>
__global__ __launch_bounds__(kBlock) void k_import(const R* __restrict__ src, R* __restrict__ dst,
                                                   Consts<R> k) {
  const int x = blockIdx.x * kBlock + threadIdx.x;
  const int y = blockIdx.y;
  if (x >= k.nx) return;
  const size_t dense = (size_t)k.nx * k.ny;
  for (int q = 0; q < 19; ++q) {
    R v = src[q * dense + (size_t)y * k.nx + x];
    if (q == 0) v -= R(1);
    dst[q * k.plane + y * k.pitch + x] = v;
  }
}

// Full-field mode: fill the fields not given by the caller from porosity
// (Kozeny-Carman, Bruggeman / ratio) or from the layered inputs.
template <typename R>
__global__ __launch_bounds__(kBlock) void k_derive_fields(R* __restrict__ phi, R* __restrict__ invk,
                                                          R* __restrict__ d, Consts<R> k, int have_phi,
                                                          int have_invk, int have_d) {
  const int x = blockIdx.x * kBlock + threadIdx.x;
  const int y = blockIdx.y;
  if (x >= k.nx) return;
  const int o = y * k.pitch + x;
  const bool porous = y >= k.ny_ch;
  if (!have_phi) phi[o] = porous ? k.phi_gdl : R(1);
  const R ph = phi[o];
  if (!have_invk) {
    if (k.kc_inv > R(0)) {
      const R om = R(1) - ph;
      invk[o] = om * om * k.kc_inv / (ph * ph * ph);
    } else {
      invk[o] = porous ? k.invk_gdl : R(0);
    }
  }
  if (!have_d) d[o] = (porous && k.deff_ratio > R(0)) ? k.deff_ratio * k.D_f : ph * sqrt(ph) * k.D_f;
}

// Copy a dense [ny][nx] caller array into a pitched workspace plane.
template <typename R>
__global__ __launch_bounds__(kBlock) void k_pitch_copy(const R* __restrict__ src, R* __restrict__ dst,
                                                       int nx, int pitch) {
  const int x = blockIdx.x * kBlock + threadIdx.x;
  const int y = blockIdx.y;
  if (x >= nx) return;
  dst[y * pitch + x] = src[(size_t)y * nx + x];
}

}  // namespace lbm

namespace lbm {

// Per-cell porosity, 1/K and O2 diffusivity as the kernels use them.
template <typename R, int MAT>
__global__ __launch_bounds__(kBlock) void k_material(const R* __restrict__ phi_f, const R* __restrict__ invk_f,
                                                     const R* __restrict__ d_f, Consts<R> k, R* phi, R* invk, R* d) {
  const int x = blockIdx.x * kBlock + threadIdx.x;
  const int y = blockIdx.y;
  if (x >= k.nx) return;
  R a, b, c;
  base_fields<R, MAT>(k, phi_f, invk_f, d_f, x, y, a, b, c);
  const size_t o = (size_t)y * k.nx + x;
  if (phi) phi[o] = a;
  if (invk) invk[o] = b;
  if (d) d[o] = c;
}

}  // namespace lbm
