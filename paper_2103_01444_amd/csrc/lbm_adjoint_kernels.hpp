// Kernels of the reverse sweep (three per-cell fields: porosity, 1/K, D_eff).
#pragma once

#include <type_traits>

#include "lbm_adjoint.hpp"
#include "lbm_kernels2d.hpp"

namespace lbm {

// Element offset the pull of population q at (x, y) reads.
template <typename R>
__device__ __forceinline__ int pull_offset(const Consts<R>& k, int q, int x, int y) {
  int xs = x - EX[q];
  int ys = y - EY[q];
  if (k.flags & F_PERIODIC_X) xs = xs < 0 ? xs + k.nx : (xs >= k.nx ? xs - k.nx : xs);
  if (k.flags & F_PERIODIC_Y) ys = ys < 0 ? ys + k.ny : (ys >= k.ny ? ys - k.ny : ys);
  const bool in = (unsigned)xs < (unsigned)k.nx && (unsigned)ys < (unsigned)k.ny;
  return in ? (q * k.plane + ys * k.pitch + xs) : (OPP[q] * k.plane + y * k.pitch + x);
}

// The adjoint of S is kept as each node's mu (the adjoint of what the node
// pulled), in the same planes as a state.  Population q of node (x, y) was
// pulled by (x + e_q), or, where that link crosses a wall, by the node itself
// as its opposite: the element of mu that holds its adjoint.
template <typename R>
__device__ __forceinline__ int puller_offset(const Consts<R>& k, int q, int x, int y) {
  int xs = x + EX[q];
  int ys = y + EY[q];
  if (k.flags & F_PERIODIC_X) xs = xs < 0 ? xs + k.nx : (xs >= k.nx ? xs - k.nx : xs);
  if (k.flags & F_PERIODIC_Y) ys = ys < 0 ? ys + k.ny : (ys >= k.ny ? ys - k.ny : ys);
  const bool in = (unsigned)xs < (unsigned)k.nx && (unsigned)ys < (unsigned)k.ny;
  return in ? (q * k.plane + ys * k.pitch + xs) : (OPP[q] * k.plane + y * k.pitch + x);
}

// Populations [Q0, Q1) of node (x, y), y the wavefront's row; inner: the
// wavefront lies one node or more inside the lattice (wave-uniform bases).
// NT: the non-temporal hint.
template <typename R, int Q0, int Q1, bool NT>
__device__ __forceinline__ void pull_part(const R* __restrict__ S, const Consts<R>& k, bool inner, int x, int y,
                                          R* f) {
  if (inner) {
    const PlaneBuffer<R> b(S, k, y);
#pragma unroll
    for (int q = Q0; q < Q1; ++q)
      f[q - Q0] = b.template load<NT ? 2 : 0>(q, -EX[q], -EY[q], uint32_t(x) * uint32_t(sizeof(R)));
  } else {
#pragma unroll
    for (int q = Q0; q < Q1; ++q) {
      if constexpr (NT)
        f[q - Q0] = __builtin_nontemporal_load(S + pull_offset(k, q, x, y));
      else
        f[q - Q0] = S[pull_offset(k, q, x, y)];
    }
  }
}

// Adjoint of the post-collision populations [Q0, Q1) of node (x, y) from mu.
template <typename R, int Q0, int Q1>
__device__ __forceinline__ void gather_part(const R* __restrict__ mu, const Consts<R>& k, bool inner, int x, int y,
                                            R* la) {
  if (inner) {
    const PlaneBuffer<R> b(mu, k, y);
#pragma unroll
    for (int q = Q0; q < Q1; ++q)
      la[q - Q0] = b.template load<0>(q, EX[q], EY[q], uint32_t(x) * uint32_t(sizeof(R)));
  } else {
#pragma unroll
    for (int q = Q0; q < Q1; ++q) la[q - Q0] = mu[puller_offset(k, q, x, y)];
  }
}

// Store [Q0, Q1) of node (x, y), y the wavefront's row.  AUX: cache policy.
template <typename R, int Q0, int Q1, int AUX>
__device__ __forceinline__ void store_part(R* __restrict__ mu, const Consts<R>& k, int x, int y, const R* v) {
  const PlaneBuffer<R> b(mu, k, y);
#pragma unroll
  for (int q = Q0; q < Q1; ++q) b.template store<AUX>(q, 0, 0, uint32_t(x) * uint32_t(sizeof(R)), v[q - Q0]);
}

// The reverse step of one node: mu = (dS'/d pulled)^T lambda at the state S.
// SEED: of J (times w = dJ dx / nx * 4 F C_ref / dt), no lambda.  NT: of S.
//
// A wavefront holds consecutive nodes of row y, lane l the node x = xl + l;
// both nodes of a boundary pair (0, 1) and (nx - 2, nx - 1) if it holds
// either.  gather(q0, la) fills la with the adjoints of the populations from
// q0 on (10 scalar ones from 9, 9 flow ones from 0); put(q0, mu) takes mu.
// g0, g1, g2: the gradient with respect to the node's (phi, 1/K, D_eff).
//
// Two passes per node: the ten scalar populations (pull, adjoint of their
// collisions), which leave the velocity's adjoint, then the nine flow ones,
// so that about 30 values are live at once.  A boundary lane runs its own
// node's collision adjoint in the common passes on its extrapolated
// populations; the lane of the feeding column takes the boundary node's
// result across lanes and runs the transposed extrapolation, while the
// boundary lane keeps what belongs to its own material.
//
// Small lattices are bound by one wavefront's chain, large ones by HBM.
// Holding all nineteen populations, the moment-matrix transposes and the
// buffer resources of 57 planes at once took 128 VGPRs and spilled: 544 bytes
// of scratch per lane in FP64 and 482 scalar-register spills; in two passes
// no instance spills vector registers.  Per reverse step at 200x40 FP64 29.8
// -> 9.2 us.  (Gradients of the spilled forms have differed from run to run.)
template <typename R, bool SEED, bool EXT, bool NT, typename Gather, typename Put>
__device__ __forceinline__ void reverse_node(const R* __restrict__ S, const R* __restrict__ phi_f,
                                             const R* __restrict__ invk_f, const R* __restrict__ d_f,
                                             const Consts<R>& k, int x, int y, int xl, bool inner, R w,
                                             const Gather& gather, const Put& put, R& g0, R& g1, R& g2) {
  const bool open = !(k.flags & F_PERIODIC_X);
  const bool react = !(k.flags & F_NO_REACTION);
  const bool cl = react && y >= k.y_cl0;
  const bool in_row = open && y < k.ny_ch;
  const bool inlet = in_row && x == 0;
  const bool outlet = open && x == k.nx - 1;
  const bool bnode = inlet || outlet;
  const int xp = inlet ? 1 : (outlet ? k.nx - 2 : x);
  const int lane_in = -xl, lane_out = k.nx - 1 - xl;  // lanes of columns 0 and nx - 1
  const bool w_in = in_row && lane_in >= 0 && lane_in < 63, w_out = open && lane_out >= 1 && lane_out < 64;
  const bool pressure = EXT && (k.flags & F_PRESSURE_INLET);

  AdjMat<R> m = adj_material<R>(k, phi_f, invk_f, d_f, xp, y);
  R f[9], g[10];
  pull_part<R, 9, 19, NT>(S, k, inner, xp, y, g);
  pull_part<R, 0, 9, NT>(S, k, inner, xp, y, f);
  // Thin-film CL (EXT): the bottom row's wall-crossing populations react as
  // the forward pull left them (column nx - 2's film for the outlet).
  const bool film = EXT && (k.flags & F_THIN_CL) && react && y == k.ny - 1;
  FilmTape<R> ft{};
  if (film) {
    ft = film_tape(g[4], g[9], m, k);
    g[4] += ft.S_T * m.sig;
    g[9] -= ft.s;
  }
  // Boundary lanes: their extrapolated populations and their own material.
  if (bnode) {
    R p[19];
#pragma unroll
    for (int q = 0; q < 19; ++q) p[q] = q < 9 ? f[q] : g[q - 9];
    AdjMat<R> mc = adj_material<R>(k, phi_f, invk_f, d_f, x, y);
    boundary_column(p, k, y, inlet, m, mc);
    if (outlet) outlet_scalar_adj_material(mc, m);
    m = mc;
#pragma unroll
    for (int q = 0; q < 19; ++q) (q < 9 ? f[q] : g[q - 9]) = p[q];
  }

  MatAdj<R> ma{};
  MacroTape<R> t = flow_macros_tape<R, EXT>(f, theta_of(g, m.isig), m, k);
  const R S18 = ((f[1] + f[3]) + (f[2] + f[4])) + ((f[5] + f[7]) + (f[6] + f[8]));
  R lux = R(0), luy = R(0), lth = R(0), lpp = R(0);
  R blx = R(0), bly = R(0);  // velocity's adjoint from the transposed extrapolation
  const R ubx = w_in ? inlet_velocity(k, y) : R(0);

  // ---- scalars ----
  R mus[10];
  if constexpr (SEED) {
    // J's adjoint: w ds_c / d(theta, c) on the CL's populations
#pragma unroll
    for (int q = 0; q < 10; ++q) mus[q] = R(0);
    if (cl) {
      const R th = theta_of(g, m.isig);
      const ReactAdj<R> r = reaction_tape(th, sum5(g + 5), m.rhocp, k);
      const R lt = theta_adj<R, EXT>(w * r.dsc_dth, th, m, k, ma);
#pragma unroll
      for (int q = 0; q < 5; ++q) {
        mus[q] = lt;
        mus[5 + q] = w * r.dsc_dc;
      }
    }
  } else {
    R la[10];
    gather(std::integral_constant<int, 9>{}, la);
    scalars_adj<R, EXT>(g, t.ux, t.uy, m, k, cl, la, mus, lux, luy, ma);
  }
  // With buoyancy the boundary nodes' temperature adjoint also has a share
  // from the flow pass, so both passes of a boundary wavefront precede the
  // exchange there.
  const bool buoyant = EXT && (k.flags & F_BUOYANCY);
  R muf[9];
  auto flow_pass = [&]() {
    if constexpr (SEED) {
#pragma unroll
      for (int q = 0; q < 9; ++q) muf[q] = R(0);
    } else {
      R la[9];
      gather(std::integral_constant<int, 0>{}, la);
      flow_adj<R, EXT>(t, m, k, la, lux, luy, muf, lth, ma);
      if (buoyant) {
        const R l = theta_adj<R, EXT>(lth, t.thb, m, k, ma);
        lth = R(0);
#pragma unroll
        for (int q = 0; q < 5; ++q) mus[q] += l;
      }
    }
  };
  if (EXT) flow_pass();

  // Exchange of the scalars' part.
  if (w_in) {
    R mub[10];
#pragma unroll
    for (int q = 0; q < 10; ++q) mub[q] = __shfl(mus[q], lane_in, 64);
    const R uxp = __shfl(t.ux, lane_in + 1, 64), uyp = __shfl(t.uy, lane_in + 1, 64);
    if (x <= 1) {
      MatAdj<R> axp{}, ab{};
      R lt1 = R(0), lc1 = R(0);
      inlet_scalars_adj<R, EXT>(mub, uxp, uyp, theta_of(g, m.isig), sum5(g + 5), pressure, m, k, blx, bly, lt1, lc1,
                                axp, ab);
      if (x == 0) {
        ma.aC += ab.aC;
      } else {
        ma.aT += axp.aT;
        ma.aC += axp.aC;
        if (EXT) ma.sig += axp.sig;
#pragma unroll
        for (int q = 0; q < 5; ++q) {
          mus[q] += mub[q] + lt1;
          mus[5 + q] += mub[5 + q] + lc1;
        }
      }
    }
  }
  if (w_out) {  // the outlet's scalars are copies, collided with column nx - 2's scalar material
    R mub[10];
#pragma unroll
    for (int q = 0; q < 10; ++q) mub[q] = __shfl(mus[q], lane_out, 64);
    const R sT = __shfl(ma.aT, lane_out, 64), sC = __shfl(ma.aC, lane_out, 64);
    const R sr = __shfl(ma.rhocp, lane_out, 64), ss = EXT ? __shfl(ma.sig, lane_out, 64) : R(0);
    if (x == k.nx - 2) {
#pragma unroll
      for (int q = 0; q < 10; ++q) mus[q] += mub[q];
      ma.aT += sT;
      ma.aC += sC;
      ma.rhocp += sr;
      if (EXT) ma.sig += ss;
    }
  }
  // A boundary node's pulled sources were never read by the forward step:
  // their adjoint is 0.
  auto put_scalars = [&]() {
    if (bnode) {
#pragma unroll
      for (int q = 0; q < 10; ++q) mus[q] = R(0);
    }
    put(std::integral_constant<int, 9>{}, mus);
  };
  if (!EXT) put_scalars();

  // ---- flow ----
  if (!EXT) flow_pass();
  if (w_in || w_out) {
    const R pp = fma_(R(0.6), S18, R(-0.4) * (t.u2 * m.iphi));
    // both boundaries in turn (nx = 3: one column feeds both)
#pragma unroll
    for (int side = 0; side < 2; ++side) {
      if (!(side == 0 ? w_in : w_out)) continue;
      const int lb = side == 0 ? lane_in : lane_out, lp = side == 0 ? lane_in + 1 : lane_out - 1;
      R mub[9];
#pragma unroll
      for (int q = 0; q < 9; ++q) mub[q] = __shfl(muf[q], lb, 64);
      const R uxp = __shfl(t.ux, lp, 64), uyp = __shfl(t.uy, lp, 64), ppp = __shfl(pp, lp, 64);
      const R ip = __shfl(m.iphi, lp, 64), phi_b = __shfl(m.phi, lb, 64), iphi_b = __shfl(m.iphi, lb, 64);
      const int xb = side == 0 ? 0 : k.nx - 1, xf = side == 0 ? 1 : k.nx - 2;
      if (x == xb || x == xf) {
        AdjMat<R> mx = m;
        mx.iphi = ip;
        MatAdj<R> axp{}, ab{};
        R lx = R(0), ly = R(0), lp1 = R(0);
        boundary_flow_adj(mub, uxp, uyp, ppp, side == 0 && !pressure, ubx, side == 0 ? k.p_in : k.p_out, mx, phi_b,
                          iphi_b, lx, ly, lp1, axp, ab);
        if (x == xb) {
          ma.phi += ab.phi;
        } else {
          ma.phi += axp.phi;
          blx += lx;
          bly += ly;
          lpp += lp1;
#pragma unroll
          for (int q = 0; q < 9; ++q) muf[q] += mub[q];
        }
      }
    }
    if (!bnode && (x == 1 || x == k.nx - 2)) {
      // xp's macros: phi p = 0.6 S - 0.4 u^2 / phi, u = v / den
      const R c = R(0.8) * lpp * m.iphi;
      ma.phi += R(0.4) * lpp * t.u2 * m.iphi * m.iphi;
      R lvx, lvy, lt = R(0), mx[9];
      flow_macros_adj<R, EXT>(t, m, k, fma_(-c, t.ux, blx), fma_(-c, t.uy, bly), R(0), R(0), lvx, lvy, lt, ma);
      flow_sums_adj(R(0), R(0.6) * lpp, R(0), R(0), R(0), lvx, lvy, R(0), R(0), mx);
#pragma unroll
      for (int q = 0; q < 9; ++q) muf[q] += mx[q];
      if (buoyant) {
        const R l = theta_adj<R, EXT>(lt, t.thb, m, k, ma);
#pragma unroll
        for (int q = 0; q < 5; ++q) mus[q] += l;
      }
    }
  }
  // Transpose of the film's update in the column that pulled it (the
  // outlet's copy came back through the exchange above); the seed adds J's
  // dependence on the film, which counts column nx - 2 twice (the outlet
  // carries its film).
  if (film && !bnode) {
    const R ls = SEED ? ((open && x == k.nx - 2) ? R(2) * w : w) : R(0);
    film_adj(ft, m, k, ls, mus[4], mus[9], ma);
  }
  if (EXT) put_scalars();
  if (bnode) {
#pragma unroll
    for (int q = 0; q < 9; ++q) muf[q] = R(0);
  }
  put(std::integral_constant<int, 0>{}, muf);

  // The gradient of this node's own material; the outlet's scalar-material
  // terms went to column nx - 2.
  if (outlet) {
    ma.aT = R(0);
    ma.aC = R(0);
    ma.rhocp = R(0);
    ma.sig = R(0);
  }
  g0 = g1 = g2 = R(0);
  material_adj<R, EXT>(k, m, ma, g0, g1, g2);
}

// One reverse step, one launch: mu_out at the state S from mu_in, gradients
// accumulated into grad (planes phi, 1/K, D_eff).  S is one state of a chain,
// read once here: non-temporal loads and plain stores leave the last-level
// cache to mu (41 steps back on lattices periodic in x, cached S and written
// through -> this, us: FP32 1537x431 1591 -> 1455, 2048x700 3028 -> 2387, FP64
// 1537x431 3043 -> 2308; with the checkpoints' replay beside it FP32 1024x256,
// 60 steps, 1311 -> 1236).
template <typename R, bool SEED, bool EXT = false>
__global__ __launch_bounds__(kBlock) void k_adj_step(const R* __restrict__ S, const R* __restrict__ mu_in,
                                                     R* __restrict__ mu_out, R* __restrict__ grad,
                                                     const R* __restrict__ phi_f, const R* __restrict__ invk_f,
                                                     const R* __restrict__ d_f, Consts<R> k, R w) {
  int bx, y;
  xcd_tile(gridDim.x, gridDim.y, bx, y);
  const int x = bx * kBlock + int(threadIdx.x) - adj_lane_shift(k.nx);
  if ((unsigned)x >= (unsigned)k.nx) return;
  const bool inner = __all(x >= 1 && x <= k.nx - 2) && y >= 1 && y <= k.ny - 2;
  R g0, g1, g2;
  reverse_node<R, SEED, EXT, true>(
      S, phi_f, invk_f, d_f, k, x, y, x - int(threadIdx.x & 63), inner, w,
      [&](auto q0, auto& la) { gather_part<R, q0(), q0() + sizeof(la) / sizeof(R)>(mu_in, k, inner, x, y, la); },
      [&](auto q0, const auto& mu) { store_part<R, q0(), q0() + sizeof(mu) / sizeof(R), 0>(mu_out, k, x, y, mu); }, g0,
      g1, g2);
  const int o = y * k.pitch + x;
  grad[o] += g0;
  grad[k.plane + o] += g1;
  grad[2 * k.plane + o] += g2;
}

// Two reverse steps in one launch, at the states S1 (first) and S0, with the
// bits of two single ones.  A workgroup takes a tile of at most kAdjX columns
// and ROWS - 2 rows.  The first step runs over the tile and a ring of one
// node, a row per wavefront, and leaves mu in LDS; the second gathers from
// there and writes the tile's.  Of the 264 bytes a node that a single FP32 step moves
// (S, mu in and out, the gradient twice, the fields) lambda's 152 and the
// gradient's 24 are halved, and the ring adds a share of S and mu.  Reverse
// sweep with its replay, per step, one -> two steps per launch: 1024x256 FP32
// 24.5 -> 18.7 us.  ROWS = 8, or 4 on lattices of fewer than 2^17 nodes,
// which leave CUs idle (200x40 FP64 13.3 -> 10.4, FP32 9.8 -> 9.3; 1024x256
// FP32 18.7 with 8, 19.7 with 4, 19.0 with 12).  With the rates and sixths
// that the FP32 gradient's error asked for (rate_at, nth) 19.2 -> 19.6 there,
// 200x40 FP64 9.8 -> 9.9 (11.0 with all model options, 10.4 before).
// Lattices without periodic axes.
constexpr int kAdjX = 60;
template <typename R, bool EXT, int ROWS>
__global__ __launch_bounds__(64 * ROWS) void k_adj_step2(const R* __restrict__ S1, const R* __restrict__ S0,
                                                             const R* __restrict__ mu_in, R* __restrict__ mu_out,
                                                             R* __restrict__ grad, const R* __restrict__ phi_f,
                                                             const R* __restrict__ invk_f,
                                                             const R* __restrict__ d_f, Consts<R> k) {
  __shared__ R lds[ROWS * 19 * 64];
  int bx, by;
  xcd_tile(gridDim.x, gridDim.y, bx, by);
  // tiles equal within one column: 30 columns or more wide, or the whole row
  const int x0 = int(int64_t(bx) * k.nx / gridDim.x), x1 = int(int64_t(bx + 1) * k.nx / gridDim.x);
  const int xl = x0 > 0 ? x0 - 1 : 0, xr = x1 < k.nx ? x1 + 1 : k.nx;  // the first step's columns
  const int i = threadIdx.x & 63, j = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int x = xl + i, y0 = by * (ROWS - 2), y = y0 - 1 + j;
  const bool row = (unsigned)y < (unsigned)k.ny;
  const bool own = x >= x0 && x < x1 && j >= 1 && j < ROWS - 1;
  R ga[3] = {R(0), R(0), R(0)}, gb[3] = {R(0), R(0), R(0)};
  if (row && x < xr) {
    const bool inner = __all(x >= 1 && x <= k.nx - 2) && y >= 1 && y <= k.ny - 2;
    R* p = lds + j * 19 * 64 + i;
    reverse_node<R, false, EXT, false>(
        S1, phi_f, invk_f, d_f, k, x, y, xl, inner, R(0),
        [&](auto q0, auto& la) { gather_part<R, q0(), q0() + sizeof(la) / sizeof(R)>(mu_in, k, inner, x, y, la); },
        [&](auto q0, const auto& mu) {
#pragma unroll
          for (int q = 0; q < int(sizeof(mu) / sizeof(R)); ++q) p[(q0() + q) * 64] = mu[q];
        },
        ga[0], ga[1], ga[2]);
  }
  __syncthreads();
  // the second step: the tile, 30 columns or more wide (or the whole row), so
  // that it holds both nodes of a boundary pair or neither
  if (!(row && own)) return;
  const bool inner = __all(x >= 1 && x <= k.nx - 2) && y >= 1 && y <= k.ny - 2;
  const R* p = lds + j * 19 * 64 + i;
  reverse_node<R, false, EXT, false>(
      S0, phi_f, invk_f, d_f, k, x, y, xl, inner, R(0),
      [&](auto q0, auto& la) {
#pragma unroll
        for (int n = 0; n < int(sizeof(la) / sizeof(R)); ++n) {
          const int q = q0() + n;
          const int xs = x + EX[q], ys = y + EY[q];
          const bool in = inner || ((unsigned)xs < (unsigned)k.nx && (unsigned)ys < (unsigned)k.ny);
          la[n] = p[in ? (EY[q] * 19 + q) * 64 + EX[q] : OPP[q] * 64];
        }
      },
      [&](auto q0, const auto& mu) {
        store_part<R, q0(), q0() + sizeof(mu) / sizeof(R), 16>(mu_out, k, x, y, mu);
      },
      gb[0], gb[1], gb[2]);
  const int o = y * k.pitch + x;
#pragma unroll
  for (int c = 0; c < 3; ++c) {
    const int n = c * k.plane + o;
    grad[n] = (grad[n] + ga[c]) + gb[c];
  }
}

// Gradient through the initial state: the O2 equilibrium at rest depends on
// b_C = 20 sqrt(3) D - 4 (Eq. 10).  mu: the first step's.
template <typename R>
__global__ __launch_bounds__(kBlock) void k_adj_init(const R* __restrict__ mu, R* __restrict__ grad, Consts<R> k) {
  const int x = blockIdx.x * kBlock + threadIdx.x;
  const int y = blockIdx.y;
  if (x >= k.nx) return;
  R l[5];
#pragma unroll
  for (int q = 0; q < 5; ++q) l[q] = mu[puller_offset(k, 14 + q, x, y)];
  grad[2 * k.plane + y * k.pitch + x] +=
      R(34.64101615137754587) * k.c_in * (-l[0] * R(0.2) + (l[1] + l[2] + l[3] + l[4]) * R(0.05));
}

// Pitched plane -> dense [ny][nx] caller array.
template <typename R>
__global__ __launch_bounds__(kBlock) void k_unpitch(const R* __restrict__ src, R* __restrict__ dst, int nx, int pitch) {
  const int x = blockIdx.x * kBlock + threadIdx.x;
  const int y = blockIdx.y;
  if (x >= nx) return;
  dst[(size_t)y * nx + x] = src[y * pitch + x];
}

template <typename R>
__global__ __launch_bounds__(kBlock) void k_fill(R* __restrict__ dst, int64_t n, R v) {
  const int64_t i = blockIdx.x * (int64_t)kBlock + threadIdx.x;
  if (i < n) dst[i] = v;
}

}  // namespace lbm
