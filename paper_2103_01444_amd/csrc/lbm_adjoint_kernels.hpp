// Kernels of the reverse sweep (three per-cell fields: porosity, 1/K, D_eff).
#pragma once

#include "lbm_adjoint.hpp"
#include "lbm_kernels2d.hpp"

namespace lbm {

// Element offset the pull of population q at (x, y) reads, and the push of
// its adjoint writes.
template <typename R>
__device__ __forceinline__ int pull_offset(const Consts<R>& k, int q, int x, int y) {
  int xs = x - EX[q];
  int ys = y - EY[q];
  if (k.flags & F_PERIODIC_X) xs = xs < 0 ? xs + k.nx : (xs >= k.nx ? xs - k.nx : xs);
  if (k.flags & F_PERIODIC_Y) ys = ys < 0 ? ys + k.ny : (ys >= k.ny ? ys - k.ny : ys);
  const bool in = (unsigned)xs < (unsigned)k.nx && (unsigned)ys < (unsigned)k.ny;
  return in ? (q * k.plane + ys * k.pitch + xs) : (OPP[q] * k.plane + y * k.pitch + x);
}

// Populations [Q0, Q1) of node (x, y): inner (the wavefront lies one node or
// more inside the lattice) through the wave-uniform bases.
template <typename R, int Q0, int Q1>
__device__ __forceinline__ void pull_part(const R* __restrict__ S, const PlaneBuffer<R>& b, const Consts<R>& k,
                                          bool inner, int x, int y, R* f) {
  if (inner) {
    const uint32_t ob = uint32_t(y * k.pitch + x) * uint32_t(sizeof(R));
#pragma unroll
    for (int q = Q0; q < Q1; ++q) f[q - Q0] = b.template load<2>(q, -EX[q], -EY[q], ob);
  } else {
#pragma unroll
    for (int q = Q0; q < Q1; ++q) f[q - Q0] = __builtin_nontemporal_load(S + pull_offset(k, q, x, y));
  }
}

template <typename R, int Q0, int Q1>
__device__ __forceinline__ void push_part(R* __restrict__ lam, const PlaneBuffer<R>& b, const Consts<R>& k,
                                          bool inner, int x, int y, const R* mu) {
  if (inner) {
    const uint32_t ob = uint32_t(y * k.pitch + x) * uint32_t(sizeof(R));
#pragma unroll
    for (int q = Q0; q < Q1; ++q) b.store(q, -EX[q], -EY[q], ob, mu[q - Q0]);
  } else {
#pragma unroll
    for (int q = Q0; q < Q1; ++q) lam[pull_offset(k, q, x, y)] = mu[q - Q0];
  }
}

// Population q of the node at element offset o.
template <typename R>
__device__ __forceinline__ R load_own(const R* __restrict__ p, const PlaneBuffer<R>& b, const Consts<R>& k, int q,
                                      int o) {
  return k.near32 ? b.template load<0>(q, 0, 0, uint32_t(o) * uint32_t(sizeof(R))) : p[q * k.plane + o];
}

// One reverse step: lam_out = (dS'/dS)^T lam_in at the state S, gradients
// accumulated into grad (planes phi, 1/K, D_eff).  SEED: lam_out = dJ/dS
// (times w = dJ dx / nx * 4 F C_ref / dt), no lam_in.
//
// Two passes per node: the ten scalar populations (pull, adjoint of their
// collisions, push), which leave the velocity's adjoint, then the nine flow
// ones, so that about 30 values are live at once.  A boundary lane runs its
// own node's collision adjoint in the common passes on its extrapolated
// populations; the lane of the feeding column takes the boundary node's
// result across lanes and runs the transposed extrapolation, while the
// boundary lane keeps what belongs to its own material.
//
// Small lattices are bound by one wavefront's chain, large ones by HBM (in
// FP32 S, lambda in and out, the gradient twice, the fields: 264 bytes a
// node).  Holding all nineteen populations, the moment-matrix transposes and
// the buffer resources of 57 planes at once took 128 VGPRs and spilled: 544
// bytes of scratch per lane in FP64 and 482 scalar-register spills.  Now 71
// (FP32) and 135 (FP64) VGPRs without a spill; per reverse step at 200x40
// FP64 29.8 -> 9.2 us, at 1024x256 FP32 (beside the replay) 18.0 -> 17.2 us.
// (Gradients of the spilled forms have differed from run to run.)
template <typename R, bool SEED, bool EXT = false>
__global__ __launch_bounds__(kBlock) void k_adj_step(const R* __restrict__ S, const R* __restrict__ lam_in,
                                                     R* __restrict__ lam_out, R* __restrict__ grad,
                                                     const R* __restrict__ phi_f, const R* __restrict__ invk_f,
                                                     const R* __restrict__ d_f, Consts<R> k, R w) {
  int bx, by;
  xcd_tile(gridDim.x, gridDim.y, bx, by);
  const int shift = adj_lane_shift(k.nx);
  const int x = bx * kBlock + int(threadIdx.x) - shift;
  const int y = by;
  if ((unsigned)x >= (unsigned)k.nx) return;
  const bool open = !(k.flags & F_PERIODIC_X);
  const bool react = !(k.flags & F_NO_REACTION);
  const bool cl = react && y >= k.y_cl0;
  const bool in_row = open && y < k.ny_ch;
  const bool inlet = in_row && x == 0;
  const bool outlet = open && x == k.nx - 1;
  const bool bnode = inlet || outlet;
  const int xp = inlet ? 1 : (outlet ? k.nx - 2 : x);
  const int l0 = (x + shift) & ~63;  // first lane of the wavefront, as an x + shift
  const bool w_in = in_row && l0 == 0, w_out = open && l0 == ((k.nx - 1 + shift) & ~63);
  const int lane_out = (k.nx - 1 + shift) & 63;
  const bool pressure = EXT && (k.flags & F_PRESSURE_INLET);
  const bool inner = k.near32 && __all(x >= 1 && x <= k.nx - 2 && y >= 1 && y <= k.ny - 2);
  const int o = y * k.pitch + x;
  const PlaneBuffer<R> bS(S, k), bi(lam_in, k), bo(lam_out, k);

  AdjMat<R> m = adj_material<R>(k, phi_f, invk_f, d_f, xp, y);
  R f[9], g[10];
  pull_part<R, 9, 19>(S, bS, k, inner, xp, y, g);
  pull_part<R, 0, 9>(S, bS, k, inner, xp, y, f);
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
#pragma unroll
    for (int q = 0; q < 10; ++q) la[q] = load_own(lam_in, bi, k, 9 + q, o);
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
#pragma unroll
      for (int q = 0; q < 9; ++q) la[q] = load_own(lam_in, bi, k, q, o);
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
    for (int q = 0; q < 10; ++q) mub[q] = __shfl(mus[q], shift, 64);
    const R uxp = __shfl(t.ux, shift + 1, 64), uyp = __shfl(t.uy, shift + 1, 64);
    if (x <= 1) {
      MatAdj<R> axp{}, ab{};
      R lt1 = R(0), lc1 = R(0);
      inlet_scalars_adj<R, EXT>(mub, uxp, uyp, theta_of(g, m.isig), sum5(g + 5), ubx, pressure, m, k, blx, bly, lt1,
                                lc1, axp, ab);
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
  auto push_scalars = [&]() {
    if (bnode) {
#pragma unroll
      for (int q = 0; q < 10; ++q) mus[q] = R(0);
    }
    push_part<R, 9, 19>(lam_out, bo, k, inner, x, y, mus);
  };
  if (!EXT) push_scalars();

  // ---- flow ----
  if (!EXT) flow_pass();
  if (w_in || w_out) {
    const R pp = fma_(R(0.6), S18, R(-0.4) * (t.u2 * m.iphi));
    // both boundaries in turn (nx = 3: one column feeds both)
#pragma unroll
    for (int side = 0; side < 2; ++side) {
      if (!(side == 0 ? w_in : w_out)) continue;
      const int lb = side == 0 ? shift : lane_out, lp = side == 0 ? shift + 1 : lane_out - 1;
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
  if (EXT) push_scalars();
  if (bnode) {
#pragma unroll
    for (int q = 0; q < 9; ++q) muf[q] = R(0);
  }
  push_part<R, 0, 9>(lam_out, bo, k, inner, x, y, muf);

  // The gradient of this node's own material; the outlet's scalar-material
  // terms went to column nx - 2.
  if (outlet) {
    ma.aT = R(0);
    ma.aC = R(0);
    ma.rhocp = R(0);
    ma.sig = R(0);
  }
  R g0 = R(0), g1 = R(0), g2 = R(0);
  material_adj<R, EXT>(k, m, ma, g0, g1, g2);
  grad[o] += g0;
  grad[k.plane + o] += g1;
  grad[2 * k.plane + o] += g2;
}

// Gradient through the initial state: the O2 equilibrium at rest depends on
// b_C = 20 sqrt(3) D - 4 (Eq. 10).
template <typename R>
__global__ __launch_bounds__(kBlock) void k_adj_init(const R* __restrict__ lam0, R* __restrict__ grad, Consts<R> k) {
  const int x = blockIdx.x * kBlock + threadIdx.x;
  const int y = blockIdx.y;
  if (x >= k.nx) return;
  const int o = y * k.pitch + x;
  const R l0 = lam0[14 * k.plane + o];
  const R l14 = lam0[15 * k.plane + o] + lam0[16 * k.plane + o] + lam0[17 * k.plane + o] + lam0[18 * k.plane + o];
  grad[2 * k.plane + o] += R(34.64101615137754587) * k.c_in * (-l0 * R(0.2) + l14 * R(0.05));
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
