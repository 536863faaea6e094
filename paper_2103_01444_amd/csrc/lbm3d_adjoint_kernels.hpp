// Kernels of the 3D reverse sweep (three per-cell fields: porosity, 1/K, D_eff).
#pragma once

#include "lbm3d_adjoint.hpp"
#include "lbm3d_kernels.hpp"

namespace lbm3 {

// Post-collision adjoints [Q0, Q1) of node (x, y, z), y and z the
// wavefront's.
template <typename R, int Q0, int Q1>
__device__ __forceinline__ void load_own(const R* __restrict__ lam, const Consts3<R>& k, int x, int y, int z,
                                         R (&la)[Q1 - Q0]) {
  const Planes3<R> b(lam, k, y, z);
#pragma unroll
  for (int q = Q0; q < Q1; ++q)
    la[q - Q0] = b.template load<0>(q, 0, 0, 0, uint32_t(x) * uint32_t(sizeof(R)));
}

// Push: the adjoint of the pulled element (x - e_q, q), or of the
// bounced-back (x, opp q), is mu[q - Q0].
template <typename R, int Q0, int Q1>
__device__ __forceinline__ void push(R* __restrict__ lam, const Consts3<R>& k, int x, int y, int z,
                                     const R (&mu)[Q1 - Q0]) {
  if (inside(k, x, y, z)) {
    const Planes3<R> b(lam, k, y, z);
#pragma unroll
    for (int q = Q0; q < Q1; ++q)
      b.template store<0>(q, -EX[q], -EY[q], -EZ[q], uint32_t(x) * uint32_t(sizeof(R)), mu[q - Q0]);
    return;
  }
#pragma unroll
  for (int q = Q0; q < Q1; ++q) lam[pull_offset(k, q, x, y, z)] = mu[q - Q0];
}

// One reverse step: lam_out = (dS'/dS)^T lam_in at the state S, gradients
// accumulated into grad (planes phi, 1/K, D_eff).  SEED: lam_out = w dJ/dS.
//
// As the 2D reverse step: the fourteen scalar populations (pull, adjoint of
// their collisions, push), then the nineteen flow ones; a boundary lane runs
// its own node on its extrapolated populations, and the lane of the feeding
// column, which the lane shift keeps in the same wavefront, takes the
// boundary node's result across lanes and runs the transposed
// extrapolation.  Bound by HBM (432 bytes a node in FP32).  The former
// kernel held all 33 populations at once (144 VGPRs) and left the boundary
// nodes to a second kernel on a second stream, joined by events at every
// step: 72 us per reverse step at 160x80x40 FP32, now 50 (4.5 TB/s).
template <typename R, bool SEED>
__global__ __launch_bounds__(kBlock3) void k3_adj_step(const R* __restrict__ S, const R* __restrict__ lam_in,
                                                       R* __restrict__ lam_out, R* __restrict__ grad,
                                                       const R* __restrict__ phi_f, const R* __restrict__ invk_f,
                                                       const R* __restrict__ d_f, Consts3<R> k, R w) {
  const int shift = lbm::adj_lane_shift(k.nx);
  int x, y, z;
  if (!node_of(k, shift, x, y, z)) return;
  const bool open = !(k.flags & F_PERIODIC_X);
  const bool cl = !(k.flags & F_NO_REACTION) && z >= k.z_cl0;
  const bool in_row = open && z < k.nz_ch;
  const bool inlet = in_row && x == 0, outlet = open && x == k.nx - 1, bnode = inlet || outlet;
  const int xp = inlet ? 1 : (outlet ? k.nx - 2 : x);
  const int l0 = (x + shift) & ~63;  // first lane of the wavefront, as an x + shift
  const bool w_in = in_row && l0 == 0, w_out = open && l0 == ((k.nx - 1 + shift) & ~63);
  const int lane_out = (k.nx - 1 + shift) & 63;
  const int o = (z * k.ny + y) * k.pitch + x;

  AdjMat3<R> m = adj_material(k, phi_f, invk_f, d_f, xp, y, z);
  R g[14];
  MacroTape3<R> t;
  {
    R f[19];
    pull_range<R, 0, 19, false>(S, k, xp, y, z, f);
    pull_range<R, 19, 33, false>(S, k, xp, y, z, g);
    if (bnode) {  // the boundary node's extrapolated populations and its own material
      R p[33];
#pragma unroll
      for (int q = 0; q < 33; ++q) p[q] = q < 19 ? f[q] : g[q - 19];
      AdjMat3<R> mc = adj_material(k, phi_f, invk_f, d_f, x, y, z);
      boundary_column(p, k, y, z, inlet, m, mc);
      if (outlet) {  // the outlet node collides with column nx-2's scalar material
        mc.aT = m.aT;
        mc.aC = m.aC;
        mc.rhocp = m.rhocp;
        mc.irc = m.irc;
      }
      m = mc;
#pragma unroll
      for (int q = 0; q < 33; ++q) (q < 19 ? f[q] : g[q - 19]) = p[q];
    }
    t = flow_macros_tape(f, m, k);
  }
  MatAdj3<R> ma{};
  Vec3<R> lu, bl;  // velocity's adjoints: of the node's collision, of the transposed extrapolation
  R lpp = R(0);
  const R ub = w_in ? inlet_velocity(k, y, z) : R(0);

  // ---- scalars ----
  {
    R mus[14];
    if constexpr (SEED) {
#pragma unroll
      for (int q = 0; q < 14; ++q) mus[q] = R(0);
      if (cl) {
        R th = R(0), c = R(0);
#pragma unroll
        for (int q = 0; q < 7; ++q) {
          th += g[q];
          c += g[7 + q];
        }
        const ReactAdj<R> r = reaction_tape(th, c, m.rhocp, k);
#pragma unroll
        for (int q = 0; q < 7; ++q) {
          mus[q] = w * r.dsc_dth;
          mus[7 + q] = w * r.dsc_dc;
        }
      }
    } else {
      R la[14];
      load_own<R, 19, 33>(lam_in, k, x, y, z, la);
      scalars_adj(g, t.u, m, k, cl, la, mus, lu, ma);
    }
    if (w_in) {
      R mub[14];
#pragma unroll
      for (int q = 0; q < 14; ++q) mub[q] = __shfl(mus[q], shift, 64);
      const Vec3<R> up{__shfl(t.u.x, shift + 1, 64), __shfl(t.u.y, shift + 1, 64), __shfl(t.u.z, shift + 1, 64)};
      if (x <= 1) {
        MatAdj3<R> axp{}, ab{};
        R th = R(0), c = R(0), lt1 = R(0), lc1 = R(0);
#pragma unroll
        for (int q = 0; q < 7; ++q) {
          th += g[q];
          c += g[7 + q];
        }
        inlet_scalars_adj(mub, up, th, c, m, k, bl, lt1, lc1, axp, ab);
        if (x == 0) {
          ma.aC += ab.aC;
        } else {
          ma.aT += axp.aT;
          ma.aC += axp.aC;
#pragma unroll
          for (int q = 0; q < 7; ++q) {
            mus[q] += mub[q] + lt1;
            mus[7 + q] += mub[7 + q] + lc1;
          }
        }
      }
    }
    if (w_out) {  // the outlet's scalars are copies
      R mub[14];
#pragma unroll
      for (int q = 0; q < 14; ++q) mub[q] = __shfl(mus[q], lane_out, 64);
      const R sT = __shfl(ma.aT, lane_out, 64), sC = __shfl(ma.aC, lane_out, 64);
      const R sr = __shfl(ma.rhocp, lane_out, 64);
      if (x == k.nx - 2) {
#pragma unroll
        for (int q = 0; q < 14; ++q) mus[q] += mub[q];
        ma.aT += sT;
        ma.aC += sC;
        ma.rhocp += sr;
      }
    }
    if (bnode) {  // its pulled sources were never read by the forward step
#pragma unroll
      for (int q = 0; q < 14; ++q) mus[q] = R(0);
    }
    push<R, 19, 33>(lam_out, k, x, y, z, mus);
  }

  // ---- flow ----
  R muf[19];
  if constexpr (SEED) {
#pragma unroll
    for (int q = 0; q < 19; ++q) muf[q] = R(0);
  } else {
    R la[19];
    load_own<R, 0, 19>(lam_in, k, x, y, z, la);
    flow_adj(t, m, k, la, lu, muf, ma);
  }
  if (w_in || w_out) {
    // both boundaries in turn (nx = 3: one column feeds both)
#pragma unroll
    for (int side = 0; side < 2; ++side) {
      if (!(side == 0 ? w_in : w_out)) continue;
      const int lb = side == 0 ? shift : lane_out, lp = side == 0 ? shift + 1 : lane_out - 1;
      R mub[19];
#pragma unroll
      for (int q = 0; q < 19; ++q) mub[q] = __shfl(muf[q], lb, 64);
      const Vec3<R> up{__shfl(t.u.x, lp, 64), __shfl(t.u.y, lp, 64), __shfl(t.u.z, lp, 64)};
      const R ppp = __shfl(t.pp, lp, 64), ip = __shfl(m.iphi, lp, 64);
      const R phi_b = __shfl(m.phi, lb, 64), iphi_b = __shfl(m.iphi, lb, 64);
      const int xb = side == 0 ? 0 : k.nx - 1, xf = side == 0 ? 1 : k.nx - 2;
      if (x == xb || x == xf) {
        MatAdj3<R> axp{}, ab{};
        Vec3<R> l;
        R lp1 = R(0);
        boundary_flow_adj(mub, up, ppp, side == 0, ub, ip, phi_b, iphi_b, l, lp1, axp, ab);
        if (x == xb) {
          ma.phi += ab.phi;
        } else {
          ma.phi += axp.phi;
          bl = axpy(R(1), l, bl);
          lpp += lp1;
#pragma unroll
          for (int q = 0; q < 19; ++q) muf[q] += mub[q];
        }
      }
    }
    if (!bnode && (x == 1 || x == k.nx - 2)) {
      // xp's macros: phi p = s / 2 - u^2 / (4 phi), u = v / den
      ma.phi += R(0.25) * lpp * t.u2 * m.iphi * m.iphi;
      const Vec3<R> lv = flow_macros_adj(t, m, k, axpy(R(-0.5) * lpp * m.iphi, t.u, bl), Vec3<R>{}, ma);
#pragma unroll
      for (int q = 1; q < 19; ++q) muf[q] += R(0.5) * lpp + along(q, lv);
    }
  }
  if (bnode) {
#pragma unroll
    for (int q = 0; q < 19; ++q) muf[q] = R(0);
  }
  push<R, 0, 19>(lam_out, k, x, y, z, muf);

  if (outlet) ma.aT = ma.aC = ma.rhocp = R(0);  // went to column nx - 2
  R g0 = R(0), g1 = R(0), g2 = R(0);
  material_adj(k, m, ma, g0, g1, g2);
  grad[o] += g0;
  grad[k.plane + o] += g1;
  grad[2 * k.plane + o] += g2;
}

// Gradient through the initial state: the O2 equilibrium at rest depends on
// a_C = sqrt(3) D (g0 = c_in (1 - 6 a_C), g_i = c_in a_C).
template <typename R>
__global__ __launch_bounds__(kBlock3) void k3_adj_init(const R* __restrict__ lam0, R* __restrict__ grad,
                                                       Consts3<R> k) {
  const int x = blockIdx.x * kBlock3 + threadIdx.x;
  const int y = blockIdx.y, z = blockIdx.z;
  if (x >= k.nx) return;
  const int o = (z * k.ny + y) * k.pitch + x;
  R l16 = R(0);
#pragma unroll
  for (int q = 27; q < 33; ++q) l16 += lam0[q * k.plane + o];
  grad[2 * k.plane + o] += R(kSqrt3) * k.c_in * (R(-6) * lam0[26 * k.plane + o] + l16);
}

template <typename R>
__global__ __launch_bounds__(kBlock3) void k3_fill(R* __restrict__ dst, int64_t n, R v) {
  const int64_t i = blockIdx.x * int64_t(kBlock3) + threadIdx.x;
  if (i < n) dst[i] = v;
}

// Pitched plane -> dense [nz][ny][nx] caller array.
template <typename R>
__global__ __launch_bounds__(kBlock3) void k3_unpitch(const R* __restrict__ src, R* __restrict__ dst, int nx, int ny,
                                                      int pitch) {
  const int x = blockIdx.x * kBlock3 + threadIdx.x;
  const int y = blockIdx.y, z = blockIdx.z;
  if (x >= nx) return;
  dst[(size_t(z) * ny + y) * nx + x] = src[(z * ny + y) * pitch + x];
}

}  // namespace lbm3
