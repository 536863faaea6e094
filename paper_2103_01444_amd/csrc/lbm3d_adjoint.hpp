// Discrete adjoint of the 3D step (reverse mode, written by hand).
//
// Same structure as the 2D adjoint: the step is S' = C(P(S)) with P the
// pull (a permutation with bounce-back) plus the inlet / outlet columns and
// C the per-node collision, so per node
//   mu_x   = (dC_x / d pre_x)^T lambda_x
//   mu_xp += (dB / d pre_xp)^T mu_b   for the boundary node b fed by xp
//   lambda_new[source of pull (x, q)] = mu_x[q].
// The collision is two-rate, so its transpose acts pair by pair on the
// symmetric / antisymmetric parts.
#pragma once

#include "lbm3d_device.hpp"
#include "lbm_adjoint.hpp"  // reaction_tape, ReactAdj, the primitives

namespace lbm3 {

using lbm::fast_rcp;
using lbm::fast_sqrt;
using lbm::fma_;
using lbm::nth;
using lbm::ReactAdj;
using lbm::reaction_tape;

constexpr double kSqrt3 = 1.7320508075688772935;

// Adjoints of the medium's quantities as the forward step uses them
// (dl = phi nu / K).
template <typename R>
struct MatAdj3 {
  R phi = R(0), dl = R(0), l0 = R(0), l1 = R(0), aT = R(0), aC = R(0), rhocp = R(0);
};

// The forward step's material with what the reverse step takes of it.
template <typename R>
struct AdjMat3 : Mat3<R> {
  R iphi, dl, irc;
};
template <typename R>
__device__ __forceinline__ AdjMat3<R> adj_material(const Consts3<R>& k, const R* __restrict__ phi_f,
                                                   const R* __restrict__ invk_f, const R* __restrict__ d_f, int x,
                                                   int y, int z) {
  AdjMat3<R> m;
  static_cast<Mat3<R>&>(m) = material<R, MAT_FULL>(k, phi_f, invk_f, d_f, x, y, z);
  m.iphi = fast_rcp(m.phi);
  m.dl = m.phi * k.nu * m.invk;
  m.irc = fast_rcp(m.rhocp);
  return m;
}

// Chain the adjoints of the derived material quantities to (phi, 1/K, D), as
// in 2D.
template <typename R>
__device__ __forceinline__ void material_adj(const Consts3<R>& k, const AdjMat3<R>& m, const MatAdj3<R>& a, R& g_phi,
                                             R& g_invk, R& g_d) {
  const R ldl = fma_(R(0.25), a.l0, a.dl);
  R linvk = m.phi * k.nu * ldl;
  if (m.invk > R(0)) linvk += R(0.5) * a.l1 * m.l1 / m.invk;  // 0 at 1/K = 0
  const R drc = k.rhocp_f - k.rhocp_s, dk = k.aT_f - k.aT_s;
  g_phi += a.phi + k.nu * m.invk * ldl - R(0.5) * a.l1 * m.l1 * m.iphi + a.aT * (dk - m.aT * drc) * m.irc +
           a.rhocp * drc;
  g_invk += linvk;
  g_d += a.aC * R(kSqrt3);  // aC = sqrt3 D
}

template <typename R>
struct Vec3 {
  R x = R(0), y = R(0), z = R(0);
};
template <typename R>
__device__ __forceinline__ R dot(const Vec3<R>& a, const Vec3<R>& b) {
  return fma_(a.x, b.x, fma_(a.y, b.y, a.z * b.z));
}
template <typename R>
__device__ __forceinline__ Vec3<R> axpy(R s, const Vec3<R>& a, const Vec3<R>& b) {
  return {fma_(s, a.x, b.x), fma_(s, a.y, b.y), fma_(s, a.z, b.z)};
}
template <typename R>
__device__ __forceinline__ Vec3<R> scale(R s, const Vec3<R>& a) {
  return {s * a.x, s * a.y, s * a.z};
}
// e_i . a and b += s e_i for velocity i (components 0, 1, -1: additions only).
template <typename R>
__device__ __forceinline__ R along(int i, const Vec3<R>& a) {
  R v = R(0);
  if (EX[i]) v = EX[i] > 0 ? v + a.x : v - a.x;
  if (EY[i]) v = EY[i] > 0 ? v + a.y : v - a.y;
  if (EZ[i]) v = EZ[i] > 0 ? v + a.z : v - a.z;
  return v;
}
template <typename R>
__device__ __forceinline__ void add_along(int i, R s, Vec3<R>& b) {
  if (EX[i]) b.x = EX[i] > 0 ? b.x + s : b.x - s;
  if (EY[i]) b.y = EY[i] > 0 ? b.y + s : b.y - s;
  if (EZ[i]) b.z = EZ[i] > 0 ? b.z + s : b.z - s;
}

// Forward intermediates of the flow macros kept for their adjoint; pp: phi p.
template <typename R>
struct MacroTape3 {
  Vec3<R> v, u, F;
  R vm, ir, iden, u2, drag, pp;
};

template <typename R>
__device__ __forceinline__ MacroTape3<R> flow_macros_tape(const R* f, const AdjMat3<R>& m, const Consts3<R>& k) {
  MacroTape3<R> t;
  R s = R(0);
#pragma unroll
  for (int i = 1; i < 19; i += 2) {
    add_along(i, f[i] - f[i + 1], t.v);
    s += f[i] + f[i + 1];
  }
  const bool body = k.flags & F_BODY_FORCE;
  if (body) {
    t.v.x += R(0.5) * m.phi * k.ax;
    t.v.y += R(0.5) * m.phi * k.ay;
  }
  t.vm = fast_sqrt(dot(t.v, t.v));
  const R r = lbm::fast_momentum_root(m.l0, m.l1, t.vm);
  t.ir = lbm::fast_rcp_inf(r);
  t.iden = lbm::fast_rcp_inf(m.l0 + r);
  t.u = scale(t.iden, t.v);
  t.u2 = dot(t.u, t.u);
  t.drag = fma_(R(2) * m.l1, t.vm * t.iden, m.dl);
  t.F = scale(-t.drag, t.u);
  if (body) {
    t.F.x += m.phi * k.ax;
    t.F.y += m.phi * k.ay;
  }
  t.pp = fma_(R(0.5), s, R(-0.25) * (t.u2 * m.iphi));
  return t;
}

// Adjoint of v -> (u, F): the adjoint of v from those of u and F.
template <typename R>
__device__ __forceinline__ Vec3<R> flow_macros_adj(const MacroTape3<R>& t, const AdjMat3<R>& m, const Consts3<R>& k,
                                                   Vec3<R> lu, const Vec3<R>& lF, MatAdj3<R>& ma) {
  const R um = t.vm * t.iden;
  const R ldrag = -dot(t.u, lF);
  lu = axpy(-t.drag, lF, lu);
  ma.dl += ldrag;
  ma.l1 = fma_(R(2) * um, ldrag, ma.l1);
  const R lum = R(2) * m.l1 * ldrag;
  const R lden = -t.iden * fma_(um, lum, dot(t.u, lu));
  const R ldr = lden * t.ir;
  ma.l0 += fma_(ldr, m.l0, lden);
  ma.l1 = fma_(R(0.5) * t.vm, ldr, ma.l1);
  const R lvm = fma_(R(0.5) * m.l1, ldr, lum * t.iden);
  Vec3<R> lv = scale(t.iden, lu);
  if (t.vm > R(0)) lv = axpy(lvm / t.vm, t.v, lv);  // a cell at rest: derivative of |v| taken as 0
  if (k.flags & F_BODY_FORCE)
    ma.phi += k.ax * fma_(R(0.5), lv.x, lF.x) + k.ay * fma_(R(0.5), lv.y, lF.y);
  return lv;
}

// Adjoint of the two scalar collisions and the CL source: g, la, mu hold the
// temperature populations in 0..6 and O2's in 7..13 (as lbm::scalars_adj).
template <typename R>
__device__ __forceinline__ void scalars_adj(const R (&g)[14], const Vec3<R>& u, const AdjMat3<R>& mt,
                                            const Consts3<R>& k, bool cl, const R (&la)[14], R (&mu)[14], Vec3<R>& lu,
                                            MatAdj3<R>& ma) {
  const R qp = R(0.9282032302755092), qm = R(1.2679491924311228);
  const R kp = R(0.5) * (R(1) - qp), km = R(0.5) * (R(1) - qm), hm = R(0.5) * qm;
  R X[2] = {R(0), R(0)};
#pragma unroll
  for (int q = 0; q < 7; ++q) {
    X[0] += g[q];
    X[1] += g[7 + q];
  }
  ReactAdj<R> rx{};
  if (cl) rx = reaction_tape(X[0], X[1], mt.rhocp, k);
  const R src[2] = {cl ? rx.S_T : R(0), cl ? -rx.s_c : R(0)};
  R lX[2], lsrc[2];
#pragma unroll
  for (int s = 0; s < 2; ++s) {
    const R* a = la + 7 * s;
    R* o = mu + 7 * s;
    const R aw = s == 0 ? mt.aT : mt.aC;
    R le = R(0), lo = R(0);
#pragma unroll
    for (int p = 0; p < 3; ++p) {
      const int i = 2 * p + 1, j = i + 1;
      const R ai = a[i] - a[0], aj = a[j] - a[0];
      const R lnp = ai + aj, lnm = ai - aj;
      le += lnp;
      lo = fma_(along(19 + i, u), lnm, lo);
      add_along(19 + i, hm * X[s] * lnm, lu);
      o[i] = fma_(kp, lnp, km * lnm);
      o[j] = fma_(kp, lnp, -km * lnm);
    }
    const R law = le * fma_(qp, X[s], src[s]);
    if (s == 0) ma.aT += law; else ma.aC += law;
    lX[s] = a[0] + fma_(qp * aw, le, hm * lo);
    lsrc[s] = fma_(aw, le, a[0]);
  }
  if (cl) {  // src_T = S_T(theta, c, rhocp), src_C = -s_c(theta, c)
    const R lsc = fma_(k.four_f_cref * rx.ehs * mt.irc, lsrc[0], -lsrc[1]);
    ma.rhocp -= rx.S_T * mt.irc * lsrc[0];
    lX[1] = fma_(rx.dsc_dc, lsc, lX[1]);
    lX[0] = fma_(rx.dsc_dth, lsc, lX[0]);
    if (k.flags & lbm::F_PHYSICAL_HEAT) lX[0] += k.four_f_cref * rx.s_c * R(2) * k.U0_slope * mt.irc * lsrc[0];
  }
#pragma unroll
  for (int s = 0; s < 2; ++s) {
    R* o = mu + 7 * s;
    o[0] = lX[s];
#pragma unroll
    for (int q = 1; q < 7; ++q) o[q] += lX[s];
  }
}

// Adjoint of the flow collision of one node.  Per opposite pair the forward
// step is (1 - s+) even + w (C + (e u)(e H)) and (1 - s-) odd + w (e G) with
//   C = 3 s+ phi p - (1.5 s+ u^2 + 3 h+ u F) / phi,
//   H = (4.5 s+ u + 9 h+ F) / phi,  G = 3 (s- u + h- F),  h = 1 - s / 2.
// la: the post-collision adjoints, lu: the velocity's from the scalars.  A
// value common to all of la passes to mu unchanged and drops out of the rest
// (the equilibrium and force terms of a node sum to zero), so la[0] is taken
// off before the weighted sums rather than left to cancel after them.
template <typename R>
__device__ __forceinline__ void flow_adj(const MacroTape3<R>& t, const AdjMat3<R>& mt, const Consts3<R>& k,
                                         const R (&la)[19], Vec3<R> lu, R (&mu)[19], MatAdj3<R>& ma) {
  const R sp = k.s_plus, sm = k.s_minus;
  const R hp = R(1) - R(0.5) * sp, hm = R(1) - R(0.5) * sm;
  const R iphi = mt.iphi;
  const Vec3<R> H = scale(iphi, axpy(R(9) * hp, t.F, scale(R(4.5) * sp, t.u)));
  // weights in units of 1/36 (2 for an axis pair, 1 for a diagonal one)
  Vec3<R> lH, lG, lT;
  R lC = R(0);
#pragma unroll
  for (int i = 1; i < 19; i += 2) {
    R le = (la[i] - la[0]) + (la[i + 1] - la[0]), lo = la[i] - la[i + 1];
    if (i < 7) {
      le += le;
      lo += lo;
    }
    lC += le;
    add_along(i, le * along(i, H), lT);
    add_along(i, le * along(i, t.u), lH);
    add_along(i, lo, lG);
  }
  const R c36 = R(1.0 / 36.0);
  lu = axpy(c36, lT, lu);
  lH = scale(c36, lH);
  lG = {nth<12>(lG.x), nth<12>(lG.y), nth<12>(lG.z)};  // three times the weighted sum
  lC *= R(1.0 / 12.0);            // likewise
  const R uF = dot(t.u, t.F);
  const R lpp = sp * lC;
  const R lw = -fma_(R(0.5) * sp, lC, R(0.25) * lpp);  // of u^2 / phi
  const R lz = -hp * lC;                               // of (u F) / phi
  ma.phi -= iphi * (dot(lH, H) + iphi * fma_(lw, t.u2, lz * uF));
  Vec3<R> lF = axpy(R(9) * hp * iphi, lH, axpy(hm, lG, scale(lz * iphi, t.u)));
  lu = axpy(R(4.5) * sp * iphi, lH, axpy(sm, lG, axpy(R(2) * lw * iphi, t.u, axpy(lz * iphi, t.F, lu))));
  const Vec3<R> lv = flow_macros_adj(t, mt, k, lu, lF, ma);
  const R lS = R(0.5) * lpp, ke = R(0.5) * (R(1) - sp), ko = R(0.5) * (R(1) - sm);
  mu[0] = (R(1) - sp) * la[0];
#pragma unroll
  for (int i = 1; i < 19; i += 2) {
    const R e = fma_(ke, la[i] + la[i + 1], lS), o = fma_(ko, la[i] - la[i + 1], along(i, lv));
    mu[i] = e + o;
    mu[i + 1] = e - o;
  }
}

// Transposed extrapolation of the inlet's scalars from column 1 (as
// lbm::inlet_scalars_adj): u, th1, c1 of column 1.
template <typename R>
__device__ __forceinline__ void inlet_scalars_adj(const R (&mu_b)[14], const Vec3<R>& u, R th1, R c1,
                                                  const AdjMat3<R>& mxp, const Consts3<R>& k, Vec3<R>& lu, R& lth1,
                                                  R& lc1, MatAdj3<R>& maxp, MatAdj3<R>& mab) {
#pragma unroll
  for (int s = 0; s < 2; ++s) {
    const R* m = mu_b + 7 * s;
    const R X = s == 0 ? th1 : c1, aw = s == 0 ? mxp.aT : mxp.aC;
    R sum = R(0);
    Vec3<R> d;
#pragma unroll
    for (int i = 1; i < 7; i += 2) {
      sum += m[i] + m[i + 1];
      add_along(19 + i, R(0.5) * (m[i] - m[i + 1]), d);
    }
    const R la = fma_(R(-6), m[0], sum);
    const R lX = -(fma_(aw, la, m[0]) + dot(u, d));
    lu = axpy(-X, d, lu);
    if (s == 0) {
      maxp.aT = fma_(-X, la, maxp.aT);
      lth1 = lX;
    } else {
      maxp.aC = fma_(-X, la, maxp.aC);
      mab.aC = fma_(k.c_in, la, mab.aC);  // + geq(c_in, u_b; aC_b)
      lc1 = lX;
    }
  }
}

// Flow part of the transposed extrapolation: adds to the adjoints of xp's
// velocity and phi p and to the materials'.  inlet: velocity (ub, 0, 0) and
// xp's pressure at b; else xp's velocity and zero pressure.
template <typename R>
__device__ __forceinline__ void boundary_flow_adj(const R (&m)[19], const Vec3<R>& u, R pp, bool inlet, R ub,
                                                  R iphi_p, R phi_b, R iphi_b, Vec3<R>& lu, R& lpp, MatAdj3<R>& maxp,
                                                  MatAdj3<R>& mab) {
  R sum = R(0), xx = R(0), yy = R(0), zz = R(0), xy = R(0), xz = R(0), yz = R(0);
  Vec3<R> d;
#pragma unroll
  for (int i = 1; i < 19; i += 2) {
    const R w = weight<R>(i);
    const R le = w * ((m[i] - m[0]) + (m[i + 1] - m[0]));  // a common value drops out, as in flow_adj
    sum += le;
    add_along(i, R(3) * w * (m[i] - m[i + 1]), d);
    if (EX[i]) xx += le;
    if (EY[i]) yy += le;
    if (EZ[i]) zz += le;
    if (EX[i] && EY[i]) xy = EX[i] * EY[i] > 0 ? xy + le : xy - le;
    if (EX[i] && EZ[i]) xz = EX[i] * EZ[i] > 0 ? xz + le : xz - le;
    if (EY[i] && EZ[i]) yz = EY[i] * EZ[i] > 0 ? yz + le : yz - le;
  }
  const R ldpp = R(3) * sum, lw = R(-1.5) * sum;
  // gradient T u and value u T u of the quadratic part, T = 4.5 sum w l e e + lw
  const R c = R(4.5);
  auto T = [&](const Vec3<R>& a) {
    return Vec3<R>{fma_(fma_(c, xx, lw), a.x, c * fma_(xy, a.y, xz * a.z)),
                   fma_(fma_(c, yy, lw), a.y, c * fma_(xy, a.x, yz * a.z)),
                   fma_(fma_(c, zz, lw), a.z, c * fma_(xz, a.x, yz * a.y))};
  };
  const Vec3<R> g = T(u);
  const R e2 = dot(u, g);
  lu = axpy(R(-2) * iphi_p, g, axpy(R(-1), d, lu));
  maxp.phi = fma_(iphi_p * iphi_p, e2, maxp.phi);
  lpp -= ldpp;
  if (inlet) {
    lpp = fma_(ldpp * iphi_p, phi_b, lpp);
    maxp.phi -= ldpp * pp * phi_b * iphi_p * iphi_p;
    mab.phi += ldpp * pp * iphi_p - iphi_b * iphi_b * ub * ub * fma_(c, xx, lw);
  } else {
    lu = axpy(R(2) * iphi_b, g, axpy(R(1), d, lu));
    mab.phi -= iphi_b * iphi_b * e2;
  }
}

}  // namespace lbm3
