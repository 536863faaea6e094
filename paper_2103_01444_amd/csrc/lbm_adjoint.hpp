// Discrete adjoint of the coupled step (reverse mode, written by hand).
//
// The forward step is S' = C(P(S)): P pulls the populations (a permutation
// with half-way bounce-back) and applies the inlet / outlet extrapolation
// columns, C collides every node.  With lambda the adjoint of S', the
// adjoint of S is obtained per node x by
//   mu_x  = (dC_x / d pre_x)^T lambda_x                       (collision)
//   mu_xp += (dB / d pre_xp)^T mu_b     for the boundary node b fed by xp
//   lambda_new[source of pull (x, q)] = mu_x[q]
// Every element of the state is pulled by exactly one node; boundary nodes,
// whose pulled values the forward step discards, have mu = 0.  Each node
// accumulates only its own gradient with respect to (porosity, 1/K, D_eff).
#pragma once

#include "lbm_device.hpp"

namespace lbm {

// 1 / a and sqrt(a) from the hardware estimates and Newton steps, within 1
// ulp (the forward step's are IEEE's: lbm_device.hpp, where the range of the
// operands is discussed).  A root below the bound of its operand's comes out
// too small, which no result can feel (it is a speed that is added to 1/2).
// FP32: 3 and 6 instructions instead of 10 and 16, FP64: 5 and 11 instead of
// 10 and 20.
template <typename R>
__device__ __forceinline__ R fast_rcp(R a) { return rcp_seed(a); }
// 1 / a of an a that may be infinite: 0.
template <typename R>
__device__ __forceinline__ R fast_rcp_inf(R a) { return rcp_seed(a, below_inf(a)); }
__device__ __forceinline__ float fast_root(float a, float c, float y) {
  const float s = c * y;
  return fma_(fma_(-s, s, a), 0.5f * y, s);
}
__device__ __forceinline__ double fast_root(double a, double c, double y) { return root_(a, c, y); }
__device__ __forceinline__ float fast_sqrt(float a) {
  return fast_root(a, a, rsq_(__builtin_fmaxf(a, 1.17549435e-38f)));
}
__device__ __forceinline__ double fast_sqrt(double a) { return fast_root(a, a, rsq_(__builtin_fmax(a, 1e-300))); }
// sqrt(l0^2 + l1 |v|), as momentum_denominator's.
template <typename R>
__device__ __forceinline__ R fast_momentum_root(R l0, R l1, R vm) {
  const R q = fma_(l1, vm, l0 * l0), c = below_inf(q);
  return fast_root(q, c, rsq_(c));
}

// Sum of the five populations g of a scalar lattice, and the temperature
// rise from the five temperature populations (isig: 1 / sigma, 1 without the
// heat-capacity ratio).
template <typename R>
__device__ __forceinline__ R sum5(const R* g) {
  return g[0] + ((g[1] + g[3]) + (g[2] + g[4]));
}
template <typename R>
__device__ __forceinline__ R theta_of(const R* g, R isig) {
  return sum5(g) * isig;
}

// The forward step's material with what the reverse step takes of it:
// 1 / phi, the linear drag coefficient dl = phi nu / K, the equilibrium
// weights a = (4 + b) / 20 of a moving scalar population and the reciprocals
// of rho c_p and sigma.
template <typename R>
struct AdjMat : Mat<R> {
  R iphi, dl, aT, aC, irc, isig;
};
template <typename R>
__device__ __forceinline__ AdjMat<R> adj_material(const Consts<R>& k, const R* __restrict__ phi_f,
                                                  const R* __restrict__ invk_f, const R* __restrict__ d_f, int x,
                                                  int y) {
  AdjMat<R> m;
  static_cast<Mat<R>&>(m) = material<R, MAT_FULL>(k, phi_f, invk_f, d_f, x, y);
  m.iphi = fast_rcp(m.phi);
  m.dl = m.phi * k.nu * m.invk;
  m.aT = fma_(R(0.05), m.bT, R(0.2));
  m.aC = fma_(R(0.05), m.bC, R(0.2));
  m.irc = fast_rcp(m.rhocp);
  m.isig = (k.flags & F_SIGMA_ENERGY) ? k.rhocp_f * m.irc : R(1);
  return m;
}
// outlet_scalar_material with the reverse step's quantities.
template <typename R>
__device__ __forceinline__ void outlet_scalar_adj_material(AdjMat<R>& mb, const AdjMat<R>& mp) {
  outlet_scalar_material(mb, mp);
  mb.aT = mp.aT;
  mb.aC = mp.aC;
  mb.irc = mp.irc;
  mb.isig = mp.isig;
}

// Lane shift of the reverse step: lane l of a row's first workgroup holds
// x = l - shift, so that columns nx - 2 and nx - 1 share a wavefront (as
// columns 0 and 1 do) at every width.
__host__ __device__ inline int adj_lane_shift(int nx) { return ((nx - 1) & 63) == 0 ? 1 : 0; }

// EXT: the instances of the reverse step that also cover Boussinesq
// buoyancy, the energy equation with the heat-capacity ratio sigma, the
// pressure-driven inlet and the thin-film CL; the default instances leave
// their terms out (and their registers free).
//
// Adjoints of the medium's quantities as the forward step uses them.
template <typename R>
struct MatAdj {
  R phi = R(0), dl = R(0), l0 = R(0), l1 = R(0), aT = R(0), aC = R(0), rhocp = R(0);
  R sig = R(0);  // heat-capacity ratio (EXT only)
};

// Chain the adjoints of the derived material quantities to (phi, 1/K, D).
template <typename R, bool EXT = false>
__device__ __forceinline__ void material_adj(const Consts<R>& k, const AdjMat<R>& m, const MatAdj<R>& a, R& g_phi,
                                             R& g_invk, R& g_d) {
  // dl = phi nu / K, l0 = 1/2 + dl / 4, l1 = c phi^-1/2 K^-1/2 (its
  // derivative in 1/K taken as 0 at 1/K = 0, the clear fluid)
  const R ldl = fma_(R(0.25), a.l0, a.dl);
  R lphi = a.phi + k.nu * m.invk * ldl - R(0.5) * a.l1 * m.l1 * m.iphi;
  R linvk = m.phi * k.nu * ldl;
  if (m.invk > R(0)) linvk += R(0.5) * a.l1 * m.l1 / m.invk;
  // rho c_p = phi rhocp_f + (1 - phi) rhocp_s; aT = sqrt 3 alpha (Eq. 19)
  const R drc = k.rhocp_f - k.rhocp_s, dk = k.aT_f - k.aT_s;
  if (EXT && (k.flags & F_SIGMA_ENERGY)) {  // aT = k_eff / (rho c_p)_f, sigma = rho c_p / (rho c_p)_f
    lphi += a.aT * dk * k.irc_f + (a.rhocp + a.sig * k.irc_f) * drc;
  } else {
    lphi += a.aT * (dk - m.aT * drc) * m.irc + a.rhocp * drc;
  }
  g_phi += lphi;
  g_invk += linvk;
  g_d += a.aC * R(1.7320508075688772935);
}

// Forward intermediates of flow_macros kept for its adjoint.
template <typename R>
struct MacroTape {
  R vx, vy, vm, ir, iden, ux, uy, u2, Fx, Fy, drag;  // ir: 1 / sqrt(l0^2 + l1 |v|)
  R ax, ay, thb;  // acceleration, and the temperature rise buoyancy takes it from (EXT)
};

// The acceleration a of flow_macros is on when the test-mode body force is,
// or (EXT) Boussinesq buoyancy.
template <typename R, bool EXT>
__device__ __forceinline__ bool accelerated(const Consts<R>& k) {
  return (k.flags & F_BODY_FORCE) || (EXT && (k.flags & F_BUOYANCY));
}

// f: the nine flow populations; th: the node's temperature rise (EXT).
template <typename R, bool EXT>
__device__ __forceinline__ MacroTape<R> flow_macros_tape(const R* f, R th, const AdjMat<R>& m, const Consts<R>& k) {
  MacroTape<R> t;
  const R b57 = f[5] - f[7], b68 = f[6] - f[8];
  t.vx = (f[1] - f[3]) + (b57 - b68);
  t.vy = (f[2] - f[4]) + (b57 + b68);
  t.ax = t.ay = t.thb = R(0);
  if (accelerated<R, EXT>(k)) {
    if (k.flags & F_BODY_FORCE) {
      t.ax = k.ax;
      t.ay = k.ay;
    }
    if (EXT && (k.flags & F_BUOYANCY)) {
      t.thb = th;
      t.ax += k.bx * th;
      t.ay += k.by * th;
    }
    t.vx += R(0.5) * m.phi * t.ax;
    t.vy += R(0.5) * m.phi * t.ay;
  }
  t.vm = fast_sqrt(fma_(t.vx, t.vx, t.vy * t.vy));
  const R r = fast_momentum_root(m.l0, m.l1, t.vm);
  t.ir = fast_rcp_inf(r);
  t.iden = fast_rcp_inf(m.l0 + r);
  t.ux = t.vx * t.iden;
  t.uy = t.vy * t.iden;
  t.u2 = fma_(t.ux, t.ux, t.uy * t.uy);
  t.drag = fma_(R(2) * m.l1, t.vm * t.iden, m.dl);
  t.Fx = -t.drag * t.ux;
  t.Fy = -t.drag * t.uy;
  if (accelerated<R, EXT>(k)) {
    t.Fx += m.phi * t.ax;
    t.Fy += m.phi * t.ay;
  }
  return t;
}

// Adjoint of v -> (u, F): from the adjoints of u and F the adjoints lvx, lvy
// of v = sum e f; the material's added to ma.  With buoyancy (EXT) the
// adjoint of the temperature rise is added to lth.
template <typename R, bool EXT>
__device__ __forceinline__ void flow_macros_adj(const MacroTape<R>& t, const AdjMat<R>& m, const Consts<R>& k, R lux,
                                                R luy, R lFx, R lFy, R& lvx, R& lvy, R& lth, MatAdj<R>& ma) {
  // F = -drag u (+ phi a), drag = dl + 2 l1 |v| / den
  const R um = t.vm * t.iden;
  const R ldrag = -fma_(t.ux, lFx, t.uy * lFy);
  lux = fma_(-t.drag, lFx, lux);
  luy = fma_(-t.drag, lFy, luy);
  ma.dl += ldrag;
  ma.l1 = fma_(R(2) * um, ldrag, ma.l1);
  const R lum = R(2) * m.l1 * ldrag;
  // u = v / den, |u| = |v| / den, den = l0 + r, r = sqrt(l0^2 + l1 |v|)
  const R lden = -t.iden * fma_(um, lum, fma_(t.ux, lux, t.uy * luy));
  const R ldr = lden * t.ir;
  ma.l0 += fma_(ldr, m.l0, lden);
  ma.l1 = fma_(R(0.5) * t.vm, ldr, ma.l1);
  const R lvm = fma_(R(0.5) * m.l1, ldr, lum * t.iden);
  lvx = lux * t.iden;
  lvy = luy * t.iden;
  if (t.vm > R(0)) {  // |v| of a cell at rest: derivative taken as 0
    const R q = lvm / t.vm;
    lvx = fma_(q, t.vx, lvx);
    lvy = fma_(q, t.vy, lvy);
  }
  if (accelerated<R, EXT>(k)) {  // a enters F as phi a and v as phi a / 2
    const R lx = fma_(R(0.5), lvx, lFx), ly = fma_(R(0.5), lvy, lFy);
    ma.phi += t.ax * lx + t.ay * ly;
    if (EXT && (k.flags & F_BUOYANCY)) lth += m.phi * (k.bx * lx + k.by * ly);
  }
}

// Share of the adjoint of theta = (sum g) / sigma that goes onto every
// population; sigma's own part to ma.
template <typename R, bool EXT>
__device__ __forceinline__ R theta_adj(R lth, R th, const AdjMat<R>& m, const Consts<R>& k, MatAdj<R>& ma) {
  if (EXT && (k.flags & F_SIGMA_ENERGY)) {
    ma.sig -= th * m.isig * lth;
    return lth * m.isig;
  }
  return lth;
}

// Reaction sensitivities: ds_c/dc, ds_c/dtheta, and S_T's.
template <typename R>
struct ReactAdj {
  R s_c, S_T, ehs, dsc_dc, dsc_dth;
};

// A rate and its derivative in T, at x = (T - T_in) / T and dx = dx/dT.
//
// The exponents of the reaction are differences of numbers of order 50 whose
// FP32 roundings are 2e-6 of the rate, the same in all cells of a catalyst
// layer of one temperature.  The forward step has them (its bits are those of
// the state); the reverse step starts from the value at T_in, computed on the
// host, and is off by 1e-7.  Error of the reverse sweep itself (against the
// 64-bit adjoint of the FP32 trajectory), 224x42 over 106 steps: d/dphi
// 4.9e-6 -> 4.7e-7, d/dD_eff 6.3e-6 -> 6.6e-7.
template <typename R>
__device__ __forceinline__ R rate_at(const RateFromInlet<R>& r, R x, R dx, R& slope) {
  const R v = r.fac * exp(fma_(r.d, x, r.ln));
  slope = v * (r.d * dx);
  return v;
}

// Tape of the CL reaction (Eqs. 12-17, Tafel or Butler-Volmer, printed or
// physical heat) and its derivatives: s_c = -(c - c_eq) expm1(-kappa), c_eq =
// exp(alpha_sum F eta / (R T)) with Butler-Volmer (0 with Tafel), S_T = 4 F
// C_ref s_c ehs / (rho c_p).  With the printed heat ehs = eta + T dU0/dT = V -
// U0(0) does not depend on T; with the physical heat ehs = -eta + T dU0/dT has
// dehs/dT = 2 dU0/dT, which the callers add to the temperature adjoint.
template <typename R, typename K>
__device__ __forceinline__ ReactAdj<R> reaction_tape(R theta, R c, R rhocp, const K& k) {
  const R T = k.T_in + theta;
  const R iT = R(1) / T;
  const R x = theta * iT, dx = k.T_in * iT * iT;
  const R eta = k.V_op - (k.U0_slope * T + k.U0_icept);
  R dkappa, dceq = R(0);
  const R kappa = rate_at(k.kappa, x, dx, dkappa);
  const R ceq = k.bv ? rate_at(k.ceq, x, dx, dceq) : R(0);
  const R em = expm1(-kappa);
  ReactAdj<R> r;
  r.s_c = -(c - ceq) * em;
  r.ehs = ((k.flags & F_PHYSICAL_HEAT) ? -eta : eta) + T * k.U0_slope;
  r.S_T = k.four_f_cref * r.s_c * r.ehs / rhocp;
  r.dsc_dc = -em;
  r.dsc_dth = (c - ceq) * (em + R(1)) * dkappa + em * dceq;
  return r;
}

// Tape of the thin-film reaction (surface_reaction: the populations g_t, g_c
// that cross the reactive wall, wall values g / a)
// and its derivatives with respect to the wall temperature T, g_c and a_c.
template <typename R>
struct FilmTape {
  R a_t, th, s, S_T, ehs, em, ds_dT, ds_dac, dehs_dT;
};

template <typename R>
__device__ __forceinline__ FilmTape<R> film_tape(R g_t, R g_c, const AdjMat<R>& m, const Consts<R>& k) {
  FilmTape<R> f;
  f.a_t = m.aT;
  const R a_c = m.aC;
  f.th = g_t / f.a_t;
  const R T = k.T_in + f.th;
  const R iT = R(1) / T;
  const R x = f.th * iT, dx = k.T_in * iT * iT;
  const R eta = k.V_op - (k.U0_slope * T + k.U0_icept);
  R dkappa, dceq = R(0);
  const R film = exp(k.ln_thin) / a_c;
  const R kappa_a = rate_at(k.kappa, x, dx, dkappa) * film;
  const R ceq = k.bv ? rate_at(k.ceq, x, dx, dceq) : R(0);
  f.em = expm1(-kappa_a);
  f.s = -(g_c - a_c * ceq) * f.em;
  const bool phys = k.flags & F_PHYSICAL_HEAT;
  f.ehs = (phys ? -eta : eta) + T * k.U0_slope;
  f.S_T = k.four_f_cref * f.s * f.ehs / m.rhocp;
  // ds/dkappa = (g_c - a_c c_eq)(em + 1), ds/dc_eq = a_c em
  const R ds_dk = (g_c - a_c * ceq) * (f.em + R(1));
  f.ds_dT = ds_dk * (dkappa * film) + a_c * f.em * dceq;
  f.ds_dac = -ds_dk * kappa_a / a_c + ceq * f.em;
  f.dehs_dT = phys ? R(2) * k.U0_slope : R(0);
  return f;
}

// Transpose of the film's update of the two populations, g_t += sigma S_T
// and g_c -= s: given the adjoints l13, l18 of the updated values, returns
// those of the incoming ones in place and adds the material adjoints.
// ls, le: adjoints of s and of the heat factor from other uses (the seed
// of J takes ls = its weight).
template <typename R>
__device__ __forceinline__ void film_adj(const FilmTape<R>& f, const AdjMat<R>& m, const Consts<R>& k, R ls, R& l13,
                                         R& l18, MatAdj<R>& ma) {
  const R sg = (k.flags & F_SIGMA_ENERGY) ? m.sig : R(1);
  const R irc = R(1) / m.rhocp;
  const R lST = sg * l13;
  if (k.flags & F_SIGMA_ENERGY) ma.sig += f.S_T * l13;
  ls += lST * k.four_f_cref * f.ehs * irc - l18;
  const R lehs = lST * k.four_f_cref * f.s * irc;
  ma.rhocp += -lST * f.S_T * irc;
  const R lT = ls * f.ds_dT + lehs * f.dehs_dT;
  l13 += lT / f.a_t;
  l18 += -ls * f.em;
  // T = T_in + g_t / a_t
  ma.aT += -lT * f.th / f.a_t;
  ma.aC += ls * f.ds_dac;
}

// Adjoint of the two scalar collisions of one node and of the CL source.
// g[0..4] temperature, g[5..9] O2 (pre-collision), la their post-collision
// adjoints; out: mu[0..9], the adjoints lux, luy of the velocity, the
// material's in ma.  The rest population is the conserved sum minus the
// moving ones, so its adjoint passes to every population unchanged and is
// taken off the moving ones' before they are relaxed.
template <typename R, bool EXT>
__device__ __forceinline__ void scalars_adj(const R (&g)[10], R ux, R uy, const AdjMat<R>& mt, const Consts<R>& k,
                                            bool cl, const R (&la)[10], R (&mu)[10], R& lux, R& luy, MatAdj<R>& ma) {
  const bool sigma = EXT && (k.flags & F_SIGMA_ENERGY);
  const R q1 = R(1.2679491924311228), q3 = R(0.9282032302755092);
  const R k1 = R(0.5) * (R(1) - q1), k3 = R(0.5) * (R(1) - q3), h1 = R(0.5) * q1;
  const R X[2] = {theta_of(g, mt.isig), sum5(g + 5)};
  ReactAdj<R> rx{};
  if (cl) rx = reaction_tape(X[0], X[1], mt.rhocp, k);
  const R src[2] = {cl ? rx.S_T : R(0), cl ? -rx.s_c : R(0)};
  R lX[2], lsrc[2];
#pragma unroll
  for (int s = 0; s < 2; ++s) {
    const R* a = la + 5 * s;
    R* o = mu + 5 * s;
    const R a1 = a[1] - a[0], a2 = a[2] - a[0], a3 = a[3] - a[0], a4 = a[4] - a[0];
    const R le1 = a1 + a3, le2 = a2 + a4, lo1 = a1 - a3, lo2 = a2 - a4, le = le1 + le2;
    const R aw = s == 0 ? mt.aT : mt.aC;
    const R law = le * fma_(q3, X[s], src[s]);
    if (s == 0) ma.aT += law; else ma.aC += law;
    lsrc[s] = fma_(aw, le, (sigma && s == 0) ? mt.sig * a[0] : a[0]);
    if (sigma && s == 0) ma.sig += src[0] * a[0];
    lX[s] = fma_(q3 * aw, le, h1 * fma_(ux, lo1, uy * lo2));
    lux = fma_(h1 * X[s], lo1, lux);
    luy = fma_(h1 * X[s], lo2, luy);
    o[0] = a[0];
    o[1] = fma_(k3, le1, k1 * lo1);
    o[2] = fma_(k3, le2, k1 * lo2);
    o[3] = fma_(k3, le1, -k1 * lo1);
    o[4] = fma_(k3, le2, -k1 * lo2);
  }
  if (cl) {  // src_T = S_T(theta, c, rho c_p), src_C = -s_c(theta, c)
    const R lsc = fma_(k.four_f_cref * rx.ehs * mt.irc, lsrc[0], -lsrc[1]);
    ma.rhocp -= rx.S_T * mt.irc * lsrc[0];
    lX[1] = fma_(rx.dsc_dc, lsc, lX[1]);
    lX[0] = fma_(rx.dsc_dth, lsc, lX[0]);
    if (k.flags & F_PHYSICAL_HEAT) lX[0] += k.four_f_cref * rx.s_c * R(2) * k.U0_slope * mt.irc * lsrc[0];
  }
#pragma unroll
  for (int s = 0; s < 2; ++s) {
    R* o = mu + 5 * s;
    const R l = o[0] + (s == 0 ? theta_adj<R, EXT>(lX[0], X[0], mt, k, ma) : lX[1]);
    o[0] = l;
#pragma unroll
    for (int i = 1; i < 5; ++i) o[i] += l;
  }
}

// Adjoints of the flow sums of a node, onto its populations.
template <typename R>
__device__ __forceinline__ void flow_sums_adj(R l0, R lS, R lA, R lN, R lM, R lJx, R lJy, R lqx, R lqy, R (&mu)[9]) {
  const R l13 = lS + (lA + lN), l24 = lS + (lA - lN), l57 = lS + lM, l68 = lS - lM;
  const R b13 = fma_(R(-2), lqx, lJx), b24 = fma_(R(-2), lqy, lJy);
  const R dx = lJx + lqx, dy = lJy + lqy, b57 = dx + dy, b68 = dy - dx;
  mu[0] = l0;
  mu[1] = l13 + b13;
  mu[3] = l13 - b13;
  mu[2] = l24 + b24;
  mu[4] = l24 - b24;
  mu[5] = l57 + b57;
  mu[7] = l57 - b57;
  mu[6] = l68 + b68;
  mu[8] = l68 - b68;
}

// a / N to the last bit or so.  The adjoint of a conserved moment passes
// through every step unchanged; fl(1 / N) would scale it by 1 + 3e-8 (FP32)
// at each.
template <int N, typename R>
__device__ __forceinline__ R nth(R a) {
  const R c = R(1.0 / N), q = c * a;
  return fma_(fma_(R(-N), q, a), c, q);
}

// Adjoint of the flow collision of one node in the sums of `collide`, S the
// sum of its moving populations: la[0..8] the post-collision adjoints, lux,
// luy the velocity's from the scalars; out: mu[0..8].
template <typename R, bool EXT>
__device__ __forceinline__ void flow_adj(const MacroTape<R>& t, const AdjMat<R>& mt, const Consts<R>& k,
                                         const R (&la)[9], R lux, R luy, R (&mu)[9], R& lth, MatAdj<R>& ma) {
  const R se = k.s_e, sq = k.s_q;
  const R ke = R(1) - se, kq = R(1) - sq, he = R(1) - R(0.5) * se, hq = R(1) - R(0.5) * sq;
  const R iphi = mt.iphi;
  // outputs -> S', A', N', M', j', q'
  const R s13 = la[1] + la[3], s24 = la[2] + la[4], s57 = la[5] + la[7], s68 = la[6] + la[8];
  const R d13 = la[1] - la[3], d24 = la[2] - la[4], d57 = la[5] - la[7], d68 = la[6] - la[8];
  const R lB = R(0.25) * (s57 + s68);
  const R lA = fma_(R(0.25), s13 + s24, -lB), lN = R(0.25) * (s13 - s24), lM2 = R(0.125) * (s57 - s68);
  const R c6 = R(1.0 / 6.0);
  const R gx = d57 - d68, gy = d57 + d68;
  const R ljx = nth<6>(d13 + gx), ljy = nth<6>(d24 + gy);
  const R lqx = c6 * fma_(R(0.5), gx, -d13), lqy = c6 * fma_(R(0.5), gy, -d24);
  const R lS = fma_(se, fma_(R(0.8), lA, -la[0]), lB);
  const R lz = (R(4.0 / 3.0) * he) * (fma_(R(0.5), lA, lB) - la[0]);  // of (u F) / phi
  const R lw = R(-0.2) * se * lA;                                      // of u^2 / phi
  // N and M: u_i P_j with P = (s_e u + (2 - s_e) F) / phi
  const R Px = iphi * fma_(R(2) * he, t.Fx, se * t.ux), Py = iphi * fma_(R(2) * he, t.Fy, se * t.uy);
  const R lPx = fma_(lN, t.ux, lM2 * t.uy), lPy = fma_(-lN, t.uy, lM2 * t.ux);
  const R uF = fma_(t.ux, t.Fx, t.uy * t.Fy);
  ma.phi -= iphi * (fma_(lPx, Px, lPy * Py) + iphi * fma_(lw, t.u2, lz * uF));
  const R e = se * iphi, h = R(2) * he * iphi, z = lz * iphi, w2 = R(2) * lw * iphi;
  R lFx = ljx - hq * lqx + h * lPx + z * t.ux;
  R lFy = ljy - hq * lqy + h * lPy + z * t.uy;
  lux += lN * Px + lM2 * Py + e * lPx + z * t.Fx + w2 * t.ux - sq * lqx;
  luy += lM2 * Px - lN * Py + e * lPy + z * t.Fy + w2 * t.uy - sq * lqy;
  R lvx, lvy;
  flow_macros_adj<R, EXT>(t, mt, k, lux, luy, lFx, lFy, lvx, lvy, lth, ma);
  flow_sums_adj(ke * la[0], lS, ke * lA, ke * lN, R(2) * ke * lM2, ljx + lvx, ljy + lvy, kq * lqx, kq * lqy, mu);
}

// Transposed extrapolation of a boundary node b from the column xp next to
// it.  Both take part: mu_b is the adjoint of b's pre-collision populations,
// (ux, uy, pp) xp's velocity and phi p.  Per boundary kind the extrapolated
// equilibrium takes the velocity (velocity inlet: fixed) and phi p
// (velocity inlet: phi_b p of xp; else phi_b times a given pressure pb).
//
// Scalar part (inlet only): mu_b[0..9], th1 and c1 of xp; adds the adjoints
// of xp's populations to lth1 and lc1 (per population) and of its velocity to
// lux, luy, and the materials'.
template <typename R, bool EXT>
__device__ __forceinline__ void inlet_scalars_adj(const R (&mu_b)[10], R ux, R uy, R th1, R c1, bool pressure,
                                                  const AdjMat<R>& mxp, const Consts<R>& k, R& lux, R& luy, R& lth1,
                                                  R& lc1, MatAdj<R>& maxp, MatAdj<R>& mab) {
#pragma unroll
  for (int s = 0; s < 2; ++s) {
    const R* m = mu_b + 5 * s;
    const R X = s == 0 ? th1 : c1, aw = s == 0 ? mxp.aT : mxp.aC;
    const R d1 = R(0.5) * (m[1] - m[3]), d2 = R(0.5) * (m[2] - m[4]);
    const R la = ((m[1] + m[3]) + (m[2] + m[4])) - R(4) * m[0];
    const R sig = (EXT && s == 0) ? mxp.sig : R(1);
    const R lX = -(fma_(aw, la, sig * m[0]) + fma_(ux, d1, uy * d2));
    lux = fma_(-X, d1, lux);
    luy = fma_(-X, d2, luy);
    if (s == 0) {
      maxp.aT = fma_(-X, la, maxp.aT);
      if (EXT) maxp.sig = fma_(-X, m[0], maxp.sig);
      lth1 = theta_adj<R, EXT>(lX, th1, mxp, k, maxp);
    } else {
      maxp.aC = fma_(-X, la, maxp.aC);
      mab.aC = fma_(k.c_in, la, mab.aC);  // + geq(c_in, u_b; aC_b)
      if (pressure) {
        lux = fma_(k.c_in, d1, lux);
        luy = fma_(k.c_in, d2, luy);
      }
      lc1 = lX;
    }
  }
}

// Flow part: mu_b[0..8]; adds to the velocity's adjoint and to lpp (of phi p
// of xp).
template <typename R>
__device__ __forceinline__ void boundary_flow_adj(const R (&m)[9], R ux, R uy, R pp, bool fixed_u, R ubx, R pb,
                                                  const AdjMat<R>& mxp, R phi_b, R iphi_b, R& lux, R& luy, R& lpp,
                                                  MatAdj<R>& maxp, MatAdj<R>& mab) {
  const R s13 = m[1] + m[3], s24 = m[2] + m[4], s57 = m[5] + m[7], s68 = m[6] + m[8];
  const R d13 = m[1] - m[3], d24 = m[2] - m[4], d57 = m[5] - m[7], d68 = m[6] - m[8];
  const R c12 = R(1.0 / 12.0), c3 = R(1.0 / 3.0);
  const R lA = s13 + s24, lB = s57 + s68;
  const R ldpp = fma_(R(-5.0 / 3.0), m[0], fma_(c3, lA, c12 * lB));
  const R ldu2 = fma_(R(-2.0 / 3.0), m[0], c12 * (lA + lB));
  const R dN = R(0.25) * (s13 - s24);
  const R lxx = ldu2 + dN, lyy = ldu2 - dN, lxy = R(0.25) * (s57 - s68);
  const R ldx = fma_(c3, d13, c12 * (d57 - d68)), ldy = fma_(c3, d24, c12 * (d57 + d68));
  const R gx = fma_(R(2) * ux, lxx, uy * lxy), gy = fma_(R(2) * uy, lyy, ux * lxy);
  const R e2 = fma_(ux * ux, lxx, fma_(uy * uy, lyy, ux * uy * lxy));
  // - (xp's equilibrium)
  lux -= fma_(mxp.iphi, gx, ldx);
  luy -= fma_(mxp.iphi, gy, ldy);
  maxp.phi = fma_(mxp.iphi * mxp.iphi, e2, maxp.phi);
  lpp -= ldpp;
  if (fixed_u) {  // velocity u_b = (ubx, 0), phi p = phi_b (phi p)_xp / phi_xp
    lpp = fma_(ldpp * mxp.iphi, phi_b, lpp);
    maxp.phi -= ldpp * pp * phi_b * mxp.iphi * mxp.iphi;
    mab.phi += ldpp * pp * mxp.iphi - iphi_b * iphi_b * ubx * ubx * lxx;
  } else {  // xp's velocity, phi p = phi_b pb
    lux += fma_(iphi_b, gx, ldx);
    luy += fma_(iphi_b, gy, ldy);
    mab.phi += ldpp * pb - iphi_b * iphi_b * e2;
  }
}

}  // namespace lbm
