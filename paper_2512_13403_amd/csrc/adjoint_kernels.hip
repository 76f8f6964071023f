// adjoint_kernels.hip -- reverse-mode derivative of the finite-volume step
// (arXiv 2512.13403, Sec. 2.3 and 6.2.4) for gfx950.
//
// With dt held fixed, the derivative of one step U^n -> U^{n+1} is applied in
// transposed form, lam^n = (dU^{n+1}/dU^n)^T lam^{n+1}, source by source in
// reverse order and then through the two RK stages:
//   lam1 = lam_a/2 + (dt/2) J(U1)^T lam_a,   lam^n = lam_a/2 + lam1 + dt J(U^n)^T lam1.
// J(U)^T v for L(U) = -sum_a (F_{a,i+1/2} - F_{a,i-1/2}) / h_a is deterministic
// (no floating-point atomics).  The periodic minmod (or first-order) HLLC scheme
// takes one kernel per axis, k_x_jtv and k_axis_jtv; the general path two passes
// per axis:
//   k_face_vjp    one thread per face: Fb = (v_right - v_left)/h, the HLLC
//                 reverse sweep gives the face-state adjoints W^L_b, W^R_b, and
//                 the minmod selections of the two slopes the face used;
//   k_cell_gather one thread per cell: sums, over the (at most four) faces
//                 whose stencil reads the cell, the reverse of
//                 W^L = W_i + minmod(..)/2, W^R = W_{i+1} - minmod(..)/2;
// and k_jtv_finish applies (dW/dU)^T per cell.  At every kink the derivative
// of the branch the forward took is used (minmod: the returned argument, or 0;
// wave-speed min/max: the selected argument, the first on ties; HLLC: the
// side and fan the face fell in).  The other limiters and solvers run in
// k_face_vjp_rt, which takes them at run time and writes each face's four
// stencil contributions instead of the minmod selections: the slope partials
// dphi/da, dphi/db of van Leer (2b^2/(a+b)^2, 2a^2/(a+b)^2), MC ((1/2, 1/2),
// (2, 0) or (0, 2), ties in that order) and superbee ((2, 0), (0, 1), (1, 0)
// or (0, 2)), and the HLL / Rusanov reverse sweeps.
#include "mg.h"
#include "mh_adjoint.h"
#include "mh_device.h"

namespace mh {

namespace {

__device__ __forceinline__ int minmod_sel(float a, float b) {
  return (a * b <= 0.0f) ? 0 : (fabsf(a) <= fabsf(b) ? 1 : 2);
}
__device__ __forceinline__ int minmod_sel(double a, double b) {
  return (a * b <= 0.0) ? 0 : (fabs(a) <= fabs(b) ? 1 : 2);
}
template <typename T>
__device__ __forceinline__ T sel_value(int s, T a, T b) {
  return s == 1 ? a : (s == 2 ? b : T(0));
}

// primitive variables of cell q, with the arithmetic of the stage kernels
// (so every limiter and wave-speed branch is taken as in the forward step)
template <typename T>
__device__ __forceinline__ void prim_at(const T* __restrict__ U, long long N, long long q, T gm1,
                                        T (&w)[5]) {
  T u[5];
#pragma unroll
  for (int f = 0; f < 5; ++f) u[f] = U[f * N + q];
  to_prim(u, gm1, w);
}

// the same as the products of to_prim, W = x y: rho 1, m (1/rho), e (g - 1)
template <typename T>
__device__ __forceinline__ void prim_factors_at(const T* __restrict__ U, long long N, long long q,
                                                T gm1, T (&x)[5], T (&y)[5]) {
  T u[5], w[5];
#pragma unroll
  for (int f = 0; f < 5; ++f) x[f] = u[f] = U[f * N + q];
  to_prim(u, gm1, w);
  y[0] = T(1);
  y[1] = y[2] = y[3] = dev_rcp(u[0]);
  x[4] = fmad(-(T(0.5) * u[0]), fmad(w[1], w[1], fmad(w[2], w[2], w[3] * w[3])), u[4]);
  y[4] = gm1;
}

// a difference that is not contracted with the product behind an operand
template <typename T>
__device__ __forceinline__ T plain_diff(T a, T b) {
#pragma clang fp contract(off)
  return a - b;
}

// Differences of W for the limiter branches of the face-wise kernels and of the x
// rows.  The stage kernels subtract rounded values of W, so where velocity or
// pressure does not change, the slope is exactly zero and the step took no branch,
// while a difference contracted with the product behind W, fma(m, 1/rho, -W_c),
// leaves the rounding error of that product, of either sign: both sides of a cell
// then take a branch, and not the same one.  fp64 subtracts rounded values, as the
// step does.  fp32 keeps the contracted differences, which decide the near-ties
// of a varying field as exact arithmetic does more often (gradient of a turbulent
// 256^3 step against 64 bits: 7.6e-4 off, 7.8e-4 with rounded differences), but
// takes no branch where W is flat: where one of the slope's two differences is zero,
// as rounded, and so is another at most two further (plateaus and their ends, pairs
// of equal cells).  (A single pair of equal neighbours in a varying fp32 field is a
// coincidence of rounding, about one in 1e5, and decided like the near-ties.)  Which product is contracted is written out,
// not left to the compiler, whose choice changes with the code around it: in the
// lowest of a face's three differences the lower cell's, in the others the upper's.
template <typename T>
constexpr bool contracted_branches = sizeof(T) == 4;
// The fields (a bit each) whose slope is flat, from the zero differences z: bits
// 5 (k + 3) .. of the difference between cells k and k + 1 of the slope's, k = -3 .. 2
__device__ __forceinline__ unsigned flat_fields(unsigned z) {
  const auto d = [&](int k) { return (z >> (5 * (k + 3))) & 31u; };
  return (d(0) & (d(-2) | d(-1) | d(1) | d(2))) | (d(-1) & (d(-3) | d(-2) | d(0) | d(1)));
}

// Reverse of the one-sided HLLC assembly of the stage kernel, for face states
// wl, wr = (rho, v_n, v_t1, v_t2, P) in the face frame.  Fb = dL/dF; writes
// dL/dwl and dL/dwr.  The forward quantities are recomputed with the stage
// kernel's own arithmetic (c = gP rsq(gP rho), S* through one reciprocal of
// rho_L(S_L - u_L) - rho_R(S_R - u_R)), so the side, fan and wave-speed
// branches are the ones the step took; the derivatives use the same
// reciprocals (dc/dP = g rsq(gP rho) / 2, dc/drho = -c / (2 rho) with
// 1/rho = gP rsq^2) instead of divisions.  Everything that belongs to the side
// K the face fell on (its energy, flux and star state) is reversed once, for
// the selected state, and handed to the left or right adjoint at the end; only
// the speeds and S* have a reverse on both sides.
template <typename T>
__device__ __forceinline__ void hllc_reverse(const T (&wl)[5], const T (&wr)[5], T g, T gm1inv,
                                             const T (&Fb)[5], T (&wlb)[5], T (&wrb)[5]) {
  const T rl = wl[0], ul = wl[1], pl = wl[4];
  const T rr = wr[0], ur = wr[1], pr = wr[4];
  const T gpl = g * pl, gpr = g * pr;
  const T rsl = dev_rsq(gpl * rl), rsr = dev_rsq(gpr * rr);
  const T cl = gpl * rsl, cr = gpr * rsr;
  const bool minL = (ul - cl) <= (ur - cr);
  const bool maxL = (ul + cl) >= (ur + cr);
  const T SL = minL ? ul - cl : ur - cr;
  const T SR = maxL ? ul + cl : ur + cr;
  const T dl = rl * (SL - ul), dr = rr * (SR - ur);
  const T num = fmad(-ur, dr, fmad(ul, dl, pr - pl));
  const T iden = dev_rcp(dl - dr);
  const T ss = num * iden;
  const bool left = (SL >= T(0)) || (ss >= T(0));
  const bool fan = (left ? -SL : SR) > T(0);
  const T rK = left ? rl : rr, uK = left ? ul : ur, pK = left ? pl : pr;
  const T aK = left ? wl[2] : wr[2], bK = left ? wl[3] : wr[3];
  const T SK = left ? SL : SR, dK = left ? dl : dr;
  const T kK = fmad(uK, uK, fmad(aK, aK, bK * bK));
  const T EK = fmad(pK, gm1inv, (T(0.5) * rK) * kK);
  const T mK = rK * uK;

  // F_K = (mK, mK uK + pK, mK aK, mK bK, uK (EK + pK))
  T mKb = fmad(Fb[3], bK, fmad(Fb[2], aK, fmad(Fb[1], uK, Fb[0])));
  T uKb = fmad(Fb[4], EK + pK, Fb[1] * mK);
  T pKb = fmad(Fb[4], uK, Fb[1]);
  T aKb = Fb[2] * mK, bKb = Fb[3] * mK, EKb = Fb[4] * uK;
  T rKb = T(0), SKb = T(0), dKb = T(0), ssb = T(0);
  if (fan) {
    const T q = dev_rcp(SK - ss);
    const T qd = q * dK;
    const T H = fmad(dK, ss, pK);
    const T G4 = fmad(SK - uK, EK, (ss - uK) * H);
    const T s[5] = {qd, qd * ss, qd * aK, qd * bK, q * G4};
    const T UK[5] = {rK, mK, rK * aK, rK * bK, EK};
    T sb[5];
#pragma unroll
    for (int f = 0; f < 5; ++f) {
      SKb = fmad(Fb[f], s[f] - UK[f], SKb);
      sb[f] = SK * Fb[f];  // the adjoint of s; that of UK is its negative
    }
    T qb = sb[4] * G4;
    const T G4b = sb[4] * q;
    SKb = fmad(G4b, EK, SKb);
    uKb = fmad(-G4b, EK + H, uKb);
    EKb = fmad(G4b, SK - uK, EKb) - sb[4];
    const T Hb = G4b * (ss - uK);
    dKb = Hb * ss;
    ssb = fmad(G4b, H, Hb * dK);
    pKb += Hb;
    const T qdb = fmad(sb[3], bK, fmad(sb[2], aK, fmad(sb[1], ss, sb[0])));
    ssb = fmad(sb[1], qd, ssb);
    qb = fmad(qdb, dK, qb);
    dKb = fmad(qdb, q, dKb);
    const T Zb = -(qb * q) * q;  // q = 1/Z, Z = SK - ss
    SKb += Zb;
    ssb -= Zb;
    rKb = -fmad(sb[3], bK, fmad(sb[2], aK, sb[0]));
    mKb -= sb[1];
    aKb = fmad(sb[2], qd - rK, aKb);
    bKb = fmad(sb[3], qd - rK, bKb);
  }
  rKb = fmad(mKb, uK, rKb);
  uKb = fmad(mKb, rK, uKb);
  // EK = pK / (g - 1) + rK kK / 2
  pKb = fmad(EKb, gm1inv, pKb);
  rKb = fmad(EKb * T(0.5), kK, rKb);
  const T Er = EKb * rK;
  uKb = fmad(Er, uK, uKb);
  aKb = fmad(Er, aK, aKb);
  bKb = fmad(Er, bK, bKb);

  // ss = num / den, den = dl - dr, d_K = rho_K (S_K - u_K)
  const T numb = ssb * iden, denb = -(ssb * ss) * iden;
  const T dlb = fmad(numb, ul, left ? dKb : T(0)) + denb;
  const T drb = fmad(-numb, ur, left ? T(0) : dKb) - denb;
  T plb = (left ? pKb : T(0)) - numb, prb = (left ? T(0) : pKb) + numb;
  T ulb = fmad(-dlb, rl, fmad(numb, dl, left ? uKb : T(0)));
  T urb = fmad(-drb, rr, fmad(-numb, dr, left ? T(0) : uKb));
  T rlb = fmad(dlb, SL - ul, left ? rKb : T(0));
  T rrb = fmad(drb, SR - ur, left ? T(0) : rKb);
  const T SLb = fmad(dlb, rl, left ? SKb : T(0));
  const T SRb = fmad(drb, rr, left ? T(0) : SKb);
  const T sll = minL ? SLb : T(0), slr = minL ? T(0) : SLb;
  const T srl = maxL ? SRb : T(0), srr = maxL ? T(0) : SRb;
  ulb += sll + srl;
  urb += slr + srr;
  const T clb = srl - sll, crb = srr - slr;
  // c = sqrt(gP / rho): dc/dP = g rsq / 2, dc/drho = -c / (2 rho), 1/rho = gP rsq^2
  plb = fmad(clb, T(0.5) * g * rsl, plb);
  rlb = fmad(-clb, (T(0.5) * cl) * (gpl * rsl * rsl), rlb);
  prb = fmad(crb, T(0.5) * g * rsr, prb);
  rrb = fmad(-crb, (T(0.5) * cr) * (gpr * rsr * rsr), rrb);
  wlb[0] = rlb; wlb[1] = ulb; wlb[2] = left ? aKb : T(0); wlb[3] = left ? bKb : T(0); wlb[4] = plb;
  wrb[0] = rrb; wrb[1] = urb; wrb[2] = left ? T(0) : aKb; wrb[3] = left ? T(0) : bKb; wrb[4] = prb;
}

// limited slope phi(a, b) of a run-time limiter with its partials on the
// branch taken (0 when ab <= 0)
template <typename T>
__device__ __forceinline__ T slope_partials(int lim, T a, T b, T& pa, T& pb) {
  pa = T(0);
  pb = T(0);
  if (lim == LIM_NONE || !(a * b > T(0))) return T(0);
  const T aa = fabs(a), ab = fabs(b);
  T m;
  if (lim == LIM_MINMOD) {
    if (aa <= ab) { pa = T(1); return a; }
    pb = T(1);
    return b;
  }
  if (lim == LIM_VANLEER) {
    const T s = a + b;
    const T is2 = T(1) / (s * s);
    pa = T(2) * b * b * is2;
    pb = T(2) * a * a * is2;
    return T(2) * a * b / s;
  }
  if (lim == LIM_MC) {
    const T cen = fabs(T(0.5) * (a + b)), t2 = fmin(T(2) * aa, T(2) * ab);
    if (cen <= t2) { pa = T(0.5); pb = T(0.5); m = cen; }
    else if (aa <= ab) { pa = T(2); m = T(2) * aa; }
    else { pb = T(2); m = T(2) * ab; }
  } else {  // superbee
    const T s1 = fmin(T(2) * aa, ab), s2 = fmin(aa, T(2) * ab);
    if (s1 >= s2) {
      if (T(2) * aa <= ab) pa = T(2); else pb = T(1);
      m = s1;
    } else {
      if (aa <= T(2) * ab) pa = T(1); else pb = T(2);
      m = s2;
    }
  }
  return a > T(0) ? m : -m;
}

// conserved state and flux of a face-frame primitive state (rho, v_n, v_t1,
// v_t2, P), and the reverse: wb += (dU/dw)^T Ub + (dF/dw)^T Fb
template <typename T>
__device__ __forceinline__ void frame_state_flux(const T (&w)[5], T gm1, T (&U)[5], T (&F)[5]) {
  const T r = w[0], u = w[1], a = w[2], b = w[3], p = w[4];
  const T E = p / gm1 + T(0.5) * r * (u * u + a * a + b * b);
  U[0] = r; U[1] = r * u; U[2] = r * a; U[3] = r * b; U[4] = E;
  F[0] = r * u; F[1] = r * u * u + p; F[2] = r * u * a; F[3] = r * u * b; F[4] = u * (E + p);
}
template <typename T>
__device__ __forceinline__ void frame_state_flux_reverse(const T (&w)[5], T gm1, const T (&Ub)[5],
                                                         const T (&Fb)[5], T (&wb)[5]) {
  const T r = w[0], u = w[1], a = w[2], b = w[3], p = w[4];
  const T q2 = u * u + a * a + b * b;
  const T E = p / gm1 + T(0.5) * r * q2;
  const T Eb = Ub[4] + Fb[4] * u;  // E enters U[4] and F[4]
  wb[0] += Ub[0] + Ub[1] * u + Ub[2] * a + Ub[3] * b +
           u * (Fb[0] + Fb[1] * u + Fb[2] * a + Fb[3] * b) + Eb * T(0.5) * q2;
  wb[1] += r * (Ub[1] + Fb[0] + T(2) * Fb[1] * u + Fb[2] * a + Fb[3] * b + Eb * u) +
           Fb[4] * (E + p);
  wb[2] += r * (Ub[2] + Fb[2] * u + Eb * a);
  wb[3] += r * (Ub[3] + Fb[3] * u + Eb * b);
  wb[4] += Fb[1] + Fb[4] * u + Eb / gm1;
}
// c = sqrt(g P / rho): wb += cb dc/dw
template <typename T>
__device__ __forceinline__ void sound_reverse(const T (&w)[5], T g, T c, T cb, T (&wb)[5]) {
  wb[4] += cb * g / (T(2) * c * w[0]);
  wb[0] -= cb * c / (T(2) * w[0]);
}

// Reverse of the HLL flux (F_L for 0 <= S_L, F_R for S_R <= 0, else the HLL
// average); Davis min/max take the left argument on ties.  Writes wlb, wrb.
template <typename T>
__device__ void hll_reverse(const T (&wl)[5], const T (&wr)[5], T g, const T (&Fb)[5],
                            T (&wlb)[5], T (&wrb)[5]) {
  const T gm1 = g - T(1);
  T UL[5], FL[5], UR[5], FR[5];
  frame_state_flux(wl, gm1, UL, FL);
  frame_state_flux(wr, gm1, UR, FR);
  const T cl = sqrt(g * wl[4] / wl[0]), cr = sqrt(g * wr[4] / wr[0]);
  const bool minL = (wl[1] - cl) <= (wr[1] - cr);
  const bool maxL = (wl[1] + cl) >= (wr[1] + cr);
  const T SL = minL ? wl[1] - cl : wr[1] - cr;
  const T SR = maxL ? wl[1] + cl : wr[1] + cr;
  T ULb[5], FLb[5], URb[5], FRb[5];
  T SLb = T(0), SRb = T(0);
  const bool lo = T(0) <= SL, hi = !lo && SR <= T(0);
  const T iD = T(1) / (SR - SL);
#pragma unroll
  for (int f = 0; f < 5; ++f) {
    wlb[f] = T(0);
    wrb[f] = T(0);
    if (lo || hi) {
      FLb[f] = lo ? Fb[f] : T(0);
      FRb[f] = hi ? Fb[f] : T(0);
      ULb[f] = URb[f] = T(0);
    } else {
      const T dU = UR[f] - UL[f];
      const T Fm = (SR * FL[f] - SL * FR[f] + SL * SR * dU) * iD;
      FLb[f] = Fb[f] * SR * iD;
      FRb[f] = -Fb[f] * SL * iD;
      URb[f] = Fb[f] * SL * SR * iD;
      ULb[f] = -URb[f];
      SLb += Fb[f] * (SR * dU - FR[f] + Fm) * iD;
      SRb += Fb[f] * (FL[f] + SL * dU - Fm) * iD;
    }
  }
  T clb = T(0), crb = T(0);
  if (minL) { wlb[1] += SLb; clb -= SLb; } else { wrb[1] += SLb; crb -= SLb; }
  if (maxL) { wlb[1] += SRb; clb += SRb; } else { wrb[1] += SRb; crb += SRb; }
  sound_reverse(wl, g, cl, clb, wlb);
  sound_reverse(wr, g, cr, crb, wrb);
  frame_state_flux_reverse(wl, gm1, ULb, FLb, wlb);
  frame_state_flux_reverse(wr, gm1, URb, FRb, wrb);
}

// Reverse of the Rusanov flux (F_L + F_R)/2 - s (U_R - U_L)/2, s = max(|v_L|
// + c_L, |v_R| + c_R): the left argument on ties, d|v|/dv = -1 for v < 0,
// else +1.  Writes wlb, wrb.
template <typename T>
__device__ void rusanov_reverse(const T (&wl)[5], const T (&wr)[5], T g, const T (&Fb)[5],
                                T (&wlb)[5], T (&wrb)[5]) {
  const T gm1 = g - T(1);
  T UL[5], FL[5], UR[5], FR[5];
  frame_state_flux(wl, gm1, UL, FL);
  frame_state_flux(wr, gm1, UR, FR);
  const T cl = sqrt(g * wl[4] / wl[0]), cr = sqrt(g * wr[4] / wr[0]);
  const bool maxL = (fabs(wl[1]) + cl) >= (fabs(wr[1]) + cr);
  const T s = maxL ? fabs(wl[1]) + cl : fabs(wr[1]) + cr;
  T ULb[5], FLb[5], URb[5], FRb[5];
  T sb = T(0);
#pragma unroll
  for (int f = 0; f < 5; ++f) {
    wlb[f] = T(0);
    wrb[f] = T(0);
    FLb[f] = FRb[f] = T(0.5) * Fb[f];
    URb[f] = -T(0.5) * s * Fb[f];
    ULb[f] = -URb[f];
    sb -= T(0.5) * Fb[f] * (UR[f] - UL[f]);
  }
  T clb = T(0), crb = T(0);
  if (maxL) {
    wlb[1] += wl[1] < T(0) ? -sb : sb;
    clb = sb;
  } else {
    wrb[1] += wr[1] < T(0) ? -sb : sb;
    crb = sb;
  }
  sound_reverse(wl, g, cl, clb, wlb);
  sound_reverse(wr, g, cr, crb, wrb);
  frame_state_flux_reverse(wl, gm1, ULb, FLb, wlb);
  frame_state_flux_reverse(wr, gm1, URb, FRb, wrb);
}

struct AxisGeom {
  int n[3];   // cells along x, y, z
  int bc;     // boundary kind of the axis
  int nf;     // faces along the axis: n (periodic) or n + 1 (outflow)
};

// cell index of (along-axis coordinate c, the other two coordinates) and the
// face record index of (face f along the axis, the other two coordinates)
template <int AX>
__device__ __forceinline__ long long cell_of(const AxisGeom& g, int c, int o1, int o2) {
  if (AX == 0) return ((long long)o2 * g.n[1] + o1) * g.n[0] + c;
  if (AX == 1) return ((long long)o2 * g.n[1] + c) * g.n[0] + o1;
  return ((long long)c * g.n[1] + o2) * g.n[0] + o1;
}
template <int AX>
__device__ __forceinline__ long long face_of(const AxisGeom& g, int f, int o1, int o2) {
  if (AX == 0) return ((long long)o2 * g.n[1] + o1) * g.nf + f;
  if (AX == 1) return ((long long)o2 * g.nf + f) * g.n[0] + o1;
  return ((long long)f * g.n[1] + o2) * g.n[0] + o1;
}
// the inverses: thread t takes face record t and cell t, so that consecutive
// lanes touch consecutive addresses (x fastest) along every axis
template <int AX>
__device__ __forceinline__ void face_coords(const AxisGeom& g, long long t, int& f, int& o1,
                                            int& o2) {
  if (AX == 0) {
    f = (int)(t % g.nf);
    const long long r = t / g.nf;
    o1 = (int)(r % g.n[1]);
    o2 = (int)(r / g.n[1]);
  } else if (AX == 1) {
    o1 = (int)(t % g.n[0]);
    const long long r = t / g.n[0];
    f = (int)(r % g.nf);
    o2 = (int)(r / g.nf);
  } else {
    o1 = (int)(t % g.n[0]);
    const long long r = t / g.n[0];
    o2 = (int)(r % g.n[1]);
    f = (int)(r / g.n[1]);
  }
}
template <int AX>
__device__ __forceinline__ void cell_coords(const AxisGeom& g, long long t, int& c, int& o1,
                                            int& o2) {
  if (AX == 0) {
    c = (int)(t % g.n[0]);
    const long long r = t / g.n[0];
    o1 = (int)(r % g.n[1]);
    o2 = (int)(r / g.n[1]);
  } else if (AX == 1) {
    o1 = (int)(t % g.n[0]);
    const long long r = t / g.n[0];
    c = (int)(r % g.n[1]);
    o2 = (int)(r / g.n[1]);
  } else {
    o1 = (int)(t % g.n[0]);
    const long long r = t / g.n[0];
    o2 = (int)(r % g.n[1]);
    c = (int)(r / g.n[1]);
  }
}
// the two other coordinates of axis AX: AX=0 -> (y, z), AX=1 -> (x, z), AX=2 -> (x, y)
template <int AX>
__device__ __forceinline__ void other_dims(const AxisGeom& g, int& d1, int& d2) {
  d1 = AX == 0 ? g.n[1] : g.n[0];
  d2 = AX == 2 ? g.n[1] : g.n[2];
}

// W of a face's four stencil cells i - 1 .. i + 2 in the face frame, and the three
// differences between them
template <typename T>
struct FaceStencil {
  T w[4][5], dm[5], dc[5], dp[5];
};
template <typename T, int AX>
__device__ __forceinline__ void face_stencil(const T* __restrict__ U, long long N,
                                             const AxisGeom& g, int i, int o1, int o2, T gm1,
                                             const int (&perm)[5], FaceStencil<T>& st) {
  T x[4][5], y[4][5];
#pragma unroll
  for (int k = 0; k < 4; ++k) {
    T xc[5], yc[5];
    prim_factors_at(U, N, cell_of<AX>(g, bc_map(i - 1 + k, g.n[AX], g.bc), o1, o2), gm1, xc, yc);
#pragma unroll
    for (int s = 0; s < 5; ++s) {
      x[k][s] = xc[perm[s]];
      y[k][s] = yc[perm[s]];
      st.w[k][s] = x[k][s] * y[k][s];
    }
  }
#pragma unroll
  for (int s = 0; s < 5; ++s) {
    if constexpr (contracted_branches<T>) {
      st.dm[s] = fmad(-x[0][s], y[0][s], st.w[1][s]);
      st.dc[s] = fmad(x[2][s], y[2][s], -st.w[1][s]);
      st.dp[s] = fmad(x[3][s], y[3][s], -st.w[2][s]);
    } else {
      st.dm[s] = plain_diff(st.w[1][s], st.w[0][s]);
      st.dc[s] = plain_diff(st.w[2][s], st.w[1][s]);
      st.dp[s] = plain_diff(st.w[3][s], st.w[2][s]);
    }
  }
}

// whether any two neighbours of the stencil are equal in any field, without which no
// slope is flat
template <typename T>
__device__ __forceinline__ bool any_equal(const T (&w)[4][5]) {
  bool e = false;
#pragma unroll
  for (int s = 0; s < 5; ++s)
    e = e || w[0][s] == w[1][s] || w[1][s] == w[2][s] || w[2][s] == w[3][s];
  return e;
}
// the face-frame fields whose slope in cell i (flat[0]) or i + 1 (flat[1]) is flat
// (flat_fields), cell i the left one of the face
template <typename T, int AX>
__device__ __forceinline__ void flat_slopes(const T* __restrict__ U, long long N, const AxisGeom& g,
                                            int i, int o1, int o2, T gm1, const int (&perm)[5],
                                            unsigned (&flat)[2]) {
  unsigned long long z = 0;
  T below[5] = {};
#pragma unroll 1
  for (int k = -3; k <= 4; ++k) {
    T t[5];
    prim_at(U, N, cell_of<AX>(g, bc_map(i + k, g.n[AX], g.bc), o1, o2), gm1, t);
    unsigned m = 0;
#pragma unroll
    for (int s = 0; s < 5; ++s) {
      m |= (t[perm[s]] == below[s] ? 1u : 0u) << s;
      below[s] = t[perm[s]];
    }
    if (k > -3) z |= (unsigned long long)m << (5 * (k + 2));
  }
  flat[0] = flat_fields((unsigned)z & 0x3fffffffu);
  flat[1] = flat_fields((unsigned)(z >> 5));
}

template <typename T, int LIM, int AX>
__global__ __launch_bounds__(256) void k_face_vjp(const T* __restrict__ U, const T* __restrict__ v,
                                                  AxisGeom g, T gamma, T ih, T* __restrict__ wbar,
                                                  int* __restrict__ flags, long long nfaces) {
  const long long t = (long long)blockIdx.x * 256 + threadIdx.x;
  if (t >= nfaces) return;
  int d1, d2;
  other_dims<AX>(g, d1, d2);
  int f, o1, o2;
  face_coords<AX>(g, t, f, o1, o2);
  const int n = g.n[AX];
  const int i = g.bc == BC_PERIODIC ? f : f - 1;  // left cell position of the face
  const long long N = (long long)g.n[0] * g.n[1] * g.n[2];
  const T gm1 = gamma - T(1);
  const T gm1inv = T(1) / gm1;
  constexpr int vn = 1 + AX, t1 = 1 + (AX + 1) % 3, t2 = 1 + (AX + 2) % 3;
  const int perm[5] = {0, vn, t1, t2, 4};
  FaceStencil<T> st;
  face_stencil<T, AX>(U, N, g, i, o1, o2, gm1, perm, st);
  const T(&w)[4][5] = st.w;
  T wl[5], wr[5];
  int fl = 0;
#pragma unroll
  for (int s = 0; s < 5; ++s) {
    const T a0 = st.dc[s], b0 = st.dm[s], a1 = st.dp[s], b1 = st.dc[s];
    const int s0 = LIM == LIM_NONE ? 0 : minmod_sel(a0, b0);
    const int s1 = LIM == LIM_NONE ? 0 : minmod_sel(a1, b1);
    wl[s] = w[1][s] + T(0.5) * sel_value(s0, a0, b0);
    wr[s] = w[2][s] - T(0.5) * sel_value(s1, a1, b1);
    fl |= (s0 << (2 * s)) | (s1 << (10 + 2 * s));
  }
  if (contracted_branches<T> && LIM != LIM_NONE && any_equal(w)) {
    unsigned flat[2];
    flat_slopes<T, AX>(U, N, g, i, o1, o2, gm1, perm, flat);
#pragma unroll
    for (int s = 0; s < 5; ++s) {
      const bool f0 = (flat[0] >> s) & 1u, f1 = (flat[1] >> s) & 1u;
      if (f0) wl[s] = w[1][s];
      if (f1) wr[s] = w[2][s];
      fl &= ~((f0 ? 3 << (2 * s) : 0) | (f1 ? 3 << (10 + 2 * s) : 0));
    }
  }
  // Fb = (v of the face's right cell - v of its left cell) / h, real cells only
  const bool has_right = g.bc == BC_PERIODIC || i + 1 <= n - 1;
  const bool has_left = g.bc == BC_PERIODIC || i >= 0;
  const long long qr = cell_of<AX>(g, bc_map(i + 1, n, g.bc), o1, o2);
  const long long ql = cell_of<AX>(g, bc_map(i, n, g.bc), o1, o2);
  T Fb[5];
#pragma unroll
  for (int s = 0; s < 5; ++s) {
    const T vr = has_right ? v[perm[s] * N + qr] : T(0);
    const T vl = has_left ? v[perm[s] * N + ql] : T(0);
    Fb[s] = (vr - vl) * ih;
  }
  T wlb[5], wrb[5];
  hllc_reverse<T>(wl, wr, gamma, gm1inv, Fb, wlb, wrb);
  const long long rec = face_of<AX>(g, f, o1, o2);
  const long long NF = (long long)g.nf * d1 * d2;
#pragma unroll
  for (int s = 0; s < 5; ++s) {
    wbar[s * NF + rec] = wlb[s];
    wbar[(5 + s) * NF + rec] = wrb[s];
  }
  flags[rec] = fl;
}

// The same for a run-time limiter `lim` and solver `rs`: writes the face's
// contributions to the W adjoint of its four stencil cells i-1+k (k = 0..3),
// per face-frame field s, to slots[(5 k + s) NF + rec]:
//   k = 0: -pb0 WLb/2
//   k = 1: WLb (1 + (pb0 - pa0)/2) + pb1 WRb/2
//   k = 2: pa0 WLb/2 + WRb (1 - (pb1 - pa1)/2)
//   k = 3: -pa1 WRb/2
// from W^L = W_i + phi(a0, b0)/2, W^R = W_{i+1} - phi(a1, b1)/2.
template <typename T, int AX>
__global__ __launch_bounds__(256) void k_face_vjp_rt(const T* __restrict__ U,
                                                     const T* __restrict__ v, AxisGeom g, T gamma,
                                                     T ih, int lim, int rs,
                                                     T* __restrict__ slots, long long nfaces) {
  const long long t = (long long)blockIdx.x * 256 + threadIdx.x;
  if (t >= nfaces) return;
  int d1, d2;
  other_dims<AX>(g, d1, d2);
  int f, o1, o2;
  face_coords<AX>(g, t, f, o1, o2);
  const int n = g.n[AX];
  const int i = g.bc == BC_PERIODIC ? f : f - 1;
  const long long N = (long long)g.n[0] * g.n[1] * g.n[2];
  const T gm1 = gamma - T(1);
  const T gm1inv = T(1) / gm1;
  constexpr int vn = 1 + AX, t1 = 1 + (AX + 1) % 3, t2 = 1 + (AX + 2) % 3;
  const int perm[5] = {0, vn, t1, t2, 4};
  FaceStencil<T> st;
  face_stencil<T, AX>(U, N, g, i, o1, o2, gm1, perm, st);
  const T(&w)[4][5] = st.w;
  T wl[5], wr[5], pa0[5], pb0[5], pa1[5], pb1[5];
#pragma unroll
  for (int s = 0; s < 5; ++s) {
    const T d0 = slope_partials(lim, st.dc[s], st.dm[s], pa0[s], pb0[s]);
    const T d1 = slope_partials(lim, st.dp[s], st.dc[s], pa1[s], pb1[s]);
    wl[s] = w[1][s] + T(0.5) * d0;
    wr[s] = w[2][s] - T(0.5) * d1;
  }
  if (contracted_branches<T> && lim != LIM_NONE && any_equal(w)) {
    unsigned flat[2];
    flat_slopes<T, AX>(U, N, g, i, o1, o2, gm1, perm, flat);
#pragma unroll
    for (int s = 0; s < 5; ++s) {
      if ((flat[0] >> s) & 1u) {
        wl[s] = w[1][s];
        pa0[s] = pb0[s] = T(0);
      }
      if ((flat[1] >> s) & 1u) {
        wr[s] = w[2][s];
        pa1[s] = pb1[s] = T(0);
      }
    }
  }
  const bool has_right = g.bc == BC_PERIODIC || i + 1 <= n - 1;
  const bool has_left = g.bc == BC_PERIODIC || i >= 0;
  const long long qr = cell_of<AX>(g, bc_map(i + 1, n, g.bc), o1, o2);
  const long long ql = cell_of<AX>(g, bc_map(i, n, g.bc), o1, o2);
  T Fb[5];
#pragma unroll
  for (int s = 0; s < 5; ++s) {
    const T vr = has_right ? v[perm[s] * N + qr] : T(0);
    const T vl = has_left ? v[perm[s] * N + ql] : T(0);
    Fb[s] = (vr - vl) * ih;
  }
  T wlb[5], wrb[5];
  if (rs == RS_HLL) hll_reverse<T>(wl, wr, gamma, Fb, wlb, wrb);
  else if (rs == RS_RUSANOV) rusanov_reverse<T>(wl, wr, gamma, Fb, wlb, wrb);
  else hllc_reverse<T>(wl, wr, gamma, gm1inv, Fb, wlb, wrb);
  const long long rec = face_of<AX>(g, f, o1, o2);
  const long long NF = (long long)g.nf * d1 * d2;
#pragma unroll
  for (int s = 0; s < 5; ++s) {
    const T L = wlb[s], R = wrb[s];
    slots[(0 + s) * NF + rec] = -T(0.5) * pb0[s] * L;
    slots[(5 + s) * NF + rec] = L + T(0.5) * (pb0[s] - pa0[s]) * L + T(0.5) * pb1[s] * R;
    slots[(10 + s) * NF + rec] = T(0.5) * pa0[s] * L + R - T(0.5) * (pb1[s] - pa1[s]) * R;
    slots[(15 + s) * NF + rec] = -T(0.5) * pa1[s] * R;
  }
}

// contribution of the face with left cell position i to the stencil slot k
// (position i - 1 + k), field s (face frame), from the reverse of
// W^L = W_i + minmod_i/2 and W^R = W_{i+1} - minmod_{i+1}/2
template <typename T>
__device__ __forceinline__ T slot_contrib(int k, int fl, int s, T WLb, T WRb) {
  // selection codes of the two slopes (1: forward difference, 2: backward,
  // 0: none); every term is a signed half of WLb or WRb or zero, so selects
  // give the same sums as multiplying by the 0/1 indicators
  const int s0 = (fl >> (2 * s)) & 3, s1 = (fl >> (10 + 2 * s)) & 3;
  const T hl = T(0.5) * WLb, hr = T(0.5) * WRb;
  switch (k) {
    case 0: return s0 == 2 ? -hl : T(0);
    case 1: return (WLb + (s0 == 2 ? hl : (s0 == 1 ? -hl : T(0)))) + (s1 == 2 ? hr : T(0));
    case 2: return ((s0 == 1 ? hl : T(0)) + WRb) + (s1 == 2 ? -hr : (s1 == 1 ? hr : T(0)));
    default: return s1 == 1 ? -hr : T(0);
  }
}

// out = c0 x0 + c1 x1 + c2 x2 + beta (dW/dU)^T w at cell q, W = (rho, v, P)
// of U (the last step of J(U)^T v)
template <typename T>
struct FinishArgs {
  T gm1, beta, c0, c1, c2;
  const T *x0, *x1, *x2;
  T* out;
  int xv;  // the x that is the v of J^T v itself (0, 1, 2), or -1
};
// the same from W and v of the cell in registers
template <typename T>
__device__ __forceinline__ void finish_prim(const T (&prim)[5], const T (&vc)[5], const T (&w)[5],
                                            long long q, long long N, const FinishArgs<T>& fa) {
  const T ir = dev_rcp(prim[0]);
  const T vx = prim[1], vy = prim[2], vz = prim[3];
  const T wr = w[0], wx = w[1], wy = w[2], wz = w[3], wp = w[4];
  const T gm1 = fa.gm1;
  T o[5];
  o[0] = wr - (wx * vx + wy * vy + wz * vz) * ir + wp * gm1 * T(0.5) * (vx * vx + vy * vy + vz * vz);
  o[1] = wx * ir - wp * gm1 * vx;
  o[2] = wy * ir - wp * gm1 * vy;
  o[3] = wz * ir - wp * gm1 * vz;
  o[4] = wp * gm1;
#pragma unroll
  for (int f = 0; f < 5; ++f) o[f] *= fa.beta;
  if (fa.x0) {
#pragma unroll
    for (int f = 0; f < 5; ++f) o[f] += fa.c0 * (fa.xv == 0 ? vc[f] : fa.x0[f * N + q]);
  }
  if (fa.x1) {
#pragma unroll
    for (int f = 0; f < 5; ++f) o[f] += fa.c1 * (fa.xv == 1 ? vc[f] : fa.x1[f * N + q]);
  }
  if (fa.x2) {
#pragma unroll
    for (int f = 0; f < 5; ++f) o[f] += fa.c2 * (fa.xv == 2 ? vc[f] : fa.x2[f * N + q]);
  }
#pragma unroll
  for (int f = 0; f < 5; ++f) fa.out[f * N + q] = o[f];
}
template <typename T>
__device__ __forceinline__ void finish_cell(const T* __restrict__ U, const T (&w)[5], long long q,
                                            long long N, const FinishArgs<T>& fa) {
  const T rho = U[q];
  const T ir = dev_rcp(rho);
  const T vx = U[N + q] * ir, vy = U[2 * N + q] * ir, vz = U[3 * N + q] * ir;
  const T wr = w[0], wx = w[1], wy = w[2], wz = w[3], wp = w[4];
  const T gm1 = fa.gm1;
  T g[5];
  g[0] = wr - (wx * vx + wy * vy + wz * vz) * ir + wp * gm1 * T(0.5) * (vx * vx + vy * vy + vz * vz);
  g[1] = wx * ir - wp * gm1 * vx;
  g[2] = wy * ir - wp * gm1 * vy;
  g[3] = wz * ir - wp * gm1 * vz;
  g[4] = wp * gm1;
#pragma unroll
  for (int f = 0; f < 5; ++f) {
    T o = fa.beta * g[f];
    if (fa.x0) o += fa.c0 * fa.x0[f * N + q];
    if (fa.x1) o += fa.c1 * fa.x1[f * N + q];
    if (fa.x2) o += fa.c2 * fa.x2[f * N + q];
    fa.out[f * N + q] = o;
  }
}

// what a gather does with its sum: add it to Wacc, store it to Wacc (the
// first axis), or add Wacc and finish the cell (the last axis; FIRST_LAST when
// it is the only one)
enum : int { GATHER_ADD = 0, GATHER_FIRST = 1, GATHER_LAST = 2, GATHER_FIRST_LAST = 3 };

// SLOTS: the face records are the four stencil contributions written by
// k_face_vjp_rt; otherwise (W^L_b, W^R_b) and the minmod selections
template <typename T, int AX, bool SLOTS, int MODE>
__global__ __launch_bounds__(256) void k_cell_gather(const T* __restrict__ wbar,
                                                     const int* __restrict__ flags, AxisGeom g,
                                                     T* __restrict__ Wacc,
                                                     const T* __restrict__ U, FinishArgs<T> fa) {
  const long long N = (long long)g.n[0] * g.n[1] * g.n[2];
  const long long t = (long long)blockIdx.x * 256 + threadIdx.x;
  if (t >= N) return;
  int d1, d2;
  other_dims<AX>(g, d1, d2);
  const int n = g.n[AX];
  int c, o1, o2;
  cell_coords<AX>(g, t, c, o1, o2);
  const long long NF = (long long)g.nf * d1 * d2;
  constexpr int vn = 1 + AX, t1 = 1 + (AX + 1) % 3, t2 = 1 + (AX + 2) % 3;
  const int perm[5] = {0, vn, t1, t2, 4};
  T acc[5] = {T(0), T(0), T(0), T(0), T(0)};
  auto add_face = [&](int f, int i) {  // record f, left cell position i
    const long long rec = face_of<AX>(g, f, o1, o2);
    const int fl = SLOTS ? 0 : flags[rec];
    for (int k = 0; k < 4; ++k) {
      if (bc_map(i - 1 + k, n, g.bc) != c) continue;
#pragma unroll
      for (int s = 0; s < 5; ++s)
        acc[s] += SLOTS ? wbar[(5 * k + s) * NF + rec]
                        : slot_contrib<T>(k, fl, s, wbar[s * NF + rec], wbar[(5 + s) * NF + rec]);
    }
  };
  if (g.bc == BC_PERIODIC && n >= 4) {
    // face c - 2 + m (wrapped) holds this cell in stencil slot k = 3 - m, so
    // every record is loaded before any sum (the slot known at compile time);
    // slot 3 reads only W^R_b, slot 0 only W^L_b; sums in face order
    long long rec[4];
#pragma unroll
    for (int m = 0; m < 4; ++m) {
      const int i = c - 2 + m;
      rec[m] = face_of<AX>(g, i < 0 ? i + n : (i >= n ? i - n : i), o1, o2);
    }
    int fl[4];
    T wl[4][5], wr[4][5];
#pragma unroll
    for (int m = 0; m < 4; ++m) {
      fl[m] = SLOTS ? 0 : flags[rec[m]];
#pragma unroll
      for (int s = 0; s < 5; ++s) {
        if (SLOTS) {
          wl[m][s] = wbar[(5 * (3 - m) + s) * NF + rec[m]];
          wr[m][s] = T(0);
        } else {
          wl[m][s] = m >= 1 ? wbar[s * NF + rec[m]] : T(0);
          wr[m][s] = m <= 2 ? wbar[(5 + s) * NF + rec[m]] : T(0);
        }
      }
    }
#pragma unroll
    for (int m = 0; m < 4; ++m)
#pragma unroll
      for (int s = 0; s < 5; ++s)
        acc[s] += SLOTS ? wl[m][s] : slot_contrib<T>(3 - m, fl[m], s, wl[m][s], wr[m][s]);
  } else if (g.bc == BC_PERIODIC) {
    for (int f = 0; f < n; ++f) add_face(f, f);
  } else {
    for (int i = max(-1, c - 2); i <= min(n - 1, c + 1); ++i) add_face(i + 1, i);
  }
  const long long q = cell_of<AX>(g, c, o1, o2);
  if (MODE == GATHER_ADD) {
#pragma unroll
    for (int s = 0; s < 5; ++s) Wacc[perm[s] * N + q] += acc[s];
  } else if (MODE == GATHER_FIRST) {
#pragma unroll
    for (int s = 0; s < 5; ++s) Wacc[perm[s] * N + q] = acc[s];
  } else {
    T w[5];
#pragma unroll
    for (int s = 0; s < 5; ++s)
      w[perm[s]] = MODE == GATHER_LAST ? Wacc[perm[s] * N + q] + acc[s] : acc[s];
    finish_cell(U, w, q, N, fa);
  }
}

// Minmod as a value and the branch it took: fwd (the forward difference a) or
// bwd (the backward difference b), neither where they disagree in sign -- the
// selections of minmod_sel.
template <typename T, int LIM>
__device__ __forceinline__ T slope_branch(T a, T b, bool& fwd, bool& bwd) {
  if (LIM == LIM_NONE) {
    fwd = bwd = false;
    return T(0);
  }
  const bool same = !(a * b <= T(0)), le = fabs(a) <= fabs(b);
  fwd = same && le;
  bwd = same && !le;
  return fwd ? a : (bwd ? b : T(0));
}

// The fused kernels reverse the slopes per cell, not per face.  With WLb of
// the face above cell c and WRb of the face below it (W^L = W_c + dW_c/2,
// W^R = W_c - dW_c/2), the slope's adjoint is dWb = (WLb - WRb)/2 and the
// cell's own term WLb + WRb; a forward branch (dW_c = W_{c+1} - W_c) adds
// dWb to cell c + 1 and takes it from c, a backward one adds it to c and takes
// it from c - 1.  Five sums and two selects per field and face, where the four
// stencil contributions of a face (slot_contrib) took about thirty.

// J(U)^T v along axis AX = 1 or 2 for periodic boundaries (n >= 4) and the
// minmod (or first-order) HLLC scheme, face reverse and gather fused: one
// thread per (x, other) column and segment of `seg` cells along the axis
// marches the faces c0 - 2 .. c1 in order, with W of the face's cells and the
// next one, the slope of the lower cell, and the open sums of two cells in
// registers.  After face f, cell f - 1 is complete: stored, added to or
// finished (with W and v from registers) as in k_cell_gather's MODE.  The next
// cell's U and v are loaded one face ahead.  Lanes take consecutive x, so
// every load and store of a wave is contiguous.
template <typename T, int LIM, int AX, int MODE>
__global__ __launch_bounds__(256) void k_axis_jtv(const T* __restrict__ U, const T* __restrict__ v,
                                                  AxisGeom g, T gamma, T ih, int seg,
                                                  T* __restrict__ Wacc, FinishArgs<T> fa) {
  static_assert(AX == 1 || AX == 2, "columns along y or z");
  constexpr bool FIN = MODE == GATHER_LAST || MODE == GATHER_FIRST_LAST;
  int d1, d2;
  other_dims<AX>(g, d1, d2);
  const int n = g.n[AX];
  const int nseg = (n + seg - 1) / seg;
  const long long t = (long long)blockIdx.x * 256 + threadIdx.x;
  if (t >= (long long)d1 * d2 * nseg) return;
  const int o1 = (int)(t % d1);
  const long long r = t / d1;
  const int o2 = (int)(r % d2), sg = (int)(r / d2);
  const int c0 = sg * seg, c1 = min(c0 + seg, n);
  const long long N = (long long)g.n[0] * g.n[1] * g.n[2];
  const long long stride = AX == 1 ? (long long)g.n[0] : (long long)g.n[0] * g.n[1];
  const long long base = cell_of<AX>(g, 0, o1, o2);
  const T gm1 = gamma - T(1);
  const T gm1inv = T(1) / gm1;
  constexpr int vn = 1 + AX, t1 = 1 + (AX + 1) % 3, t2 = 1 + (AX + 2) % 3;
  const int perm[5] = {0, vn, t1, t2, 4};
  auto wrapc = [&](int c) { return c < 0 ? c + n : (c >= n ? c - n : c); };
  // fields in the face frame, (rho, v_n, v_t1, v_t2, P or E)
  auto load_raw = [&](const T* __restrict__ src, int c, T (&out)[5]) {
    const T* s = src + base + wrapc(c) * stride;
#pragma unroll
    for (int k = 0; k < 5; ++k) out[k] = s[perm[k] * N];
  };
  auto prim = [&](const T (&u)[5], T (&w)[5]) {  // to_prim in the face frame
    T ug[5], wg[5];
#pragma unroll
    for (int k = 0; k < 5; ++k) ug[perm[k]] = u[k];
    to_prim(ug, gm1, wg);
#pragma unroll
    for (int k = 0; k < 5; ++k) w[k] = wg[perm[k]];
  };
  // W of cells f - 1 (finish only), f, f + 1, f + 2; v of f - 1, f, f + 1;
  // the slope of cell f with its branch
  T wm[5], w0[5], w1[5], w2[5], vm[5], v0[5], v1[5], dw[5], un[5], vnx[5];
  bool fwd[5], bwd[5];
  {
    T tmp[5];
    load_raw(U, c0 - 3, tmp);
    prim(tmp, wm);
    load_raw(U, c0 - 2, tmp);
    prim(tmp, w0);
    load_raw(U, c0 - 1, tmp);
    prim(tmp, w1);
    load_raw(U, c0, un);
    load_raw(v, c0 - 2, v0);
    load_raw(v, c0 - 1, vnx);
#pragma unroll
    for (int k = 0; k < 5; ++k) {
      dw[k] = slope_branch<T, LIM>(plain_diff(w1[k], w0[k]), plain_diff(w0[k], wm[k]), fwd[k],
                                   bwd[k]);
      vm[k] = T(0);
    }
  }
  // WRb of the face below cell f, the open sum of cell f - 1, and what cell
  // f - 1's forward branch adds to cell f
  T wrp[5], open[5], e1p[5];
#pragma unroll
  for (int k = 0; k < 5; ++k) wrp[k] = open[k] = e1p[k] = T(0);
  for (int f = c0 - 2; f <= c1; ++f) {
    prim(un, w2);
#pragma unroll
    for (int k = 0; k < 5; ++k) v1[k] = vnx[k];
    if (f < c1) {
      load_raw(U, f + 3, un);
      load_raw(v, f + 2, vnx);
    }
    T acc[5];
    const bool emit = f - 1 >= c0;
    const long long q = base + (long long)(f - 1) * stride;
    if (emit && (MODE == GATHER_ADD || MODE == GATHER_LAST)) {
#pragma unroll
      for (int k = 0; k < 5; ++k) acc[k] = Wacc[perm[k] * N + q];
    } else {
#pragma unroll
      for (int k = 0; k < 5; ++k) acc[k] = T(0);
    }
    T wl[5], wr[5], dn[5], Fb[5], wlb[5], wrb[5];
    bool fwn[5], bwn[5];
#pragma unroll
    for (int k = 0; k < 5; ++k) {
      dn[k] = slope_branch<T, LIM>(plain_diff(w2[k], w1[k]), plain_diff(w1[k], w0[k]), fwn[k],
                                   bwn[k]);
      wl[k] = fmad(T(0.5), dw[k], w0[k]);
      wr[k] = fmad(T(-0.5), dn[k], w1[k]);
      Fb[k] = (v1[k] - v0[k]) * ih;
    }
    hllc_reverse<T>(wl, wr, gamma, gm1inv, Fb, wlb, wrb);
    T done[5];
#pragma unroll
    for (int k = 0; k < 5; ++k) {
      const T dwb = T(0.5) * (wlb[k] - wrp[k]);
      const T e1 = fwd[k] ? dwb : T(0), e2 = bwd[k] ? dwb : T(0);
      done[k] = open[k] - e2;  // cell f - 1
      open[k] = ((wlb[k] + wrp[k]) + (e2 - e1)) + e1p[k];
      e1p[k] = e1;
      wrp[k] = wrb[k];
    }
    if (emit) {
      if (!FIN) {
#pragma unroll
        for (int k = 0; k < 5; ++k) Wacc[perm[k] * N + q] = acc[k] + done[k];
      } else {
        T pg[5], vg[5], wg[5];
#pragma unroll
        for (int k = 0; k < 5; ++k) {
          pg[perm[k]] = wm[k];
          vg[perm[k]] = vm[k];
          wg[perm[k]] = acc[k] + done[k];
        }
        finish_prim(pg, vg, wg, q, N, fa);
      }
    }
#pragma unroll
    for (int k = 0; k < 5; ++k) {
      wm[k] = w0[k];
      w0[k] = w1[k];
      w1[k] = w2[k];
      dw[k] = dn[k];
      fwd[k] = fwn[k];
      bwd[k] = bwn[k];
      vm[k] = v0[k];
      v0[k] = v1[k];
    }
  }
}

// J(U)^T v along x for periodic boundaries (nx >= 4) and the minmod (or
// first-order) HLLC scheme: a thread per cell c, which reverses the face above
// it (between c and c + 1).  A workgroup holds `rpb` whole rows (`len` = nx
// cells each, the ends wrapping inside the row, no face computed twice), or,
// for rows beyond XROW_MAX, one piece of a row: `cells` cells with three more
// on either side (`len` = cells + 6), of which the outer ones only lend their
// state, slope or face.  State, v, the slope, WRb and the slope's
// contributions pass between neighbours through LDS, and each is computed
// once, where a lane per face of 61-cell pieces converted every cell four
// times.
// In fp32 the limiter's differences are formed with one rounding from the
// neighbour's factors (velocity m / rho, pressure (g - 1) e), W_{c+1} - W_c =
// fma(m, 1/rho, -W_c).  A cell's backward difference then rounds W_{c-1}'s
// product for the face above it and its own for the face below it, so at a
// near-tie the two faces may take different branches; each face's own branch is
// reversed.
constexpr int XROW_MAX = 512;
constexpr int XLDS = 16;  // values per thread in LDS

template <typename T, int LIM, int MODE>
__global__ __launch_bounds__(XROW_MAX) void k_x_jtv(const T* __restrict__ U,
                                                    const T* __restrict__ v, AxisGeom g, T gamma,
                                                    T ih, int len, int rpb, int cells, int npieces,
                                                    T* __restrict__ Wacc, FinishArgs<T> fa) {
  static_assert(MODE == GATHER_FIRST || MODE == GATHER_FIRST_LAST, "x is the first axis, if any");
  extern __shared__ __align__(16) unsigned char x_jtv_lds[];
  const int nt = blockDim.x;
  T* const A = reinterpret_cast<T*>(x_jtv_lds);  // [6][nt]: rho, m, 1/rho, e (fp64: W); then WRb
  T* const B = A + 6 * nt;                       // [5][nt]: v; then the forward contribution
  T* const C = B + 5 * nt;                       // [5][nt]: lower-face slope; then the backward one
  const int n = g.n[0], tid = threadIdx.x;
  const long long nrows = (long long)g.n[1] * g.n[2];
  const long long N = nrows * n;
  const bool whole = npieces == 1;
  const int lr = tid / len, j = tid - lr * len;
  const long long row =
      whole ? (long long)blockIdx.x * rpb + lr : (long long)(blockIdx.x / npieces);
  const int x0 = whole ? 0 : (int)(blockIdx.x % npieces) * cells - 3;
  const bool active = lr < rpb && row < nrows;
  // LDS columns of the cells below and above (a piece's end cells stay put)
  const int tm = j > 0 ? tid - 1 : (whole ? tid + len - 1 : tid);
  const int tp = j < len - 1 ? tid + 1 : (whole ? tid - (len - 1) : tid);
  int c = x0 + j;
  if (!whole) c = c < 0 ? c + n : (c >= n ? c % n : c);
  const long long q = row * n + c;
  const T gm1 = gamma - T(1);
  const T gm1inv = T(1) / gm1;
  const bool own = active && (whole || (j >= 3 && j < 3 + cells && x0 + j < n));
  // u: rho, m, e with P = (g - 1) e; w the primitives
  T u[5], ir, w[5], vc[5], dw[5], wp[5];
  bool fwd[5], bwd[5], fwl[5], bwl[5];  // branches at the face above and below
  if (active) {
#pragma unroll
    for (int f = 0; f < 5; ++f) {
      u[f] = U[f * N + q];
      vc[f] = v[f * N + q];
    }
    to_prim(u, gm1, w);  // the arithmetic of the stage kernels
    ir = dev_rcp(u[0]);
    u[4] = fmad(-(T(0.5) * u[0]), fmad(w[1], w[1], fmad(w[2], w[2], w[3] * w[3])), u[4]);
    if constexpr (contracted_branches<T>) {
      A[tid] = u[0];
      A[5 * nt + tid] = u[4];
      A[4 * nt + tid] = ir;
#pragma unroll
      for (int f = 1; f < 4; ++f) A[f * nt + tid] = u[f];
    } else {
#pragma unroll
      for (int f = 0; f < 5; ++f) A[f * nt + tid] = w[f];
    }
#pragma unroll
    for (int f = 0; f < 5; ++f) B[f * nt + tid] = vc[f];
  }
  __syncthreads();
  if (active) {
    if constexpr (contracted_branches<T>) {
      const T irp = A[4 * nt + tp], irm = A[4 * nt + tm];
      T a[5], b[5], bl[5];  // forward, and backward as the upper and the lower face take it
      bool equal = false;
#pragma unroll
      for (int f = 0; f < 5; ++f) {
        const int k = f == 4 ? 5 : f;
        const T up = A[k * nt + tp], um = A[k * nt + tm];
        T wm;
        if (f == 0) {
          wp[f] = up;
          wm = um;
          a[f] = up - w[f];
          b[f] = bl[f] = w[f] - um;
        } else {
          const T sp = f == 4 ? gm1 : irp, s0 = f == 4 ? gm1 : ir, sm = f == 4 ? gm1 : irm;
          wp[f] = up * sp;
          wm = um * sm;
          a[f] = fmad(up, sp, -w[f]);
          b[f] = fmad(-um, sm, w[f]);
          bl[f] = fmad(u[f], s0, -wm);
        }
        equal = equal || wp[f] == w[f] || wm == w[f];
      }
      if (LIM != LIM_NONE && equal) {
        // (rare, and so read again, one cell after another: its registers are the
        // whole kernel's)  A flat slope's zero is given no branch.
        unsigned z = 0;
        T below[5] = {};
#pragma unroll 1
        for (int k = -3; k <= 3; ++k) {
          const int at = c + k;
          T t[5];
          prim_at(U, N, row * n + (at < 0 ? at + n : (at >= n ? at - n : at)), gm1, t);
          unsigned m = 0;
#pragma unroll
          for (int f = 0; f < 5; ++f) {
            m |= (t[f] == below[f] ? 1u : 0u) << f;
            below[f] = t[f];
          }
          if (k > -3) z |= m << (5 * (k + 2));
        }
        const unsigned flat = flat_fields(z);
#pragma unroll
        for (int f = 0; f < 5; ++f)
          if ((flat >> f) & 1u) a[f] = T(0);
      }
#pragma unroll
      for (int f = 0; f < 5; ++f) {
        dw[f] = slope_branch<T, LIM>(a[f], b[f], fwd[f], bwd[f]);
        C[f * nt + tid] = slope_branch<T, LIM>(a[f], bl[f], fwl[f], bwl[f]);
      }
    } else {
#pragma unroll
      for (int f = 0; f < 5; ++f) {
        wp[f] = A[f * nt + tp];
        dw[f] = slope_branch<T, LIM>(plain_diff(wp[f], w[f]), plain_diff(w[f], A[f * nt + tm]),
                                     fwd[f], bwd[f]);
        fwl[f] = fwd[f];
        bwl[f] = bwd[f];
        C[f * nt + tid] = dw[f];
      }
    }
  }
  __syncthreads();
  T wlb[5], wrb[5];
  if (active) {
    T wl[5], wr[5], Fb[5];
#pragma unroll
    for (int f = 0; f < 5; ++f) {
      wl[f] = fmad(T(0.5), dw[f], w[f]);
      wr[f] = fmad(T(-0.5), C[f * nt + tp], wp[f]);
      Fb[f] = (B[f * nt + tp] - vc[f]) * ih;
    }
    hllc_reverse<T>(wl, wr, gamma, gm1inv, Fb, wlb, wrb);
#pragma unroll
    for (int f = 0; f < 5; ++f) A[f * nt + tid] = wrb[f];
  }
  __syncthreads();
  T sum[5];
  if (active) {
#pragma unroll
    for (int f = 0; f < 5; ++f) {
      const T wrp = A[f * nt + tm];
      const T hl = T(0.5) * wlb[f], hr = T(0.5) * wrp;
      const T e1 = (fwd[f] ? hl : T(0)) - (fwl[f] ? hr : T(0));
      const T e2 = (bwd[f] ? hl : T(0)) - (bwl[f] ? hr : T(0));
      sum[f] = (wlb[f] + wrp) + (e2 - e1);
      B[f * nt + tid] = e1;
      C[f * nt + tid] = e2;
    }
  }
  __syncthreads();
  if (!own) return;
#pragma unroll
  for (int f = 0; f < 5; ++f) sum[f] = (sum[f] + B[f * nt + tm]) - C[f * nt + tp];
  if (MODE == GATHER_FIRST) {
#pragma unroll
    for (int f = 0; f < 5; ++f) Wacc[f * N + q] = sum[f];
  } else {
    finish_prim(w, vc, sum, q, N, fa);
  }
}

// rows per workgroup of k_x_jtv for whole rows of n <= XROW_MAX cells: the
// count that wastes the fewest lanes of its last wave, near 256 threads
inline int x_rows_per_block(int n) {
  int best = 1;
  double score = -1.0;
  for (int r = 1; r * n <= XROW_MAX; ++r) {
    const int t = r * n, w = (t + 63) / 64 * 64;
    const double s = (double)t / w - 1e-4 * (t < 256 ? 256 - t : t - 256);
    if (s > score) {
      score = s;
      best = r;
    }
  }
  return best;
}

// out = c0 x0 + c1 x1 + c2 x2 + beta (dW/dU)^T Wacc, W = (rho, v, P) of U
template <typename T>
__global__ __launch_bounds__(256) void k_jtv_finish(const T* __restrict__ U,
                                                    const T* __restrict__ Wacc, long long N,
                                                    FinishArgs<T> fa) {
  const long long q = (long long)blockIdx.x * 256 + threadIdx.x;
  if (q >= N) return;
  T w[5];
#pragma unroll
  for (int f = 0; f < 5; ++f) w[f] = Wacc[f * N + q];
  finish_cell(U, w, q, N, fa);
}

// g += weight (dL/dB)^T v for the flux-correction field B (B at a cell is
// added to the flux through its upper face on each axis a; a face's flux
// leaves the cell below with -1/h_a and enters the cell above with +1/h_a):
// per axis, d = v(i+1) - v(i), with v beyond the last cell 0 for outflow
// (periodic: wrapped), plus v(0) at the first cell with outflow, whose B
// also sits on the face below it
template <typename T>
__global__ __launch_bounds__(256) void k_flux_corr_vjp(const T* __restrict__ v, int nx, int ny,
                                                       int nz, int bcx, int bcy, int bcz, T wx,
                                                       T wy, T wz, T* g) {
  const long long N = (long long)nx * ny * nz;
  const long long q = (long long)blockIdx.x * 256 + threadIdx.x;
  if (q >= N) return;
  const int i = (int)(q % nx), j = (int)((q / nx) % ny), k = (int)(q / ((long long)nx * ny));
  const long long sx = 1, sy = nx, sz = (long long)nx * ny;
  const int n[3] = {nx, ny, nz}, c[3] = {i, j, k}, bc[3] = {bcx, bcy, bcz};
  const long long st[3] = {sx, sy, sz};
  const T w[3] = {wx, wy, wz};
#pragma unroll
  for (int f = 0; f < 5; ++f) {
    const T* vf = v + f * N;
    T acc = T(0);
#pragma unroll
    for (int a = 0; a < 3; ++a) {
      T up;
      if (c[a] + 1 < n[a]) up = vf[q + st[a]];
      else up = bc[a] == BC_PERIODIC ? vf[q - (long long)(n[a] - 1) * st[a]] : T(0);
      T d = up - vf[q];
      if (bc[a] != BC_PERIODIC && c[a] == 0) d += vf[q];
      acc += w[a] * d;
    }
    g[f * N + q] += acc;
  }
}

template <typename T>
__global__ __launch_bounds__(256) void k_fill(T* y, long long n, T v) {
  const long long q = (long long)blockIdx.x * 256 + threadIdx.x;
  if (q < n) y[q] = v;
}

// ---------------------------------------------------------------- sources

// OU acceleration at (x, y, z) from the row records and X phase factors,
// the same separable sum the stage kernel evaluates
template <typename T>
__device__ __forceinline__ void ou_accel(const T* __restrict__ rows, const T* __restrict__ tabx,
                                         int R, int nx, int ny, int x, int y, int z, T (&a)[3]) {
  const T* pq = rows + ((long long)z * ny + y) * 6 * (R + 1);
#pragma unroll
  for (int c = 0; c < 3; ++c) a[c] = pq[2 * c];
  for (int n = 1; n <= R; ++n) {
    const T xr = tabx[2 * ((long long)n * nx + x)], xi = tabx[2 * ((long long)n * nx + x) + 1];
#pragma unroll
    for (int c = 0; c < 3; ++c) a[c] += xr * pq[6 * n + 2 * c] - xi * pq[6 * n + 2 * c + 1];
  }
}

// reverse of the kick m += rho a dt, E += (m_old . a) dt (the acceleration
// does not depend on the state): lam_rho += sum_c lam_m_c a_c dt,
// lam_m_c += lam_E a_c dt
template <typename T>
__device__ __forceinline__ void kick_vjp_cell(const T (&a)[3], T dt, const T (&li)[5],
                                              T (&lo)[5]) {
  const T Eb = li[4];
  T rb = li[0];
#pragma unroll
  for (int c = 0; c < 3; ++c) {
    const T mb = li[1 + c];
    rb += mb * a[c] * dt;
    lo[1 + c] = mb + Eb * a[c] * dt;
  }
  lo[0] = rb;
  lo[4] = Eb;
}

template <typename T>
__global__ __launch_bounds__(256) void k_force_kick_vjp(const T* __restrict__ rows,
                                                        const T* __restrict__ tabx, int R, int nx,
                                                        int ny, int nz, T dt,
                                                        const T* __restrict__ lin, T* lout) {
  const long long N = (long long)nx * ny * nz;
  const long long q = (long long)blockIdx.x * 256 + threadIdx.x;
  if (q >= N) return;
  const int x = (int)(q % nx), y = (int)((q / nx) % ny), z = (int)(q / ((long long)nx * ny));
  T a[3];
  ou_accel(rows, tabx, R, nx, ny, x, y, z, a);
  T li[5], lo[5];
#pragma unroll
  for (int f = 0; f < 5; ++f) li[f] = lin[f * N + q];
  kick_vjp_cell(a, dt, li, lo);
#pragma unroll
  for (int f = 0; f < 5; ++f) lout[f * N + q] = lo[f];
}

__device__ __forceinline__ int wrapi(int i, int n) { return i < 0 ? i + n : (i >= n ? i - n : i); }

// reverse of the gravity kick at U (before the kick) with g = -grad phi:
// lam as for any kick, and accb_c = lam_m_c rho dt + lam_E m_c dt
template <typename T>
__global__ __launch_bounds__(256) void k_grav_kick_vjp(const T* __restrict__ U,
                                                       const T* __restrict__ phi, int n, T i2h,
                                                       T dt, const T* __restrict__ lin, T* lout,
                                                       T* __restrict__ accb) {
  const long long N = (long long)n * n * n;
  const long long q = (long long)blockIdx.x * 256 + threadIdx.x;
  if (q >= N) return;
  const int i = (int)(q % n), j = (int)((q / n) % n), k = (int)(q / ((long long)n * n));
  const long long n2 = (long long)n * n;
  const long long row = (long long)k * n2 + (long long)j * n;
  T a[3];
  a[0] = -(phi[row + wrapi(i + 1, n)] - phi[row + wrapi(i - 1, n)]) * i2h;
  a[1] = -(phi[(long long)k * n2 + (long long)wrapi(j + 1, n) * n + i] -
           phi[(long long)k * n2 + (long long)wrapi(j - 1, n) * n + i]) * i2h;
  a[2] = -(phi[(long long)wrapi(k + 1, n) * n2 + (long long)j * n + i] -
           phi[(long long)wrapi(k - 1, n) * n2 + (long long)j * n + i]) * i2h;
  const T rho = U[q], Eb = lin[4 * N + q];
  T rb = lin[q];
#pragma unroll
  for (int c = 0; c < 3; ++c) {
    const T mb = lin[(1 + c) * N + q];
    rb += mb * a[c] * dt;
    lout[(1 + c) * N + q] = mb + Eb * a[c] * dt;
    accb[c * N + q] = mb * rho * dt + Eb * U[(1 + c) * N + q] * dt;
  }
  lout[q] = rb;
  lout[4 * N + q] = Eb;
}

// reverse of g_c,i = -(phi_{i+1} - phi_{i-1}) / (2h): phib_j = sum_c (accb_c,j+1 - accb_c,j-1) / (2h)
template <typename T>
__global__ __launch_bounds__(256) void k_grad_adjoint(const T* __restrict__ accb, int n, T i2h,
                                                      T* __restrict__ phib) {
  const long long N = (long long)n * n * n;
  const long long q = (long long)blockIdx.x * 256 + threadIdx.x;
  if (q >= N) return;
  const int i = (int)(q % n), j = (int)((q / n) % n), k = (int)(q / ((long long)n * n));
  const long long n2 = (long long)n * n;
  const long long row = (long long)k * n2 + (long long)j * n;
  phib[q] = ((accb[row + wrapi(i + 1, n)] - accb[row + wrapi(i - 1, n)]) +
             (accb[N + (long long)k * n2 + (long long)wrapi(j + 1, n) * n + i] -
              accb[N + (long long)k * n2 + (long long)wrapi(j - 1, n) * n + i]) +
             (accb[2 * N + (long long)wrapi(k + 1, n) * n2 + (long long)j * n + i] -
              accb[2 * N + (long long)wrapi(k - 1, n) * n2 + (long long)j * n + i])) * i2h;
}

// lam_rho += s x
template <typename T>
__global__ __launch_bounds__(256) void k_axpy(T* y, const T* __restrict__ x, long long n, T s) {
  const long long q = (long long)blockIdx.x * 256 + threadIdx.x;
  if (q < n) y[q] += s * x[q];
}

// reverse of exact cooling E' = ek + rho Tn(rho, T)/(g-1), T = (g-1)(E - ek)/rho,
// ek = |m|^2/(2 rho), using the partial derivatives of the branch taken
template <typename T>
__device__ __forceinline__ void cool_vjp_cell(const T* __restrict__ U, long long N, long long q,
                                              T gm1, T dt, const CoolParams<T>& c,
                                              const T (&li)[5], T (&lo)[5]) {
  const T rho = U[q], mx = U[N + q], my = U[2 * N + q], mz = U[3 * N + q], E = U[4 * N + q];
  const T ek = T(0.5) * (mx * mx + my * my + mz * mz) / rho;
  const T Tin = gm1 * (E - ek) / rho;
  // the forward map (same branch decisions as the forward kernel) and its partials
  const T k2 = c.k2r * rho;
  T Tn, dT, dr;
  if (Tin >= c.tc) {
    const T k1 = c.k1r * rho;
    const T st = sqrt(Tin);
    const T t1 = (st - c.sqrt_tc) / k1;
    if (dt <= t1) {
      const T s = st - k1 * dt;
      Tn = s * s;
      dT = s / st;
      dr = -T(2) * s * c.k1r * dt;
    } else {
      const T w = T(1) + k2 * (dt - t1);
      Tn = c.tc - c.ts * log(w);
      dT = c.ts * k2 / (w * T(2) * st * k1);
      dr = -c.ts / w * (c.k2r * (dt - t1) + k2 * t1 / rho);
    }
  } else {
    const T e = exp((c.tc - Tin) * c.its);
    const T w = e + k2 * dt;
    Tn = c.tc - c.ts * log(w);
    dT = e / w;
    dr = -c.ts / w * c.k2r * dt;
  }
  if (Tn < c.tfloor) {
    Tn = c.tfloor;
    dT = T(0);
    dr = T(0);
  }
  const T Eb = li[4];
  T ekb = Eb;
  T rhob = li[0] + Eb * Tn / gm1;
  const T Tnb = Eb * rho / gm1;
  const T Tb = Tnb * dT;
  rhob += Tnb * dr;
  const T Einb = Tb * gm1 / rho;
  ekb -= Tb * gm1 / rho;
  rhob -= Tb * Tin / rho;
  rhob -= ekb * ek / rho;
  lo[0] = rhob;
  lo[1] = li[1] + ekb * mx / rho;
  lo[2] = li[2] + ekb * my / rho;
  lo[3] = li[3] + ekb * mz / rho;
  lo[4] = Einb;
}


template <typename T>
__global__ __launch_bounds__(256) void k_cool_vjp(const T* __restrict__ U, long long N, T gm1, T dt,
                                                  CoolParams<T> c, const T* __restrict__ lin,
                                                  T* lout) {
  const long long q = (long long)blockIdx.x * 256 + threadIdx.x;
  if (q >= N) return;
  T li[5], lo[5];
#pragma unroll
  for (int f = 0; f < 5; ++f) li[f] = lin[f * N + q];
  cool_vjp_cell(U, N, q, gm1, dt, c, li, lo);
#pragma unroll
  for (int f = 0; f < 5; ++f) lout[f * N + q] = lo[f];
}

// cooling reverse then forcing-kick reverse in one pass (the order of the
// reverse sweep without gravity): the intermediate adjoint stays in registers
template <typename T>
__global__ __launch_bounds__(256) void k_cool_force_vjp(const T* __restrict__ U, T gm1, T dt,
                                                        CoolParams<T> c,
                                                        const T* __restrict__ rows,
                                                        const T* __restrict__ tabx, int R, int nx,
                                                        int ny, int nz, const T* __restrict__ lin,
                                                        T* lout) {
  const long long N = (long long)nx * ny * nz;
  const long long q = (long long)blockIdx.x * 256 + threadIdx.x;
  if (q >= N) return;
  const int x = (int)(q % nx), y = (int)((q / nx) % ny), z = (int)(q / ((long long)nx * ny));
  T li[5], lm[5], lo[5];
#pragma unroll
  for (int f = 0; f < 5; ++f) li[f] = lin[f * N + q];
  cool_vjp_cell(U, N, q, gm1, dt, c, li, lm);
  T a[3];
  ou_accel(rows, tabx, R, nx, ny, x, y, z, a);
  kick_vjp_cell(a, dt, lm, lo);
#pragma unroll
  for (int f = 0; f < 5; ++f) lout[f * N + q] = lo[f];
}

inline unsigned nblk(long long n) { return (unsigned)((n + 255) / 256); }

}  // namespace

// Cells per column segment of the fused march: a segment costs its cells plus
// three faces it shares with its neighbours, and a SIMD works through
// ceil(waves / 1024) segments of 64 columns; fewer than 2.2 (fp64, which holds
// two waves by its registers: 1.4) waves leave it waiting on loads, so that
// shorter segments gain nothing more below that.  Fixed 64-cell segments ran a
// 32^3 march on four workgroups; one adjoint step from kept stages, fixed ->
// rule: 64^3 fp32 362 -> 63 us, 128^3 fp32 405 -> 205 us and fp64 593 ->
// 399 us, 256^3 1.60 ms and 3.1 ms either way.
template <typename T>
inline int march_segment(long long columns, int n) {
  const double least_waves = sizeof(T) == 4 ? 2.2 : 1.4;
  int best = n;
  double least = 1e300;
  for (int nseg = (n + 127) / 128; nseg <= n; ++nseg) {
    const int seg = (n + nseg - 1) / nseg;
    const long long threads = columns * ((n + seg - 1) / seg);
    const double waves = (double)((threads + 65535) / 65536);
    const double cost = (seg + 3.0) * (waves > least_waves ? waves : least_waves);
    if (cost < least) {
      least = cost;
      best = seg;
    }
  }
  return best;
}

// J(U)^T v into out = c0 x0 + c1 x1 + beta J^T v (x0, x1 may be NULL)
template <typename T>
hipError_t adj_jtv(const AdjointBuffers<T>& B, const StageGeom& geom, int limiter, int riemann,
                   T gamma,
                   const double* h, const T* U, const T* v, T beta, T c0, const T* x0, T c1,
                   const T* x1, T c2, const T* x2, T* out, hipStream_t s) {
  const long long N = (long long)geom.nx * geom.ny * geom.nz;
  const int nn[3] = {geom.nx, geom.ny, geom.nz};
  const bool rt = adj_runtime_scheme(limiter, riemann);
  const FinishArgs<T> fa{gamma - T(1), beta, c0, c1, c2, x0, x1, x2, out,
                         x0 == v ? 0 : (x1 == v ? 1 : (x2 == v ? 2 : -1))};
  // the axes with fluxes (a periodic axis of one cell has none: its fluxes
  // cancel exactly); the first one's gather stores the W adjoint, the last
  // one's adds the others and finishes the cell
  int active[3], na = 0;
  for (int ax = 0; ax < 3; ++ax)
    if (!(geom.bc[ax] == BC_PERIODIC && nn[ax] == 1)) active[na++] = ax;
  if (na == 0) {
    hipLaunchKernelGGL((k_fill<T>), dim3(nblk(5 * N)), dim3(256), 0, s, B.Wacc, 5 * N, T(0));
    hipLaunchKernelGGL((k_jtv_finish<T>), dim3(nblk(N)), dim3(256), 0, s, U, B.Wacc, N, fa);
    return hipGetLastError();
  }
  for (int ia = 0; ia < na; ++ia) {
    const int ax = active[ia];
    const int mode = na == 1 ? GATHER_FIRST_LAST
                             : (ia == 0 ? GATHER_FIRST : (ia == na - 1 ? GATHER_LAST : GATHER_ADD));
    AxisGeom ag{{geom.nx, geom.ny, geom.nz}, geom.bc[ax], 0};
    ag.nf = geom.bc[ax] == BC_PERIODIC ? nn[ax] : nn[ax] + 1;
    const long long nfaces = (long long)ag.nf * (N / nn[ax]);
    const T ih = (T)(1.0 / h[ax]);
#define MH_GATHER(AX, SL)                                                                     \
  do {                                                                                        \
    if (mode == GATHER_ADD)                                                                   \
      hipLaunchKernelGGL((k_cell_gather<T, AX, SL, GATHER_ADD>), dim3(nblk(N)), dim3(256), 0, \
                         s, B.wbar, B.flags, ag, B.Wacc, U, fa);                              \
    else if (mode == GATHER_FIRST)                                                            \
      hipLaunchKernelGGL((k_cell_gather<T, AX, SL, GATHER_FIRST>), dim3(nblk(N)), dim3(256),  \
                         0, s, B.wbar, B.flags, ag, B.Wacc, U, fa);                           \
    else if (mode == GATHER_LAST)                                                             \
      hipLaunchKernelGGL((k_cell_gather<T, AX, SL, GATHER_LAST>), dim3(nblk(N)), dim3(256),   \
                         0, s, B.wbar, B.flags, ag, B.Wacc, U, fa);                           \
    else                                                                                      \
      hipLaunchKernelGGL((k_cell_gather<T, AX, SL, GATHER_FIRST_LAST>), dim3(nblk(N)),        \
                         dim3(256), 0, s, B.wbar, B.flags, ag, B.Wacc, U, fa);                \
  } while (0)
#define MH_FACE(AX)                                                                           \
  do {                                                                                        \
    if (rt) {                                                                                 \
      hipLaunchKernelGGL((k_face_vjp_rt<T, AX>), dim3(nblk(nfaces)), dim3(256), 0, s, U, v,   \
                         ag, gamma, ih, limiter, riemann, B.wbar, nfaces);                    \
      MH_GATHER(AX, true);                                                                    \
    } else {                                                                                  \
      if (limiter == LIM_NONE)                                                                \
        hipLaunchKernelGGL((k_face_vjp<T, LIM_NONE, AX>), dim3(nblk(nfaces)), dim3(256), 0,   \
                           s, U, v, ag, gamma, ih, B.wbar, B.flags, nfaces);                  \
      else                                                                                    \
        hipLaunchKernelGGL((k_face_vjp<T, LIM_MINMOD, AX>), dim3(nblk(nfaces)), dim3(256), 0, \
                           s, U, v, ag, gamma, ih, B.wbar, B.flags, nfaces);                  \
      MH_GATHER(AX, false);                                                                   \
    }                                                                                         \
  } while (0)
    // periodic with at least four cells, minmod or first order: face reverse
    // and gather fused, rows along x, column marches along y and z
    const bool march = !rt && geom.bc[ax] == BC_PERIODIC && nn[ax] >= 4;
    if (march && ax == 0) {
      const int n = nn[0];
      const long long rows = N / n;
      const int npieces = n <= XROW_MAX ? 1 : (n + XROW_MAX - 7) / (XROW_MAX - 6);
      const int rpb = npieces == 1 ? x_rows_per_block(n) : 1;
      const int cells = (n + npieces - 1) / npieces;
      const int len = npieces == 1 ? n : cells + 6;
      const unsigned threads = (unsigned)((rpb * len + 63) / 64 * 64);
      const unsigned blocks =
          (unsigned)(npieces == 1 ? (rows + rpb - 1) / rpb : rows * npieces);
      const size_t lds = XLDS * threads * sizeof(T);
#define MH_XJTV_MODE(LM, MODE)                                                                \
  hipLaunchKernelGGL((k_x_jtv<T, LM, MODE>), dim3(blocks), dim3(threads), lds, s, U, v, ag,   \
                     gamma, ih, len, rpb, cells, npieces, B.Wacc, fa)
#define MH_XJTV(LM)                                                                           \
  do {                                                                                        \
    if (mode == GATHER_FIRST) MH_XJTV_MODE(LM, GATHER_FIRST);                                 \
    else MH_XJTV_MODE(LM, GATHER_FIRST_LAST);                                                 \
  } while (0)
      if (limiter == LIM_NONE) MH_XJTV(LIM_NONE);
      else MH_XJTV(LIM_MINMOD);
#undef MH_XJTV
#undef MH_XJTV_MODE
    } else if (march) {
      const int seg = march_segment<T>(N / nn[ax], nn[ax]);
      const long long threads = (N / nn[ax]) * ((nn[ax] + seg - 1) / seg);
#define MH_MARCH(AX, LM)                                                                      \
  do {                                                                                        \
    if (mode == GATHER_ADD)                                                                   \
      hipLaunchKernelGGL((k_axis_jtv<T, LM, AX, GATHER_ADD>), dim3(nblk(threads)), dim3(256), \
                         0, s, U, v, ag, gamma, ih, seg, B.Wacc, fa);                         \
    else if (mode == GATHER_FIRST)                                                            \
      hipLaunchKernelGGL((k_axis_jtv<T, LM, AX, GATHER_FIRST>), dim3(nblk(threads)),          \
                         dim3(256), 0, s, U, v, ag, gamma, ih, seg, B.Wacc, fa);              \
    else if (mode == GATHER_LAST)                                                             \
      hipLaunchKernelGGL((k_axis_jtv<T, LM, AX, GATHER_LAST>), dim3(nblk(threads)),           \
                         dim3(256), 0, s, U, v, ag, gamma, ih, seg, B.Wacc, fa);              \
    else                                                                                      \
      hipLaunchKernelGGL((k_axis_jtv<T, LM, AX, GATHER_FIRST_LAST>), dim3(nblk(threads)),     \
                         dim3(256), 0, s, U, v, ag, gamma, ih, seg, B.Wacc, fa);              \
  } while (0)
      if (ax == 1) {
        if (limiter == LIM_NONE) MH_MARCH(1, LIM_NONE);
        else MH_MARCH(1, LIM_MINMOD);
      } else {
        if (limiter == LIM_NONE) MH_MARCH(2, LIM_NONE);
        else MH_MARCH(2, LIM_MINMOD);
      }
#undef MH_MARCH
    } else if (ax == 0) MH_FACE(0);
    else if (ax == 1) MH_FACE(1);
    else MH_FACE(2);
#undef MH_FACE
#undef MH_GATHER
  }
  return hipGetLastError();
}

template <typename T>
hipError_t adj_flux_corr_vjp(const T* v, const StageGeom& g, const double* h, double weight,
                             T* grad, hipStream_t s) {
  const long long N = (long long)g.nx * g.ny * g.nz;
  hipLaunchKernelGGL((k_flux_corr_vjp<T>), dim3(nblk(N)), dim3(256), 0, s, v, g.nx, g.ny, g.nz,
                     g.bc[0], g.bc[1], g.bc[2], (T)(weight / h[0]), (T)(weight / h[1]),
                     (T)(weight / h[2]), grad);
  return hipGetLastError();
}

template <typename T>
hipError_t adj_force_kick_vjp(const T* rows, const T* tabx, int R, const StageGeom& g, T dt,
                              const T* lin, T* lout, hipStream_t s) {
  const long long N = (long long)g.nx * g.ny * g.nz;
  hipLaunchKernelGGL((k_force_kick_vjp<T>), dim3(nblk(N)), dim3(256), 0, s, rows, tabx, R, g.nx,
                     g.ny, g.nz, dt, lin, lout);
  return hipGetLastError();
}

template <typename T>
hipError_t adj_cool_vjp(const T* U, long long N, T gm1, T dt, const CoolParams<T>& c, const T* lin,
                        T* lout, hipStream_t s) {
  hipLaunchKernelGGL((k_cool_vjp<T>), dim3(nblk(N)), dim3(256), 0, s, U, N, gm1, dt, c, lin, lout);
  return hipGetLastError();
}

template <typename T>
hipError_t adj_cool_force_vjp(const T* U, T gm1, T dt, const CoolParams<T>& c, const T* rows,
                              const T* tabx, int R, const StageGeom& g, const T* lin, T* lout,
                              hipStream_t s) {
  const long long N = (long long)g.nx * g.ny * g.nz;
  hipLaunchKernelGGL((k_cool_force_vjp<T>), dim3(nblk(N)), dim3(256), 0, s, U, gm1, dt, c, rows,
                     tabx, R, g.nx, g.ny, g.nz, lin, lout);
  return hipGetLastError();
}

// reverse of the gravity step at Ub (the state the kick acted on), with the
// potential phi solved from Ub: lout from lin, using a second multigrid solve
// with the same operator for the adjoint of A^+ (Sec. 6.2.4)
template <typename T>
hipError_t adj_gravity_vjp(const AdjointBuffers<T>& B, MGLayout& mgL, char* mgws,
                           const mh_physics_desc& p, const T* Ub, const T* phi, int n, double h,
                           T dt, const T* lin, T* lout, DevClock* clk, hipStream_t s) {
  const long long N = (long long)n * n * n;
  if (mgL.fft) return fft_gravity_vjp<T>(mgws, mgL, h, p.grav_G, Ub, dt, lin, lout, B.accb, s);
  const T i2h = (T)(1.0 / (2.0 * h));
  hipLaunchKernelGGL((k_grav_kick_vjp<T>), dim3(nblk(N)), dim3(256), 0, s, Ub, phi, n, i2h, dt,
                     lin, lout, B.accb);
  hipLaunchKernelGGL((k_grad_adjoint<T>), dim3(nblk(N)), dim3(256), 0, s, B.accb, n, i2h, B.phib);
  hipError_t e = mg_set_rhs<T>(mgws, mgL, B.phib, 1.0, clk, s);
  if (e != hipSuccess) return e;
  e = mg_set_guess<T>(mgws, mgL, (const T*)nullptr, s);
  if (e != hipSuccess) return e;
  e = mg_solve<T>(mgws, mgL, p, clk, nullptr, s);
  if (e != hipSuccess) return e;
  const T* x = reinterpret_cast<const T*>(mgws + mg_phi_offset(mgL));
  hipLaunchKernelGGL((k_axpy<T>), dim3(nblk(N)), dim3(256), 0, s, lout, x, N,
                     (T)(4.0 * M_PI * p.grav_G));
  return hipGetLastError();
}

#define ADJ_INSTANTIATE(T)                                                                       \
  template hipError_t adj_jtv<T>(const AdjointBuffers<T>&, const StageGeom&, int, int, T,        \
                                 const double*, const T*, const T*, T, T, const T*, T, const T*, \
                                 T, const T*, T*, hipStream_t);                                  \
  template hipError_t adj_flux_corr_vjp<T>(const T*, const StageGeom&, const double*, double,   \
                                           T*, hipStream_t);                                   \
  template hipError_t adj_force_kick_vjp<T>(const T*, const T*, int, const StageGeom&, T,        \
                                            const T*, T*, hipStream_t);                          \
  template hipError_t adj_cool_vjp<T>(const T*, long long, T, T, const CoolParams<T>&, const T*, \
                                      T*, hipStream_t);                                          \
  template hipError_t adj_cool_force_vjp<T>(const T*, T, T, const CoolParams<T>&, const T*,     \
                                            const T*, int, const StageGeom&, const T*, T*,     \
                                            hipStream_t);                                      \
  template hipError_t adj_gravity_vjp<T>(const AdjointBuffers<T>&, MGLayout&, char*,             \
                                         const mh_physics_desc&, const T*, const T*, int, double, \
                                         T, const T*, T*, DevClock*, hipStream_t);
ADJ_INSTANTIATE(float)
ADJ_INSTANTIATE(double)
#undef ADJ_INSTANTIATE

}  // namespace mh
