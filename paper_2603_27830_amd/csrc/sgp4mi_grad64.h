// One point's forward pass and its derivatives in double, for the VJP and the
// Jacobian.
//
// The state is a function of six mean quantities only: the semi-major axis a,
// the components ax, ay of the (long-period corrected) eccentricity vector,
// the mean longitude U from the node, the node and the inclination i.  On the
// way lie six polar quantities (radius mrt, rates mvt and rvdot, and the
// angles u, node, i of the corrected orientation), whose partial derivatives
// with respect to (a, r_l, p_L, beta, e sin E, u) are some twenty scalars.  A
// derivative in either direction is those scalars, the implicit derivative at
// Kepler's root (dpsi = (dU + sin psi dax - cos psi day) / D) and the frame of
// the orbit: with U, V the radial and transverse unit vectors and W the
// normal,
//   dU =  (du + cos i dnode) V + (sin u di - sin i cos u dnode) W
//   dV = -(du + cos i dnode) U + (cos u di + sin i sin u dnode) W.
// So nothing is differentiated per element or per inclination constant inside
// the point (the constants that depend on the inclination alone enter through
// one inclination derivative).
//
// Constants are read from LDS (c: the record's doubles of one satellite, then
// the extras below).  As scalar operands the 40 doubles overflow the scalar
// file and come back through lane reads (374 of ~1,400 vector instructions of
// the VJP's point); as LDS reads they cost no vector instruction.
#pragma once

#include "sgp4mi_point.h"

namespace sgp4mi {

// Per-satellite extras behind the record's doubles: d(Lcof)/di, d(aycof)/di.
enum Grad64Const : int { kLcofI = kNRec, kAycofI, kNGrad64 };

// The extras from the record (the clamp of 1 + cos i as in initialisation).
__device__ __forceinline__ void grad64_extras(double* c, double j3oj2) {
  const double ci = c[kCosi], si = c[kSini];
  double den = 1.0 + ci, dden = -si;
  if (fabs(den) <= 1.5e-12) {
    den = 1.5e-12;
    dden = 0.0;
  }
  const double num = si * (3.0 + 5.0 * ci), dnum = ci * (3.0 + 5.0 * ci) - 5.0 * si * si;
  c[kLcofI] = -0.25 * j3oj2 * (dnum - num * dden / den) / den;
  c[kAycofI] = -0.5 * j3oj2 * ci;
}

// What the derivatives need of a point's forward pass.
struct Point64 {
  // secular
  double t, cMdf, sMdf, x, x3, cM, dsM, A, Ld;
  double a, ra, e, om0, sw, cw, tau, ax, ay;
  bool clamped;
  // Kepler and the orbit in its plane
  double sp, cp, iD, ecE, esE, om, rl, irl, ia, sr, betal, ibeta, rdotl, rvdotl, w, iopb, sinu, cosu;
  // short period
  double s2, c2, ipl, k1, k2, qk, g1, bk, mrt, mvt, rvdot;
  // orientation
  double ssu, csu, sinc, cinc, snod, cnod;
};

// The forward kernel's model, in two parts; each returns the point's code (0,
// 1, 4, 6).
//
// Every quotient is a product of three reciprocals: 1 / sqrt(a), 1 / D and
// 1 / beta (r_l = a D, p_L = a beta^2).  The simplified-drag sets take the
// general expressions (their records hold zeros for the terms they leave out,
// and those constants have no derivatives).
__device__ __forceinline__ uint32_t point64_secular(const double* c, double t_abs, Point64& p, double* U) {
  const double t = t_abs - c[kEpochMin];
  p.t = t;
  const double Mdf = fma(c[kMdot], t, c[kM0]);
  sincos_any(Mdf, &p.sMdf, &p.cMdf);
  p.x = fma(c[kEta], p.cMdf, 1.0);
  p.x3 = p.x * p.x * p.x - c[kDM0];
  const double dMa = fma(c[kMcof], p.x3, c[kArgpcof] * t);
  const double M = Mdf + dMa;
  const double argp = fma(c[kArgpdot], t, c[kArgp0]) - dMa;
  double sM = p.sMdf;
  p.cM = p.cMdf;
  if (fabs(dMa) > kRotMax) sincos_any(M, &sM, &p.cM);
  else rotate_small(&sM, &p.cM, dMa);
  p.dsM = sM - c[kSinM0];
  p.A = fma(-t, fma(t, fma(t, fma(t, c[kD4], c[kD3]), c[kD2]), c[kC1]), 1.0);
  p.Ld = t * t * fma(t, fma(t, fma(t, c[kT5cof], c[kT4cof]), c[kT3cof]), c[kT2cof]);
  const double a = c[kA0pp] * p.A * p.A;
  p.a = a;
  double e = c[kE0] - fma(c[kBC5], p.dsM, c[kBC4] * t);
  if (!(e >= -0.001 && e < 1.0)) return 1;
  p.clamped = e < 1.0e-6;
  e = fmax(e, 1.0e-6);
  p.e = e;
  sincos_any(argp, &p.sw, &p.cw);
  const double ra = rsq(a);
  p.ia = ra * ra;
  const double ax = e * p.cw;
  p.om0 = fma(-e, e, 1.0);
  p.tau = p.ia * rcp(p.om0);
  const double ay = e * p.sw + p.tau * c[kAycof];
  p.ax = ax;
  p.ay = ay;
  *U = fma(c[kN0pp], p.Ld, M) + argp + p.tau * c[kLcof] * ax;
  p.ra = ra;
  return 0;
}

// From the mean elements on.
__device__ __forceinline__ uint32_t point64_orbit(const double* c, const Grav& g, double t, double U, Point64& p) {
  const double a = p.a, ax = p.ax, ay = p.ay, ra = p.ra;
  double sp, cp;
  const double eb = fabs(ax) + fabs(ay);
  bool in = eb <= kepler_small<double>();
  in = in & (fabs(U) <= kTableMax);
  const bool small = __all(in);
  const double iD0 = kepler64(U, ax, ay, eb, small, &sp, &cp);
  p.sp = sp;
  p.cp = cp;
  p.ecE = ax * cp + ay * sp;
  p.esE = ax * sp - ay * cp;
  const double D = 1.0 - p.ecE;
  p.iD = rcp_from(D, iD0);
  p.om = 1.0 - (ax * ax + ay * ay);
  if (!(a * p.om >= 0.0)) return 4;
  p.rl = a * D;
  p.irl = p.ia * p.iD;
  p.sr = ra * p.iD;  // sqrt(a) / r_l
  p.rdotl = p.sr * p.esE;
  p.ibeta = rsq(p.om);
  p.betal = p.om * p.ibeta;
  p.rvdotl = p.sr * p.betal;
  p.iopb = rcp(1.0 + p.betal);
  p.w = p.esE * p.iopb;
  p.sinu = p.iD * (sp - ay - ax * p.w);
  p.cosu = p.iD * (cp - ax + ay * p.w);
  p.s2 = 2.0 * p.sinu * p.cosu;
  p.c2 = 1.0 - 2.0 * p.sinu * p.sinu;
  p.ipl = p.ia * (p.ibeta * p.ibeta);
  p.k1 = g.k2 * p.ipl;
  p.k2 = p.k1 * p.ipl;
  p.qk = ra * p.ia * p.k1;
  const double c41h = 1.5 * c[kC41], x1 = c[kX1];
  p.g1 = x1 * p.c2 + c41h;
  p.bk = 1.0 - p.k2 * p.betal * c41h;
  p.mrt = p.rl * p.bk + 0.5 * p.k1 * x1 * p.c2;
  p.mvt = p.rdotl - p.qk * x1 * p.s2;
  p.rvdot = p.rvdotl + p.qk * p.g1;
  const double du = -0.25 * p.k2 * c[kX7] * p.s2;
  const double kc = 1.5 * p.k2 * c[kCosi];
  const double dinc = kc * c[kSini] * p.c2;
  double dnode = kc * p.s2;
  p.ssu = p.sinu;
  p.csu = p.cosu;
  p.sinc = c[kSini];
  p.cinc = c[kCosi];
  rotate_node64(&p.ssu, &p.csu, du, &p.sinc, &p.cinc, dinc, &dnode, c[kI0], small);
  const double node = fma(t, fma(t, c[kNodecf], c[kNodedot]), c[kNode0]);
  sincos_any(node + dnode, &p.snod, &p.cnod);
  return p.mrt < 1.0 ? 6u : 0u;
}

// du at fixed psi for a change of ax and of ay.
__device__ __forceinline__ void u_partials(const Point64& p, double* u_x, double* u_y) {
  const double wb = p.w * p.iopb * p.ibeta;
  const double wx = p.sp * p.iopb + wb * p.ax, wy = wb * p.ay - p.cp * p.iopb;
  *u_x = p.iD * (p.cosu * (-p.w - p.ax * wx) - p.sinu * (p.ay * wx - 1.0));
  *u_y = p.iD * (p.cosu * (-1.0 - p.ax * wy) - p.sinu * (p.w + p.ay * wy));
}

// ------------------------------------------------------------------- VJP --
// Adjoint sums of one satellite.  The record's other constants follow from
// these: t2cof = 1.5 C1 (its adjoint is added to C1's), sin M0 enters only as
// bC5 (sin M - sin M0) (its adjoint is bC5 times E0's), and those that depend
// on the inclination alone share kAInc.
enum Adj64 : int {
  kAM0, kAMdot, kAArgp0, kAArgpdot, kANode0, kANodedot, kANodecf, kAC1, kABC4, kAArgpcof, kAEta, kAMcof, kADM0, kAD2,
  kAD3, kAD4, kABC5, kAT3cof, kAT4cof, kAT5cof, kAN0pp, kAA0pp, kAE0, kAInc, kNAdj64
};
__device__ constexpr int kAdjRec[kAInc] = {kM0,  kMdot, kArgp0, kArgpdot, kNode0, kNodedot, kNodecf, kC1,
                                           kBC4, kArgpcof, kEta, kMcof, kDM0, kD2, kD3, kD4,
                                           kBC5, kT3cof, kT4cof, kT5cof, kN0pp, kA0pp, kE0};

// One lane's adjoint sums: a column of LDS, [kNAdj64][64] per wavefront.  Held
// in registers the sums take 48 of them over the whole point, which is the
// difference between two and three wavefronts per SIMD.
struct Adj64Sums {
  double* col;
  __device__ __forceinline__ void clear() const {
#pragma unroll
    for (int k = 0; k < kNAdj64; ++k) col[64 * k] = 0.0;
  }
  __device__ __forceinline__ void add(int k, double x) const { unsafeAtomicAdd(col + 64 * k, x); }
};

// A vector's components along the orbit's radial, transverse and normal unit
// vectors: rotations by the node, the inclination and the argument of latitude.
__device__ __forceinline__ void to_frame(const Point64& p, const double x[3], double* u, double* v, double* w) {
  const double x1 = p.cnod * x[0] + p.snod * x[1], x2 = p.cnod * x[1] - p.snod * x[0];
  const double x3 = p.cinc * x2 + p.sinc * x[2];
  *w = p.cinc * x[2] - p.sinc * x2;
  *u = p.csu * x1 + p.ssu * x3;
  *v = p.csu * x3 - p.ssu * x1;
}

__device__ __forceinline__ void point64_reverse(const double* c, const Grav& g, const Point64& p, const double gr[3],
                                                const double gv[3], const Adj64Sums& cb) {
  // the state's adjoint in the orbit's frame, then that of the polar quantities
  double rU, rV, rW, vU, vV, vW;
  to_frame(p, gr, &rU, &rV, &rW);
  to_frame(p, gv, &vU, &vV, &vW);
  const double rr = g.radius * p.mrt, vm = g.vkms * p.mvt, vr = g.vkms * p.rvdot;
  const double mb = g.radius * rU, vb = g.vkms * vU, wb = g.vkms * vV;
  const double ub = rr * rV + vm * vV - vr * vU;
  const double s1 = rr * rW + vm * vW, s0 = vr * vW;
  const double ib = p.ssu * s1 + p.csu * s0;
  const double nb = p.cinc * ub + p.sinc * (p.ssu * s0 - p.csu * s1);

  // polar quantities -> u, p_L, r_l, beta, e sin E, a
  const double x1 = c[kX1], x7 = c[kX7], ci = c[kCosi], si = c[kSini];
  const double c41h = 1.5 * c[kC41];
  const double q2 = 2.0 * p.qk * x1;
  const double nk3 = 3.0 * ci * p.k2, ik3 = nk3 * si;
  const double u_b = ub * (1.0 - 0.5 * x7 * p.k2 * p.c2) - mb * (p.k1 * x1 * p.s2) + nb * (nk3 * p.c2) -
                     ib * (ik3 * p.s2) - q2 * (vb * p.c2 + wb * p.s2);
  const double pl_b = p.ipl * (mb * (2.0 * p.rl * c41h * p.betal * p.k2 - 0.5 * x1 * p.c2 * p.k1) +
                               ub * (0.5 * x7 * p.k2 * p.s2) - nb * (nk3 * p.s2) - ib * (ik3 * p.c2) +
                               vb * (p.qk * x1 * p.s2) - wb * (p.qk * p.g1));
  const double rl_b = mb * p.bk - p.irl * (vb * p.rdotl + wb * p.rvdotl);
  const double be_b = wb * p.sr - mb * (p.rl * c41h * p.k2);
  const double es_b = vb * p.sr;
  double a_b = p.ia * (vb * (0.5 * p.rdotl + 1.5 * p.qk * x1 * p.s2) + wb * (0.5 * p.rvdotl - 1.5 * p.qk * p.g1)) +
               rl_b * (1.0 - p.ecE) + pl_b * p.om;
  // Kepler's equation at its root, then ax and ay at fixed psi
  double u_x, u_y;
  u_partials(p, &u_x, &u_y);
  const double arl = p.a * rl_b;
  const double U_b = p.iD * (arl * p.esE + p.ecE * es_b + p.betal * p.iD * u_b);
  const double be2 = be_b * p.ibeta + 2.0 * p.a * pl_b;
  double ax_b = -arl * p.cp + p.sp * (es_b + U_b) - p.ax * be2 + u_x * u_b;
  const double ay_b = -arl * p.sp - p.cp * (es_b + U_b) - p.ay * be2 + u_y * u_b;
  // inclination: the short-period coefficients and the J3 terms
  const double cs = ci * si;
  const double i_b = mb * (cs * (9.0 * p.rl * p.k2 * p.betal + p.k1 * p.c2)) + ub * (3.5 * cs * p.k2 * p.s2) -
                     nb * (1.5 * si * p.k2 * p.s2) + ib * (1.0 + 1.5 * p.k2 * p.c2 * (ci * ci - si * si)) -
                     vb * (2.0 * cs * p.qk * p.s2) + wb * (cs * p.qk * (2.0 * p.c2 - 9.0)) +
                     p.tau * (ay_b * c[kAycofI] + U_b * p.ax * c[kLcofI]);
  // long-period terms
  const double tau_b = (U_b * c[kLcof] * p.ax + ay_b * c[kAycof]) * (p.tau * p.tau);
  ax_b += U_b * p.tau * c[kLcof];
  const double e_b = ax_b * p.cw + ay_b * p.sw + 2.0 * tau_b * p.a * p.e;
  const double w_b = p.e * (ay_b * p.cw - ax_b * p.sw) + U_b;
  a_b -= tau_b * p.om0;

  // secular drag and gravity
  const double t = p.t, t2 = t * t;
  const double es = p.clamped ? 0.0 : e_b;
  const double aA = a_b * p.A;
  const double A_b = 2.0 * c[kA0pp] * aA;
  const double Ld_b = U_b * c[kN0pp];
  double M_b = U_b;
  cb.add(kAE0, es);
  cb.add(kAA0pp, aA * p.A);
  cb.add(kAN0pp, U_b * p.Ld);
  cb.add(kABC4, -(es * t));
  cb.add(kAC1, 1.5 * Ld_b * t2 - A_b * t);
  cb.add(kAInc, i_b);
  const double t3 = t2 * t, t4 = t3 * t;
  cb.add(kAT3cof, Ld_b * t3);
  cb.add(kAT4cof, Ld_b * t4);
  cb.add(kAT5cof, Ld_b * (t4 * t));
  cb.add(kAD2, -(A_b * t2));
  cb.add(kAD3, -(A_b * t3));
  cb.add(kAD4, -(A_b * t4));
  cb.add(kABC5, -(es * p.dsM));
  M_b -= es * c[kBC5] * p.cM;
  const double dMa_b = M_b - w_b;
  cb.add(kAArgpcof, dMa_b * t);
  cb.add(kAMcof, dMa_b * p.x3);
  const double dm = dMa_b * c[kMcof];
  cb.add(kADM0, -(dm));
  const double x_b = 3.0 * dm * p.x * p.x;
  cb.add(kAEta, x_b * p.cMdf);
  M_b -= x_b * c[kEta] * p.sMdf;
  cb.add(kAM0, M_b);
  cb.add(kAMdot, M_b * t);
  cb.add(kAArgp0, w_b);
  cb.add(kAArgpdot, w_b * t);
  cb.add(kANode0, nb);
  cb.add(kANodedot, nb * t);
  cb.add(kANodecf, nb * t2);
}

// -------------------------------------------------------------- Jacobian --
// The secular values of a point that only the elements' tangents need, set
// aside in LDS (a column per lane, [kNParked64][64] per wavefront) while
// Kepler's equation and the columns take the registers.
constexpr int kNParked64 = 14;
__device__ __forceinline__ void park(double* col, const Point64& p) {
  const double x[kNParked64] = {p.t, p.cMdf, p.sMdf, p.x, p.x3, p.cM, p.dsM, p.A, p.Ld, p.e, p.om0, p.sw, p.cw, p.tau};
#pragma unroll
  for (int k = 0; k < kNParked64; ++k) col[64 * k] = x[k];
}
__device__ __forceinline__ void unpark(const double* col, Point64& p) {
  double* const x[kNParked64] = {&p.t, &p.cMdf, &p.sMdf, &p.x, &p.x3, &p.cM, &p.dsM, &p.A, &p.Ld, &p.e, &p.om0, &p.sw,
                                 &p.cw, &p.tau};
#pragma unroll
  for (int k = 0; k < kNParked64; ++k) *x[k] = col[64 * k];
}

// The state's derivative columns with respect to a, ax, ay, U, the inclination
// (where it enters by itself) and the node: d (r, v) / d each, km and km/s.
enum Col64 : int { kColA, kColAx, kColAy, kColU, kColI, kColNode, kNCol64 };
struct Columns64 {
  double d[kNCol64][6];
};

__device__ __forceinline__ void point64_columns(const double* c, const Grav& g, const Point64& p, Columns64& o) {
  const double wx = p.snod * p.sinc, wy = -p.cnod * p.sinc;
  const double xmx = -p.snod * p.cinc, xmy = p.cnod * p.cinc;
  const double U[3] = {xmx * p.ssu + p.cnod * p.csu, xmy * p.ssu + p.snod * p.csu, p.sinc * p.ssu};
  const double V[3] = {xmx * p.csu - p.cnod * p.ssu, xmy * p.csu - p.snod * p.ssu, p.sinc * p.csu};
  const double W[3] = {wx, wy, p.cinc};
  const double rr = g.radius * p.mrt;
  // tangents of the polar quantities to a column of the state
  auto column = [&](int k, double dm, double du, double dn, double di, double dv, double dw) {
    const double al = du + p.cinc * dn, sn = p.sinc * dn;
    const double be = p.ssu * di - p.csu * sn, ga = p.csu * di + p.ssu * sn;
    const double r0 = g.radius * dm, r1 = rr * al, r2 = rr * be;
    const double v0 = g.vkms * (dv - p.rvdot * al), v1 = g.vkms * (dw + p.mvt * al);
    const double v2 = g.vkms * (p.mvt * be + p.rvdot * ga);
#pragma unroll
    for (int q = 0; q < 3; ++q) {
      o.d[k][q] = r0 * U[q] + r1 * V[q] + r2 * W[q];
      o.d[k][3 + q] = v0 * U[q] + v1 * V[q] + v2 * W[q];
    }
  };
  // the node turns the state about the pole
  {
    const double x = rr * U[0], y = rr * U[1];
    const double vx = g.vkms * (p.mvt * U[0] + p.rvdot * V[0]), vy = g.vkms * (p.mvt * U[1] + p.rvdot * V[1]);
    o.d[kColNode][0] = -y;
    o.d[kColNode][1] = x;
    o.d[kColNode][2] = 0.0;
    o.d[kColNode][3] = -vy;
    o.d[kColNode][4] = vx;
    o.d[kColNode][5] = 0.0;
  }
  const double x1 = c[kX1], x7 = c[kX7], ci = c[kCosi], si = c[kSini], c41h = 1.5 * c[kC41], cs = ci * si;
  column(kColI, cs * (9.0 * p.rl * p.k2 * p.betal + p.k1 * p.c2), 3.5 * cs * p.k2 * p.s2, -1.5 * si * p.k2 * p.s2,
         1.0 + 1.5 * p.k2 * p.c2 * (ci * ci - si * si), -2.0 * cs * p.qk * p.s2, cs * p.qk * (2.0 * p.c2 - 9.0));
  // partial derivatives with respect to u, p_L (over p_L), r_l, beta and e sin E
  const double nk3 = 3.0 * ci * p.k2, ik3 = nk3 * si, xk = p.qk * x1, q2 = 2.0 * xk;
  const double m_u = -p.k1 * x1 * p.s2, u_u = 1.0 - 0.5 * x7 * p.k2 * p.c2, n_u = nk3 * p.c2, i_u = -ik3 * p.s2;
  const double v_u = -q2 * p.c2, w_u = -q2 * p.s2;
  const double mb = p.rl * c41h * p.k2;
  const double m_p = p.ipl * (2.0 * mb * p.betal - 0.5 * x1 * p.c2 * p.k1), u_p = p.ipl * (0.5 * x7 * p.k2 * p.s2);
  const double n_p = -p.ipl * nk3 * p.s2, i_p = -p.ipl * ik3 * p.c2, v_p = p.ipl * xk * p.s2, w_p = -p.ipl * p.qk * p.g1;
  const double v_r = -p.rdotl * p.irl, w_r = -p.rvdotl * p.irl;
  {
    const double D = 1.0 - p.ecE;
    column(kColA, p.bk * D + m_p * p.om, u_p * p.om, n_p * p.om, i_p * p.om,
           p.ia * (0.5 * p.rdotl + 1.5 * xk * p.s2) + v_r * D + v_p * p.om,
           p.ia * (0.5 * p.rvdotl - 1.5 * p.qk * p.g1) + w_r * D + w_p * p.om);
  }
  double u_x, u_y;
  u_partials(p, &u_x, &u_y);
  // psi's column scaled by d psi = (dU + sin psi dax - cos psi day) / D, and
  // the changes at fixed psi
  const double bi = p.betal * p.iD * p.iD;
  auto plane = [&](int k, double dpsi, double drl, double desE, double dbeta, double dpl, double du) {
    const double r = p.a * (p.esE * p.iD * dpsi + drl), es = p.sr * (p.ecE * p.iD * dpsi + desE), u = bi * dpsi + du;
    column(k, p.bk * r - mb * dbeta + m_p * dpl + m_u * u, u_u * u + u_p * dpl, n_u * u + n_p * dpl, i_u * u + i_p * dpl,
           v_r * r + es + v_p * dpl + v_u * u, w_r * r + p.sr * dbeta + w_p * dpl + w_u * u);
  };
  plane(kColU, 1.0, 0.0, 0.0, 0.0, 0.0, 0.0);
  plane(kColAx, p.sp, -p.cp, p.sp, -p.ax * p.ibeta, -2.0 * p.a * p.ax, u_x);
  plane(kColAy, -p.cp, -p.sp, -p.cp, -p.ay * p.ibeta, -2.0 * p.a * p.ay, u_y);
}

// Element m's tangent of the state (m as the element rows: n, e, i, node, argp,
// M, B*); dc: the record's derivatives with respect to it.
__device__ __forceinline__ void element_tangent(int m, const double* dc, const double* c, const Point64& p,
                                                const Columns64& col, double d[6]) {
  if (m == 3) {  // the node at epoch turns the state, nothing else
#pragma unroll
    for (int q = 0; q < 6; ++q) d[q] = col.d[kColNode][q];
    return;
  }
  const double t = p.t;
  // argp at epoch enters the drag terms only through C4 and C3, M at epoch only
  // through the terms at epoch: their other derivatives are zero
  const bool all = m != 4 && m != 5;
  const double Mdf_t = all ? fma(dc[kMdot], t, dc[kM0]) : m == 5 ? 1.0 : 0.0;
  double dMa_t = 0.0;
  if (m != 5) dMa_t = dc[kArgpcof] * t;
  if (m != 4) {
    const double x_t = all ? dc[kEta] * p.cMdf - c[kEta] * p.sMdf * Mdf_t : -c[kEta] * p.sMdf;
    dMa_t += c[kMcof] * (3.0 * p.x * p.x * x_t - dc[kDM0]);
    if (all) dMa_t += dc[kMcof] * p.x3;
  }
  const double M_t = Mdf_t + dMa_t;
  const double w_t = (m == 4 ? 1.0 : all ? dc[kArgpdot] * t : 0.0) - dMa_t;
  double e_t = -c[kBC5] * (p.cM * M_t - (m == 4 ? 0.0 : dc[kSinM0]));
  if (m != 5) e_t -= dc[kBC4] * t;
  if (all) e_t += dc[kE0] - dc[kBC5] * p.dsM;
  double a_t = 0.0, L_t = M_t + w_t;
  if (all) {
    const double A_t = -t * fma(t, fma(t, fma(t, dc[kD4], dc[kD3]), dc[kD2]), dc[kC1]);
    a_t = p.A * (dc[kA0pp] * p.A + 2.0 * c[kA0pp] * A_t);
    const double Ld_t = t * t * fma(t, fma(t, fma(t, dc[kT5cof], dc[kT4cof]), dc[kT3cof]), dc[kT2cof]);
    L_t += dc[kN0pp] * p.Ld + c[kN0pp] * Ld_t;
  }
  if (p.clamped) e_t = 0.0;
  // long-period terms
  const double tau_t = p.tau * p.tau * (2.0 * p.a * p.e * e_t - p.om0 * a_t);
  const double ax_t = p.cw * e_t - p.e * p.sw * w_t;
  double ay_t = p.sw * e_t + p.e * p.cw * w_t + c[kAycof] * tau_t;
  double U_t = L_t + c[kLcof] * (p.ax * tau_t + p.tau * ax_t);
  if (m == 2) {
    ay_t += p.tau * c[kAycofI];
    U_t += p.tau * p.ax * c[kLcofI];
  }
#pragma unroll
  for (int q = 0; q < 6; ++q) {
    d[q] = ax_t * col.d[kColAx][q] + ay_t * col.d[kColAy][q] + U_t * col.d[kColU][q];
    if (all) d[q] += a_t * col.d[kColA][q];
    if (m == 2) d[q] += col.d[kColI][q];
  }
  if (all) {
    const double node_t = t * fma(t, dc[kNodecf], dc[kNodedot]);
#pragma unroll
    for (int q = 0; q < 6; ++q)
      if (q != 2 && q != 5) d[q] += node_t * col.d[kColNode][q];
  }
}

}  // namespace sgp4mi
