// dcf_common.hpp -- device-side data structures and the per-face numerics of
// the finite-volume compressible Navier-Stokes right-hand side (gfx950, FP64).
//
// Paper correspondence:
//   conserved vector and total energy ............ Section 2.1, Eq. (2)
//   convective fluxes F^c, G^c, H^c ................ Eq. (3)
//   dissipative fluxes (stress, heat flux) ......... Eqs. (4)-(5), Fourier law
//   semi-discrete update with cell widths .......... Eq. (6)
//   WENO-type reconstruction + HLLC Riemann solver . Section 2.1 / Section 3.1
//   halo-cell boundary conditions .................. Section 3.2
// Schemes named but not written out in the paper use their published
// definitions: WENO5-JS (Jiang & Shu 1996, eps = 1e-6, power 2), HLLC
// (Toro, Spruce & Speares 1994) with Davis wave speeds, 4th-order central
// differences for the dissipative fluxes, and three-stage TVD Runge-Kutta
// (Shu & Osher 1988).
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

namespace dcf {

constexpr int NH = 3;  // halo layers per active axis (Section 2.2)

enum : int {
  BC_PERIODIC = 0, BC_WALL = 1, BC_POROUS = 2, BC_ZEROGRAD = 3, BC_DIRICHLET = 4, BC_DISTURB = 5
};
__host__ __device__ __forceinline__ bool is_wall(int k) {
  return k == BC_WALL || k == BC_POROUS || k == BC_DISTURB;
}
enum : int { VISC_NONE = 0, VISC_POWER = 1, VISC_SUTHERLAND = 2 };
enum : int { SRC_NONE = 0, SRC_MASSFLUX = 1 };
enum : int { SCHEME_WENO5 = 0, SCHEME_TENO6A = 1 };
enum : int { QR = 0, QU = 1, QV = 2, QW = 3, QP = 4, QT = 5, QMU = 6, NQ = 7 };

// Everything a kernel needs about one solve, passed by value.
struct Dev {
  int ndim, nv;
  int n[3], h[3], N[3];  // interior cells, halo layers, box cells per axis
  int ho[3];             // array index of interior cell 0 along each axis
  long ncell, nbox;      // interior cells; box cells (N0 N1 N2)
  long nboxp;            // elements of one box array (rows padded to 16 doubles)
  long sb[3];            // box strides per axis
  // grid metrics per axis (device arrays): widths, 1/width, dxi/dx at
  // centres (n) and at faces (n+1)
  const double *dx[3], *idx[3], *mc[3], *mf[3];
  const double *xm[3];   // cell-centre coordinates (midpoint of the two faces)
  double Lx;             // the x cell widths summed in index order (an x line's length)
  double vol;            // product of the axes' lengths, each summed so
  // gas
  double gamma, R, Pr, cp, mu_ref, T_ref, vparam;
  double gm1i, cpPr;     // 1/(gamma - 1) and cp/Pr
  double iR, iTref;      // 1/R and 1/T_ref
  int visc;
  // boundaries
  int bck[6];
  double Tw[6];          // wall temperature; 0 = adiabatic wall
  int doff[6];           // disturbance wall: offset of (A, kappa) in K, else -1
  const double *dir[6];
  int pface, pb, pe;
  double pinf;
  const double *K;       // boundary parameters: porous K_i, then (A, kappa) per disturbance face
  int source;
  // workspace
  double *Q[NQ];         // primitive box arrays
  double *F[3];          // face fluxes per direction, 5 components each
  long fcount[3];        // faces per direction (component stride of F)
  int fn[3][3];          // face-array extents per direction
  unsigned *flags;
  int scheme;            // SCHEME_WENO5 or SCHEME_TENO6A (face reconstruction and
                         // order of the central dissipative stencils)
};

// Primitive box arrays a kernel writes besides its main output (null Q[0]:
// none).
struct BoxOut {
  double *Q[NQ] = {};
};

__device__ __forceinline__ bool finite_pos(double x) { return x > 0.0 && x < 1.0e300; }

// Box arrays: interior cell 0 of each row sits on a 128-byte boundary (x
// offset 16 doubles, row pitch a multiple of 16), so tiles of 16 cells along
// x load whole cache lines.
__host__ __device__ __forceinline__ long bidx(const Dev &g, int i, int j, int k) {
  return (long)(k + g.ho[2]) * g.sb[2] + (long)(j + g.ho[1]) * g.sb[1] + (i + g.ho[0]);
}

// Box position of ghost cell number gi (ghost cells enumerated z-plane by
// z-plane: whole halo planes, then per interior plane its halo rows and the
// 2 h0 x-halo cells of each interior row).
__host__ __device__ __forceinline__ void ghost_position(const Dev &g, unsigned gi, int p[3]) {
  const unsigned N0 = g.N[0], h0 = g.h[0], h1 = g.h[1], h2 = g.h[2];
  const unsigned n0 = g.n[0], n1 = g.n[1], n2 = g.n[2];
  const unsigned plane = N0 * (unsigned)g.N[1];
  const unsigned lowz = h2 * plane, inner = plane - n0 * n1;
  unsigned x, y, z;
  if (gi < lowz || gi >= lowz + n2 * inner) {  // a whole halo plane
    const unsigned r0 = gi < lowz ? gi : gi - n2 * inner;
    z = r0 / plane;
    if (gi >= lowz) z += n2;
    const unsigned r = r0 % plane;
    y = r / N0;
    x = r % N0;
  } else {
    const unsigned r0 = gi - lowz;
    z = h2 + r0 / inner;
    unsigned r = r0 % inner;
    const unsigned lowy = h1 * N0, mid = 2u * h0;
    if (r < lowy) {
      y = r / N0;
      x = r % N0;
    } else if (r < lowy + n1 * mid) {
      r -= lowy;
      y = h1 + r / mid;
      const unsigned m = r % mid;
      x = m < h0 ? m : n0 + m;
    } else {
      r -= lowy + n1 * mid;
      y = h1 + n1 + r / N0;
      x = r % N0;
    }
  }
  p[0] = (int)x - g.h[0];
  p[1] = (int)y - g.h[1];
  p[2] = (int)z - g.h[2];
}

// Reciprocal from the hardware estimate refined by two Newton-Raphson steps
// e = 1 - x r, r <- r + r e (each squares the relative error): within about
// an ulp of 1/x for normal x, at half the instructions of an IEEE division.
// Zero or non-finite x gives a non-finite result.
__device__ __forceinline__ double rcp_nr(double x) {
  double r = __builtin_amdgcn_rcp(x);
  double e = fma(-x, r, 1.0);
  r = fma(r, e, r);
  e = fma(-x, r, 1.0);
  return fma(r, e, r);
}

// 1/sqrt(x) for normal x > 0, likewise: the hardware estimate and two Newton
// steps y <- y + y (1 - x y^2) / 2.  Negative x gives NaN.
__device__ __forceinline__ double rsq_nr(double x) {
  const double hx = 0.5 * x;
  double y = __builtin_amdgcn_rsq(x);
  y = fma(y, fma(-hx * y, y, 0.5), y);
  return fma(y, fma(-hx * y, y, 0.5), y);
}

// Sound speed c = sqrt(gamma p / rho), written gamma p y with
// y = 1 / sqrt(gamma p rho) = 1 / (rho c) so that it needs no division.
__device__ __forceinline__ double sound_speed(double gamma, double rho, double p, double &y) {
  const double gp = gamma * p;
  y = rsq_nr(gp * rho);
  return gp * y;
}
__device__ __forceinline__ double sound_speed(double gamma, double rho, double p) {
  double y;
  return sound_speed(gamma, rho, p, y);
}

// x^w for x > 0 (else NaN) as exp(w log x), for results within the normal
// range: with x = m 2^e, m in [sqrt(1/2), sqrt(2)), and s = (m - 1)/(m + 1),
// log m = 2 atanh s = 2 s sum_k s^{2k} / (2k + 1), |s| < 0.1716; and exp as 2^n
// times the Taylor series of the remainder, |r| <= log(2)/2.  Both series are cut
// below 3e-17 of their sum; what the leading terms of w log x and of the last sum
// lose to rounding is carried in a second word.  Error of x^0.7 in ulp, largest
// and rms: 0.8 and 0.29 over x in [1/2, 2] and over [0.05, 20] (exp and log of
// the math library 1.0 and 0.31, 2.9 and 0.50), at 113 instead of 150
// instructions.
__device__ __forceinline__ double pow_positive(double x, double w) {
  double m = __builtin_amdgcn_frexp_mant(x);  // [1/2, 1)
  int e = __builtin_amdgcn_frexp_exp(x);
  const bool low = m < 0.70710678118654752;
  m = low ? m + m : m;
  e = low ? e - 1 : e;
  const double ln2 = 0.69314718055994531, ln2lo = 2.3190468138462996e-17;
  const double a = m - 1.0, b = m + 1.0, rb = rcp_nr(b);
  const double s = a * rb, z = s * s, s2 = s + s;
  double t = 1.0 / 19.0;
  t = fma(t, z, 1.0 / 17.0);
  t = fma(t, z, 1.0 / 15.0);
  t = fma(t, z, 1.0 / 13.0);
  t = fma(t, z, 1.0 / 11.0);
  t = fma(t, z, 1.0 / 9.0);
  t = fma(t, z, 1.0 / 7.0);
  t = fma(t, z, 1.0 / 5.0);
  t = fma(t, z, 1.0 / 3.0);
  // log x = h + s2 + small; |h| >= |s2| or h = 0
  const double de = (double)e, h = de * ln2;
  const double small = fma(s2 * z, t, fma(fma(-s, b, a), rb + rb, fma(de, ln2, -h) + de * ln2lo));
  const double l = h + s2, llo = ((h - l) + s2) + small;
  const double y = w * l, ylo = fma(w, l, -y) + w * llo;
  const double n = __builtin_rint(y * 1.4426950408889634);
  const double r0 = fma(n, -ln2, y), rlo = fma(n, -ln2lo, ylo), r = r0 + rlo;
  double p = 1.0 / 6227020800.0;
  p = fma(p, r, 1.0 / 479001600.0);
  p = fma(p, r, 1.0 / 39916800.0);
  p = fma(p, r, 1.0 / 3628800.0);
  p = fma(p, r, 1.0 / 362880.0);
  p = fma(p, r, 1.0 / 40320.0);
  p = fma(p, r, 1.0 / 5040.0);
  p = fma(p, r, 1.0 / 720.0);
  p = fma(p, r, 1.0 / 120.0);
  p = fma(p, r, 1.0 / 24.0);
  p = fma(p, r, 1.0 / 6.0);
  p = fma(p, r, 0.5);
  // 1 + r0 and what it loses to rounding, so that the last sum alone rounds
  const double hi = 1.0 + r0, lo = (1.0 - hi) + r0;
  p = hi + fma(r * r, p, lo + rlo);
  p = __builtin_amdgcn_ldexp(p, (int)n);
  return x > 0.0 ? p : __builtin_nan("");
}

// Dynamic viscosity: power law, or Sutherland's law (Section 3.2).
__device__ __forceinline__ double viscosity(const Dev &g, double T, int law) {
  if (law == VISC_POWER) return g.mu_ref * pow_positive(T * g.iTref, g.vparam);
  if (law == VISC_SUTHERLAND) {
    // t^{3/2} (1 + s) / (t + s) with t^{3/2} = t^2 / sqrt(t)
    double t = T * g.iTref;
    double s = g.vparam * g.iTref;
    return g.mu_ref * (1.0 + s) * (t * t * rsq_nr(t)) * rcp_nr(t + s);
  }
  return 0.0;
}

__device__ __forceinline__ double viscosity(const Dev &g, double T) {
  return viscosity(g, T, g.visc);
}

// WENO5-JS (Section 2.1): both reconstructions at the face between v2 and
// v3, left-biased from v0..v4 and right-biased from v5..v1.  The nonlinear
// weights d_k / (eps + beta_k)^2 are normalised after multiplying through by
// the product of the three denominators, and the two values share one
// reciprocal: y_L = N_L D_R r, y_R = N_R D_L r with r = 1 / (6 D_L D_R)
// (the candidates are kept at six times the third-order reconstructions).
// The mirrored stencils share work: the left stencils (1..3) and (2..4) are
// the right stencils (3..1) and (4..2), with the same second differences, and
// the left candidates 1 and 2 equal the right candidates 2 and 1.
__device__ __forceinline__ void weno5_pair(double v0, double v1, double v2, double v3, double v4,
                                           double v5, double &yl, double &yr) {
  const double eps = 1.0e-6;
  const double c1312 = 13.0 / 12.0;
  // first differences over the faces, second differences over cells (0,1,2),
  // (1,2,3), (2,3,4), (3,4,5)
  const double e0 = v1 - v0, e1 = v2 - v1, e2 = v3 - v2, e3 = v4 - v3, e4 = v5 - v4;
  const double d0 = e1 - e0, d1 = e2 - e1, d2 = e3 - e2, d3 = e4 - e3;
  // candidates as six times their offset from the own cell's value (v2 on the
  // left, v3 on the right)
  const double al0 = fma(5.0, e1, -2.0 * e0), al1 = fma(2.0, e2, e1), al2 = fma(4.0, e2, -e3);
  const double ar0 = fma(-5.0, e3, 2.0 * e4), ar1 = fma(-2.0, e2, -e3), ar2 = fma(-4.0, e2, e1);
  // first-derivative terms of the smoothness indicators, per side
  const double sl0 = fma(3.0, e1, -e0), sl1 = e1 + e2, sl2 = fma(-3.0, e2, e3);
  const double sr0 = fma(-3.0, e3, e4), sr1 = e2 + e3, sr2 = fma(3.0, e2, -e1);
  // u_k = (eps + beta_k)^2 / d_k, the square of (eps + beta_k) / sqrt(d_k)
  // with 1 / sqrt(d_k) folded into the constants (d = 0.1, 0.6, 0.3); the
  // weights d_k / (eps + beta_k)^2 times the product of all three
  // denominators are then the products of the other two u (the common
  // factor d_0 d_1 d_2 cancels in the normalisation)
  constexpr double is1 = 3.162277660168379, is6 = 1.2909944487358056,
                   is3 = 1.8257418583505538;  // 1 / sqrt(d_k)
  const double r0 = d0 * d0, r1 = d1 * d1, r2 = d2 * d2, r3 = d3 * d3;
  auto usq = [&](double r, double s, double sc) {
    const double t = fma(c1312 * sc, r, fma(0.25 * sc, s * s, eps * sc));
    return t * t;
  };
  const double ul0 = usq(r0, sl0, is1), ul1 = usq(r1, sl1, is6), ul2 = usq(r2, sl2, is3);
  const double ur0 = usq(r3, sr0, is1), ur1 = usq(r2, sr1, is6), ur2 = usq(r1, sr2, is3);
  const double wl0 = ul1 * ul2, wl1 = ul0 * ul2, wl2 = ul0 * ul1;
  const double wr0 = ur1 * ur2, wr1 = ur0 * ur2, wr2 = ur0 * ur1;
  const double nl = wl0 * al0 + wl1 * al1 + wl2 * al2, dl = wl0 + wl1 + wl2;
  const double nr = wr0 * ar0 + wr1 * ar1 + wr2 * ar2, dr = wr0 + wr1 + wr2;
  const double r = rcp_nr(6.0 * dl * dr);
  yl = fma(nl * dr, r, v2);
  yr = fma(nr * dl, r, v3);
}

// The side whose state a face takes (0 <= SL: left; SR < 0: right; else left
// where 0 <= S*), and whether its wave term counts (SL < 0 <= SR): on the sign
// bits, as none of the three speeds is -0 (192 x 128 x 128: 0.2 % over a selection
// by S* alone, 0.7 % with S* clamped to [SL, SR]).
__device__ __forceinline__ bool hllc_left(double SL, double Ss, double SR) {
  return (__double2hiint(SL) & (__double2hiint(SR) | __double2hiint(Ss))) >= 0;
}
__device__ __forceinline__ bool hllc_subsonic(double SL, double SR) {
  return (__double2hiint(SL) & ~__double2hiint(SR)) < 0;
}

// HLLC flux in the face frame.  q = (rho, u_n, u_t1, u_t2, p) on each side;
// F = (mass, normal momentum, t1 momentum, t2 momentum, energy).  Ties at
// 0 <= S select the left-side state.  Star state written with one
// reciprocal r = 1/(S_K - S*):
//   U*_K = r [rho (S-u), rho (S-u) S*, rho (S-u) v, rho (S-u) w,
//             E (S-u) + (S*-u)(rho (S-u) S* + p)].
__device__ __forceinline__ void hllc(const double *qL, const double *qR, double gamma,
                                     double gm1i, double *F) {
  double rL = qL[0], uL = qL[1], vL = qL[2], wL = qL[3], pL = qL[4];
  double rR = qR[0], uR = qR[1], vR = qR[2], wR = qR[3], pR = qR[4];
  double cL = sound_speed(gamma, rL, pL);
  double cR = sound_speed(gamma, rR, pR);
  double SL = fmin(uL - cL, uR - cR);
  double SR = fmax(uL + cL, uR + cR);
  double mL = rL * (SL - uL), mR = rR * (SR - uR);
  double Ss = fma(pR - pL + uL * mL - uR * mR, rcp_nr(mL - mR), 0.0);  // (+0, not -0)
  // On a supersonic face the upwind side's wave term vanishes, F = F(U_K), also
  // where S* points the other way: where a reconstructed pressure is not
  // positive its sound speed is NaN, fmin and fmax leave that side out, and S*
  // need not lie between SL and SR (selections only: a branch would end the
  // block in which this arithmetic and the reconstructions hide each other's
  // latencies).
  const bool left = hllc_left(SL, Ss, SR);
  const double SLm = fmin(SL, 0.0), SRp = fmax(SR, 0.0);
  double r = left ? rL : rR, u = left ? uL : uR, v = left ? vL : vR, w = left ? wL : wR;
  double p = left ? pL : pR, S = left ? SL : SR, m = left ? mL : mR;
  const double Sw = left ? SLm : SRp;
  double E = p * gm1i + 0.5 * r * (u * u + v * v + w * w);
  double inv = rcp_nr(S - Ss);
  double Us0 = m * inv;
  double Us4 = (E * (S - u) + (Ss - u) * (m * Ss + p)) * inv;
  double fm = r * u;
  F[0] = fm + Sw * (Us0 - r);
  F[1] = fm * u + p + Sw * (Us0 * Ss - fm);
  F[2] = F[0] * v;  // the star state keeps the side's tangential velocities
  F[3] = F[0] * w;
  F[4] = u * (E + p) + Sw * (Us4 - E);
}

// TENO6-A (Fu, Hu & Adams: targeted ENO, six points, adaptive dissipation):
// both reconstructions at the face between v2 and v3, the left one centred on
// v2 (cells v0 .. v5) and the right one its mirror image centred on v3 (cells
// v5 .. v0).  Per side, with (a .. f) the six cells and c the centre:
// third-order candidates on (b c d), (c d e) and (a b c) and a fourth-order
// one on (c d e f), sixth-order linear weights (0.45, 0.3, 0.05, 0.2); the
// Jiang-Shu indicators of the candidates and of the six-point polynomial
// (integrals over the centre cell) give tau6 = |b6 - (b0 + b2 + 4 b1) / 6|
// and the measures gamma_k = (1 + tau6 / (b_k + 1e-40))^6; a candidate whose
// share gamma_k / sum gamma is below the cut-off C_T is dropped (tested as
// gamma_k < C_T sum gamma), the kept ones are combined with their linear
// weights renormalised.
// C_T = 10^-floor(10.5 - 3.5 (1 - (1-m)^4 (1+4m))), m = 1 - min(1, eta/0.17),
// eta the smallest of Ren's measures (|2 a b| + e) / (a^2 + b^2 + e) over the
// neighbouring differences (a, b) of the four inner cells,
// e = 0.9 * 0.17 * (1e-3)^2 / (1 - 0.9 * 0.17); the mirrored differences give
// the same measures, so C_T is shared by both sides.  Reciprocals are the
// refined hardware ones (no IEEE division), one for the least ratio, one for a
// side's four measures and one for both values: 5 per component where each
// quotient had its own, 14.
// The flux launches are bound by the issue of this arithmetic (VALU busy 87 % in
// the x + y launch, 80 % in z + update: 192 x 128 x 128, 489 and 320 us): x + y
// faces of 256 x 128 x 128 in 638 us, 748 with the 14 reciprocals and 115 VGPRs
// (4 wavefronts per SIMD; 95 and 5 now), z faces + update 422 and 473.
__device__ __forceinline__ void teno6a_pair(double v0, double v1, double v2, double v3, double v4,
                                            double v5, double &yl, double &yr) {
  constexpr double c1312 = 13.0 / 12.0;
  // first differences over the faces, second differences over the cells
  const double e0 = v1 - v0, e1 = v2 - v1, e2 = v3 - v2, e3 = v4 - v3, e4 = v5 - v4;
  double ct;
  {
    const double Cr = 0.17, xi = 1.0e-3;
    const double ee = 0.9 * Cr * xi * xi / (1.0 - 0.9 * Cr);
    // the least of four ratios n_k / d_k, compared over common denominators:
    // one reciprocal
    const double f0 = e0 * e0, f1 = e1 * e1, f2 = e2 * e2, f3 = e3 * e3, f4 = e4 * e4;
    const double n0 = fabs(2.0 * e1 * e0) + ee, n1 = fabs(2.0 * e2 * e1) + ee;
    const double n2 = fabs(2.0 * e3 * e2) + ee, n3 = fabs(2.0 * e4 * e3) + ee;
    const double g0 = f1 + (f0 + ee), g1 = f2 + (f1 + ee), g2 = f3 + (f2 + ee),
                 g3 = f4 + (f3 + ee);
    const double na = fmin(n0 * g1, n1 * g0), ga = g0 * g1;
    const double nb = fmin(n2 * g3, n3 * g2), gb = g2 * g3;
    const double eta = fmin(na * gb, nb * ga) * rcp_nr(ga * gb);
    const double m = 1.0 - fmin(1.0, eta * (1.0 / Cr));
    const double om = 1.0 - m, om2 = om * om;
    const double bbar = 10.5 - 3.5 * (1.0 - om2 * om2 * (1.0 + 4.0 * m));
    ct = bbar >= 8.0 ? 1.0e-8 : 1.0e-7;
    ct = bbar >= 9.0 ? 1.0e-9 : ct;
    ct = bbar >= 10.0 ? 1.0e-10 : ct;
  }
  const double d0 = e1 - e0, d1 = e2 - e1, d2 = e3 - e2, d3 = e4 - e3;
  const double r0 = c1312 * (d0 * d0), r1 = c1312 * (d1 * d1), r2 = c1312 * (d2 * d2),
               r3 = c1312 * (d3 * d3);
  // One side, cells a .. f along its own direction, differences ea = b - a ..
  // ef = f - e, ra, rb, rc = 13/12 (second difference)^2 of (a b c), (b c d),
  // (c d e): six times the offset's numerator over the sum of the kept weights.
  // (b3 and b6 stay forms in the cell values: where the data are uniform to
  // rounding their own rounding decides the cut-off, and there the selection is
  // to stay as it is defined by these forms.)
  auto side = [ct](double a, double b, double c, double d, double e, double f, double ea,
                   double eb, double ec, double ed, double ef, double ra, double rb, double rc,
                   double &N, double &W) {
    const double t0 = eb + ec, t1 = fma(-3.0, ec, ed), t2 = fma(3.0, eb, -ea);
    const double b0 = fma(0.25 * t0, t0, rb);
    const double b1 = fma(0.25 * t1, t1, rc);
    const double b2 = fma(0.25 * t2, t2, ra);
    const double b3 = (c * (2107.0 * c - 9402.0 * d + 7042.0 * e - 1854.0 * f) +
                       d * (11003.0 * d - 17246.0 * e + 4642.0 * f) +
                       e * (7043.0 * e - 3882.0 * f) + 547.0 * f * f) * (1.0 / 240.0);
    const double b6 =
        (a * (271779.0 * a - 2380800.0 * b + 4086352.0 * c - 3462252.0 * d + 1458762.0 * e -
              245620.0 * f) +
         b * (5653317.0 * b - 20427884.0 * c + 17905032.0 * d - 7727988.0 * e +
              1325006.0 * f) +
         c * (19510972.0 * c - 35817664.0 * d + 15929912.0 * e - 2792660.0 * f) +
         d * (17195652.0 * d - 15880404.0 * e + 2863984.0 * f) +
         e * (3824847.0 * e - 1429976.0 * f) + 139633.0 * f * f) * (1.0 / 120960.0);
    const double tau = fabs(b6 - (b0 + b2 + 4.0 * b1) * (1.0 / 6.0));
    // (1 + tau / beta)^6: the four reciprocals from one
    const double h0 = b0 + 1.0e-40, h1 = b1 + 1.0e-40, h2 = b2 + 1.0e-40, h3 = b3 + 1.0e-40;
    const double h01 = h0 * h1, h23 = h2 * h3;
    const double R = tau * rcp_nr(h01 * h23);
    const double R01 = R * h23, R23 = R * h01;
    auto gam = [](double x, double y) {
      const double r = fma(x, y, 1.0), rr = r * r;
      return rr * rr * rr;
    };
    const double g0 = gam(R01, h1), g1 = gam(R01, h0), g2 = gam(R23, h3), g3 = gam(R23, h2);
    const double lim = ct * (g0 + g1 + g2 + g3);
    const double w0 = g0 < lim ? 0.0 : 0.45, w1 = g1 < lim ? 0.0 : 0.3;
    const double w2 = g2 < lim ? 0.0 : 0.05, w3 = g3 < lim ? 0.0 : 0.2;
    // candidates: (b c d), (c d e), (a b c), (c d e f)
    const double q0 = fma(2.0, ec, eb), q1 = fma(4.0, ec, -ed), q2 = fma(5.0, eb, -2.0 * ea);
    const double q3 = fma(4.5, ec, fma(0.5, ef, -2.0 * ed));
    N = w0 * q0 + w1 * q1 + w2 * q2 + w3 * q3;
    W = w0 + w1 + w2 + w3;
  };
  double Nl, Wl, Nr, Wr;
  // (the sides one after the other, and evaluated here: interleaved, or sunk to
  // the flux with those of the other components, they take the registers of two
  // wavefronts per SIMD instead of four)
  asm volatile("" : "+v"(ct));
  side(v0, v1, v2, v3, v4, v5, e0, e1, e2, e3, e4, r0, r1, r2, Nl, Wl);
  asm volatile("" : "+v"(Nl), "+v"(Wl));
  __builtin_amdgcn_sched_barrier(0);
  side(v5, v4, v3, v2, v1, v0, -e4, -e3, -e2, -e1, -e0, r3, r2, r1, Nr, Wr);
  const double r = rcp_nr(6.0 * Wl * Wr);
  yl = fma(Nl * Wr, r, v2);
  yr = fma(Nr * Wl, r, v3);
  asm volatile("" : "+v"(yl), "+v"(yr));
  __builtin_amdgcn_sched_barrier(0);
}

// 6th-order central interpolation and derivatives in index space: face value
// and face derivative from the six cells around a face, cell derivative from
// three cells either side.
__device__ __forceinline__ double interp6(double a, double b, double c, double d, double e,
                                          double f) {
  return (150.0 * (c + d) - 25.0 * (b + e) + 3.0 * (a + f)) * (1.0 / 256.0);
}
__device__ __forceinline__ double dface6(double a, double b, double c, double d, double e,
                                         double f) {
  return (2250.0 * (d - c) - 125.0 * (e - b) + 9.0 * (f - a)) * (1.0 / 1920.0);
}
__device__ __forceinline__ double dcell6(double m3, double m2, double m1, double p1, double p2,
                                         double p3) {
  return (45.0 * (p1 - m1) - 9.0 * (p2 - m2) + (p3 - m3)) * (1.0 / 60.0);
}

// 4th-order central interpolation and derivatives in index space.
__device__ __forceinline__ double interp4(double a, double b, double c, double d) {
  return (9.0 * (b + c) - (a + d)) * (1.0 / 16.0);
}
__device__ __forceinline__ double dface4(double a, double b, double c, double d) {
  return (27.0 * (c - b) - (d - a)) * (1.0 / 24.0);
}
__device__ __forceinline__ double dcell4(double m2, double m1, double p1, double p2) {
  return (8.0 * (p1 - m1) - (p2 - m2)) * (1.0 / 12.0);
}

// Workgroups are dispatched round-robin over the 8 XCDs (each with its own
// L2).  This bijection of [0, nb) gives XCD x a contiguous range of logical
// tile indices, so neighbouring tiles that share halo cells meet in one L2.
__device__ __forceinline__ unsigned xcd_remap(unsigned L, unsigned nb) {
  const unsigned x = L % 8u, i = L / 8u, per = nb / 8u, rem = nb % 8u;
  return x < rem ? x * (per + 1u) + i : rem * (per + 1u) + (x - rem) * per + i;
}

// As xcd_remap, but spreading chunks of C consecutive logical tiles round
// robin over the XCDs (chunk k on XCD k mod 8): tiles of one chunk share an
// L2 while the work of any region is spread over all XCDs.  Blocks past the
// last whole round of 8 chunks keep their index.
__device__ __forceinline__ unsigned xcd_chunk_remap(unsigned P, unsigned nb, unsigned C) {
  const unsigned full = nb / (8u * C) * (8u * C);
  if (P >= full) return P;
  const unsigned x = P % 8u, i = P / 8u;
  return ((i / C) * 8u + x) * C + i % C;
}

__host__ __device__ __forceinline__ constexpr int tan1(int d) { return d == 0 ? 1 : 0; }
__host__ __device__ __forceinline__ constexpr int tan2(int d) { return d == 2 ? 1 : 2; }

}  // namespace dcf
