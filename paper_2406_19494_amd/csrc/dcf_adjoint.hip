// dcf_adjoint.hip -- hand-written reverse mode (VJP) of one TVD-RK3 step of
// the finite-volume right-hand side (Eq. (6)), through the halo-cell boundary
// conditions including the differentiable porous wall (Section 3.2), so that
// gradients of a cost along a trajectory reach the wall parameters (the
// end-to-end optimisation of Section 1).
//
// Per stage (state V, stage output W = a Un + b (V + dt R(V))), given the
// stage-output adjoint Wb:
//   Rb = b dt Wb,  Fb(face) = Rb(right cell)/dx - Rb(left cell)/dx (formed
//                  per face from Wb inside the flux adjoint kernels),
//   Qb = sum over faces of (dF/dQ)^T Fb        (convective + dissipative),
//   Qb += D_t^T Gb   (tangential derivatives were cell-centred, then
//                     interpolated: their adjoint Gb is gathered along t),
//   Tb += mu'(T) mub, then the halo fill is transposed (ghosts along two axes
//   into those along one, these into their sources and, for the walls'
//   parameters, into dJ/dK), and Vb = b Wb + (dQ/dU)^T Qb.
// Every scatter of the reverse pass is done as a deterministic gather: face
// adjoints are accumulated in LDS tiles offset by offset (one writer per
// cell per phase), and the tile only writes the cells all of whose faces it
// computed; no atomics anywhere, so results are bitwise reproducible.
#include "dcf_adjoint.hpp"
#include "dcf_cells.hpp"
#include "dcf_kernels.hpp"

namespace dcf {

// Tile shape of direction D for workgroups of NWV wavefronts (TF faces per line x
// TW lines): x-faces run along the lanes, a line per wavefront; y and z tiles take
// 8 neighbouring x-lines so that a cell row is read and written in 64-byte
// segments, 8 faces of them per wavefront.  A tile completes TF - 5 cells per
// line; the faces of the other 5 are computed twice.
template <int D, int NWV> struct TileShape {
  static constexpr int TF = D == 0 ? 64 : 8 * NWV;
  static constexpr int TW = D == 0 ? NWV : 8;
};

// ---------------------------------------------------------------------------
// Reverse of WENO5-JS at one face (the arithmetic of weno5_pair): the adjoints
// c[0..5] that the six cells v0..v5 receive from the adjoints ylb, yrb of the
// two reconstructed values.  Both sides share the differences; a side without
// adjoint (the downwind side of a supersonic face) is skipped.
// ---------------------------------------------------------------------------
// One side: a, s the candidates' offsets (times six) and first-derivative terms
// of its three stencils, d and r = d^2 their second differences; ab and sb
// receive the adjoints of a and (a quarter) of s, db / (13/3 / sqrt(d_k)) those
// of d.
__device__ __forceinline__ void weno5_side_vjp(const double *a, const double *s, const double *d,
                                               const double *r, double yb, double *ab, double *sb,
                                               double *db) {
  // t_k = (eps + beta_k) / sqrt(d_k), u_k = t_k^2, weights w_k = u_i u_j
  // (i, j != k), offset of the value N / (6 W)
  constexpr double eps = 1.0e-6, c1312 = 13.0 / 12.0;
  // 1 / sqrt(d_k), d = 0.1, 0.6, 0.3
  constexpr double sc[3] = {3.162277660168379, 1.2909944487358056, 1.8257418583505538};
  double h[3], t[3], u[3];
#pragma unroll
  for (int k = 0; k < 3; ++k) {
    h[k] = (0.25 * sc[k]) * s[k];
    t[k] = fma(c1312 * sc[k], r[k], fma(h[k], s[k], eps * sc[k]));
    u[k] = t[k] * t[k];
  }
  const double w0 = u[1] * u[2], w1 = u[0] * u[2], w2 = u[0] * u[1];
  const double iW = rcp_nr(w0 + w1 + w2);
  const double o = (w0 * a[0] + w1 * a[1] + w2 * a[2]) * iW;  // six times the offset
  const double nb = (yb * (1.0 / 6.0)) * iW;
  ab[0] = nb * w0;
  ab[1] = nb * w1;
  ab[2] = nb * w2;
  const double w0b = nb * (a[0] - o), w1b = nb * (a[1] - o), w2b = nb * (a[2] - o);
  const double ub[3] = {w1b * u[2] + w2b * u[1], w0b * u[2] + w2b * u[0],
                        w0b * u[1] + w1b * u[0]};
#pragma unroll
  for (int k = 0; k < 3; ++k) {
    const double tu = t[k] * ub[k];  // half of the adjoint of t_k
    sb[k] = h[k] * tu;
    db[k] = d[k] * tu;
  }
}

__device__ __forceinline__ void weno5_vjp(double v0, double v1, double v2, double v3, double v4,
                                          double v5, double ylb, double yrb, double *c) {
  const double e0 = v1 - v0, e1 = v2 - v1, e2 = v3 - v2, e3 = v4 - v3, e4 = v5 - v4;
  const double d0 = e1 - e0, d1 = e2 - e1, d2 = e3 - e2, d3 = e4 - e3;
  const double r0 = d0 * d0, r1 = d1 * d1, r2 = d2 * d2, r3 = d3 * d3;
  // adjoint of the second differences of stencil k: k4[k] db[k]
  constexpr double c13 = 13.0 / 3.0;
  constexpr double k4[3] = {c13 * 3.162277660168379, c13 * 1.2909944487358056,
                            c13 * 1.8257418583505538};
  double e0b = 0.0, e1b = 0.0, e2b = 0.0, e3b = 0.0, e4b = 0.0;
  double d0b = 0.0, d1b = 0.0, d2b = 0.0, d3b = 0.0;
  double ab[3], sb[3], db[3];
  if (ylb != 0.0) {
    const double a[3] = {fma(5.0, e1, -2.0 * e0), fma(2.0, e2, e1), fma(4.0, e2, -e3)};
    const double s[3] = {fma(3.0, e1, -e0), e1 + e2, fma(-3.0, e2, e3)};
    const double d[3] = {d0, d1, d2}, r[3] = {r0, r1, r2};
    weno5_side_vjp(a, s, d, r, ylb, ab, sb, db);
    e0b = -2.0 * ab[0] - 4.0 * sb[0];
    e1b = fma(5.0, ab[0], ab[1]) + fma(12.0, sb[0], 4.0 * sb[1]);
    e2b = fma(4.0, ab[2], 2.0 * ab[1]) + fma(-12.0, sb[2], 4.0 * sb[1]);
    e3b = fma(4.0, sb[2], -ab[2]);
    d0b = k4[0] * db[0];
    d1b = k4[1] * db[1];
    d2b = k4[2] * db[2];
  }
  if (yrb != 0.0) {
    const double a[3] = {fma(-5.0, e3, 2.0 * e4), fma(-2.0, e2, -e3), fma(-4.0, e2, e1)};
    const double s[3] = {fma(-3.0, e3, e4), e2 + e3, fma(3.0, e2, -e1)};
    const double d[3] = {d3, d2, d1}, r[3] = {r3, r2, r1};
    weno5_side_vjp(a, s, d, r, yrb, ab, sb, db);
    e4b = 2.0 * ab[0] + 4.0 * sb[0];
    e3b += fma(-5.0, ab[0], -ab[1]) + fma(-12.0, sb[0], 4.0 * sb[1]);
    e2b += fma(-4.0, ab[2], -2.0 * ab[1]) + fma(12.0, sb[2], 4.0 * sb[1]);
    e1b += fma(-4.0, sb[2], ab[2]);
    d3b = k4[0] * db[0];
    d2b = fma(k4[1], db[1], d2b);
    d1b = fma(k4[2], db[2], d1b);
  }
  e0b -= d0b;
  e1b += d0b - d1b;
  e2b += d1b - d2b;
  e3b += d2b - d3b;
  e4b += d3b;
  c[0] = -e0b;
  c[1] = e0b - e1b;
  c[2] = e1b - e2b + ylb;
  c[3] = e2b - e3b + yrb;
  c[4] = e3b - e4b;
  c[5] = e4b;
}

// Reverse of the HLLC flux (same branch choices as the forward: Davis wave
// speeds with the left candidate kept on ties and a NaN one left out, the upwind
// side of a supersonic face, else 0 <= S* selects the left side).
__device__ void hllc_vjp(const double *qL, const double *qR, double gamma, double gm1i,
                         const double *Fb, double *qLb, double *qRb) {
  double rL = qL[0], uL = qL[1], vL = qL[2], wL = qL[3], pL = qL[4];
  double rR = qR[0], uR = qR[1], vR = qR[2], wR = qR[3], pR = qR[4];
  double EL = pL * gm1i + 0.5 * rL * (uL * uL + vL * vL + wL * wL);
  double ER = pR * gm1i + 0.5 * rR * (uR * uR + vR * vR + wR * wR);
  // wave speeds, star speed and star reciprocal in the forward's arithmetic
  // (same branch decisions)
  double yL, yR;  // 1 / (rho c) per side
  double cL = sound_speed(gamma, rL, pL, yL);
  double cR = sound_speed(gamma, rR, pR, yR);
  double aL = uL - cL, bL = uR - cR;
  double SL = fmin(aL, bL);
  const bool selL = SL != aL;
  double aR = uL + cL, bR = uR + cR;
  double SR = fmax(aR, bR);
  const bool selR = SR != aR;
  double mL = rL * (SL - uL), mR = rR * (SR - uR);
  double Nn = pR - pL + uL * mL - uR * mR, Dd = mL - mR;
  const double iDd = rcp_nr(Dd);
  double Ss = fma(Nn, iDd, 0.0);
  const bool left = hllc_left(SL, Ss, SR);
  double r = left ? rL : rR, u = left ? uL : uR, v = left ? vL : vR, w = left ? wL : wR;
  double p = left ? pL : pR, E = left ? EL : ER, SK = left ? SL : SR, m = left ? mL : mR;
  double inv = rcp_nr(SK - Ss);
  // a supersonic face (0 <= SL: left, or SR < 0: right) has the flux of its
  // side alone: the wave term has weight S = 0 there, and the adjoint of the
  // clamped speed is dropped (selections only, as in the forward)
  const bool sub = hllc_subsonic(SL, SR);
  const double S = sub ? SK : 0.0;
  double Us0 = m * inv;
  double A4 = m * Ss + p;
  double N4 = E * (SK - u) + (Ss - u) * A4;
  double Us4 = N4 * inv;
  double fm = r * u;
  const double F0 = Fb[0], F1 = Fb[1], F2 = Fb[2], F3 = Fb[3], F4 = Fb[4];
  double Sb = F0 * (Us0 - r) + F1 * (Us0 * Ss - fm) + F2 * (Us0 * v - r * v) +
              F3 * (Us0 * w - r * w) + F4 * (Us4 - E);
  double Us0b = S * (F0 + F1 * Ss + F2 * v + F3 * w);
  double Ssb = F1 * S * Us0;
  double Us4b = S * F4;
  double fmb = F0 + F1 * (u - S) + F2 * v + F3 * w;
  double rb = -S * (F0 + F2 * v + F3 * w);
  double ub = F1 * fm + F4 * (E + p);
  double vb = F2 * (fm + S * Us0 - S * r);
  double wb = F3 * (fm + S * Us0 - S * r);
  double pb = F1 + F4 * u;
  double Eb = F4 * (u - S);
  double N4b = Us4b * inv, invb = Us4b * N4;
  Eb += N4b * (SK - u);
  Sb += N4b * E;
  ub -= N4b * (E + A4);
  Ssb += N4b * (A4 + (Ss - u) * m);
  double mb = N4b * (Ss - u) * Ss;
  pb += N4b * (Ss - u);
  mb += Us0b * inv;
  invb += Us0b * m;
  double db = -invb * inv * inv;
  Sb = sub ? Sb + db : 0.0;
  Ssb -= db;
  rb += fmb * u;
  ub += fmb * r;
  pb += Eb * gm1i;
  rb += Eb * 0.5 * (u * u + v * v + w * w);
  ub += Eb * r * u;
  vb += Eb * r * v;
  wb += Eb * r * w;
  const double kb[5] = {rb, ub, vb, wb, pb};
#pragma unroll
  for (int m = 0; m < 5; ++m) {
    qLb[m] = left ? kb[m] : 0.0;
    qRb[m] = left ? 0.0 : kb[m];
  }
  double mLb = left ? mb : 0.0, mRb = left ? 0.0 : mb;
  double SLb = left ? Sb : 0.0, SRb = left ? 0.0 : Sb;
  double Nnb = Ssb * iDd, Ddb = -Ssb * Ss * iDd;
  qRb[4] += Nnb;
  qLb[4] -= Nnb;
  qLb[1] += Nnb * mL;
  mLb += Nnb * uL + Ddb;
  qRb[1] -= Nnb * mR;
  mRb += -Nnb * uR - Ddb;
  qLb[0] += mLb * (SL - uL);
  SLb += mLb * rL;
  qLb[1] -= mLb * rL;
  qRb[0] += mRb * (SR - uR);
  SRb += mRb * rR;
  qRb[1] -= mRb * rR;
  const double tLR = selL ? SLb : 0.0, tLL = selL ? 0.0 : SLb;  // S_L = u - c of a side
  const double tRR = selR ? SRb : 0.0, tRL = selR ? 0.0 : SRb;  // S_R = u + c of a side
  qLb[1] += tLL + tRL;
  qRb[1] += tLR + tRR;
  const double cLb = tRL - tLL, cRb = tRR - tLR;
  // c = sqrt(gamma p / rho): dc/dp = gamma / (2 rho c) = gamma y / 2 and
  // dc/drho = -c / (2 rho) = -c^2 y / 2 (a side whose c is NaN set no speed)
  yL = fmax(yL, 0.0);
  yR = fmax(yR, 0.0);
  qLb[4] += cLb * (0.5 * gamma) * yL;
  qLb[0] -= cLb * (0.5 * fmax(cL * cL, 0.0)) * yL;
  qRb[4] += cRb * (0.5 * gamma) * yR;
  qRb[0] -= cRb * (0.5 * fmax(cR * cR, 0.0)) * yR;
}

// Flux adjoint at face f of direction D from the stage-output adjoint Wb:
// with Rb = b dt Wb (the right-hand-side adjoint, 5-component flux layout),
// Fb[m] = Rb_m(cell f)/dx_f - Rb_m(cell f-1)/dx_{f-1}.
// With the mass-flux body force f = -sum_c V_c R_rhou(c) / W every cell's
// x-momentum right-hand side also carries the force's dependence on the face
// fluxes: its adjoint gets -f-bar V_c / W.  Between the two cells of a face
// these terms cancel (V_c / dx is the face's area); the boundary faces keep
// theirs, as in the forward's boundary-flux form.
template <int NDIM>
__device__ __forceinline__ void face_adjoint(const Dev &g, const AdjBuffers &A, int D,
                                             const int *pos, int f, double *Fb) {
  const long nc = g.ncell;
  const double s = A.bcoef * A.dtp[0];
  const long vo[5] = {0, nc, 2 * nc, 3 * nc, (long)(NDIM + 1) * nc};
  // both cells' loads are issued unconditionally (at clamped positions, in
  // bounds) and together; only the sums depend on the cell existing
  const bool hr = f < g.n[D], hl = f >= 1;
  int cpos[3] = {pos[0], pos[1], pos[2]};
  cpos[D] = hr ? f : g.n[D] - 1;
  const long cr = ((long)cpos[2] * g.n[1] + cpos[1]) * g.n[0] + cpos[0];
  cpos[D] = hl ? f - 1 : 0;
  const long cl = ((long)cpos[2] * g.n[1] + cpos[1]) * g.n[0] + cpos[0];
  const double idr = g.idx[D][hr ? f : g.n[D] - 1], idl = g.idx[D][hl ? f - 1 : 0];
  double wr[5], wl[5];
#pragma unroll
  for (int m = 0; m < 5; ++m) {
    const bool on = m < 2 || m == 4 || m <= NDIM;
    wr[m] = on ? A.Wb[vo[m] + cr] : 0.0;
    wl[m] = on ? A.Wb[vo[m] + cl] : 0.0;
  }
#pragma unroll
  for (int m = 0; m < 5; ++m) {
    Fb[m] = 0.0;
    if (!(m < 2 || m == 4 || m <= NDIM)) continue;
    const double r = Fb[m] + (s * wr[m]) * idr;
    Fb[m] = hr ? r : Fb[m];
    const double l = Fb[m] - (s * wl[m]) * idl;
    Fb[m] = hl ? l : Fb[m];
  }
  if (g.source == SRC_MASSFLUX && !(hr && hl)) {
    double area = A.src[1] / g.vol;
#pragma unroll
    for (int e = 0; e < NDIM; ++e)
      if (e != D) area *= g.dx[e][pos[e]];
    Fb[1] += hr ? -area : area;
  }
}

// Tile geometry for direction D: tile index -> first face and line origin.
struct Tile {
  int f0;       // first face of the tile along D
  int c0, c1;   // cells written by the tile along D: [c0, c1)
  int line[3];  // tangential position of this thread's line (pos[D] unused)
  int lane_line, lane_face;
  unsigned lg;  // line group of the tile
  bool line_ok;
  bool valid;   // the workgroup has a tile
};

// P: the workgroup's index among the nb workgroups of direction D (the
// hardware index modulo 8 must equal P modulo 8: the XCD order below assumes
// it); t.valid is false for workgroups beyond the direction's tile count
template <int OLO, int OHI, int D, int NWV>
__device__ __forceinline__ Tile make_tile(const Dev &g, unsigned P, unsigned nb) {
  constexpr int TF = TileShape<D, NWV>::TF, TW = TileShape<D, NWV>::TW;
  constexpr int SPAN = OHI - OLO;
  constexpr int CPT = TF - SPAN;  // cells completed per tile line
  const int T1 = tan1(D), T2 = tan2(D);
  const int nt1 = g.n[T1], nt2 = g.n[T2];
  const int cmin = OLO;                         // first cell receiving contributions
  const int ncell_line = g.n[D] + 1 + SPAN;     // cells [OLO, n + OHI]
  const unsigned tiles_d = (unsigned)(ncell_line + CPT - 1) / CPT;
  const unsigned lines = (unsigned)nt1 * nt2;  // (ncell < 2^31)
  // y/z tiles: the two line groups that share each 128-byte row segment (and
  // the tiles along D of both, which share halo rows) run on one XCD, with
  // such chunks dealt round robin so that every XCD gets wall and free-stream
  // regions alike; x tiles keep the hardware order
  const unsigned tile = D == 0 ? P : xcd_chunk_remap(P, nb, 2u * tiles_d);
  const unsigned lg = tile / tiles_d;  // line group
  const int td = (int)(tile - lg * tiles_d);
  Tile t;
  t.valid = lg < (lines + TW - 1) / TW;
  const int tid = threadIdx.x;
  if (D == 0) {
    t.lane_face = tid % TF;
    t.lane_line = tid / TF;
  } else {
    t.lane_line = tid % TW;
    t.lane_face = tid / TW;
  }
  const unsigned ln = lg * TW + t.lane_line;  // line index over (t1 fastest, t2)
  t.line_ok = ln < lines;
  const int bq = t.line_ok && nt2 > 1 ? (int)(ln / (unsigned)nt1) : 0;
  const int a = t.line_ok ? (int)ln - bq * nt1 : 0;
  t.line[D] = 0;
  t.line[T1] = a;
  t.line[T2] = bq;
  t.c0 = cmin + td * CPT;
  t.c1 = min(t.c0 + CPT, g.n[D] + OHI + 1);
  t.f0 = t.c0 - OHI;
  t.lg = lg;
  return t;
}

// Tiles of direction D in workgroups of nwv wavefronts.
template <int OLO, int OHI>
__host__ inline unsigned tile_count(const Dev &g, int D, int nwv) {
  const int TF = D == 0 ? 64 : 8 * nwv, TW = D == 0 ? nwv : 8;
  constexpr int SPAN = OHI - OLO;
  const int CPT = TF - SPAN;
  const int ncell_line = g.n[D] + 1 + SPAN;
  const long tiles_d = (ncell_line + CPT - 1) / CPT;
  const long lines = (long)g.n[tan1(D)] * g.n[tan2(D)];
  return (unsigned)(tiles_d * ((lines + TW - 1) / TW));
}

// Wavefronts per workgroup for directions d0 .. d1 - 1: 4, or 8 where y and z
// tiles twice as long leave fewer wavefronts in all (65 x 49 x 33, whose y lines
// take one tile of 8 instead of three of 4: a training step 487 us, 501 with 4;
// at equal counts 4 starts and ends sooner, 1024 x 256: 304 and 307).
__host__ inline int dir_waves(const Dev &g, int d0, int d1) {
  unsigned long w4 = 0, w8 = 0;
  for (int D = d0; D < d1; ++D) {
    w4 += 4ul * tile_count<-3, 2>(g, D, 4);
    w8 += 8ul * tile_count<-3, 2>(g, D, 8);
  }
  return w8 < w4 ? 8 : 4;
}

// ---------------------------------------------------------------------------
// Adjoint of the fluxes along D, one tile of faces per workgroup:
//  * convective: WENO5-JS + HLLC reversed per face, contributions to the
//    cells f-3 .. f+2 (rho, velocity, p);
//  * dissipative (VISC): the face stress / heat flux reversed to face-level
//    adjoints, expanded over the cells f-2 .. f+1 into velocity, T, mu and
//    the adjoint Gb of the cell-centred tangential velocity derivatives.
// Both share the face adjoint from Wb and one LDS window of cells
// (f0-3 .. f0+TF+1 per line); the tile writes each completed cell once.
// Bound by the latency of a face's chain (loads, reconstructions, Riemann
// solver, their reverse component by component) at 4 wavefronts per SIMD, 121
// VGPRs in 2D: 5 with 96 spill and are slower by a quarter.  1024 x 256, both
// directions: 54.7 us, 62 with staged gathers between barriers, stencils read
// when needed and 113 instead of 76 FP64 instructions per reversed side;
// 65 x 49 x 33, three directions: 73 us, 119 in three launches.
// ---------------------------------------------------------------------------
// LDS of one tile: each wavefront's accumulators, NCH channels of the cells its
// 64 faces touch.  A wavefront holds 64 faces of one line (x) or 8 faces of 8
// lines (y, z: line fastest), so the cell at offset o of its lane's face is
// entry lane + ST o: consecutive entries for consecutive lanes.
template <int NDIM, int D, bool VISC, int NWV> struct DirLds {
  static constexpr int TF = TileShape<D, NWV>::TF, TW = TileShape<D, NWV>::TW;
  static constexpr int NOFF = 6, NCW = TF + 5;
  static constexpr int CP = 1 + NDIM, CT = 2 + NDIM, CMU = 3 + NDIM, CG = 4 + NDIM;
  static constexpr int NCH = VISC ? CG + 2 * (NDIM - 1) : CP + 1;
  static constexpr int ST = D == 0 ? 1 : TW, RW = 64 + (NOFF - 1) * ST;
  static constexpr int SIZE = NWV * NCH * RW;  // doubles
};

// One tile of direction D.  ALL: the tiles of every direction run in one launch,
// so a y or z tile writes its completed cells' Qb contributions to the side
// arrays Qby or Qbz (set, never added) instead of adding them to the Qb that
// the x tiles set; k_ghost_vjp (ghost cells) and k_interior_vjp (interior
// cells) add them.
template <int NDIM, int D, bool VISC, bool ALL, int NWV>
__device__ __forceinline__ void dir_vjp_tile(const Dev &g, const AdjBuffers &A, unsigned P,
                                             unsigned nb, double *lds) {
  using L = DirLds<NDIM, D, VISC, NWV>;
  constexpr bool SIDE = ALL && D > 0;
  constexpr int OLO = -3, OHI = 2, NOFF = L::NOFF, SPAN = OHI - OLO;
  constexpr int TW = L::TW;
  constexpr int NCW = L::NCW;  // window cells per line
  constexpr int T1 = tan1(D), T2 = tan2(D);
  // accumulator channels, active axes only: rho, the NDIM global velocity
  // components, p, then T, mu and Gb(T1,T1), Gb(T1,D) (Gb(T2,T2), Gb(T2,D))
  // for each active tangential axis when viscous
  constexpr int CP = L::CP, CT = L::CT, CMU = L::CMU, CG = L::CG;
  constexpr int NCH = L::NCH, ST = L::ST, RW = L::RW;
  const int lane = threadIdx.x % 64, wave = threadIdx.x / 64;
  // [channel][entry] of this wavefront, which alone touches it before the
  // write-out: LDS operations of a wavefront are in order, no barriers
  double *acc = lds + wave * NCH * RW;
  Tile t = make_tile<OLO, OHI, D, NWV>(g, P, nb);
  if (!t.valid) return;  // uniform across the workgroup
  // (the convective channels 0 .. CP are set by the first pass)
  for (int i = lane; i < (NCH - CT) * RW; i += 64) acc[CT * RW + i] = 0.0;

  const int f = t.f0 + t.lane_face;
  const bool active = t.line_ok && f >= 0 && f <= g.n[D];
  const int qi[5] = {QR, QU + D, QU + T1, QU + T2, QP};
  constexpr int ch[5] = {0, 1 + D, 1 + T1, 1 + T2, CP};  // face frame -> channel (active m)
  double qLb[5] = {0, 0, 0, 0, 0}, qRb[5] = {0, 0, 0, 0, 0};
  double Fb[5] = {0, 0, 0, 0, 0};
  long base = 0;
  const long s = g.sb[D];
  // the next component's stencil, read again ahead of its use (all of them held
  // since the first pass would not fit the registers)
  double nv[NOFF] = {0, 0, 0, 0, 0, 0};
  // for the dissipative flux: face velocities and their differences (face frame)
  // from the same reads, T and mu of the four inner cells
  double uf[3] = {0, 0, 0}, dn[3] = {0, 0, 0}, Tc[4] = {0, 0, 0, 0}, muc[4] = {0, 0, 0, 0};
  auto fetch = [&](int m) {
    const double *Qm = g.Q[qi[m]] + base;
#pragma unroll
    for (int o = 0; o < NOFF; ++o) nv[o] = Qm[(o - 3) * s];
  };
  if (active) {
    int pos[3] = {t.line[0], t.line[1], t.line[2]};
    pos[D] = f;
    face_adjoint<NDIM>(g, A, D, pos, f, Fb);
    base = bidx(g, pos[0], pos[1], pos[2]);
    double qL[5], qR[5];
#pragma unroll
    for (int m = 0; m < 5; ++m) {
      const bool act = !((m == 2 && T1 >= NDIM) || (m == 3 && T2 >= NDIM));
      if (!act) {
        qL[m] = qR[m] = 0.0;
        continue;
      }
      const double *Qm = g.Q[qi[m]];
      double v0 = Qm[base - 3 * s], v1 = Qm[base - 2 * s], v2 = Qm[base - s];
      double v3 = Qm[base], v4 = Qm[base + s], v5 = Qm[base + 2 * s];
      weno5_pair(v0, v1, v2, v3, v4, v5, qL[m], qR[m]);
    }
    double Fr[5] = {Fb[0], Fb[1 + D], Fb[1 + T1], Fb[1 + T2], Fb[4]};
    fetch(0);
    hllc_vjp(qL, qR, g.gamma, g.gm1i, Fr, qLb, qRb);
  }
  // convective, per component: reverse the two reconstructions, then sum the
  // contributions to cells f-3 .. f+2 per window cell by lane shuffles, in a
  // fixed order of faces (deterministic, no atomics)
#pragma unroll
  for (int m = 0; m < 5; ++m) {
    const bool act = !((m == 2 && T1 >= NDIM) || (m == 3 && T2 >= NDIM));
    if (!act) continue;  // uniform across the block
    double c[NOFF] = {0, 0, 0, 0, 0, 0};
    const double v0 = nv[0], v1 = nv[1], v2 = nv[2], v3 = nv[3], v4 = nv[4], v5 = nv[5];
    const int next = m + 1 + (m == 1 && T1 >= NDIM ? 1 : 0) +
                     ((m == 1 && T1 >= NDIM) || m == 2 ? (T2 >= NDIM ? 1 : 0) : 0);
    if (active) {
      if (next < 5) {
        fetch(next);
      } else if constexpr (VISC) {
#pragma unroll
        for (int o = 0; o < 4; ++o) {
          Tc[o] = g.Q[QT][base + (o - 2) * s];
          muc[o] = g.Q[QMU][base + (o - 2) * s];
        }
      }
      if (VISC && m >= 1 && m <= 3) {
        uf[m - 1] = interp4(v1, v2, v3, v4);
        dn[m - 1] = dface4(v1, v2, v3, v4);
      }
      weno5_vjp(v0, v1, v2, v3, v4, v5, qLb[m], qRb[m], c);
    }
    // entry L (and 64 + L for the last SPAN cells) takes offset o from lane
    // L - ST o, in a fixed order of faces
    double s0 = 0.0, s1 = 0.0;
#pragma unroll
    for (int o = 0; o < NOFF; ++o) {
      const double x0 = __shfl(c[o], lane - ST * o);
      const double x1 = __shfl(c[o], 64 + lane - ST * o);
      if (lane >= ST * o) s0 += x0;
      if (ST * o > lane) s1 += x1;
    }
    acc[ch[m] * RW + lane] = s0;
    if (lane < SPAN * ST) acc[ch[m] * RW + 64 + lane] = s1;
  }
  if constexpr (VISC) {
    // face-level adjoints of the dissipative flux
    double ufb[3] = {0, 0, 0}, dnb[3] = {0, 0, 0}, dTb = 0.0, mufb = 0.0;
    double divtb = 0.0, dtnb[3] = {0, 0, 0};
    double mfD = 0.0;
    if (active) {
      mfD = g.mf[D][f];
      double muf = interp4(muc[0], muc[1], muc[2], muc[3]);
#pragma unroll
      for (int c = 0; c < 3; ++c) dn[c] *= mfD;
      double dT = dface4(Tc[0], Tc[1], Tc[2], Tc[3]) * mfD;
      double divt = 0.0, dtn[3] = {0.0, 0.0, 0.0};
#pragma unroll
      for (int r = 0; r < 2; ++r) {
        const int tt = r == 0 ? T1 : T2;
        if (tt >= NDIM) continue;
        // cell-centred tangential derivatives d u_tt / d x_tt and d u_D /
        // d x_tt of the stage's primitive box, with the operands and
        // arithmetic of the forward flux kernels (the same values bitwise)
        const double *Ut = g.Q[QU + tt], *Ud = g.Q[QU + D];
        const long stt = g.sb[tt];
        const double mct = g.mc[tt][t.line[tt]];
        double gtt[4], gtn[4];
#pragma unroll
        for (int o = 0; o < 4; ++o) {
          long cb = base + (o - 2) * s;
          gtt[o] = dcell4(Ut[cb - 2 * stt], Ut[cb - stt], Ut[cb + stt], Ut[cb + 2 * stt]) * mct;
          gtn[o] = dcell4(Ud[cb - 2 * stt], Ud[cb - stt], Ud[cb + stt], Ud[cb + 2 * stt]) * mct;
        }
        divt += interp4(gtt[0], gtt[1], gtt[2], gtt[3]);
        dtn[1 + r] = interp4(gtn[0], gtn[1], gtn[2], gtn[3]);
      }
      // (component 0 normal, 1 along T1, 2 along T2)
      constexpr bool on[3] = {true, T1 < NDIM, T2 < NDIM};
      double brk[3];
      brk[0] = (4.0 / 3.0) * dn[0] - (2.0 / 3.0) * divt;
      brk[1] = on[1] ? dtn[1] + dn[1] : 0.0;
      brk[2] = on[2] ? dtn[2] + dn[2] : 0.0;
      const double cpPr = g.cpPr;
      // reverse
      const double enb = -Fb[4];
      const double Fm[3] = {Fb[1 + D], Fb[1 + T1], Fb[1 + T2]};
      double taub[3];
#pragma unroll
      for (int c = 0; c < 3; ++c) {
        taub[c] = -Fm[c] + enb * uf[c];
        ufb[c] = enb * (muf * brk[c]);
      }
      dTb = enb * (muf * cpPr);
      mufb = enb * dT * cpPr + taub[0] * brk[0] + taub[1] * brk[1] + taub[2] * brk[2];
      dnb[0] = taub[0] * muf * (4.0 / 3.0);
      divtb = -taub[0] * muf * (2.0 / 3.0);
#pragma unroll
      for (int c = 1; c < 3; ++c)
        if (on[c]) dnb[c] = dtnb[c] = taub[c] * muf;
    }
    // cells f-2 .. f+1 are the entries at offsets 1 .. 4, one offset at a time:
    // neighbouring faces update the same cells at consecutive offsets
    const double I4[4] = {-1.0 / 16.0, 9.0 / 16.0, 9.0 / 16.0, -1.0 / 16.0};
    const double D4[4] = {1.0 / 24.0, -27.0 / 24.0, 27.0 / 24.0, -1.0 / 24.0};
#pragma unroll
    for (int o = 0; o < 4; ++o) {
      __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
      __builtin_amdgcn_wave_barrier();
      if (active) {
        double *w = acc + lane + ST * (1 + o);
        const double dm = D4[o] * mfD, im = I4[o];
#pragma unroll
        for (int c = 0; c < 3; ++c)
          if (c == 0 || (c == 1 && T1 < NDIM) || (c == 2 && T2 < NDIM))
            w[ch[1 + c] * RW] += ufb[c] * im + dnb[c] * dm;
        w[CT * RW] += dTb * dm;
        w[CMU * RW] += mufb * im;
        if constexpr (T1 < NDIM) {
          w[CG * RW] += divtb * im;
          w[(CG + 1) * RW] += dtnb[1] * im;
        }
        if constexpr (T2 < NDIM) {
          w[(CG + 2) * RW] += divtb * im;
          w[(CG + 3) * RW] += dtnb[2] * im;
        }
      }
    }
  }
  __syncthreads();  // every line's window complete before the write-out
  // write the completed cells: window cell w <-> cell t.f0 + OLO + w
  for (int i = threadIdx.x; i < TW * NCW; i += 64 * NWV) {
    // x-lines: consecutive threads take consecutive cells of a line;
    // otherwise consecutive lines (x-neighbours) of one cell position
    const int ll = D == 0 ? i / NCW : i % TW, w = D == 0 ? i % NCW : i / TW;
    const int cell = t.f0 + OLO + w;
    if (cell < t.c0 || cell >= t.c1) continue;
    const unsigned ln = t.lg * TW + ll;
    if (ln >= (unsigned)g.n[T1] * g.n[T2]) continue;
    int p[3];
    p[D] = cell;
    p[T2] = g.n[T2] > 1 ? (int)(ln / (unsigned)g.n[T1]) : 0;
    p[T1] = (int)ln - p[T2] * g.n[T1];
    const long b = bidx(g, p[0], p[1], p[2]);
    const bool ghost = cell < 0 || cell >= g.n[D];
    // the window cell's sum: x tiles, its line's entry; y and z tiles, the
    // wavefront whose faces start at or before it and the one before that
    double sum[NCH];
    if constexpr (D == 0) {
#pragma unroll
      for (int k = 0; k < NCH; ++k) sum[k] = lds[(ll * NCH + k) * RW + w];
    } else {
      const int wv = w / 8, x = w % 8;
      const bool own = wv < NWV, before = wv > 0 && x < SPAN;
      const double *a0 = lds + (own ? wv : NWV - 1) * NCH * RW + x * TW + ll;
      const double *a1 = lds + (before ? wv - 1 : 0) * NCH * RW + ((before ? x : 0) + 8) * TW + ll;
#pragma unroll
      for (int k = 0; k < NCH; ++k)
        sum[k] = (before ? a1[k * RW] : 0.0) + (own ? a0[k * RW] : 0.0);
    }
    if constexpr (SIDE) {
      double *const *Qs = D == 1 ? A.Qby : A.Qbz;
      Qs[QR][b] = sum[0];
#pragma unroll
      for (int c = 0; c < NDIM; ++c) Qs[QU + c][b] = sum[1 + c];
      Qs[QP][b] = sum[CP];
      if constexpr (VISC) {
        Qs[QT][b] = sum[CT];
        Qs[QMU][b] = sum[CMU];
      } else {
        Qs[QT][b] = 0.0;
      }
    } else if (D == 0 || ghost) {
      // first writer of this cell in the stage: set every component the
      // later kernels accumulate into
      A.Qb[QR][b] = sum[0];
#pragma unroll
      for (int c = 0; c < NDIM; ++c) A.Qb[QU + c][b] = sum[1 + c];
      A.Qb[QP][b] = sum[CP];
      if constexpr (VISC) {
        A.Qb[QT][b] = sum[CT];
        A.Qb[QMU][b] = sum[CMU];
      } else {
        A.Qb[QT][b] = 0.0;
      }
    } else {
      A.Qb[QR][b] += sum[0];
#pragma unroll
      for (int c = 0; c < NDIM; ++c) A.Qb[QU + c][b] += sum[1 + c];
      A.Qb[QP][b] += sum[CP];
      if constexpr (VISC) {
        A.Qb[QT][b] += sum[CT];
        A.Qb[QMU][b] += sum[CMU];
      }
    }
    if constexpr (VISC) {
      // derivative adjoints: d u_D / d x_t is this kernel's alone (set); the
      // diagonal d u_t / d x_t is shared with the kernel of every earlier
      // direction other than t, which covered the cells interior along D
      constexpr bool sh1 = D >= 2 || (D == 1 && T1 != 0), sh2 = D >= 2 || (D == 1 && T2 != 0);
      // (tiles of all directions in one launch: the later direction's share of
      // a diagonal is set in Gs)
      if constexpr (T1 < NDIM) {
        double &d1 = (ALL && sh1 ? A.Gs[T1] : A.Gb[3 * T1 + T1])[b];
        d1 = (!ALL && sh1 && !ghost ? d1 : 0.0) + sum[CG];
        A.Gb[3 * T1 + D][b] = sum[CG + 1];
      }
      if constexpr (T2 < NDIM) {
        double &d2 = (ALL && sh2 ? A.Gs[T2] : A.Gb[3 * T2 + T2])[b];
        d2 = (!ALL && sh2 && !ghost ? d2 : 0.0) + sum[CG + 2];
        A.Gb[3 * T2 + D][b] = sum[CG + 3];
      }
    }
  }
}

// One direction per launch (1D, 3D).
template <int NDIM, int D, bool VISC, int NWV>
__global__ void __launch_bounds__(64 * NWV) __attribute__((amdgpu_waves_per_eu(4)))
k_dir_vjp(Dev g, AdjBuffers A) {
  __shared__ double lds[DirLds<NDIM, D, VISC, NWV>::SIZE];
  dir_vjp_tile<NDIM, D, VISC, false, NWV>(g, A, blockIdx.x, gridDim.x, lds);
}

// The tiles of every direction of a stage in one launch, so that the
// directions' tiles share the CUs (each alone leaves the FP64 units idle while
// its workgroups wait on memory).  Workgroups are dealt in groups of 8, the
// directions in turn while they have tiles left: group c of a direction holds
// its tiles 8c .. 8c+7, so that a tile's index modulo 8 is its hardware index
// modulo 8 (its XCD) as in a launch of its own.  The y and z tiles write their
// cell contributions to Qby and Qbz; the x tiles set Qb.
struct DirGroups {
  unsigned c[3];  // groups of 8 workgroups per direction (0: no such axis)
};

// Group number grp -> direction and group within it.
__device__ __forceinline__ void dir_of_group(const DirGroups &G, int nd, unsigned grp, int &dir,
                                             unsigned &ci) {
  // rounds of nd groups while every direction has some, then of those left
  unsigned lo = 0u;  // groups per direction dealt so far
  for (;;) {
    unsigned left = 0u, m = 0xffffffffu;
    for (int d = 0; d < nd; ++d)
      if (G.c[d] > lo) {
        ++left;
        m = G.c[d] < m ? G.c[d] : m;
      }
    const unsigned span = left * (m - lo);
    if (grp < span || left <= 1u) {
      const unsigned k = grp % left;
      ci = lo + grp / left;
      unsigned seen = 0u;
      dir = 0;
      for (int d = 0; d < nd; ++d)
        if (G.c[d] > lo) {
          if (seen == k) dir = d;
          ++seen;
        }
      return;
    }
    grp -= span;
    lo = m;
  }
}

template <int NDIM, bool VISC, int NWV>
__global__ void __launch_bounds__(64 * NWV) __attribute__((amdgpu_waves_per_eu(4)))
k_dir_vjp_all(Dev g, AdjBuffers A, DirGroups G) {
  constexpr int SX = DirLds<NDIM, 0, VISC, NWV>::SIZE, SY = DirLds<NDIM, 1, VISC, NWV>::SIZE;
  __shared__ double lds[SX > SY ? SX : SY];  // (z tiles as y tiles)
  unsigned ci;
  int dir;
  dir_of_group(G, NDIM, blockIdx.x / 8u, dir, ci);
  const unsigned P = ci * 8u + blockIdx.x % 8u;
  if (dir == 0) dir_vjp_tile<NDIM, 0, VISC, true, NWV>(g, A, P, 8u * G.c[0], lds);
  else if (NDIM == 2 || dir == 1)
    dir_vjp_tile<NDIM, 1, VISC, true, NWV>(g, A, P, 8u * G.c[1], lds);
  else if constexpr (NDIM == 3)
    dir_vjp_tile<NDIM, 2, VISC, true, NWV>(g, A, P, 8u * G.c[2], lds);
}

// ---------------------------------------------------------------------------
// Gather of the tangential-derivative adjoints (transpose of the
// cell-centred 4th-order difference along t), then mu'(T) folding: on the
// ghost cells in k_ghost_vjp, on the interior cells inside k_interior_vjp.
// ---------------------------------------------------------------------------
// d mu / dT from T and mu(T): omega mu / T (power law), mu (1.5/t - 1/(t+s))
// / T_ref with t = T/T_ref, s = S/T_ref (Sutherland).
__device__ __forceinline__ double dviscosity(const Dev &g, double T, double mu) {
  if (g.visc == VISC_POWER) return g.vparam * mu / T;
  if (g.visc == VISC_SUTHERLAND) {
    double t = T / g.T_ref;
    double s = g.vparam / g.T_ref;
    return mu * (1.5 / t - 1.0 / (t + s)) / g.T_ref;
  }
  return 0.0;
}

// Gather of the tangential-derivative adjoints at box cell p: y = x + k along
// t contributes coef(k) mc(y) Gb(y) where y is interior along t; the metric
// factors of the (at most four) neighbours along each axis are shared by the
// NDIM velocity components.  G: the axes along which p is a ghost, as bits.
// Along those only the two inward neighbours can be interior; a cell that is a
// ghost along two axes has no derivative adjoint, so along the other axes of an
// edge there is nothing to gather.  ALL3: the diagonals' second shares are in Gs.
template <int NDIM, unsigned G, bool ALL3>
__device__ __forceinline__ void tangential_gather(const Dev &g, const AdjBuffers &A, const int *p,
                                                  long b, double *add) {
  constexpr bool edge = (G & (G - 1u)) != 0u;
  constexpr int ks[4] = {-1, 1, -2, 2};
  constexpr double cf[4] = {8.0 / 12.0, -8.0 / 12.0, -1.0 / 12.0, 1.0 / 12.0};
  // Every load is issued first, so all of them are in flight together, then
  // the terms of the interior neighbours are summed in the order of the
  // definition (selects, no branches).  A neighbour that is not an interior
  // cell reads the cell itself and the metric at the cell's (clamped)
  // position instead, in bounds either way; an interior cell's neighbours
  // all lie in the box (two of its three ghost layers at most).
  double mct[NDIM][4], gv[NDIM][4][NDIM];
  bool in[NDIM][4];
#pragma unroll
  for (int t = 0; t < NDIM; ++t) {
    const bool ghost = (G >> t) & 1u;
    if (edge && !ghost) continue;
    const long st = g.sb[t];
    const int pt = ghost ? min(max(p[t], 0), g.n[t] - 1) : p[t];
    const int s = ghost && p[t] >= 0 ? -1 : 1;  // inwards
#pragma unroll
    for (int r = 0; r < (ghost ? 2 : 4); ++r) {
      const int k = ghost ? s * (r + 1) : ks[r];
      const int yt = p[t] + k;
      in[t][r] = yt >= 0 && yt < g.n[t];
      mct[t][r] = g.mc[t][in[t][r] ? yt : pt];
      if (ghost) mct[t][r] *= (double)s;
      const long bb = (G == 0u || in[t][r]) ? b + k * st : b;
#pragma unroll
      for (int phi = 0; phi < NDIM; ++phi) gv[t][r][phi] = A.Gb[3 * t + phi][bb];
      if constexpr (ALL3) gv[t][r][t] += A.Gs[t][bb];
    }
  }
#pragma unroll
  for (int phi = 0; phi < NDIM; ++phi) add[phi] = 0.0;
#pragma unroll
  for (int t = 0; t < NDIM; ++t) {
    const bool ghost = (G >> t) & 1u;
    if (edge && !ghost) continue;
#pragma unroll
    for (int r = 0; r < (ghost ? 2 : 4); ++r) {
      const double w = (ghost ? cf[2 * r + 1] : cf[r]) * mct[t][r];
#pragma unroll
      for (int phi = 0; phi < NDIM; ++phi) {
        const double sum = add[phi] + w * gv[t][r][phi];
        add[phi] = in[t][r] ? sum : add[phi];
      }
    }
  }
}

// Adjoint components carried through the halo fill: rho, the active
// velocities, p, T (mu-bar is folded into T-bar first).
template <int NDIM> struct HaloQ {
  static constexpr int nq = NDIM + 3;
  static constexpr int qs[6] = {QR, QU, NDIM >= 2 ? QV : QP,
                                NDIM == 3 ? QW : (NDIM == 2 ? QP : QT), NDIM == 3 ? QP : QT, QT};
};

// A ghost adjoint mapped to its contribution to the source: copies pass
// through; walls: p_g = p_s, u_g = -u_s (plus a prescribed normal part that
// depends on the state only through the porous p_w, taken separately);
// isothermal: rho_g = p_g / (R T_g), T_g = 2 T_w - T_s; adiabatic:
// rho_g = rho_s, T_g = T_s.  rg, pg: the ghost's density and pressure.
template <int NDIM>
__device__ __forceinline__ void ghost_transform(const Dev &g, bool wall, bool iso,
                                                const double *gbm, double rg, double pg,
                                                double *cs) {
  constexpr int nq = HaloQ<NDIM>::nq, iP = nq - 2, iT = nq - 1;
#pragma unroll
  for (int i = 0; i < nq; ++i) cs[i] = gbm[i];
  if (!wall) return;
#pragma unroll
  for (int c = 0; c < NDIM; ++c) cs[1 + c] = -gbm[1 + c];
  if (iso) {
    const double rb = gbm[0];
    cs[0] = 0.0;
    cs[iP] = gbm[iP] + rb * rg / pg;
    cs[iT] = -(gbm[iT] - rb * rg * rg * g.R / pg);
  }
}

// Wall columns of a disturbance face of axis d: those inside along its first
// tangential axis, and along the second all that the fill along d covers.
__host__ inline long disturb_cols(const Dev &g, int d) {
  const int t2 = tan2(d);
  return (long)g.n[tan1(d)] * (t2 < d ? g.N[t2] : g.n[t2]);
}

// The ghost layers of side `side` along an axis of n cells that copy (and
// mirror) cell i: layers m0 .. m0 + cnt - 1 (cnt 0: none).  The zero-gradient
// copy fills all three layers from one cell; Dirichlet ghosts copy none.
__device__ __forceinline__ void halo_images(int kind, int side, int i, int n, int &m0, int &cnt) {
  const int lo = i, hi = n - 1 - i;
  m0 = (kind == BC_PERIODIC) == (side == 0) ? hi : lo;
  cnt = m0 < 3 ? 1 : 0;
  if (kind == BC_ZEROGRAD) {
    cnt = (side == 0 ? lo : hi) == 0 ? 3 : 0;
    m0 = 0;
  }
  if (kind == BC_DIRICHLET) cnt = 0;
}

// Adds the edges along axes D and E that fold into the ghost at p to its
// velocity adjoints.
template <int NDIM, int D, int E, bool ALL3>
__device__ __forceinline__ void edge_ghosts(const Dev &g, const AdjBuffers &A, const int *p,
                                            double *qb) {
  if constexpr (E > D && E < NDIM) {
    unsigned mask = 0u;
#pragma unroll
    for (int side = 0; side < 2; ++side) {
      int m0, cnt;
      halo_images(g.bck[2 * E + side], side, p[E], g.n[E], m0, cnt);
      mask |= (cnt == 3 ? 7u : (cnt ? 1u << m0 : 0u)) << (3 * side);
    }
    while (mask) {
      const int bit = __ffs(mask) - 1;
      mask &= mask - 1u;
      const int side = bit >= 3 ? 1 : 0, m = bit - 3 * side;
      const bool wall = side ? is_wall(g.bck[2 * E + 1]) : is_wall(g.bck[2 * E]);
      int pe[3] = {p[0], p[1], p[2]};
      pe[E] = side == 0 ? -1 - m : g.n[E] + m;
      double add[NDIM];
      tangential_gather<NDIM, (1u << D) | (1u << E), ALL3>(g, A, pe, bidx(g, pe[0], pe[1], pe[2]),
                                                          add);
#pragma unroll
      for (int phi = 0; phi < NDIM; ++phi) qb[QU + phi] += wall ? -add[phi] : add[phi];
    }
  }
}

// The ghost at p, a ghost along axis D.
template <int NDIM, int D, bool ALL3>
__device__ __forceinline__ void ghost_vjp(const Dev &g, const AdjBuffers &A, int want_dk,
                                          const int *p) {
  const long b = bidx(g, p[0], p[1], p[2]);
  const bool visc = g.visc != VISC_NONE;
  // every load first (Qb, Qby and Gb may overlap as far as the compiler
  // knows, which would serialise loads behind stores), then the stores
  const bool gather = NDIM >= 2 && A.Gb[0] != nullptr;
  double qb[NQ];
#pragma unroll
  for (int q = 0; q < NQ; ++q) {
    qb[q] = 0.0;
    if ((q == QW && NDIM < 3) || (q == QMU && !visc)) continue;
    if ((NDIM == 2 || ALL3) && D == 1) qb[q] = A.Qby[q][b];
    else if (ALL3 && D == 2) qb[q] = A.Qbz[q][b];
    else qb[q] = A.Qb[q][b];
  }
  const double Tq = g.Q[QT][b], muq = g.Q[QMU][b];  // (every box array exists)
  if (visc) qb[QT] += dviscosity(g, Tq, muq) * qb[QMU];
  if (gather) {
    double add[NDIM];
    tangential_gather<NDIM, 1u << D, ALL3>(g, A, p, b, add);
#pragma unroll
    for (int phi = 0; phi < NDIM; ++phi) qb[QU + phi] += add[phi];
  }
  // the edges folded into this ghost: the layers of both sides of an axis e
  // after D, as bits 3 side + layer; each lane takes its next one per pass
  if (gather) edge_ghosts<NDIM, D, 1, ALL3>(g, A, p, qb);
  if (gather) edge_ghosts<NDIM, D, 2, ALL3>(g, A, p, qb);
  // the (A, kappa) of a z disturbance wall act on its edge columns too, those
  // whose x lies inside: the layer-0 source's thread sums the column
  if (NDIM == 3 && D == 1 && want_dk) {
#pragma unroll 1
    for (int side = 0; side < 2; ++side) {
      const int kind = g.bck[4 + side];
      if (kind != BC_DISTURB || p[2] != ghost_source(kind, side, 0, g.n[2])) continue;
      double vsum = 0.0;
      if (gather)
#pragma unroll 1
        for (int m = 0; m < 3; ++m) {
          const int pe[3] = {p[0], p[1], side == 0 ? -1 - m : g.n[2] + m};
          double add[NDIM];
          tangential_gather<NDIM, 6u, ALL3>(g, A, pe, bidx(g, pe[0], pe[1], pe[2]), add);
          vsum += add[NDIM - 1];
        }
      A.dpart[(4 + side) * A.dcols + (long)(p[1] + 3) * g.n[0] + p[0]] = vsum;
    }
  }
#pragma unroll
  for (int i = 0; i < HaloQ<NDIM>::nq; ++i) {
    const int q = HaloQ<NDIM>::qs[i];
    A.Qb[q][b] = qb[q];
  }
}

// Ghost cells along exactly one axis: their complete adjoint, before the
// interior cells collect it.  The flux tiles' contribution (Qb, or the side
// array of the axis' direction), the tangential gather, mu'(T) folded into T,
// and the ghosts along a second axis (the edges of the box) that copy this
// cell: the halo fill runs along x, then y, then z, so its transpose folds z
// ghosts first, and an edge's adjoint is a tangential gather alone (velocity
// components: no face flux reads an edge, and no derivative that is a ghost
// along two axes has an adjoint, so corners have none).
// Launch and memory latency bound, a thread per ghost (1024 x 256: 5.7 us; this
// kernel and the collection in k_interior_vjp, 13.3 to 15.1 us, took the place
// of a 4.9 us gather and a transpose launch of 6.2 us per axis; 65 x 49 x 33:
// 10.4 us and 9.4 to 17.4 for 7.2 and three of 7.0).
template <int NDIM, bool ALL3>
__global__ void __launch_bounds__(64)
k_ghost_vjp(Dev g, AdjBuffers A, int want_dk) {
  long t = (long)blockIdx.x * blockDim.x + threadIdx.x;
  const long n0 = g.n[0], n1 = g.n[1], n2 = g.n[2];
  // ghost number c (side, layer) of an axis of n cells -> its position
  auto at = [](int c, int n) { return c < 3 ? c - 3 : n + c - 3; };
  if (t < 6 * n1 * n2) {  // x ghosts: a line's six together
    const long line = t / 6;
    const int p[3] = {at((int)(t % 6), g.n[0]), (int)(line % n1), (int)(line / n1)};
    ghost_vjp<NDIM, 0, ALL3>(g, A, want_dk, p);
    return;
  }
  // y, then z ghosts: x fastest
  t -= 6 * n1 * n2;
  if constexpr (NDIM >= 2) {
    if (t < 6 * n0 * n2) {
      const long row = t / n0;
      const int p[3] = {(int)(t % n0), at((int)(row % 6), g.n[1]), (int)(row / 6)};
      ghost_vjp<NDIM, 1, ALL3>(g, A, want_dk, p);
      return;
    }
    t -= 6 * n0 * n2;
  }
  if constexpr (NDIM == 3) {
    if (t < 6 * n0 * n1) {
      const long row = t / n0;
      const int p[3] = {(int)(t % n0), (int)(row % n1), at((int)(row / n1), g.n[2])};
      ghost_vjp<NDIM, 2, ALL3>(g, A, want_dk, p);
    }
  }
}

// Contributions of the ghosts that copy interior cell p (box index b), added to
// its adjoint qb (HaloQ order), and through the walls' parameters to dJ/dK.
// Face by face, as most faces have none of a wavefront's cells (a pass per lane
// over the faces it is near cost 24 against 15 us at 1024 x 256).
template <int NDIM, int d>
__device__ __forceinline__ void collect_ghosts(const Dev &g, const AdjBuffers &A, const int *p,
                                               long b, double *dJdK, double *qb) {
  using H = HaloQ<NDIM>;
  constexpr int nq = H::nq, iP = nq - 2;
  const int n = g.n[d], i = p[d];
  const long sd = g.sb[d];
#pragma unroll 1
  for (int side = 0; side < 2; ++side) {
    const int face = 2 * d + side;
    const int kind = g.bck[face];
    int m0, cnt;
    halo_images(kind, side, i, n, m0, cnt);
    if (cnt == 0) continue;
    // box index of ghost layer 0 and the step to the next layer
    const long G0 = b + ((side == 0 ? -1 : n) - i) * sd, gs = side == 0 ? -sd : sd;
    if (cnt == 3) {  // copies, all of this cell
#pragma unroll
      for (int q = 0; q < nq; ++q) {
        const double *Q = A.Qb[H::qs[q]] + G0;
        qb[q] += (Q[0] + Q[gs]) + Q[2 * gs];
      }
      continue;
    }
    const bool wall = is_wall(kind), iso = wall && g.Tw[face] > 0.0;
    const long G = G0 + m0 * gs;
    double gb[6], cs[6];
#pragma unroll
    for (int q = 0; q < nq; ++q) gb[q] = A.Qb[H::qs[q]][G];
    const double rg = g.Q[QR][G], pg = g.Q[QP][G];
    ghost_transform<NDIM>(g, wall, iso, gb, rg, pg, cs);
#pragma unroll
    for (int q = 0; q < nq; ++q) qb[q] += cs[q];
    if ((kind != BC_POROUS && kind != BC_DISTURB) || m0 != 0) continue;
    // the wall cell of a porous or disturbance column (the source of ghost
    // layer 0): the sum of the layers' normal-velocity adjoints
    constexpr int t1 = tan1(d), t2 = tan2(d);
    const int a = p[t1], bq = p[t2];
    const double *Qn = A.Qb[QU + d] + G0;
    const double vsum = Qn[0] + Qn[gs] + Qn[2 * gs];
    if (kind == BC_DISTURB) {
      if (dJdK) A.dpart[face * A.dcols + (long)(bq + (t2 < d ? 3 : 0)) * g.n[t1] + a] = vsum;
    } else if (face == g.pface && a >= g.pb && a < g.pe) {
      // v_g[d] = 2 sigma v_n - v_s[d], v_n = -K (p_w - p_inf)/p_inf
      const int kk = bq * (g.pe - g.pb) + (a - g.pb);
      const double vnb = (side == 0 ? 2.0 : -2.0) * vsum;
      qb[iP] += -g.K[kk] / g.pinf * vnb;
      if (dJdK) dJdK[kk] += -(g.Q[QP][b] - g.pinf) / g.pinf * vnb;
    }
  }
}

// dJ/d(A, kappa) of one disturbance face from the sums of its columns'
// normal-velocity ghost adjoints (one block, fixed summation order:
// deterministic): v_g[d] = 2 sigma A sin(phi) - v_s[d], phi = 2 pi kappa x.
__global__ void __launch_bounds__(256) k_disturb_sum(Dev g, const double *part, long cols,
                                                     int face, double *out) {
  __shared__ double sh[2][256];
  double v[2] = {0.0, 0.0};
  const int t1 = tan1(face / 2);
  const double th0 = g.K[g.doff[face]], th1 = g.K[g.doff[face] + 1];
  for (long i = threadIdx.x; i < cols; i += 256) {
    const double xd = g.xm[t1][i % g.n[t1]];
    const double ph = 2.0 * M_PI * xd * th1, w = (face % 2 == 0 ? 2.0 : -2.0) * part[i];
    v[0] += w * sin(ph);
    v[1] += w * th0 * cos(ph) * 2.0 * M_PI * xd;
  }
  sh[0][threadIdx.x] = v[0];
  sh[1][threadIdx.x] = v[1];
  __syncthreads();
  for (int w = 128; w > 0; w >>= 1) {
    if ((int)threadIdx.x < w) {
      sh[0][threadIdx.x] += sh[0][threadIdx.x + w];
      sh[1][threadIdx.x] += sh[1][threadIdx.x + w];
    }
    __syncthreads();
  }
  if (threadIdx.x == 0) {
    out[0] += sh[0][0];
    out[1] += sh[1][0];
  }
}

// ---------------------------------------------------------------------------
// Mass-flux body force of a stage, adjoint side: the source adds f to the
// x-momentum and f u to the energy right-hand side of every cell, so with
// Rb = b dt Wb, f-bar = sum_c (Rb_rhou(c) + Rb_E(c) u(c)), into src[1].  Two
// passes, fixed-shape trees (deterministic); the second also adds the forward's
// force partials (f into src[0]).  (One launch whose last workgroup adds the
// partial sums took 12.9 us, its fences most of it.)
// ---------------------------------------------------------------------------
__global__ void __launch_bounds__(256) k_force_adj_partial(Dev g, AdjBuffers A) {
  __shared__ double sh[4];
  const double s = A.bcoef * A.dtp[0];
  const long nc = g.ncell;
  const int nd = g.ndim;
  const unsigned n0 = g.n[0], n01 = n0 * (unsigned)g.n[1];
  double v = 0.0;
  for (long c = (long)blockIdx.x * 256 + threadIdx.x; c < nc; c += (long)gridDim.x * 256) {
    const unsigned cu = (unsigned)c;
    const int k = (int)(cu / n01), j = (int)((cu % n01) / n0), i = (int)(cu % n0);
    const double rb1 = s * A.Wb[nc + c], rbE = s * A.Wb[(long)(nd + 1) * nc + c];
    v += rb1 + rbE * g.Q[QU][bidx(g, i, j, k)];
  }
  v = block_total<256>(v, sh);
  if (threadIdx.x == 0) A.spart[blockIdx.x] = v;
}

__global__ void __launch_bounds__(256) k_force_adj_final(Dev g, AdjBuffers A, int nparts,
                                                         const double *fpart, int nfpart) {
  __shared__ double sh[4];
  double fb = 0.0, f = 0.0;
  for (int x = threadIdx.x; x < nparts; x += 256) fb += A.spart[x];
  for (int x = threadIdx.x; x < nfpart; x += 256) f += fpart[x];
  fb = block_total<256>(fb, sh);
  f = block_total<256>(f, sh);
  if (threadIdx.x == 0) {
    A.src[1] = fb;
    if (fpart) A.src[0] = -f / g.vol;
  }
}

// ---------------------------------------------------------------------------
// Interior: Vb = b Wb + (dQ/dU)^T Qb, with Q = (rho, u, v, w, p, T(p, rho)).
// In the first stage (fold != 0, V = Un) Vb also takes the Un terms of the
// later stages' combinations, a3 W3 + a2 W2 (their output adjoints, still
// held), so no accumulator crosses the stages.
// ---------------------------------------------------------------------------
template <int NDIM, bool ALL3>
__global__ void __launch_bounds__(256)
k_interior_vjp(Dev g, AdjBuffers A, const double *V,
                                                      const double *Wb, double a, double b,
                                                      double *Vb, const double *w3, double a3,
                                                      const double *w2, double a2, int fold,
                                                      double *dJdK) {
  constexpr int nd = NDIM;
  const unsigned cu = blockIdx.x * blockDim.x + threadIdx.x;  // ncell < 2^31
  if (cu >= (unsigned)g.ncell) return;
  const long c = cu;
  const long nc = g.ncell;
  const unsigned n0 = g.n[0], n01 = n0 * (unsigned)g.n[1];
  const int k = (int)(cu / n01), j = (int)((cu % n01) / n0), i = (int)(cu % n0);
  const long bx = bidx(g, i, j, k);
  // the cell's state and stage-output adjoints (and the fold's inputs)
  // first: every load of the kernel before the first store (Vb may be an
  // input array as far as the compiler knows), as few round trips as the
  // branches allow
  double Vc[nd + 2], wv[nd + 2], f3[nd + 2], f2[nd + 2];
#pragma unroll
  for (int v = 0; v < nd + 2; ++v) {
    const long x = (long)v * nc + c;
    Vc[v] = V[x];
    wv[v] = Wb[x];
    f3[v] = fold ? w3[x] : 0.0;
    f2[v] = fold ? w2[x] : 0.0;
  }
  // the primitive adjoint of the cell: the flux adjoints' (x tiles plus, with
  // all directions in one launch, the side arrays), the tangential gather,
  // mu'(T) folded into T, and the ghosts that copy the cell
  double rb = A.Qb[QR][bx], pb = A.Qb[QP][bx], Tb = A.Qb[QT][bx];
  double ub[3] = {A.Qb[QU][bx], nd >= 2 ? A.Qb[QV][bx] : 0.0, nd >= 3 ? A.Qb[QW][bx] : 0.0};
  const bool visc = g.visc != VISC_NONE;
  double mub = visc ? A.Qb[QMU][bx] : 0.0;
  const int pc[3] = {i, j, k};
  if constexpr (NDIM == 2 || ALL3) {
    rb += A.Qby[QR][bx];
#pragma unroll
    for (int q = 0; q < NDIM; ++q) ub[q] += A.Qby[QU + q][bx];
    pb += A.Qby[QP][bx];
    Tb += A.Qby[QT][bx];
    if (visc) mub += A.Qby[QMU][bx];
  }
  if constexpr (ALL3) {
    rb += A.Qbz[QR][bx];
#pragma unroll
    for (int q = 0; q < NDIM; ++q) ub[q] += A.Qbz[QU + q][bx];
    pb += A.Qbz[QP][bx];
    Tb += A.Qbz[QT][bx];
    if (visc) mub += A.Qbz[QMU][bx];
  }
  if (NDIM >= 2 && A.Gb[0] != nullptr) {
    double add[NDIM];
    tangential_gather<NDIM, 0u, ALL3>(g, A, pc, bx, add);
#pragma unroll
    for (int phi = 0; phi < NDIM; ++phi) ub[phi] += add[phi];
  }
  const double Tq = g.Q[QT][bx], muq = g.Q[QMU][bx];  // (every box array exists)
  if (visc) Tb += dviscosity(g, Tq, muq) * mub;
  bool rim = false;  // within three cells of a face
#pragma unroll
  for (int d = 0; d < NDIM; ++d) rim |= min(pc[d], g.n[d] - 1 - pc[d]) < 3;
  if (rim) {
    double qb[6] = {};
    if constexpr (NDIM == 3) collect_ghosts<NDIM, 2>(g, A, pc, bx, dJdK, qb);
    if constexpr (NDIM >= 2) collect_ghosts<NDIM, 1>(g, A, pc, bx, dJdK, qb);
    collect_ghosts<NDIM, 0>(g, A, pc, bx, dJdK, qb);
    rb += qb[0];
#pragma unroll
    for (int q = 0; q < NDIM; ++q) ub[q] += qb[1 + q];
    pb += qb[HaloQ<NDIM>::nq - 2];
    Tb += qb[HaloQ<NDIM>::nq - 1];
  }
  if (g.source == SRC_MASSFLUX)  // energy source f u: u-bar += Rb_E f
    ub[0] += (A.bcoef * A.dtp[0] * wv[nd + 1]) * A.src[0];
  double rho = Vc[0];
  double ir = 1.0 / rho;
  double u[3] = {Vc[1] * ir, nd >= 2 ? Vc[2] * ir : 0.0, nd >= 3 ? Vc[3] * ir : 0.0};
  double E = Vc[nd + 1];
  double k2 = u[0] * u[0] + u[1] * u[1] + u[2] * u[2];
  double p = (g.gamma - 1.0) * (E - 0.5 * rho * k2);
  double T = p / (rho * g.R);
  pb += Tb / (rho * g.R);
  rb -= Tb * T * ir;
  const double gm1 = g.gamma - 1.0;
  double Ub[5];
  Ub[0] = rb + gm1 * 0.5 * k2 * pb;
#pragma unroll
  for (int d = 0; d < nd; ++d) {
    Ub[1 + d] = ub[d] * ir - gm1 * u[d] * pb;
    Ub[0] -= ub[d] * u[d] * ir;
  }
  Ub[nd + 1] = gm1 * pb;
#pragma unroll
  for (int v = 0; v < nd + 2; ++v) {
    const long x = (long)v * nc + c;
    const double w = wv[v];
    double vb = b * w + Ub[v];
    if (fold) {
      const double accv = ((0.0 + a3 * f3[v]) + a2 * f2[v]) + a * w;
      Vb[x] = accv + vb;
    } else {
      Vb[x] = vb;
    }
  }
}

// ---------------------------------------------------------------------------
// Host sequencing.
// ---------------------------------------------------------------------------
using AdjKernel = void (*)(Dev, AdjBuffers);
using AdjAllKernel = void (*)(Dev, AdjBuffers, DirGroups);

template <bool VISC, int NWV> static AdjKernel dir_kernel_t(int nd, int D) {
  if (nd == 1) return k_dir_vjp<1, 0, VISC, 4>;  // (x tiles: 4 lines)
  if (D == 0) return k_dir_vjp<3, 0, VISC, 4>;
  return D == 1 ? k_dir_vjp<3, 1, VISC, NWV> : k_dir_vjp<3, 2, VISC, NWV>;
}
static AdjKernel dir_kernel(int nd, int D, bool visc, int nwv) {
  if (nwv == 8) return visc ? dir_kernel_t<true, 8>(nd, D) : dir_kernel_t<false, 8>(nd, D);
  return visc ? dir_kernel_t<true, 4>(nd, D) : dir_kernel_t<false, 4>(nd, D);
}
template <int NWV> static AdjAllKernel all_kernel(int nd, bool visc) {
  if (nd == 3) return visc ? k_dir_vjp_all<3, true, NWV> : k_dir_vjp_all<3, false, NWV>;
  return visc ? k_dir_vjp_all<2, true, NWV> : k_dir_vjp_all<2, false, NWV>;
}

static inline unsigned blocks(long n) { return (unsigned)((n + 255) / 256 > 0 ? (n + 255) / 256 : 1); }

#define DCF_TRY(x)                    \
  do {                                \
    hipError_t e_ = (x);              \
    if (e_ != hipSuccess) return e_;  \
  } while (0)

// dJ/d(A, kappa) of the disturbance faces of axis d from the columns' sums.
static hipError_t disturb_sums(const Dev &g, const AdjBuffers &A, int d, double *dJdK,
                               hipStream_t st) {
  if (!dJdK) return hipSuccess;
  for (int side = 0; side < 2; ++side) {
    const int face = 2 * d + side;
    if (g.bck[face] != BC_DISTURB) continue;
    k_disturb_sum<<<1, 256, 0, st>>>(g, A.dpart + face * A.dcols, disturb_cols(g, d), face,
                                     dJdK + g.doff[face]);
    DCF_TRY(hipGetLastError());
  }
  return hipSuccess;
}

// Reverse of one stage: Vb = b Wb + R'(V)^T (b dt Wb), accumulators as in
// k_interior_vjp.  Needs g.Q to hold nothing on entry (recomputed here), and
// the adjoint boxes (Qb, Gb) zero wherever no kernel of a stage writes them
// (cleared once with the workspace; the kernels keep it so).
static hipError_t stage_vjp(const Dev &g, const AdjBuffers &A0, const double *V, const double *Wb,
                            const double *dt, double a, double b, double *Vb,
                            const double *w3, double a3, const double *w2, double a2,
                            int fold, double *dJdK,
                            hipStream_t st, bool have_box) {
  const bool visc = g.visc != VISC_NONE;
  AdjBuffers A = A0;
  A.Wb = Wb;
  A.dtp = dt;
  A.bcoef = b;
  if (!have_box) DCF_TRY(launch_prim_halo(g, V, st));  // the stage's primitive box
  if (g.source == SRC_MASSFLUX) {
    // the stage's body force f (as the forward stage computed it) and f-bar
    StageArgs F = {};
    F.Uin = V;
    if (stage_force_from_state(g)) {
      DCF_TRY(launch_stage_force(g, F, A.spart + RED_BLOCKS, st));
    } else {
      DCF_TRY(launch_force_direct(g, A.spart, A.src, st));
    }
    const unsigned nb = (unsigned)std::min<long>((g.ncell + 255) / 256, RED_BLOCKS);
    k_force_adj_partial<<<nb, 256, 0, st>>>(g, A);
    k_force_adj_final<<<1, 256, 0, st>>>(g, A, (int)nb, F.fpart, F.nfpart);
    DCF_TRY(hipGetLastError());
  }
  const bool all3 = adjoint_all3(g);
  if (g.ndim == 2 || all3) {
    DirGroups G = {};
    unsigned nblk = 0u;
    const int nwv = dir_waves(g, 0, g.ndim);
    for (int D = 0; D < g.ndim; ++D) {
      G.c[D] = (tile_count<-3, 2>(g, D, nwv) + 7u) / 8u;
      nblk += 8u * G.c[D];
    }
    auto k = nwv == 8 ? all_kernel<8>(g.ndim, visc) : all_kernel<4>(g.ndim, visc);
    k<<<nblk, 64 * nwv, 0, st>>>(g, A, G);
    DCF_TRY(hipGetLastError());
  } else {
    for (int D = 0; D < g.ndim; ++D) {
      const int nwv = D == 0 ? 4 : dir_waves(g, D, D + 1);
      hipLaunchKernelGGL(dir_kernel(g.ndim, D, visc, nwv), dim3(tile_count<-3, 2>(g, D, nwv)),
                         dim3(64 * nwv), 0, st, g, A);
      DCF_TRY(hipGetLastError());
    }
  }
  const bool dist_z = g.ndim == 3 && (g.bck[4] == BC_DISTURB || g.bck[5] == BC_DISTURB);
  if (visc || g.ndim == 2 || all3 || dist_z) {  // (else the tiles left the ghosts complete)
    auto gk = g.ndim == 1 ? k_ghost_vjp<1, false>
                          : (g.ndim == 2 ? k_ghost_vjp<2, false>
                                         : (all3 ? k_ghost_vjp<3, true> : k_ghost_vjp<3, false>));
    long ng = 0;
    for (int d = 0; d < g.ndim; ++d) ng += 6L * (g.ncell / g.n[d]);
    gk<<<(unsigned)((ng + 63) / 64), 64, 0, st>>>(g, A, dJdK ? 1 : 0);
    DCF_TRY(hipGetLastError());
  }
  auto ik = g.ndim == 1 ? k_interior_vjp<1, false>
                        : (g.ndim == 2 ? k_interior_vjp<2, false>
                                       : (all3 ? k_interior_vjp<3, true>
                                               : k_interior_vjp<3, false>));
  ik<<<blocks(g.ncell), 256, 0, st>>>(g, A, V, Wb, a, b, Vb, w3, a3, w2, a2, fold, dJdK);
  DCF_TRY(hipGetLastError());
  for (int d = g.ndim - 1; d >= 0; --d) DCF_TRY(disturb_sums(g, A, d, dJdK, st));
  return hipSuccess;
}

hipError_t vjp_step(Dev g, const AdjBuffers &A, const double *Un, const double *U1,
                    const double *U2, const double *dt, const double *lam1, double *lam0,
                    double *dJdK, hipStream_t st, const Dev *boxes) {
  const bool have = boxes != nullptr;  // stage boxes cached by the forward recompute
  const Dev &g3 = have ? boxes[2] : g, &g2 = have ? boxes[1] : g, &g1 = have ? boxes[0] : g;
  // stage 3: W = Un/3 + 2/3 (U2 + dt R(U2))
  DCF_TRY(stage_vjp(g3, A, U2, lam1, dt, 1.0 / 3.0, 2.0 / 3.0, A.Ub2, nullptr, 0.0, nullptr, 0.0,
                    0, dJdK, st, have));
  // stage 2: W = 3/4 Un + 1/4 (U1 + dt R(U1))
  DCF_TRY(stage_vjp(g2, A, U1, A.Ub2, dt, 0.75, 0.25, A.Ub1, nullptr, 0.0, nullptr, 0.0, 0, dJdK,
                    st, have));
  // stage 1: W = Un + dt R(Un)
  // (Un enters stage 3 with weight 1/3 and stage 2 with 3/4)
  DCF_TRY(stage_vjp(g1, A, Un, A.Ub1, dt, 0.0, 1.0, lam0, lam1, 1.0 / 3.0, A.Ub2, 0.75, 1, dJdK,
                    st, have));
  return hipSuccess;
}

}  // namespace dcf
