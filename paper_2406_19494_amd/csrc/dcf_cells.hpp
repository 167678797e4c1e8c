// dcf_cells.hpp -- per-cell device functions shared by the kernels: conversion
// between conserved and primitive variables, the ghost-cell chain of the halo
// fill, the signal rate of the CFL step, and workgroup reductions.
#pragma once

#include "dcf_common.hpp"

namespace dcf {

// ---------------------------------------------------------------------------
// Primitives from conserved variables (Eq. (2), ideal gas).
// ---------------------------------------------------------------------------
// From (rho, rho u, rho v, rho w, E) with zeros for unused momenta.
template <int NDIM>
__device__ __forceinline__ void prim_of_state_t(const Dev &g, const double *s, double *q) {
  double rho = s[0];
  double ir = rcp_nr(rho);
  double u = s[1] * ir;
  double v = NDIM >= 2 ? s[2] * ir : 0.0;
  double w = NDIM >= 3 ? s[3] * ir : 0.0;
  double E = s[4];
  double p = (g.gamma - 1.0) * (E - 0.5 * rho * (u * u + v * v + w * w));
  q[QR] = rho;
  q[QU] = u;
  q[QV] = v;
  q[QW] = w;
  q[QP] = p;
  q[QT] = p * ir * g.iR;
}
__device__ __forceinline__ void prim_of_state(const Dev &g, const double *s, double *q) {
  if (g.ndim == 3) prim_of_state_t<3>(g, s, q);
  else if (g.ndim == 2) prim_of_state_t<2>(g, s, q);
  else prim_of_state_t<1>(g, s, q);
}

__device__ __forceinline__ void cons_to_prim(const Dev &g, const double *U, long c, double *q) {
  const int nd = g.ndim;
  const long nc = g.ncell;
  double rho = U[c];
  double ir = rcp_nr(rho);
  double u = U[nc + c] * ir;
  double v = nd >= 2 ? U[2 * nc + c] * ir : 0.0;
  double w = nd >= 3 ? U[3 * nc + c] * ir : 0.0;
  double E = U[(long)(nd + 1) * nc + c];
  double p = (g.gamma - 1.0) * (E - 0.5 * rho * (u * u + v * v + w * w));
  q[QR] = rho;
  q[QU] = u;
  q[QV] = v;
  q[QW] = w;
  q[QP] = p;
  q[QT] = p * ir * g.iR;
}

// ---------------------------------------------------------------------------
// Primitive box with halos.  The halo fill of the paper (values assigned to
// halo cells, Section 3.2) is applied axis by axis, x then y then z, each
// over the full extent of the axes filled before; a ghost thread resolves
// that chain for its own cell: it follows the source cells back to the
// interior (or to a Dirichlet profile) and applies the per-axis ghost
// transforms in x, y, z order.
// ---------------------------------------------------------------------------
// Source cell of ghost layer m (0 nearest the face) on side `side` of an axis of
// n cells.
__device__ __forceinline__ int ghost_source(int kind, int side, int m, int n) {
  if (kind == BC_PERIODIC) return side == 0 ? n - 1 - m : m;
  if (kind == BC_ZEROGRAD) return side == 0 ? 0 : n - 1;
  return side == 0 ? m : n - 1 - m;  // walls mirror
}

// Sources of the ghost chain: the conserved state (the source cell is
// converted here), the primitive box once its interior is filled, or the LDS
// window of a tile once its interior and periodic cells are (the source's
// primitives and mu are copied).  A window holds the images of periodic axes,
// so it is addressed by the source without their wrap.
struct FromState {
  const double *U;
  __device__ __forceinline__ void load(const Dev &g, const int *s, const int *, double *q,
                                       double &mu) const {
    cons_to_prim(g, U, ((long)s[2] * g.n[1] + s[1]) * g.n[0] + s[0], q);
    mu = -1.0;
  }
  __device__ __forceinline__ double pressure(const Dev &g, const int *w, const int *) const {
    double q[6];
    cons_to_prim(g, U, ((long)w[2] * g.n[1] + w[1]) * g.n[0] + w[0], q);
    return q[QP];
  }
};
struct FromBox {
  __device__ __forceinline__ void load(const Dev &g, const int *s, const int *, double *q,
                                       double &mu) const {
    const int nd = g.ndim;
    const long sb = bidx(g, s[0], s[1], s[2]);
    q[QR] = g.Q[QR][sb];
    q[QU] = g.Q[QU][sb];
    q[QV] = nd >= 2 ? g.Q[QV][sb] : 0.0;
    q[QW] = nd >= 3 ? g.Q[QW][sb] : 0.0;
    q[QP] = g.Q[QP][sb];
    if (g.visc != VISC_NONE) {
      q[QT] = g.Q[QT][sb];
      mu = g.Q[QMU][sb];
    } else {
      q[QT] = q[QP] * rcp_nr(q[QR]) * g.iR;  // as prim_of_state, to the bit
      mu = -1.0;
    }
  }
  __device__ __forceinline__ double pressure(const Dev &g, const int *w, const int *) const {
    return g.Q[QP][bidx(g, w[0], w[1], w[2])];
  }
};

// Window of a tile: NP arrays of PS values (rho, the NDIM velocities, p and,
// viscous, T, mu), x and y from (x0, y0) with pitch W.
template <int NDIM, bool VISC> struct FromWindow {
  const double *lds;
  int x0, y0, W, PS;
  __device__ __forceinline__ void load(const Dev &g, const int *, const int *sw, double *q,
                                       double &mu) const {
    const double *v = lds + (NDIM >= 2 ? (sw[1] - y0) * W : 0) + sw[0] - x0;
    q[QR] = v[0];
    q[QU] = v[PS];
    q[QV] = NDIM >= 2 ? v[2 * PS] : 0.0;
    q[QW] = NDIM >= 3 ? v[3 * PS] : 0.0;
    q[QP] = v[(NDIM + 1) * PS];
    if (VISC) {
      q[QT] = v[(NDIM + 2) * PS];
      mu = v[(NDIM + 3) * PS];
    } else {
      q[QT] = q[QP] * rcp_nr(q[QR]) * g.iR;
      mu = -1.0;
    }
  }
  __device__ __forceinline__ double pressure(const Dev &g, const int *, const int *ww) const {
    return lds[(NDIM + 1) * PS + (NDIM >= 2 ? (ww[1] - y0) * W : 0) + ww[0] - x0];
  }
};

// Primitives of ghost cell p through the halo-fill chain: follow the source
// cells back to the interior (or to a Dirichlet profile), then apply the
// per-axis ghost transforms in x, y, z order.  mu is left negative unless the
// source's is still valid (copied and no transform changed T).
template <int NDIM, class Src>
__device__ __forceinline__ void ghost_value(const Dev &g, const int *p, const Src &src, double *q,
                                            double &mu) {
  constexpr int nd = NDIM;
  int s[3] = {p[0], p[1], p[2]};
  int sw[3] = {p[0], p[1], p[2]};  // the source without the wrap of periodic axes
  int side[3] = {0, 0, 0};
  bool gh[3] = {false, false, false};
  int top = -1;
#pragma unroll
  for (int d = 0; d < nd; ++d) {
    if (p[d] < 0 || p[d] >= g.n[d]) {
      gh[d] = true;
      side[d] = p[d] < 0 ? 0 : 1;
      int m = side[d] == 0 ? -1 - p[d] : p[d] - g.n[d];
      int kind = g.bck[2 * d + side[d]];
      if (kind == BC_DIRICHLET)
        top = d;
      else
        s[d] = ghost_source(kind, side[d], m, g.n[d]);
      if (kind != BC_PERIODIC) sw[d] = s[d];
    }
  }
  mu = -1.0;  // mu of the source while no transform changed T
  int start = 0;
  if (top >= 0) {
#pragma unroll
    for (int d = 0; d < nd; ++d) {  // (static register indices)
      if (d != top) continue;
      const int t1 = tan1(d), t2 = tan2(d);
      int a = t1 < nd ? (t1 < d ? p[t1] : s[t1]) : 0;
      int bb = t2 < nd ? (t2 < d ? p[t2] : s[t2]) : 0;
      a = min(max(a, 0), g.n[t1] - 1);
      bb = min(max(bb, 0), g.n[t2] - 1);
      const long nt = (long)g.n[t1] * g.n[t2];
      const long o = (long)bb * g.n[t1] + a;
      const double *P = g.dir[2 * d + side[d]];
      q[QR] = P[o];
      q[QU] = P[nt + o];
      q[QV] = P[2 * nt + o];
      q[QW] = P[3 * nt + o];
      q[QP] = P[4 * nt + o];
    }
    q[QT] = q[QP] / (q[QR] * g.R);
    mu = -1.0;  // recomputed by the caller
    start = top + 1;
  } else {
    src.load(g, s, sw, q, mu);  // the interior source cell
  }
#pragma unroll
  for (int d = 0; d < nd; ++d) {
    if (d < start || !gh[d]) continue;
    const int face = 2 * d + side[d];
    const int kind = g.bck[face];
    if (!is_wall(kind)) continue;  // copies keep the value
    double src_n = q[QU + d];
    q[QU] = -q[QU];
    q[QV] = -q[QV];
    q[QW] = -q[QW];
    const int t1 = tan1(d), t2 = tan2(d);
    const int a = t1 < nd ? (t1 < d ? p[t1] : s[t1]) : 0;
    const int bb = t2 < nd ? (t2 < d ? p[t2] : s[t2]) : 0;
    const double sigma = side[d] == 0 ? 1.0 : -1.0;
    if (kind == BC_POROUS && face == g.pface) {
      if (a >= g.pb && a < g.pe && bb >= 0 && bb < g.n[t2]) {
        // Darcy transpiration through the porous strip: inward-normal
        // velocity -K (p_w - p_inf)/p_inf, p_w of the first interior cell.
        int w[3];
        w[d] = side[d] == 0 ? 0 : g.n[d] - 1;
        w[t1] = a;
        w[t2] = bb;
        int ww[3];
        ww[d] = w[d];
        ww[t1] = t1 < nd ? (t1 < d ? p[t1] : sw[t1]) : 0;
        ww[t2] = t2 < nd ? (t2 < d ? p[t2] : sw[t2]) : 0;
        const double pw = src.pressure(g, w, ww);
        int kk = bb * (g.pe - g.pb) + (a - g.pb);
        double vn = -g.K[kk] * (pw - g.pinf) / g.pinf;
        q[QU + d] = 2.0 * sigma * vn - src_n;
      }
    } else if (kind == BC_DISTURB && a >= 0 && a < g.n[t1]) {
      // Disturbance wall (Section 3.2, Eq. (8)): prescribed inward-normal
      // velocity A sin(2 pi kappa x) at the wall-face centre, (A, kappa)
      // taken from the boundary parameters.
      const double *th = g.K + g.doff[face];
      double vn = th[0] * sin(2.0 * M_PI * g.xm[t1][a] * th[1]);
      q[QU + d] = 2.0 * sigma * vn - src_n;
    }
    if (g.Tw[face] > 0.0) {  // isothermal; adiabatic keeps rho and T
      double Tg = 2.0 * g.Tw[face] - q[QT];
      if (!(Tg > 0.0)) atomicOr(g.flags, 1u);
      q[QT] = Tg;
      q[QR] = q[QP] / (g.R * Tg);
      mu = -1.0;
    }
  }
}

// Ghost cell p written into the box (index b).
template <int NDIM, class Src>
__device__ __forceinline__ void ghost_chain_t(const Dev &g, const int *p, long b, const Src &src) {
  double q[6], mu;
  ghost_value<NDIM>(g, p, src, q, mu);
  g.Q[QR][b] = q[QR];
  g.Q[QU][b] = q[QU];
  if (NDIM >= 2) g.Q[QV][b] = q[QV];
  if (NDIM >= 3) g.Q[QW][b] = q[QW];
  g.Q[QP][b] = q[QP];
  if (g.visc != VISC_NONE) {
    g.Q[QT][b] = q[QT];
    g.Q[QMU][b] = mu >= 0.0 ? mu : viscosity(g, q[QT]);
  }
}
template <class Src>
__device__ __forceinline__ void ghost_chain(const Dev &g, const int *p, long b, const Src &src) {
  if (g.ndim == 3) ghost_chain_t<3>(g, p, b, src);
  else if (g.ndim == 2) ghost_chain_t<2>(g, p, b, src);
  else ghost_chain_t<1>(g, p, b, src);
}

// Signal rate of one cell, sum_d (|u_d| + c)/dx_d + 2 nu_eff sum_d 1/dx_d^2
// (nu_eff = max(4/3, gamma/Pr) mu/rho); dt = cfl / max over cells.
__device__ __forceinline__ double cell_sigma(const Dev &g, const double *q, const int *pos,
                                             int law) {
  double y;  // 1 / (rho cs)
  double cs = sound_speed(g.gamma, q[QR], q[QP], y);
  double conv = 0.0, inv2 = 0.0;
  for (int d = 0; d < g.ndim; ++d) {
    double id = g.idx[d][pos[d]];
    conv += (fabs(q[QU + d]) + cs) * id;
    inv2 += id * id;
  }
  double sig = conv;
  if (law != VISC_NONE) {
    double mu = viscosity(g, q[QT], law);
    double nu = fmax(4.0 / 3.0, g.gamma / g.Pr) * mu * (cs * y);  // mu / rho
    sig += 2.0 * nu * inv2;
  }
  if (!(sig < 1.0e300)) sig = 1.0e300;  // non-finite: flagged elsewhere
  return sig;
}

__device__ __forceinline__ double cell_sigma(const Dev &g, const double *q, const int *pos) {
  return cell_sigma(g, q, pos, g.visc);
}

// Maximum over a workgroup of NT threads (whole wavefronts): within each
// 64-lane wavefront by lane exchanges, then over the wavefronts through LDS
// (sh: NT / 64 doubles).  The maximum is exact, so its value does not depend
// on the order.
template <int NT = 256>
__device__ __forceinline__ double block_max(double v, double *sh) {
#pragma unroll
  for (int off = 32; off > 0; off >>= 1) v = fmax(v, __shfl_xor(v, off, 64));
  __syncthreads();  // a previous call's readers of sh are done
  if (threadIdx.x % 64 == 0) sh[threadIdx.x / 64] = v;
  __syncthreads();
  double m = sh[0];
#pragma unroll
  for (int w = 1; w < NT / 64; ++w) m = fmax(m, sh[w]);
  return m;
}

// Sum over a workgroup of NT threads, likewise; a fixed order (pairs of lanes,
// then the wavefronts in turn).
template <int NT>
__device__ __forceinline__ double block_total(double v, double *sh) {
#pragma unroll
  for (int off = 32; off > 0; off >>= 1) v += __shfl_xor(v, off, 64);
  __syncthreads();  // a previous call's readers of sh are done
  if (threadIdx.x % 64 == 0) sh[threadIdx.x / 64] = v;
  __syncthreads();
  double m = sh[0];
#pragma unroll
  for (int w = 1; w < NT / 64; ++w) m += sh[w];
  return m;
}

}  // namespace dcf
