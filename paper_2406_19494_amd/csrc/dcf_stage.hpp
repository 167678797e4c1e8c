// dcf_stage.hpp -- device code of the fused Runge-Kutta stage: the flux of one
// face in its own frame, the primitives of a cell or ghost cell converted while
// a tile is loaded, and the update of one cell.
#pragma once

#include "dcf_cells.hpp"
#include "dcf_kernels.hpp"

namespace dcf {

// The step size of a stage (all NT threads; sh: NT / 64 doubles).
template <int NT>
__device__ __forceinline__ double stage_dt(const StageArgs &A, bool first, double *sh) {
  if (A.Rout) return 0.0;
  if (!A.part) return A.dt[0];
  double m = 0.0;
  for (int b = threadIdx.x; b < A.nparts; b += NT) m = fmax(m, A.part[b]);
  m = block_max<NT>(m, sh);
  const double dt = fmin(A.dt_max, A.cfl / m);
  if (first && threadIdx.x == 0) A.dt_out[0] = dt;
  return dt;
}

// The body force from the partial sums of k_force3 (all NT threads; sh: NT / 64
// doubles): f = -(volume sum of the x-momentum right-hand side) / volume.
template <int NT>
__device__ __forceinline__ double stage_force(const Dev &g, const StageArgs &A, double *sh) {
  if (!A.fpart) return 0.0;
  double v = 0.0;
  for (int b = threadIdx.x; b < A.nfpart; b += NT) v += A.fpart[b];
  return -block_total<NT>(v, sh) / g.vol;
}

// Primitives (rho, u, v, w, p, T, mu) of cell p of the state U when it is an
// interior cell or its image along periodic axes (at most three cells
// outside); false for the other ghost cells, which follow the halo chain.
template <int NDIM, bool VISC>
__device__ __forceinline__ bool load_prims(const Dev &g, const double *U, const int *p,
                                           double *q) {
  int w[3] = {0, 0, 0};
  bool inside = true, own = true;
#pragma unroll
  for (int d = 0; d < NDIM; ++d) {
    const int n = g.n[d];
    int x = p[d];
    own = own && x >= 0 && x < n;
    if (g.bck[2 * d] == BC_PERIODIC) x = x < 0 ? x + n : (x >= n ? x - n : x);
    inside = inside && x >= 0 && x < n;
    w[d] = x;
  }
  if (!inside) return false;
  const long nc = g.ncell;
  const long c = ((long)w[2] * g.n[1] + w[1]) * g.n[0] + w[0];
  double s[5];
  s[0] = U[c];
  s[1] = U[nc + c];
  s[2] = NDIM >= 2 ? U[2 * nc + c] : 0.0;
  s[3] = NDIM >= 3 ? U[3 * nc + c] : 0.0;
  s[4] = U[(NDIM + 1) * nc + c];
  prim_of_state_t<NDIM>(g, s, q);
  if (own && !(finite_pos(q[QR]) && finite_pos(q[QP]))) atomicOr(g.flags, 1u);
  if (VISC) q[QMU] = viscosity(g, q[QT]);
  return true;
}

// Total flux F = F^c - F^d (Eq. (6)) at one face in the face's own frame:
// G = (mass, normal, first and second tangential momentum, energy).  P(m, o)
// is primitive m (rho, u_n, u_t1, u_t2, p, T, mu) of the cell at offset o from
// the face (o = -3 .. 2; the face lies between offsets -1 and 0); Dv(r, o) the
// tangential velocity derivatives of that cell: r = 0 the tangential
// divergence d u_t1/d t1 + d u_t2/d t2, r = 1, 2 d u_n/d t1, d u_n/d t2.  mf is
// d xi/d n at the face.  False when the flux is not finite.
template <int NDIM, bool VISC, int SCH, bool PRELOAD, class PA, class DA>
__device__ __forceinline__ bool frame_flux(const Dev &g, const PA &P, const DA &Dv, double mf,
                                           double *G) {
  constexpr bool SIX = SCH == SCHEME_TENO6A;
  constexpr bool on[7] = {true, true, NDIM >= 2, NDIM >= 3, true, VISC, VISC};
  // PRELOAD: the reconstructions' stencils first, and the other loads before
  // the Riemann solver, so that a face waits for LDS twice instead of 20 times
  // (at 80 VGPRs; without, each variable's are read where they are used)
  double v[7][6];
  auto load = [&](int m) {
#pragma unroll
    for (int o = -3; o < 3; ++o)
      v[m][o + 3] = on[m] && (m < 5 || SIX || (o >= -2 && o < 2)) ? P(m, o) : 0.0;
  };
  double dv[3][6];
  auto load_d = [&](int r) {
#pragma unroll
    for (int o = -3; o < 3; ++o) dv[r][o + 3] = SIX || (o >= -2 && o < 2) ? Dv(r, o) : 0.0;
  };
  if (PRELOAD) {
#pragma unroll
    for (int m = 0; m < 5; ++m) load(m);
    __builtin_amdgcn_sched_barrier(0);  // (the scheduler would sink them to their uses)
  }
  double qL[5], qR[5];
#pragma unroll
  for (int m = 0; m < 5; ++m) {
    if (!on[m]) {
      qL[m] = qR[m] = 0.0;
      continue;
    }
    if (!PRELOAD) load(m);
    const double *x = v[m];
    if (SIX)
      teno6a_pair(x[0], x[1], x[2], x[3], x[4], x[5], qL[m], qR[m]);
    else
      weno5_pair(x[0], x[1], x[2], x[3], x[4], x[5], qL[m], qR[m]);
  }
  if (SIX) {
    // interpolation limiter: a side whose reconstructed density or pressure
    // is not positive takes its own cell's primitives (first order)
    if (!(qL[0] > 0.0 && qL[4] > 0.0))
#pragma unroll
      for (int m = 0; m < 5; ++m) qL[m] = v[m][2];
    if (!(qR[0] > 0.0 && qR[4] > 0.0))
#pragma unroll
      for (int m = 0; m < 5; ++m) qR[m] = v[m][3];
  }
  if (PRELOAD && VISC) {
    __builtin_amdgcn_sched_barrier(0);
    load(5);
    load(6);
#pragma unroll
    for (int r = 0; r < NDIM && NDIM > 1; ++r) load_d(r);
    __builtin_amdgcn_sched_barrier(0);
  }
  hllc(qL, qR, g.gamma, g.gm1i, G);
  // Dissipative flux (Eqs. (4)-(5), Fourier's law): 4th-order (TENO6-A:
  // 6th-order) central interpolation and differences
  double tn = 0.0, t1 = 0.0, t2 = 0.0, en = 0.0;
  if constexpr (VISC) {
    auto face = [&](const double *x) {
      return SIX ? interp6(x[0], x[1], x[2], x[3], x[4], x[5])
                 : interp4(x[1], x[2], x[3], x[4]);
    };
    auto diff = [&](const double *x) {
      return (SIX ? dface6(x[0], x[1], x[2], x[3], x[4], x[5])
                  : dface4(x[1], x[2], x[3], x[4])) * mf;
    };
    auto tangential = [&](int r) {
      if (!PRELOAD) load_d(r);
      return face(dv[r]);
    };
    if (!PRELOAD) {
      asm volatile("" ::: "memory");  // read again, not held since
#pragma unroll
      for (int m = 1; m < 7; ++m)
        if (m != 4) load(m);
    }
    const double muf = face(v[6]);
    tn = (4.0 / 3.0) * diff(v[1]);
    if constexpr (NDIM >= 2) tn -= (2.0 / 3.0) * tangential(0);
    tn *= muf;
    en = face(v[1]) * tn + muf * g.cpPr * diff(v[5]);
    if constexpr (NDIM >= 2) {
      t1 = muf * (tangential(1) + diff(v[2]));
      en += face(v[2]) * t1;
    }
    if constexpr (NDIM >= 3) {
      t2 = muf * (tangential(2) + diff(v[3]));
      en += face(v[3]) * t2;
    }
  }
  G[1] -= tn;
  G[2] -= t1;
  G[3] -= t2;
  G[4] -= en;
  return fabs(G[0]) + fabs(G[4]) < 1.0e300;
}

// What the update of one cell reads, loaded before the face fluxes so that the
// memory round trip passes while they are computed.
template <int NDIM> struct CellIn {
  double un[NDIM + 2], ui[NDIM + 2], id[NDIM];
};

template <int NDIM>
__device__ __forceinline__ void load_cell(const Dev &g, const StageArgs &A, const int *p,
                                          CellIn<NDIM> &in) {
  const long nc = g.ncell;
  const long c = ((long)(NDIM >= 3 ? p[2] : 0) * g.n[1] + (NDIM >= 2 ? p[1] : 0)) * g.n[0] + p[0];
#pragma unroll
  for (int v = 0; v < NDIM + 2; ++v) {
    in.un[v] = A.Un[v * nc + c];
    in.ui[v] = A.Uin[v * nc + c];
  }
#pragma unroll
  for (int d = 0; d < NDIM; ++d) in.id[d] = g.idx[d][p[d]];
}

// The stage update of the cell at p from its right-hand side R (rho, the
// three momenta, E): source, then Uout = a Un + b (Uin + dt R), or R itself.
// Returns the signal rate of the new state when want_sigma.
template <int NDIM>
__device__ __forceinline__ double update_state(const Dev &g, const StageArgs &A, const int *p,
                                               const CellIn<NDIM> &in, double dt, double *R,
                                               bool want_sigma) {
  constexpr int NV = NDIM + 2;
  const long nc = g.ncell;
  const long c = ((long)(NDIM >= 3 ? p[2] : 0) * g.n[1] + (NDIM >= 2 ? p[1] : 0)) * g.n[0] + p[0];
  if (A.force) {
    const double f = A.force[0];
    R[1] += f;
    R[4] += f * (in.ui[1] * rcp_nr(in.ui[0]));
  }
  if (A.Rout) {
#pragma unroll
    for (int v = 0; v < NV; ++v) A.Rout[v * nc + c] = R[v == NV - 1 ? 4 : v];
    return 0.0;
  }
  double st[5] = {0.0, 0.0, 0.0, 0.0, 0.0};
#pragma unroll
  for (int v = 0; v < NV; ++v) {
    const double uo = A.a * in.un[v] + A.b * (in.ui[v] + dt * R[v == NV - 1 ? 4 : v]);
    A.Uout[v * nc + c] = uo;
    st[v == NV - 1 ? 4 : v] = uo;
  }
  if (!want_sigma) return 0.0;
  double q[6];
  prim_of_state_t<NDIM>(g, st, q);
  return cell_sigma(g, q, p);
}

}  // namespace dcf
