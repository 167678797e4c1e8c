// dcf_stage.hip -- one launch per Runge-Kutta stage: a tile's cells and ghost
// cells are converted to primitives while they are loaded, every face flux of
// the tile is computed from LDS, and the stage update writes the new state.
#include <algorithm>

#include "dcf_stage.hpp"

namespace dcf {

// ---------------------------------------------------------------------------
// 1D.  A line of fewer than 1024 cells is stepped by one workgroup, one cell and
// one face per thread, with the state in registers: all stages of all steps of
// a call in one launch (a stage of 200 cells takes 1.5 us, a launch by itself
// 3.5; 10 CFL steps of 200 cells in a call: 393 us with five launches a stage,
// 57 so).  What bounds it is the chain of one face's flux and the barriers
// between its stages.  Longer lines take a launch per stage, in tiles of 255
// cells (256 faces): 4001 cells, 4 steps: 165 us with split launches, 68 so,
// launches and their starts.
// ---------------------------------------------------------------------------
template <bool VISC> struct Line1 {
  static constexpr int NP = VISC ? 5 : 3;  // rho, u, p (, T, mu)
};

// Flux of the face before window cell w (prims [NP][pitch]) into fl [3][fpitch].
template <bool VISC, int SCH>
__device__ __forceinline__ void line_face(const Dev &g, const double *w, int pitch, double mf,
                                          double *fl, int fpitch) {
  auto P = [&](int m, int o) {
    const int a = m < 2 ? m : (m == 4 ? 2 : m - 2);  // rho, u, p, T, mu
    return w[a * pitch + o];
  };
  auto Dv = [&](int, int) { return 0.0; };
  double G[5];
  if (!frame_flux<1, VISC, SCH, false>(g, P, Dv, mf, G)) atomicOr(g.flags, 1u);
  fl[0] = G[0];
  fl[fpitch] = G[1];
  fl[2 * fpitch] = G[4];
}

template <bool VISC>
__device__ __forceinline__ void line_store(const double *q, double *w, int pitch) {
  w[0] = q[QR];
  w[pitch] = q[QU];
  w[2 * pitch] = q[QP];
  if (VISC) {
    w[3 * pitch] = q[QT];
    w[4 * pitch] = q[QMU];
  }
}

// Ghost sources of a line whose interior is in the window.
template <bool VISC> struct FromLine {
  const double *w;  // of cell 0
  int pitch;
  __device__ __forceinline__ void load(const Dev &g, const int *s, const int *, double *q,
                                       double &mu) const {
    const double *v = w + s[0];
    q[QR] = v[0];
    q[QU] = v[pitch];
    q[QV] = q[QW] = 0.0;
    q[QP] = v[2 * pitch];
    q[QT] = VISC ? v[3 * pitch] : q[QP] * rcp_nr(q[QR]) * g.iR;
    mu = VISC ? v[4 * pitch] : -1.0;
  }
  __device__ __forceinline__ double pressure(const Dev &g, const int *s, const int *) const {
    return w[2 * pitch + s[0]];
  }
};

// nsteps steps of the line (n < NT) from U with step dt[0]; with cfl > 0 each
// step's CFL step replaces it and the last one goes to dt_next.  U1, U2
// (nullable): the stage states of the last step; nstages = 2 makes only those.
template <bool VISC, int SCH, int NT>
__device__ __forceinline__ void line_steps(const Dev &g, const LineArgs &A, double *lds) {
  constexpr int NP = Line1<VISC>::NP, PITCH = NT + 6;
  double *win = lds, *fl = lds + NP * PITCH;  // windows [NP][NT + 6], faces [3][NT]
  __shared__ double sh[NT / 64];
  const int t = threadIdx.x, n = g.n[0];
  const bool cell = t < n;
  const int pos[3] = {t, 0, 0};
  const double id = cell ? g.idx[0][t] : 0.0, mf = VISC ? g.mf[0][min(t, n)] : 0.0;
  double u[3] = {1.0, 0.0, 1.0}, un[3];
  if (cell)
#pragma unroll
    for (int v = 0; v < 3; ++v) u[v] = A.U[v * n + t];
  double dt = A.part ? 0.0 : A.dt[0];
  if (A.part) {  // the CFL step of these partial maxima
    double m = 0.0;
    for (int b = t; b < A.nparts; b += NT) m = fmax(m, A.part[b]);
    dt = A.cfl_first / block_max<NT>(m, sh);
    if (t == 0) A.dt_first[0] = dt;
  }
#pragma unroll 1
  for (int step = 0; step < A.nsteps; ++step) {
#pragma unroll
    for (int v = 0; v < 3; ++v) un[v] = u[v];
    double sig = 0.0;
#pragma unroll 1
    for (int k = 0; k < A.nstages; ++k) {
      const double a = k == 0 ? 0.0 : (k == 1 ? 0.75 : 1.0 / 3.0);
      const double b = k == 0 ? 1.0 : (k == 1 ? 0.25 : 2.0 / 3.0);
      double st[5] = {u[0], u[1], 0.0, 0.0, u[2]}, q[NQ];
      if (cell) {
        prim_of_state_t<1>(g, st, q);
        if (!(finite_pos(q[QR]) && finite_pos(q[QP]))) atomicOr(g.flags, 1u);
        if (VISC) q[QMU] = viscosity(g, q[QT]);
        line_store<VISC>(q, win + 3 + t, PITCH);
      }
      __syncthreads();
      if (t < 6) {
        const int p[3] = {t < 3 ? t - 3 : n + t - 3, 0, 0};
        double mu;
        ghost_value<1>(g, p, FromLine<VISC>{win + 3, PITCH}, q, mu);
        if (VISC) q[QMU] = mu >= 0.0 ? mu : viscosity(g, q[QT]);
        line_store<VISC>(q, win + 3 + p[0], PITCH);
      }
      __syncthreads();
      if (t <= n) line_face<VISC, SCH>(g, win + 3 + t, PITCH, mf, fl + t, NT);
      __syncthreads();
      if (cell) {
#pragma unroll
        for (int v = 0; v < 3; ++v) {
          double R = 0.0;
          R -= (fl[v * NT + t + 1] - fl[v * NT + t]) * id;
          u[v] = a * un[v] + b * (u[v] + dt * R);
        }
        double *keep = k == 0 ? A.U1 : (k == 1 ? A.U2 : nullptr);
        if (keep && step == A.nsteps - 1)
#pragma unroll
          for (int v = 0; v < 3; ++v) keep[v * n + t] = u[v];
        if (A.cfl > 0.0 && k == 2) {
          double sn[5] = {u[0], u[1], 0.0, 0.0, u[2]};
          prim_of_state_t<1>(g, sn, q);
          sig = cell_sigma(g, q, pos);
        }
      }
    }
    if (A.cfl > 0.0) dt = fmin(A.dt_max, A.cfl / block_max<NT>(sig, sh));
  }
  if (cell && A.nstages == 3)
#pragma unroll
    for (int v = 0; v < 3; ++v) A.U[v * n + t] = u[v];
  if (A.cfl > 0.0 && t == 0) A.dt_next[0] = dt;
}

template <bool VISC, int SCH, int NT>
__global__ void __launch_bounds__(NT) k_line(Dev g, LineArgs A) {
  __shared__ double lds[Line1<VISC>::NP * (NT + 6) + 3 * NT];
  line_steps<VISC, SCH, NT>(g, A, lds);
}

// One stage of a tile of 255 cells of a longer line.
template <bool VISC, int SCH>
__device__ __forceinline__ void stage1_tile(const Dev &g, const StageArgs &A, unsigned tile,
                                            double *lds) {
  constexpr int T = 255, NT = 256, NP = Line1<VISC>::NP, PITCH = T + 6;
  double *win = lds, *fl = lds + NP * PITCH;
  __shared__ double sh[NT / 64];
  const int t = threadIdx.x, n = g.n[0], i0 = (int)tile * T;
  const int pc[3] = {i0 + t, 0, 0};
  const bool cell = t < T && pc[0] < n;
  CellIn<1> in;
  if (cell) load_cell<1>(g, A, pc, in);
  const double dt = stage_dt<NT>(A, tile == 0, sh);
  const double mf = VISC ? g.mf[0][min(i0 + t, n)] : 0.0;
  for (int w = t; w < PITCH; w += NT) {
    const int p[3] = {i0 + w - 3, 0, 0};
    if (p[0] > n + 2) continue;
    double q[NQ], mu;
    if (!load_prims<1, VISC>(g, A.Uin, p, q)) {
      ghost_value<1>(g, p, FromState{A.Uin}, q, mu);
      if (VISC) q[QMU] = viscosity(g, q[QT]);
    }
    line_store<VISC>(q, win + w, PITCH);
  }
  __syncthreads();
  if (i0 + t <= n) line_face<VISC, SCH>(g, win + t + 3, PITCH, mf, fl + t, NT);
  __syncthreads();
  double sig = 0.0;
  if (cell) {
    double R[5] = {0.0, 0.0, 0.0, 0.0, 0.0};
#pragma unroll
    for (int v = 0; v < 3; ++v) {
      double r = 0.0;
      r -= (fl[v * NT + t + 1] - fl[v * NT + t]) * in.id[0];
      R[v == 2 ? 4 : v] = r;
    }
    sig = update_state<1>(g, A, pc, in, dt, R, A.dtpart != nullptr);
  }
  if (A.dtpart) {
    const double m = block_max<NT>(sig, sh);
    if (t == 0) A.dtpart[tile] = m;
  }
}

template <bool VISC, int SCH>
__global__ void __launch_bounds__(256) k_stage1(Dev g, StageArgs A) {
  __shared__ double lds[Line1<VISC>::NP * 261 + 3 * 256];
  stage1_tile<VISC, SCH>(g, A, blockIdx.x, lds);
}

// ---------------------------------------------------------------------------
// 2D: tiles of TX x TY cells, a window cell and a face per thread.  Bound by the
// latency of a tile's phases (window, derivatives, faces, update) at two
// workgroups of 8 wavefronts per CU: VALU busy 37 %, 48 % of a wavefront's
// cycles waiting for data, 23 MB of HBM traffic.  1024 x 256: 22 to 24 us per
// stage, 32 with ghost, x flux and y flux + update launches; 256 x 64: 8.0 and
// 18.
// ---------------------------------------------------------------------------
// SMALL: 12 x 8 cells and 4 wavefronts, else 16 x 16 cells and 8 wavefronts.
template <bool VISC, int SCH, bool SMALL> struct Tile2 {
  static constexpr int TX = SMALL ? 12 : 16, TY = SMALL ? 8 : 16;  // cells
  static constexpr int W = TX + 6, H = TY + 6;    // window cells
  static constexpr int NP = VISC ? 6 : 4;         // rho, u, v, p (, T, mu)
  // the derivative cells along a face's axis: offsets -2 .. 1 (fourth order)
  // or -3 .. 2 around each face
  static constexpr int HD = SCH == SCHEME_TENO6A ? 3 : 2;
  static constexpr int WX = TX + 2 * HD, NX = TY * WX;  // of the x faces, [TY][WX]
  static constexpr int WY = TY + 2 * HD, NY = WY * TX;  // of the y faces, [WY][TX]
  static constexpr int FX = TY * (TX + 1), FY = (TY + 1) * TX, NF = FX + FY;  // faces
  static constexpr int PR = 0;                    // [NP][H][W]
  static constexpr int DX = NP * W * H;           // [2][NX]: dv/dy, du/dy
  static constexpr int DY = DX + (VISC ? 2 * NX : 0);  // [2][NY]: du/dx, dv/dx
  static constexpr int FL = DY + (VISC ? 2 * NY : 0);  // [4][NF]
  static constexpr int SM = FL + 4 * NF;          // metrics: mf x, mf y, mc x, mc y
  static constexpr int MFY = TX + 1, MCX = MFY + TY + 1, MCY = MCX + TX;
  static constexpr int SIZE = SM + MCY + TY;      // doubles
  static constexpr int NT = SMALL ? 256 : 512;    // threads
  static_assert(W * H <= NT, "one window cell per thread");
};

template <bool VISC, int SCH, bool SMALL>
__device__ __forceinline__ void stage2_tile(const Dev &g, const StageArgs &A, unsigned tile,
                                            unsigned nbx, double *lds) {
  using L = Tile2<VISC, SCH, SMALL>;
  constexpr int TX = L::TX, TY = L::TY, W = L::W, WH = L::W * L::H, HD = L::HD, NT = L::NT;
  const int tid = threadIdx.x;
  const int i0 = (int)(tile % nbx) * TX, j0 = (int)(tile / nbx) * TY;
  const int nx = g.n[0], ny = g.n[1];
  double *pr = lds + L::PR, *sm = lds + L::SM;
  __shared__ double shx[NT / 64];
  // the inputs of this thread's cell
  const int tx = tid % TX, ty = tid / TX;
  const int pc[3] = {i0 + tx, j0 + ty, 0};
  const bool cell = ty < TY && pc[0] < nx && pc[1] < ny;
  CellIn<2> in;
  if (cell) load_cell<2>(g, A, pc, in);
  const double dt = stage_dt<NT>(A, tile == 0, shx);
  // metrics of the tile's faces and cells
  if (tid < TX + 1) sm[tid] = g.mf[0][min(i0 + tid, nx)];
  else if (tid >= 64 && tid <= 64 + TY) sm[L::MFY + tid - 64] = g.mf[1][min(j0 + tid - 64, ny)];
  else if (tid >= 128 && tid < 128 + TX) sm[L::MCX + tid - 128] = g.mc[0][min(i0 + tid - 128, nx - 1)];
  else if (tid >= 192 && tid < 192 + TY) sm[L::MCY + tid - 192] = g.mc[1][min(j0 + tid - 192, ny - 1)];
  // primitives of the window: the interior cells and periodic images from the
  // state, then (tiles at a boundary) the other ghost cells from the window
  auto store = [&](int w, const int *p, const double *q) {
    pr[w] = q[QR];
    pr[WH + w] = q[QU];
    pr[2 * WH + w] = q[QV];
    pr[3 * WH + w] = q[QP];
    if (VISC) {
      pr[4 * WH + w] = q[QT];
      pr[5 * WH + w] = q[QMU];
    }
    if (A.box.Q[0]) {
      // the box of Uin, each cell by the tile that holds its nearest
      // interior cell
      const int ci = min(max(p[0], 0), nx - 1), cj = min(max(p[1], 0), ny - 1);
      if (ci >= i0 && ci < i0 + TX && cj >= j0 && cj < j0 + TY) {
        const long b = bidx(g, p[0], p[1], 0);
        A.box.Q[QR][b] = q[QR];
        A.box.Q[QU][b] = q[QU];
        A.box.Q[QV][b] = q[QV];
        A.box.Q[QP][b] = q[QP];
        if (VISC) {
          A.box.Q[QT][b] = q[QT];
          A.box.Q[QMU][b] = q[QMU];
        }
      }
    }
  };
  bool ghost = false;
  const int pw[3] = {i0 + tid % W - 3, j0 + tid / W - 3, 0};
  if (tid < WH && pw[0] <= nx + 2 && pw[1] <= ny + 2) {
    double q[NQ];
    if (load_prims<2, VISC>(g, A.Uin, pw, q)) store(tid, pw, q);
    else ghost = true;
  }
  __syncthreads();
  if (i0 < 3 || j0 < 3 || i0 + TX + 3 > nx || j0 + TY + 3 > ny) {  // uniform
    if (ghost) {
      double q[NQ], mu;
      ghost_value<2>(g, pw, FromWindow<2, VISC>{pr, i0 - 3, j0 - 3, W, WH}, q, mu);
      if (VISC) q[QMU] = mu >= 0.0 ? mu : viscosity(g, q[QT]);
      store(tid, pw, q);
    }
    __syncthreads();
  }
  if constexpr (VISC) {
    // tangential velocity derivatives at the cells of the face stencils
    auto diff = [&](int w, int s) {  // pr + w: a velocity; s: window stride
      const double *v = pr + w;
      if (SCH == SCHEME_TENO6A)
        return dcell6(v[-3 * s], v[-2 * s], v[-s], v[s], v[2 * s], v[3 * s]);
      return dcell4(v[-2 * s], v[-s], v[s], v[2 * s]);
    };
    for (int d = tid; d < L::NX + L::NY; d += NT) {
      const bool yd = d >= L::NX;
      const int e = yd ? d - L::NX : d;
      int lx, ly;  // window position
      double m;
      if (!yd) {   // x faces: derivatives along y
        const int r = e / L::WX;
        ly = r + 3;
        lx = e % L::WX + 3 - HD;
        m = sm[L::MCY + r];
      } else {     // y faces: derivatives along x
        const int c = e % TX;
        lx = c + 3;
        ly = e / TX + 3 - HD;
        m = sm[L::MCX + c];
      }
      const int w = ly * W + lx, s = yd ? 1 : W;
      const int un = yd ? 2 * WH : WH, ut = yd ? WH : 2 * WH;  // normal, tangential velocity
      double *out = lds + (yd ? L::DY : L::DX) + e;
      out[0] = diff(ut + w, s) * m;
      out[yd ? L::NY : L::NX] = diff(un + w, s) * m;
    }
    __syncthreads();
  }
  // one face per thread (and a few for a second round): the x faces row by
  // row, then the y faces
  double *fl = lds + L::FL;
  for (int f = tid; f < L::NF; f += NT) {
    const bool yf = f >= L::FX;
    const int e = yf ? f - L::FX : f;
    const int r = yf ? e / TX : e / (TX + 1), c = yf ? e % TX : e % (TX + 1);
    if (i0 + c > nx - (yf ? 1 : 0) || j0 + r > ny - (yf ? 0 : 1)) continue;
    const double *q0 = pr + (r + 3) * W + c + 3;
    const int s = yf ? W : 1;
    const int on = yf ? 2 * WH : WH, ot = yf ? WH : 2 * WH;
    const double *d0 = lds + (yf ? L::DY + (r + HD) * TX + c : L::DX + r * L::WX + c + HD);
    const int sd = yf ? TX : 1, nd = yf ? L::NY : L::NX;
    const double mf = sm[yf ? L::MFY + r : c];
    auto P = [&](int m, int o) {
      const int a = m == 0 ? 0 : (m == 1 ? on : (m == 2 ? ot : (m - 1) * WH));
      return q0[a + o * s];
    };
    auto Dv = [&](int k, int o) { return d0[k * nd + o * sd]; };
    double G[5];
    if (!frame_flux<2, VISC, SCH, false>(g, P, Dv, mf, G)) atomicOr(g.flags, 1u);
    fl[f] = G[0];
    fl[L::NF * (yf ? 2 : 1) + f] = G[1];
    fl[L::NF * (yf ? 1 : 2) + f] = G[2];
    fl[L::NF * 3 + f] = G[4];
  }
  __syncthreads();
  double sig = 0.0;
  if (cell) {
    double R[5];
#pragma unroll
    for (int m = 0; m < 4; ++m) {
      const double *fx = fl + L::NF * m + ty * (TX + 1) + tx;
      const double *fy = fl + L::NF * m + L::FX + ty * TX + tx;
      double r = 0.0;
      r -= (fx[1] - fx[0]) * in.id[0];
      r -= (fy[TX] - fy[0]) * in.id[1];
      R[m == 3 ? 4 : m] = r;
    }
    R[3] = 0.0;
    sig = update_state<2>(g, A, pc, in, dt, R, A.dtpart != nullptr);
  }
  if (A.dtpart) {
    const double m = block_max<NT>(sig, shx);
    if (tid == 0) A.dtpart[tile] = m;
  }
}

// 4 waves per SIMD: a face's flux takes ~125 VGPRs and the stage waits on its
// dependent chains; at 5 waves (96 VGPRs) it is slower by a quarter (1024 x 256:
// 29.3 against 23.2 us).  TENO6-A takes 144: in 16 x 16 tiles 128 with 14 spilled
// let a CU hold two workgroups instead of one (512^2: 134 against 149 us a step),
// the small tiles keep the compiler's choice (256^2: 45 against 47).
template <bool VISC, int SCH, bool SMALL>
__global__ void __launch_bounds__(SMALL ? 256 : 512)
__attribute__((amdgpu_waves_per_eu(SCH == SCHEME_WENO5 || !SMALL ? 4 : 1)))
k_stage2(Dev g, StageArgs A, unsigned nbx) {
  __shared__ double lds[Tile2<VISC, SCH, SMALL>::SIZE];
  const unsigned tile = xcd_remap(blockIdx.x, gridDim.x);
  stage2_tile<VISC, SCH, SMALL>(g, A, tile, nbx, lds);
}

// ---------------------------------------------------------------------------
// 3D: a workgroup of 8 wavefronts, one per CU, takes columns of 15 x 16 cells
// and marches along z over a range of planes.
//  * Wavefronts 0-3 own the columns (16 x 16 of them: x = 15 is a halo column).
//    Each thread keeps the primitives of six planes around plane j in
//    registers, which are the stencil of its z face; it computes the face above
//    plane j, updates its cell of plane j - 1 and makes its part of the
//    derivatives of plane j + 1.
//  * Wavefronts 4-7 keep the other halo columns and compute the 256 x faces and
//    255 y faces of plane j, two per thread.
// What one kind needs of the other's goes through LDS, in as many buffers as
// let every plane have a single barrier: the two wavefronts of a SIMD then
// issue from different work, and FP64 issue is what bounds the stage.
//
// The two kinds run loops of their own with the same number of barriers, so
// that the windows of the one and the face stencils of the other never share
// registers (in one loop they do not fit 256 VGPRs: 250 spills per plane, 1250
// us per stage of 192 x 128 x 128).  So: 335 to 353 us, VALU busy 60 %, 1.0 GB of
// HBM traffic, for 522 us and 2.3 GB in ghost, x + y flux, z flux + update and
// force launches; 64^3: 50 us for 53.
// ---------------------------------------------------------------------------
template <bool VISC> struct Col3 {
  static constexpr int TX = 15, TY = 16;
  static constexpr int W = TX + 6, WH = W * (TY + 6);   // window
  static constexpr int VX = TX + 4, VY = TY + 4;        // window of the viscous terms
  static constexpr int FX = TY * (TX + 1), NF = FX + (TY + 1) * TX;  // x faces, all faces
  static constexpr int NHV = 3 * TY + 4 * TX;           // halo columns of the viscous terms
  static constexpr int NH = WH - 16 * TY;               // halo columns
  static constexpr int PC = 0;                          // [2][3][WH]: rho, w, p of plane k in k % 2
  static constexpr int PV = PC + 2 * 3 * WH;            // [3][2][WH]: u, v of plane k in k % 3
  static constexpr int FL = PV + 3 * 2 * WH;            // [2][5][NF]: faces of plane k in k % 2
  static constexpr int MF = FL + 2 * 5 * NF;            // mf x [TX + 1], mf y [TY + 1]
  static constexpr int SH = MF + TX + TY + 2;           // [8]: reductions
  static constexpr int NTM = VX * VY, NAX = TY * VX, NAY = VY * TX;
  static constexpr int TM = SH + 8;                     // [2][2][VY][VX]: T, mu
  // derivatives of the x faces [3][TY][VX] and y faces [3][VY][TX]
  static constexpr int NA = 3 * NAX + 3 * NAY;
  static constexpr int AX = TM + (VISC ? 4 * NTM : 0);  // [2][NA]
  // velocities of one plane: u [TY][VX], v [VY][TX], w [VY][VX]
  static constexpr int NC = NAX + NAY + NTM;
  static constexpr int CB = AX + (VISC ? 2 * NA : 0);   // [2][NC]
  static constexpr int SIZE = CB + (VISC ? 2 * NC : 0);  // doubles
};

// Halo column h of a tile, relative to its first cell: those within two cells
// along x (h < 48), then along y (h < 108), then the outer layers and corners.
__device__ __forceinline__ void halo_column(int h, int &x, int &y) {
  if (h < 48) {
    const int k = h % 3;
    x = k < 2 ? k - 2 : 16;
    y = h / 3;
  } else if (h < 108) {
    const int k = (h - 48) / 15;
    x = (h - 48) % 15;
    y = k < 2 ? k - 2 : 14 + k;
  } else if (h < 140) {
    x = (h - 108) % 2 ? 17 : -3;
    y = (h - 108) / 2;
  } else if (h < 170) {
    x = (h - 140) % 15;
    y = h < 155 ? -3 : 18;
  } else {  // corners: 6 rows of 6
    const int r = (h - 170) / 6, s = (h - 170) % 6;
    x = s < 3 ? s - 3 : 12 + s;
    y = r < 3 ? r - 3 : 13 + r;
  }
}

// Interior index that the halo chain copies into position x of axis d (x itself
// inside), for faces that are periodic, zero-gradient or no-slip walls; sets
// the bit 2 d + side of mask behind a wall.
__device__ __forceinline__ int source_index(const Dev &g, int d, int x, int &mask) {
  const int n = g.n[d];
  int y = x;
  if (x < 0) {
    const int kind = g.bck[2 * d];
    y = kind == BC_PERIODIC ? x + n : (kind == BC_ZEROGRAD ? 0 : -1 - x);
    if (kind == BC_WALL) mask |= 1 << (2 * d);
  }
  if (x >= n) {
    const int kind = g.bck[2 * d + 1];
    y = kind == BC_PERIODIC ? x - n : (kind == BC_ZEROGRAD ? n - 1 : 2 * n - 1 - x);
    if (kind == BC_WALL) mask |= 2 << (2 * d);
  }
  return y;
}

// A column of cells, interior or ghost: byte offset of its source cell within
// a plane (planes below 2^32 bytes: a scalar base and a 32-bit lane offset per
// load) and the walls it lies behind along x and y.
struct Column {
  unsigned off;
  int mask;  // -1: outside the ghost layers
};
__device__ __forceinline__ Column make_column(const Dev &g, int px, int py) {
  Column c = {0u, -1};
  if (px < -3 || px > g.n[0] + 2 || py < -3 || py > g.n[1] + 2) return c;
  c.mask = 0;
  const int wx = source_index(g, 0, px, c.mask), wy = source_index(g, 1, py, c.mask);
  c.off = 8u * ((unsigned)wy * (unsigned)g.n[0] + (unsigned)wx);
  return c;
}
__device__ __forceinline__ double at(const double *base, unsigned off) {
  return *(const double *)((const char *)base + off);
}

// Conserved variables of a column's source at plane k (uniform) into s.
// Returns the mask of the walls that the cell lies behind, -1 (s not loaded)
// outside the ghost layers.
__device__ __forceinline__ int load_raw(const Dev &g, const double *U, Column c, int k,
                                        double *s) {
  if (c.mask < 0 || k < -3 || k > g.n[2] + 2) return -1;
  int zmask = 0;
  const int w = source_index(g, 2, k, zmask);
  const double *base = U + (long)w * ((long)g.n[0] * g.n[1]);
#pragma unroll
  for (int v = 0; v < 5; ++v) s[v] = at(base + v * g.ncell, c.off);
  return c.mask | zmask;
}

// Primitives (without mu) of what load_raw left, through the walls' ghost
// transforms in x, y, z order.
__device__ __forceinline__ void raw_prims(const Dev &g, int mask, const double *s, double *q) {
  prim_of_state_t<3>(g, s, q);
  if (mask == 0) return;
#pragma unroll 1
  for (int face = 0; face < 6; ++face) {
    if (!(mask >> face & 1)) continue;
    q[QU] = -q[QU];
    q[QV] = -q[QV];
    q[QW] = -q[QW];
    if (g.Tw[face] > 0.0) {
      const double Tg = 2.0 * g.Tw[face] - q[QT];
      if (!(Tg > 0.0)) atomicOr(g.flags, 1u);
      q[QT] = Tg;
      q[QR] = q[QP] / (g.R * Tg);
    }
  }
}

__device__ __forceinline__ int buf2(int k) { return k & 1; }
__device__ __forceinline__ int buf3(int k) { return (k + 3) % 3; }  // k >= -3

// Of the columns' wavefronts: planes [k0, k1) of the tile at (i0, j0).  Returns
// the largest signal rate of this thread's cells (A.dtpart).
template <int LAW, int SCH>
__device__ __forceinline__ double column_waves(const Dev &g, const StageArgs &A, int i0, int j0,
                                               int k0, int k1, double dt, double force,
                                               double *lds) {
  constexpr bool VISC = LAW != VISC_NONE;
  using L = Col3<VISC>;
  constexpr int W = L::W, WH = L::WH, VX = L::VX, TX = L::TX;
  const int tx = threadIdx.x % 16, ty = threadIdx.x / 16;
  const int px = i0 + tx, py = j0 + ty;
  const Column col = make_column(g, px, py);
  const bool own = tx < TX, cell = own && px < g.n[0] && py < g.n[1];
  const double mcx = VISC ? g.mc[0][min(px, g.n[0] - 1)] : 0.0;
  const double mcy = VISC ? g.mc[1][min(py, g.n[1] - 1)] : 0.0;
  const double idx = g.idx[0][min(px, g.n[0] - 1)], idy = g.idx[1][min(py, g.n[1] - 1)];
  const long np = (long)g.n[0] * g.n[1];
  const int w = (ty + 3) * W + tx + 3;                           // window position
  const int wx = ty * VX + tx + 2, wy = (ty + 2) * TX + tx, wt = (ty + 2) * VX + tx + 2;
  // primitives (rho, u, v, w, p) of planes j-2 .. j+3, T and mu of j-1 .. j+2,
  // the x and y derivatives of the z faces of j-1 .. j+2
  double q[5][6], tm[2][4], cw[3][4], s[5];
  // the last z face, and its difference to the one before
  double F[5] = {0.0, 0.0, 0.0, 0.0, 0.0}, dz[5] = {0.0, 0.0, 0.0, 0.0, 0.0};

  auto convert = [&](int k, int mask, const double *raw, double *qn) {
    qn[QR] = qn[QP] = 1.0;
    qn[QU] = qn[QV] = qn[QW] = 0.0;
    if (mask >= 0) raw_prims(g, mask, raw, qn);
    if (cell && k >= k0 && k < k1 && !(finite_pos(qn[QR]) && finite_pos(qn[QP])))
      atomicOr(g.flags, 1u);
  };
  auto transport = [&](int i, int o) {  // T, mu of window plane i into tm[.][o]
    tm[0][o] = q[4][i] * rcp_nr(q[0][i]) * g.iR;
    tm[1][o] = viscosity(g, tm[0][o], LAW);
  };
  auto put_velocities = [&](int k, int i) {  // window plane i = plane k
    double *c = lds + L::CB + buf2(k) * L::NC;
    c[wx] = q[1][i];
    if (own) c[L::NAX + wy] = q[2][i];
    c[L::NAX + L::NAY + wt] = q[3][i];
  };
  auto put_uv = [&](int k, int i) {
    double *p = lds + L::PV + buf3(k) * 2 * WH + w;
    p[0] = q[1][i];
    p[WH] = q[2][i];
  };
  auto d4 = [&](const double *v, int st) {
    return dcell4(v[-2 * st], v[-st], v[st], v[2 * st]);
  };
  auto derivatives_z = [&](int k, int o) {  // of the z faces, plane k
    const double *c = lds + L::CB + buf2(k) * L::NC;
    if (!own) return;
    cw[0][o] = d4(c + wx, 1) * mcx + d4(c + L::NAX + wy, TX) * mcy;
    cw[1][o] = d4(c + L::NAX + L::NAY + wt, 1) * mcx;
    cw[2][o] = d4(c + L::NAX + L::NAY + wt, VX) * mcy;
  };
  auto load_state = [&](int k, double *un, double *ui) {
#pragma unroll
    for (int v = 0; v < 5; ++v) {
      un[v] = at(A.Un + (v * g.ncell + k * np), col.off);
      ui[v] = at(A.Uin + (v * g.ncell + k * np), col.off);
    }
  };
  // cell of plane k from its x and y faces in LDS and the difference dz of its
  // z faces: Uout = a Un + b (Uin + dt R), or R itself
  auto update = [&](int k) {
    double un[5], ui[5];
    load_state(k, un, ui);
    const double *FL = lds + L::FL + buf2(k) * 5 * L::NF;
    const double idz = g.idx[2][k];
    double R[5];
#pragma unroll
    for (int m = 0; m < 5; ++m) {
      const double *fx = FL + L::NF * m + ty * (TX + 1) + tx;
      const double *fy = FL + L::NF * m + L::FX + ty * TX + tx;
      double r = 0.0;
      r -= (fx[1] - fx[0]) * idx;
      r -= (fy[TX] - fy[0]) * idy;
      r -= dz[m] * idz;
      R[m] = r;
    }
    if (A.fpart) {
      R[1] += force;
      R[4] += force * (ui[1] * rcp_nr(ui[0]));
    }
    double st[5];
#pragma unroll
    for (int v = 0; v < 5; ++v) {
      st[v] = A.Rout ? R[v] : A.a * un[v] + A.b * (ui[v] + dt * R[v]);
      double *out = (A.Rout ? A.Rout : A.Uout) + (v * g.ncell + k * np);
      *(double *)((char *)out + col.off) = st[v];
    }
    if (!A.dtpart) return 0.0;
    double qn[NQ];
    prim_of_state_t<3>(g, st, qn);
    const int pc[3] = {px, py, k};
    return cell_sigma(g, qn, pc, LAW);
  };

  // the window of j = k0 - 1: planes k0-3 .. k0+2, all loads in flight at once
  {
    double raw[6][5];
    int mask[6];
#pragma unroll
    for (int i = 0; i < 6; ++i) mask[i] = load_raw(g, A.Uin, col, k0 - 3 + i, raw[i]);
#pragma unroll
    for (int i = 0; i < 6; ++i) {
      double qn[NQ];
      convert(k0 - 3 + i, mask[i], raw[i], qn);
#pragma unroll
      for (int c = 0; c < 5; ++c) q[c][i] = qn[c];  // QR .. QP
    }
  }
  put_uv(k0, 3);
  if constexpr (VISC) {
    put_velocities(k0 - 2, 1);
    __syncthreads();
    derivatives_z(k0 - 2, 0);
    put_velocities(k0 - 1, 2);
    transport(1, 0);
    transport(2, 1);
    __syncthreads();
    derivatives_z(k0 - 1, 1);
    put_velocities(k0, 3);
    transport(3, 2);
    transport(4, 3);
    __syncthreads();
    derivatives_z(k0, 2);
    put_velocities(k0 + 1, 4);
    __syncthreads();
  }
  double sig = 0.0;
#pragma unroll 1
  for (int j = k0 - 1; j < k1; ++j) {
    if constexpr (VISC) {
      derivatives_z(j + 2, 3);
      if (j + 1 < k1) {
        // the x and y faces' derivatives of plane j+1 at this column
        const double mcz = g.mc[2][j + 1];
        const double *v = lds + L::PV + buf3(j + 1) * 2 * WH + w;
        const double uz = dcell4(q[1][1], q[1][2], q[1][4], q[1][5]) * mcz;
        const double vz = dcell4(q[2][1], q[2][2], q[2][4], q[2][5]) * mcz;
        const double wz = dcell4(q[3][1], q[3][2], q[3][4], q[3][5]) * mcz;
        double *ax = lds + L::AX + buf2(j + 1) * L::NA + wx;
        ax[0] = d4(v + WH, W) * mcy + wz;
        ax[L::NAX] = d4(v, W) * mcy;
        ax[2 * L::NAX] = uz;
        if (own) {
          double *ay = lds + L::AX + buf2(j + 1) * L::NA + 3 * L::NAX + wy;
          ay[0] = d4(v, 1) * mcx + wz;
          ay[L::NAY] = d4(v + WH, 1) * mcx;
          ay[2 * L::NAY] = vz;
        }
      }
    }
    if (j > k0 && cell) sig = fmax(sig, update(j - 1));
    const int mask = load_raw(g, A.Uin, col, j + 4, s);  // in flight during the z face
    if (cell) {  // z face j + 1
      constexpr int qi[5] = {0, 3, 1, 2, 4};
      auto P = [&](int m, int o) {
        return m >= 5 ? tm[m >= 5 ? m - 5 : 0][(o + 2) & 3] : q[qi[m < 5 ? m : 0]][o + 3];
      };
      auto Dv = [&](int k, int o) { return cw[k][(o + 2) & 3]; };
      double G[5];
      if (!frame_flux<3, VISC, SCH, true>(g, P, Dv, g.mf[2][j + 1], G)) atomicOr(g.flags, 1u);
      const double Fn[5] = {G[0], G[2], G[3], G[1], G[4]};
#pragma unroll
      for (int m = 0; m < 5; ++m) {
        dz[m] = Fn[m] - F[m];
        F[m] = Fn[m];
      }
    }
    // for the next plane
    {
      double *p = lds + L::PC + buf2(j + 1) * 3 * WH + w;
      p[0] = q[0][3];
      p[WH] = q[3][3];
      p[2 * WH] = q[4][3];
      put_uv(j + 2, 4);
    }
    if constexpr (VISC) {
      double *p = lds + L::TM + buf2(j + 1) * 2 * L::NTM + wt;
      p[0] = tm[0][2];
      p[L::NTM] = tm[1][2];
      put_velocities(j + 3, 5);
#pragma unroll
      for (int i = 0; i < 3; ++i) {
        tm[0][i] = tm[0][i + 1];
        tm[1][i] = tm[1][i + 1];
#pragma unroll
        for (int c = 0; c < 3; ++c) cw[c][i] = cw[c][i + 1];
      }
      transport(5, 3);
    }
    double qn[NQ];
    convert(j + 4, mask, s, qn);
#pragma unroll
    for (int c = 0; c < 5; ++c) {
#pragma unroll
      for (int i = 0; i < 5; ++i) q[c][i] = q[c][i + 1];
      q[c][5] = qn[c];  // QR .. QP
    }
    __syncthreads();
  }
  if (cell) sig = fmax(sig, update(k1 - 1));
  return sig;
}

// Of the other wavefronts: halo columns, x and y faces.
template <int LAW, int SCH>
__device__ __forceinline__ void face_waves(const Dev &g, const StageArgs &A, int i0, int j0,
                                           int k0, int k1, double *lds) {
  constexpr bool VISC = LAW != VISC_NONE;
  using L = Col3<VISC>;
  constexpr int W = L::W, WH = L::WH, VX = L::VX, TX = L::TX, TY = L::TY;
  const int t = threadIdx.x - 256;
  int hx = 0, hy = 0;
  halo_column(min(t, L::NH - 1), hx, hy);
  const bool halo = t < L::NH, vhalo = VISC && t < L::NHV, xh = t < 48;
  Column col = make_column(g, i0 + hx, j0 + hy);
  if (!halo) col.mask = -1;
  const int w = (hy + 3) * W + hx + 3;
  const int wx = hy * VX + hx + 2, wy = (hy + 2) * TX + hx, wt = (hy + 2) * VX + hx + 2;
  // the metric of a halo column's tangential derivative
  const double mch = !vhalo ? 0.0
                     : (xh ? g.mc[1][min(j0 + hy, g.n[1] - 1)] : g.mc[0][min(i0 + hx, g.n[0] - 1)]);
  if (t < TX + 1) lds[L::MF + t] = g.mf[0][min(i0 + t, g.n[0])];
  else if (t >= 64 && t < 64 + TY + 1)
    lds[L::MF + TX + 1 + t - 64] = g.mf[1][min(j0 + t - 64, g.n[1])];
  // primitives (rho, u, v, w, p) of planes j+1, j+2, j+3; of planes j-1 and j
  // the velocities (u, w) beside x, (v, w) beside y
  double P1[5], P2[5], P3[5], H[2][2], s[5];
  auto convert = [&](int mask, const double *raw, double *p) {
    double qn[NQ] = {1.0, 0.0, 0.0, 0.0, 1.0, 1.0, 0.0};
    if (mask >= 0) raw_prims(g, mask, raw, qn);
#pragma unroll
    for (int c = 0; c < 5; ++c) p[c] = qn[c];  // QR .. QP
  };
  auto put_velocities = [&](int k, double a, double b) {
    if (!vhalo) return;
    double *c = lds + L::CB + buf2(k) * L::NC;
    c[xh ? wx : L::NAX + wy] = a;
    c[L::NAX + L::NAY + wt] = b;
  };
  auto put_uv = [&](int k, const double *p) {
    if (!halo) return;
    double *v = lds + L::PV + buf3(k) * 2 * WH + w;
    v[0] = p[QU];
    v[WH] = p[QV];
  };
  auto along = [&](const double *p) { return xh ? p[QU] : p[QV]; };
  {
    double raw[5][5], p[5];
    int mask[5];
#pragma unroll
    for (int i = 0; i < 5; ++i) mask[i] = load_raw(g, A.Uin, col, k0 - 2 + i, raw[i]);
#pragma unroll
    for (int i = 0; i < 2; ++i) {
      convert(mask[i], raw[i], p);
      H[i][0] = along(p);
      H[i][1] = p[QW];
    }
    convert(mask[2], raw[2], P1);
    convert(mask[3], raw[3], P2);
    convert(mask[4], raw[4], P3);
  }
  put_uv(k0, P1);
  if constexpr (VISC) {
    put_velocities(k0 - 2, H[0][0], H[0][1]);
    __syncthreads();
    put_velocities(k0 - 1, H[1][0], H[1][1]);
    __syncthreads();
    put_velocities(k0, along(P1), P1[QW]);
    __syncthreads();
    put_velocities(k0 + 1, along(P2), P2[QW]);
    __syncthreads();
  }
#pragma unroll 1
  for (int j = k0 - 1; j < k1; ++j) {
    if (VISC && vhalo && j + 1 < k1) {
      // the derivatives of plane j+1 at the halo column
      const double mcz = g.mc[2][j + 1];
      const double *v = lds + L::PV + buf3(j + 1) * 2 * WH + w;
      auto d4 = [&](const double *p, int st) {
        return dcell4(p[-2 * st], p[-st], p[st], p[2 * st]);
      };
      const double az = dcell4(H[0][0], H[1][0], along(P2), along(P3)) * mcz;
      const double bz = dcell4(H[0][1], H[1][1], P2[QW], P3[QW]) * mcz;
      const int st = xh ? W : 1, un = xh ? 0 : WH, ut = xh ? WH : 0;
      double *a = lds + L::AX + buf2(j + 1) * L::NA + (xh ? wx : 3 * L::NAX + wy);
      const int na = xh ? L::NAX : L::NAY;
      a[0] = d4(v + ut, st) * mch + bz;
      a[na] = d4(v + un, st) * mch;
      a[2 * na] = az;
    }
    // for the next plane
    if (halo) {
      double *p = lds + L::PC + buf2(j + 1) * 3 * WH + w;
      p[0] = P1[QR];
      p[WH] = P1[QW];
      p[2 * WH] = P1[QP];
    }
    put_uv(j + 2, P2);
    if (vhalo) {
      double *p = lds + L::TM + buf2(j + 1) * 2 * L::NTM + wt;
      const double T = P1[QP] * rcp_nr(P1[QR]) * g.iR;
      p[0] = T;
      p[L::NTM] = viscosity(g, T, LAW);
      put_velocities(j + 3, along(P3), P3[QW]);
    }
    H[0][0] = H[1][0];
    H[0][1] = H[1][1];
    H[1][0] = along(P1);
    H[1][1] = P1[QW];
#pragma unroll
    for (int c = 0; c < 5; ++c) {
      P1[c] = P2[c];
      P2[c] = P3[c];
    }
    const int mask = load_raw(g, A.Uin, col, j + 4, s);  // in flight during the faces
    if (j >= k0) {
      // both faces in one straight line of code; a thread without a y face
      // repeats another's
      double G[2][5];
      bool ok[2], fine[2];
      int fo[2];
#pragma unroll
      for (int it = 0; it < 2; ++it) {
        constexpr int NY = L::NF - L::FX;
        const int e = it == 1 && t >= NY ? NY - 1 : t;
        const int fr = it == 1 ? e / TX : e / 16, fc = it == 1 ? e % TX : e % 16;
        ok[it] = i0 + fc <= g.n[0] - it && j0 + fr < g.n[1] + it;
        fo[it] = it == 1 ? L::FX + e : e;
        const int f = (fr + 3) * W + fc + 3;
        const double *c0 = lds + L::PC + buf2(j) * 3 * WH + f;
        const double *v0 = lds + L::PV + buf3(j) * 2 * WH + f;
        const double *t0 = lds + L::TM + buf2(j) * 2 * L::NTM + (fr + 2) * VX + fc + 2;
        const double *d0 = lds + L::AX + buf2(j) * L::NA +
                           (it == 1 ? 3 * L::NAX + (fr + 2) * TX + fc : fr * VX + fc + 2);
        asm volatile("" ::: "memory");
        auto P = [&](int m, int o) {
          const int wo = o * (it == 1 ? W : 1);
          if (m >= 5) return t0[(m - 5) * L::NTM + o * (it == 1 ? VX : 1)];
          if (m == 1) return v0[(it == 1 ? WH : 0) + wo];
          if (m == 2) return v0[(it == 1 ? 0 : WH) + wo];
          return c0[(m == 0 ? 0 : (m == 3 ? WH : 2 * WH)) + wo];
        };
        auto Dv = [&](int k, int o) {
          return it == 1 ? d0[k * L::NAY + o * TX] : d0[k * L::NAX + o];
        };
        fine[it] = frame_flux<3, VISC, SCH, true>(
            g, P, Dv, lds[L::MF + (it == 1 ? TX + 1 + fr : fc)], G[it]);
      }
      if ((ok[0] && !fine[0]) || (ok[1] && !fine[1])) atomicOr(g.flags, 1u);
#pragma unroll
      for (int it = 0; it < 2; ++it) {
        if (!ok[it]) continue;
        double *F = lds + L::FL + buf2(j) * 5 * L::NF + fo[it];
        F[0] = G[it][0];
        F[L::NF * (it == 1 ? 2 : 1)] = G[it][1];
        F[L::NF * (it == 1 ? 1 : 2)] = G[it][2];
        F[L::NF * 3] = G[it][3];
        F[L::NF * 4] = G[it][4];
      }
    }
    convert(mask, s, P3);
    __syncthreads();
  }
}

// The plane-tiles, counted plane by plane along z within a tile, are divided
// evenly over the workgroups: a workgroup's range is a few runs of planes.
template <int LAW, int SCH>
__device__ __forceinline__ void stage3_range(const Dev &g, const StageArgs &A, unsigned wg,
                                             unsigned long r0, unsigned long r1, unsigned nbx,
                                             double *lds) {
  constexpr bool VISC = LAW != VISC_NONE;
  using L = Col3<VISC>;
  const double dt = stage_dt<512>(A, wg == 0, lds + L::SH);
  const double force = stage_force<512>(g, A, lds + L::SH);
  const unsigned nz = g.n[2];
  double sig = 0.0;
  auto run = [&](auto kind) {
#pragma unroll 1
    for (unsigned long r = r0; r < r1;) {
      const unsigned tile = (unsigned)(r / nz);
      const int k0 = (int)(r % nz), k1 = (int)min((unsigned long)nz, k0 + (r1 - r));
      kind((int)(tile % nbx) * L::TX, (int)(tile / nbx) * L::TY, k0, k1);
      r += (unsigned)(k1 - k0);
    }
  };
  // a loop over the runs for each kind: in a common one, what either computes
  // from its thread's position would be kept in registers through the other's
  // planes.  The barriers of the two pair up.
  if (__builtin_amdgcn_readfirstlane(threadIdx.x) < 256)
    run([&](int i0, int j0, int k0, int k1) {
      sig = fmax(sig, column_waves<LAW, SCH>(g, A, i0, j0, k0, k1, dt, force, lds));
    });
  else
    run([&](int i0, int j0, int k0, int k1) { face_waves<LAW, SCH>(g, A, i0, j0, k0, k1, lds); });
  if (A.dtpart) {
    const double m = block_max<512>(sig, lds + L::SH);
    if (threadIdx.x == 0) A.dtpart[wg] = m;
  }
}

// How a grid's plane-tiles are divided (stage3_split): ranges of len, or (len =
// 0) every tile's planes in nch nearly equal chunks.
struct Split3 {
  unsigned nbx, len, nch, groups;
};
__device__ __forceinline__ void split_range(const Dev &g, const Split3 &s, unsigned wg,
                                            unsigned long &r0, unsigned long &r1) {
  const unsigned long nz = (unsigned long)g.n[2];
  if (s.len) {
    const unsigned long total = (unsigned long)s.nbx * ((g.n[1] + 15) / 16) * nz;
    r0 = (unsigned long)wg * s.len;
    r1 = min(r0 + s.len, total);
  } else {
    const unsigned long tile = wg / s.nch, c = wg % s.nch;
    r0 = tile * nz + c * nz / s.nch;
    r1 = tile * nz + (c + 1) * nz / s.nch;
  }
}

template <int LAW, int SCH>
__global__ void __launch_bounds__(512) __attribute__((amdgpu_waves_per_eu(2)))
k_stage3(Dev g, StageArgs A, Split3 s) {
  __shared__ double lds[Col3<LAW != VISC_NONE>::SIZE];
  const unsigned wg = xcd_remap(blockIdx.x, gridDim.x);
  unsigned long r0, r1;
  split_range(g, s, wg, r0, r1);
  stage3_range<LAW, SCH>(g, A, wg, r0, r1, s.nbx, lds);
}

// ---------------------------------------------------------------------------
// 3D body force of the constant-mass-flux source from the state alone.  The
// volume sum of the unforced x-momentum right-hand side telescopes along every
// grid line to its two boundary faces (periodic lines contribute nothing), so
// one thread takes one boundary face of a non-periodic axis: its stencil is
// three interior cells and their images behind the boundary.  Partial sums per
// workgroup; the stage's workgroups add them up (stage_force).
// ---------------------------------------------------------------------------
// d u_phi / d x_t at the interior cell w, 4th order.
template <int PHI, int T>
__device__ __forceinline__ double cell_derivative(const Dev &g, const double *U, const int *w) {
  double v[4];
  constexpr int ks[4] = {-2, -1, 1, 2};
#pragma unroll
  for (int i = 0; i < 4; ++i) {
    int mask = 0;
    int s[3] = {w[0], w[1], w[2]};
    s[T] = source_index(g, T, w[T] + ks[i], mask);
    const long c = ((long)s[2] * g.n[1] + s[1]) * g.n[0] + s[0];
    const double x = U[(1 + PHI) * g.ncell + c] * rcp_nr(U[c]);
    v[i] = mask ? -x : x;
  }
  return dcell4(v[0], v[1], v[2], v[3]) * g.mc[T][w[T]];
}

// x-momentum flux of the boundary face of direction D on the given side, on
// the line through p.
template <int LAW, int D>
__device__ __forceinline__ double boundary_xmom(const Dev &g, const double *U, const int *p,
                                                int side) {
  constexpr bool VISC = LAW != VISC_NONE;
  constexpr int T1 = tan1(D), T2 = tan2(D);
  constexpr int qi[7] = {QR, QU + D, QU + T1, QU + T2, QP, QT, QMU};
  const int n = g.n[D], face = 2 * D + side;
  const bool wall = g.bck[face] == BC_WALL;
  double q[7][6], d[2][6];  // face frame, offsets -3 .. 2
#pragma unroll
  for (int m = 0; m < 3; ++m) {  // distance from the face
    int w[3] = {p[0], p[1], p[2]};
    w[D] = side ? n - 1 - m : m;
    const long c = ((long)w[2] * g.n[1] + w[1]) * g.n[0] + w[0];
    double s[5], qc[NQ];
#pragma unroll
    for (int v = 0; v < 5; ++v) s[v] = U[v * g.ncell + c];
    prim_of_state_t<3>(g, s, qc);
    if (VISC) qc[QMU] = viscosity(g, qc[QT], LAW);
    double dv = 0.0;
    if (VISC && m < 2) {
      if constexpr (D == 0) dv = cell_derivative<T1, T1>(g, U, w) + cell_derivative<T2, T2>(g, U, w);
      else dv = cell_derivative<D, 0>(g, U, w);
    }
    const int oi = side ? 2 - m : 3 + m;  // this cell; below, its image
#pragma unroll
    for (int k = 0; k < 7; ++k) q[k][oi] = qc[qi[k]];
    d[0][oi] = d[1][oi] = dv;
    if (wall) {
      qc[QU] = -qc[QU];
      qc[QV] = -qc[QV];
      qc[QW] = -qc[QW];
      dv = -dv;
      if (g.Tw[face] > 0.0) {
        const double Tg = 2.0 * g.Tw[face] - qc[QT];
        qc[QT] = Tg;
        qc[QR] = qc[QP] / (g.R * Tg);
        if (VISC) qc[QMU] = viscosity(g, Tg, LAW);
      }
    }
    // a wall's image lies at the same distance; the zero-gradient images are
    // all of the first cell
#pragma unroll
    for (int k = 0; k < 3; ++k) {
      if (wall ? k != m : m != 0) continue;
      const int og = side ? 3 + k : 2 - k;
#pragma unroll
      for (int e = 0; e < 7; ++e) q[e][og] = qc[qi[e]];
      d[0][og] = d[1][og] = dv;
    }
  }
  auto P = [&](int m, int o) { return q[m][o + 3]; };
  auto Dv = [&](int r, int o) { return r < 2 ? d[r & 1][o + 3] : 0.0; };
  double G[5];
  (void)frame_flux<3, VISC, SCHEME_WENO5, true>(g, P, Dv, g.mf[D][side ? n : 0], G);
  return G[D == 0 ? 1 : 2];
}

template <int LAW>
__global__ void __launch_bounds__(256) k_force3(Dev g, const double *U, double *part) {
  __shared__ double sh[4];
  double v = 0.0;
  unsigned nl[3], tot = 0;
  for (int D = 0; D < 3; ++D) {
    nl[D] = g.bck[2 * D] == BC_PERIODIC ? 0u : 2u * g.n[tan1(D)] * g.n[tan2(D)];
    tot += nl[D];
  }
  for (unsigned x = blockIdx.x * 256u + threadIdx.x; x < tot; x += gridDim.x * 256u) {
    unsigned l = x;
    int D = 0;
    while (l >= nl[D]) l -= nl[D++];
    const int side = l >= nl[D] / 2 ? 1 : 0;
    l -= side ? nl[D] / 2 : 0;
    const int t1 = tan1(D), t2 = tan2(D);
    const int a = (int)(l % (unsigned)g.n[t1]), b = (int)(l / (unsigned)g.n[t1]);
    const double area = g.dx[t1][a] * g.dx[t2][b];
    double F;
    if (D == 0) {
      const int p[3] = {0, a, b};
      F = boundary_xmom<LAW, 0>(g, U, p, side);
    } else if (D == 1) {
      const int p[3] = {a, 0, b};
      F = boundary_xmom<LAW, 1>(g, U, p, side);
    } else {
      const int p[3] = {a, b, 0};
      F = boundary_xmom<LAW, 2>(g, U, p, side);
    }
    v += side ? -area * F : area * F;
  }
  v = block_total<256>(v, sh);
  if (threadIdx.x == 0) part[blockIdx.x] = v;
}

// ---------------------------------------------------------------------------
// Host side.
// ---------------------------------------------------------------------------
// Small tiles up to 2^16 cells: there 16 x 16 tiles leave CUs without one, and
// a tile's second round of faces (32 of 544) waits alone; above, their extra
// halo conversions and idle lanes come to cost more.  Steps, small against 16 x 16
// tiles, in us: 64^2 24.0 and 30.7, 200^2 25.4 and 28.9, 300 x 200 28.5 and 28.9,
// 512 x 128 29.1 and 30.5; beyond the line the rounds of tiles decide: 300^2 32.0
// and 35.1, 340^2 41.2 and 35.8, 360^2 45.3 and 49.7, 512 x 256 45.4 and 38.3.
static bool stage2_small(const Dev &g) { return g.ncell <= 65536; }

static unsigned tiles_along(int n, int t) { return (unsigned)((n + t - 1) / t); }
template <bool SMALL> static unsigned stage2_nbx_t(const Dev &g) {
  return tiles_along(g.n[0], Tile2<true, SCHEME_WENO5, SMALL>::TX);
}
template <bool SMALL> static unsigned stage2_tiles_t(const Dev &g) {
  return stage2_nbx_t<SMALL>(g) * tiles_along(g.n[1], Tile2<true, SCHEME_WENO5, SMALL>::TY);
}

// 3D grids with the WENO5-JS scheme whose faces are periodic, zero-gradient or
// plain walls (the ghost cells the column kernel makes while it loads).
static bool stage3_takes(const Dev &g) {
  if (g.ndim != 3 || g.scheme != SCHEME_WENO5) return false;
  if ((long)g.n[0] * g.n[1] >= 1L << 29) return false;  // 32-bit offsets in a plane
  for (int f = 0; f < 6; ++f)
    if (g.bck[f] != BC_PERIODIC && g.bck[f] != BC_ZEROGRAD && g.bck[f] != BC_WALL) return false;
  return true;
}

// A run of planes costs its length and about 1.8 planes for its start (12 us
// against 6.5 per plane).  Either the planes of all tiles are divided over the
// 256 CUs (a range then spans parts of one more tile than its length needs), or
// each tile's nz planes into nch chunks, in rounds of 256 workgroups.  (64^3: 12
// chunks per tile 50 us, ranges of 5 planes 54 us; 192 x 128 x 128: ranges of 52
// planes 353 us, 7 chunks per tile 420 us.)
// (slots: the workgroups in flight, a share of 256 for a member of a batch.)
// (plane_times: the cost of the division found, in planes.)
static Split3 stage3_split(const Dev &g, unsigned slots = 256, double *plane_times = nullptr) {
  const unsigned nz = g.n[2];
  const unsigned tiles = tiles_along(g.n[0], Col3<true>::TX) * tiles_along(g.n[1], Col3<true>::TY);
  const unsigned long total = (unsigned long)tiles * nz;
  Split3 s = {tiles_along(g.n[0], Col3<true>::TX), 0u, 1u, 0u};
  if (total <= slots) {  // a plane each
    s.nch = nz;
    s.groups = (unsigned)total;
    if (plane_times) *plane_times = 2.8;
    return s;
  }
  double cost = 1e300;
  // (more rounds than a few only add starts)
  const unsigned cmax = 8u * slots / tiles + 8u;
  for (unsigned c = 1; c <= nz && c <= cmax; ++c) {
    const unsigned long n = (unsigned long)tiles * c;
    const double t = (double)((n + slots - 1) / slots) * ((nz + c - 1) / c + 1.8);
    if (t < cost) {
      cost = t;
      s.nch = c;
    }
  }
  s.groups = tiles * s.nch;
  const unsigned len = (unsigned)((total + slots - 1) / slots);
  const unsigned runs = len % nz == 0 ? len / nz : (len - 1) / nz + 2;
  if (len + 1.8 * runs < cost) {
    cost = len + 1.8 * runs;
    s.len = len;
    s.groups = (unsigned)((total + len - 1) / len);
  }
  if (plane_times) *plane_times = cost;
  return s;
}

// The column kernel against the split launches, in plane times of 5.8 us.  A
// plane of a tile costs that whatever part of its 15 x 16 columns the grid has,
// and a grid of few planes per CU pays for whole ones; the split launches cost
// 20 us a stage (13 more for a right-hand side alone, which fuses less) and 88 ps
// for every cell of their tiles (16 wide along x, 15 deep along z), twice that
// beyond 2^19, where their arrays leave the caches.  The body force by itself
// costs the column form 5 us more (k_force3 against the face fluxes at hand).
// Where at least two thirds of the tiles' columns are the grid's own the column
// form is kept: ahead or even by itself (64^3: 46 us a stage, 47 split), and up
// to 1.3 times ahead in batches, whose members take the kernels that they take
// alone.  Steps in us, columns and split: 256 x 4 x 256: 324 and 186;
// 128 x 17 x 128: 202 and 161; 46 x 17 x 200: 158 and 116; 64^3 with the body
// force: 174 and 162; 128 x 16 x 128: 124 and 158; 256 x 20 x 256: 639 and 646.
static bool stage3_wins(const Dev &g, double split_start) {
  const bool force = g.source != SRC_NONE;
  const long nx = g.n[0], ny = g.n[1], nz = g.n[2];
  const long tiles = (nx + 14) / 15 * ((ny + 15) / 16);
  if (!force && 3 * nx * ny >= 2 * 240 * tiles) return true;
  const double cells = (double)((nx + 15) / 16 * 16 * ny) * (double)((nz + 14) / 15 * 15);
  const double split = split_start - (force ? 0.95 : 0.0) + cells / 65536.0 +
                       std::max(0.0, cells - 524288.0) / 65536.0;
  double columns;
  (void)stage3_split(g, 256, &columns);
  return columns <= split;
}

// Large 2D grids with TENO6-A take the split launches: bound by FP64 issue, they
// run at 5 to 6 wavefronts per SIMD there and the stage's tiles at 4, while the
// launches they take more matter less and less (512^2: 134 us a step in one
// launch a stage, 147 split; 540^2: 159 and 156; 700^2: 255 and 225; 2048^2: 1952
// and 1628; a right-hand side alone, one launch for three, 700^2: 80 and 82,
// 1024^2: 159 and 154), and earlier with the body force, which the one launch
// needs a halo fill and a reduction for (256^2: 116 and 114, 400^2: 186 and 153).
static bool stage2_wins(const Dev &g, long most, long most_force) {
  return g.scheme != SCHEME_TENO6A || g.ncell <= (g.source == SRC_NONE ? most : most_force);
}

bool stage_fused(const Dev &g) {
  if (g.ndim == 3) return stage3_takes(g) && stage3_wins(g, 3.5);
  return g.ndim == 1 || stage2_wins(g, 300000, 100000);
}
bool rhs_fused(const Dev &g) {
  if (g.ndim == 3) return stage3_takes(g) && stage3_wins(g, 5.75);
  return g.ndim == 1 || stage2_wins(g, 800000, 150000);
}
unsigned stage_tiles(const Dev &g) {
  if (g.ndim == 1) return tiles_along(g.n[0], 255);
  if (g.ndim == 3) return stage3_split(g).groups;
  return stage2_small(g) ? stage2_tiles_t<true>(g) : stage2_tiles_t<false>(g);
}

template <bool VISC, int SCH>
static void launch_stage2(const Dev &g, const StageArgs &A, hipStream_t st) {
  if (stage2_small(g))
    k_stage2<VISC, SCH, true><<<stage2_tiles_t<true>(g), 256, 0, st>>>(g, A,
                                                                      stage2_nbx_t<true>(g));
  else
    k_stage2<VISC, SCH, false><<<stage2_tiles_t<false>(g), 512, 0, st>>>(
        g, A, stage2_nbx_t<false>(g));
}

template <bool VISC>
static void launch_stage_v(const Dev &g, const StageArgs &A, hipStream_t st) {
  if (g.scheme == SCHEME_TENO6A) launch_stage2<VISC, SCHEME_TENO6A>(g, A, st);
  else launch_stage2<VISC, SCHEME_WENO5>(g, A, st);
}

// Boundary faces of the non-periodic axes, 256 to a workgroup.
static unsigned force_groups(const Dev &g) {
  unsigned long faces = 0;
  for (int D = 0; D < 3; ++D)
    if (g.bck[2 * D] != BC_PERIODIC) faces += 2ul * g.n[tan1(D)] * g.n[tan2(D)];
  return (unsigned)std::min<unsigned long>((faces + 255) / 256, RED_BLOCKS);
}

bool stage_force_from_state(const Dev &g) { return stage3_takes(g); }

hipError_t launch_stage_force(const Dev &g, StageArgs &A, double *part, hipStream_t st) {
  const unsigned nb = force_groups(g);
  A.fpart = part;
  A.nfpart = (int)nb;
  if (!nb) return hipSuccess;
  if (g.visc == VISC_POWER) k_force3<VISC_POWER><<<nb, 256, 0, st>>>(g, A.Uin, part);
  else if (g.visc == VISC_SUTHERLAND) k_force3<VISC_SUTHERLAND><<<nb, 256, 0, st>>>(g, A.Uin, part);
  else k_force3<VISC_NONE><<<nb, 256, 0, st>>>(g, A.Uin, part);
  return hipGetLastError();
}

hipError_t launch_stage(const Dev &g, const StageArgs &A, hipStream_t st) {
  if (g.ndim == 3 && !stage3_takes(g)) return hipErrorInvalidValue;
  if (g.ndim == 1) {
    const unsigned n = tiles_along(g.n[0], 255);
    const bool v = g.visc != VISC_NONE;
    if (g.scheme == SCHEME_TENO6A) {
      if (v) k_stage1<true, SCHEME_TENO6A><<<n, 256, 0, st>>>(g, A);
      else k_stage1<false, SCHEME_TENO6A><<<n, 256, 0, st>>>(g, A);
    } else {
      if (v) k_stage1<true, SCHEME_WENO5><<<n, 256, 0, st>>>(g, A);
      else k_stage1<false, SCHEME_WENO5><<<n, 256, 0, st>>>(g, A);
    }
    return hipGetLastError();
  }
  if (g.ndim == 3) {
    const Split3 s = stage3_split(g);
    if (g.visc == VISC_POWER)
      k_stage3<VISC_POWER, SCHEME_WENO5><<<s.groups, 512, 0, st>>>(g, A, s);
    else if (g.visc == VISC_SUTHERLAND)
      k_stage3<VISC_SUTHERLAND, SCHEME_WENO5><<<s.groups, 512, 0, st>>>(g, A, s);
    else
      k_stage3<VISC_NONE, SCHEME_WENO5><<<s.groups, 512, 0, st>>>(g, A, s);
    return hipGetLastError();
  }
  if (g.visc != VISC_NONE) launch_stage_v<true>(g, A, st);
  else launch_stage_v<false>(g, A, st);
  return hipGetLastError();
}

// Lines that one workgroup steps: at 1023 cells a stage takes as long there as
// a launch per stage would (the body force needs the whole line's fluxes first
// and takes that path).
bool line_resident(const Dev &g) {
  return g.ndim == 1 && g.n[0] < 1024 && g.source == SRC_NONE;
}

template <bool VISC, int SCH>
static void launch_line_t(const Dev &g, const LineArgs &A, hipStream_t st) {
  if (g.n[0] < 256) k_line<VISC, SCH, 256><<<1, 256, 0, st>>>(g, A);
  else if (g.n[0] < 512) k_line<VISC, SCH, 512><<<1, 512, 0, st>>>(g, A);
  else k_line<VISC, SCH, 1024><<<1, 1024, 0, st>>>(g, A);
}

hipError_t launch_line(const Dev &g, const LineArgs &A, hipStream_t st) {
  if (!line_resident(g)) return hipErrorInvalidValue;
  const bool v = g.visc != VISC_NONE;
  if (g.scheme == SCHEME_TENO6A) {
    if (v) launch_line_t<true, SCHEME_TENO6A>(g, A, st);
    else launch_line_t<false, SCHEME_TENO6A>(g, A, st);
  } else {
    if (v) launch_line_t<true, SCHEME_WENO5>(g, A, st);
    else launch_line_t<false, SCHEME_WENO5>(g, A, st);
  }
  return hipGetLastError();
}

// ---------------------------------------------------------------------------
// Batched stages: tile x of solve y in workgroup (x, y); a workgroup beyond
// its solve's tiles returns before any barrier.
// ---------------------------------------------------------------------------
__device__ __forceinline__ StageArgs batch_args(const BatchEntry &e, int stage, double cfl) {
  StageArgs A = {};
  A.Un = e.U;
  A.Uin = stage == 0 ? e.U : (stage == 1 ? e.U1 : e.U2);
  A.Uout = stage == 0 ? e.U1 : (stage == 1 ? e.U2 : e.U);
  A.dt = e.dt;
  A.a = stage == 0 ? 0.0 : (stage == 1 ? 0.75 : 1.0 / 3.0);
  A.b = stage == 0 ? 1.0 : (stage == 1 ? 0.25 : 2.0 / 3.0);
  if (stage == 0 && cfl > 0.0) {
    A.part = e.part;
    A.nparts = (int)e.nb_dt;
    A.cfl = cfl;
    A.dt_max = 1.0e300;
    A.dt_out = e.dt;
  }
  return A;
}

// The member of this workgroup: the last that starts at or before it.  (Launches
// are packed: a workgroup without a tile would still take its place, in 3D a
// whole CU's LDS, and the others would be dealt unevenly.  Eight boxes of 12^3
// to 18^3: 65 us a step, 105 with every member's workgroups filled up to the
// largest.)
__device__ __forceinline__ const BatchEntry &batch_member(const BatchEntry *tab, int n) {
  int lo = 0, hi = n - 1;
  while (lo < hi) {
    const int mid = (lo + hi + 1) / 2;
    if (tab[mid].st_first <= blockIdx.x) lo = mid;
    else hi = mid - 1;
  }
  return tab[lo];
}

// The batch takes 16 x 16 tiles for every member (8 boundary layers of 256 x 64
// to 384 x 96: 79.8 us per step, 81.7 with 12 x 8): its members fill the chip
// together.
template <bool VISC>
__global__ void __launch_bounds__(512) __attribute__((amdgpu_waves_per_eu(4)))
kb_stage2(const BatchEntry *tab, int n, int stage, double cfl) {
  __shared__ double lds[Tile2<VISC, SCHEME_WENO5, false>::SIZE];
  const BatchEntry &e = batch_member(tab, n);
  const unsigned wg = blockIdx.x - e.st_first;
  if (wg >= e.st_tiles) return;
  const StageArgs A = batch_args(e, stage, cfl);
  stage2_tile<VISC, SCHEME_WENO5, false>(e.g, A, wg, e.st_nbx, lds);
}

// 1D members: lines short enough are stepped whole by one workgroup each, the
// others (st_tiles > 0) stage by stage.
template <bool VISC>
__global__ void __launch_bounds__(1024) kb_line(const BatchEntry *tab, double cfl) {
  __shared__ double lds[Line1<VISC>::NP * 1030 + 3 * 1024];
  const BatchEntry &e = tab[blockIdx.x];
  if (e.st_tiles) return;
  LineArgs A = {};
  A.U = e.U;
  A.dt = e.dt;
  A.nsteps = 1;
  A.nstages = 3;
  if (cfl > 0.0) {
    A.part = e.part;
    A.nparts = (int)e.nb_dt;
    A.cfl_first = cfl;
    A.dt_first = e.dt;
  }
  line_steps<VISC, SCHEME_WENO5, 1024>(e.g, A, lds);
}
template <bool VISC>
__global__ void __launch_bounds__(256) kb_stage1(const BatchEntry *tab, int n, int stage,
                                                 double cfl) {
  __shared__ double lds[Line1<VISC>::NP * 261 + 3 * 256];
  const BatchEntry &e = batch_member(tab, n);
  const unsigned wg = blockIdx.x - e.st_first;
  if (wg >= e.st_tiles) return;
  const StageArgs A = batch_args(e, stage, cfl);
  stage1_tile<VISC, SCHEME_WENO5>(e.g, A, wg, lds);
}

// 3D members whose stages run as one launch; each viscosity law has its kernel,
// a workgroup of another member's law returns.
template <int LAW>
__global__ void __launch_bounds__(512) __attribute__((amdgpu_waves_per_eu(2)))
kb_stage3(const BatchEntry *tab, int n, int stage, double cfl) {
  __shared__ double lds[Col3<LAW != VISC_NONE>::SIZE];
  const BatchEntry &e = batch_member(tab, n);
  const unsigned wg = blockIdx.x - e.st_first;
  if (wg >= e.st_tiles || e.g.visc != LAW) return;
  const StageArgs A = batch_args(e, stage, cfl);
  const Split3 s = {e.st_nbx, e.st_len, e.st_nch, e.st_tiles};
  unsigned long r0, r1;
  split_range(e.g, s, wg, r0, r1);
  stage3_range<LAW, SCHEME_WENO5>(e.g, A, wg, r0, r1, s.nbx, lds);
}

unsigned long stage_work(const Dev &g) {
  if (g.ndim != 3 || !stage_fused(g)) return 0;
  return (unsigned long)tiles_along(g.n[0], Col3<true>::TX) * tiles_along(g.n[1], Col3<true>::TY) *
         (unsigned long)g.n[2];
}

// (3D: the 256 CUs are shared in proportion to the members' plane-tiles, so that
// members of different sizes end together: five Taylor-Green boxes of 22 x 29 x 31
// to 32 x 43 x 45: 150 us a step, 220 with equal shares.)
void stage_entry_sizes(BatchEntry &e, unsigned long work) {
  e.st_tiles = e.st_nbx = e.st_len = e.st_nch = 0;
  if (!stage_fused(e.g)) return;
  if (e.g.ndim == 1) {
    e.st_tiles = line_resident(e.g) ? 0u : stage_tiles(e.g);
  } else if (e.g.ndim == 3) {
    const unsigned share = (unsigned)(256ul * stage_work(e.g) / work);
    const Split3 s = stage3_split(e.g, std::max(1u, share));
    e.st_tiles = s.groups;
    e.st_nbx = s.nbx;
    e.st_len = s.len;
    e.st_nch = s.nch;
  } else {
    e.st_tiles = stage2_tiles_t<false>(e.g);
    e.st_nbx = stage2_nbx_t<false>(e.g);
  }
}

hipError_t launch_batch_stages(const BatchEntry *tab, const BatchEntry *h, int n, double cfl,
                               hipStream_t st) {
  bool any = false, law[3] = {false, false, false};
  for (int i = 0; i < n; ++i)
    if (h[i].st_tiles) any = law[h[i].g.visc] = true;
  const unsigned all = h[n - 1].st_first + h[n - 1].st_tiles;
  const bool v = h[0].g.visc != VISC_NONE;
  if (h[0].g.ndim == 1) {
    bool lines = false;
    for (int i = 0; i < n; ++i) lines = lines || !h[i].st_tiles;
    if (lines) {
      if (v) kb_line<true><<<(unsigned)n, 1024, 0, st>>>(tab, cfl);
      else kb_line<false><<<(unsigned)n, 1024, 0, st>>>(tab, cfl);
    }
    for (int stage = 0; stage < 3 && any; ++stage) {
      if (v) kb_stage1<true><<<all, 256, 0, st>>>(tab, n, stage, cfl);
      else kb_stage1<false><<<all, 256, 0, st>>>(tab, n, stage, cfl);
    }
    return hipGetLastError();
  }
  if (!any) return hipSuccess;
  for (int stage = 0; stage < 3; ++stage) {
    if (h[0].g.ndim == 2) {
      if (v) kb_stage2<true><<<all, 512, 0, st>>>(tab, n, stage, cfl);
      else kb_stage2<false><<<all, 512, 0, st>>>(tab, n, stage, cfl);
      continue;
    }
    if (law[VISC_NONE]) kb_stage3<VISC_NONE><<<all, 512, 0, st>>>(tab, n, stage, cfl);
    if (law[VISC_POWER]) kb_stage3<VISC_POWER><<<all, 512, 0, st>>>(tab, n, stage, cfl);
    if (law[VISC_SUTHERLAND])
      kb_stage3<VISC_SUTHERLAND><<<all, 512, 0, st>>>(tab, n, stage, cfl);
  }
  return hipGetLastError();
}

}  // namespace dcf
