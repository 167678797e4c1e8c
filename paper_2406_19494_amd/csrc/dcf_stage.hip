// dcf_stage.hip -- one launch per Runge-Kutta stage: a tile's cells and ghost
// cells are converted to primitives while they are loaded, every face flux of
// the tile is computed from LDS, and the stage update writes the new state.
#include <algorithm>

#include "dcf_stage.hpp"

namespace dcf {

// ---------------------------------------------------------------------------
// 2D: tiles of 16 x 16 cells.
// ---------------------------------------------------------------------------
template <bool VISC, int SCH> struct Tile2 {
  static constexpr int T = 16, W = T + 6;         // cells, window cells per axis
  static constexpr int NP = VISC ? 6 : 4;         // rho, u, v, p (, T, mu)
  // offsets of the derivative cells along the face's axis: -2 .. 1 (fourth
  // order) or -3 .. 2 around each of the 17 faces
  static constexpr int HD = SCH == SCHEME_TENO6A ? 3 : 2, WD = T + 2 * HD;
  static constexpr int NF = T * (T + 1);          // faces per direction
  static constexpr int PR = 0;                    // [NP][W][W]
  static constexpr int DX = NP * W * W;           // [2][T][WD]: dv/dy, du/dy
  static constexpr int DY = DX + (VISC ? 2 * T * WD : 0);  // [2][WD][T]: du/dx, dv/dx
  static constexpr int FL = DY + (VISC ? 2 * T * WD : 0);  // [4][2 NF]
  static constexpr int SIZE = FL + 4 * 2 * NF;    // doubles
  static constexpr int NT = 576;                  // 9 wavefronts: one face per thread
};

template <bool VISC, int SCH>
__device__ __forceinline__ void stage2_tile(const Dev &g, const StageArgs &A, unsigned tile,
                                            unsigned nbx, double *lds) {
  using L = Tile2<VISC, SCH>;
  constexpr int T = L::T, W = L::W, WD = L::WD, HD = L::HD, NF = L::NF, NT = L::NT;
  constexpr int WW = W * W;
  const int tid = threadIdx.x;
  const int i0 = (int)(tile % nbx) * T, j0 = (int)(tile / nbx) * T;
  const int nx = g.n[0], ny = g.n[1];
  double *pr = lds + L::PR;
  __shared__ double shx[NT / 64];
  const double dt = stage_dt<NT>(A, tile == 0, shx);
  // primitives of the window
  for (int w = tid; w < WW; w += NT) {
    const int ly = w / W, lx = w % W;
    const int p[3] = {i0 + lx - 3, j0 + ly - 3, 0};
    if (p[0] > nx + 2 || p[1] > ny + 2) continue;
    double q[NQ];
    load_prims<2, VISC>(g, A.Uin, p, q);
    pr[w] = q[QR];
    pr[WW + w] = q[QU];
    pr[2 * WW + w] = q[QV];
    pr[3 * WW + w] = q[QP];
    if (VISC) {
      pr[4 * WW + w] = q[QT];
      pr[5 * WW + w] = q[QMU];
    }
    if (A.box.Q[0]) {
      // the box of Uin, each cell by the tile that holds its nearest
      // interior cell
      const int ci = min(max(p[0], 0), nx - 1), cj = min(max(p[1], 0), ny - 1);
      if (ci / T == i0 / T && cj / T == j0 / T) {
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
  }
  __syncthreads();
  if constexpr (VISC) {
    // tangential velocity derivatives at the cells of the face stencils
    auto cell = [&](int w, int s) {  // pr + w: a velocity; s: window stride
      const double *v = pr + w;
      if (SCH == SCHEME_TENO6A)
        return dcell6(v[-3 * s], v[-2 * s], v[-s], v[s], v[2 * s], v[3 * s]);
      return dcell4(v[-2 * s], v[-s], v[s], v[2 * s]);
    };
    for (int d = tid; d < 2 * T * WD; d += NT) {
      const bool yd = d >= T * WD;
      const int e = yd ? d - T * WD : d;
      int lx, ly;  // window position
      double m;
      if (!yd) {   // x faces: derivatives along y
        const int r = e / WD;
        ly = r + 3;
        lx = e % WD + 3 - HD;
        m = g.mc[1][min(j0 + r, ny - 1)];
      } else {     // y faces: derivatives along x
        const int c = e % T;
        lx = c + 3;
        ly = e / T + 3 - HD;
        m = g.mc[0][min(i0 + c, nx - 1)];
      }
      const int w = ly * W + lx, s = yd ? 1 : W;
      const int un = yd ? 2 * WW : WW, ut = yd ? WW : 2 * WW;  // normal, tangential velocity
      double *out = lds + (yd ? L::DY : L::DX) + e;
      out[0] = cell(ut + w, s) * m;
      out[T * WD] = cell(un + w, s) * m;
    }
    __syncthreads();
  }
  // one face per thread: 16 rows of 17 x faces, then 17 rows of 16 y faces
  double *fl = lds + L::FL;
  for (int f = tid; f < 2 * NF; f += NT) {
    const bool yf = f >= NF;
    const int e = yf ? f - NF : f;
    const int r = yf ? e / T : e / (T + 1), c = yf ? e % T : e % (T + 1);
    if (i0 + c > nx - (yf ? 1 : 0) || j0 + r > ny - (yf ? 0 : 1)) continue;
    const double *q0 = pr + (r + 3) * W + c + 3;
    const int s = yf ? W : 1;
    const int on = yf ? 2 * WW : WW, ot = yf ? WW : 2 * WW;
    const double *d0 = lds + (yf ? L::DY + (r + HD) * T + c : L::DX + r * WD + c + HD);
    const int sd = yf ? T : 1;
    const double mf = VISC ? (yf ? g.mf[1][j0 + r] : g.mf[0][i0 + c]) : 0.0;
    auto P = [&](int m, int o) {
      const int a = m == 0 ? 0 : (m == 1 ? on : (m == 2 ? ot : (m - 1) * WW));
      return q0[a + o * s];
    };
    auto Dv = [&](int k, int o) { return d0[k * T * WD + o * sd]; };
    double G[5];
    frame_flux<2, VISC, SCH>(g, P, Dv, mf, G);
    fl[f] = G[0];
    fl[2 * NF * (yf ? 2 : 1) + f] = G[1];
    fl[2 * NF * (yf ? 1 : 2) + f] = G[2];
    fl[2 * NF * 3 + f] = G[4];
  }
  __syncthreads();
  double sig = 0.0;
  const int tx = tid % T, ty = tid / T;
  const int p[3] = {i0 + tx, j0 + ty, 0};
  if (ty < T && p[0] < nx && p[1] < ny) {
    const double idx = g.idx[0][p[0]], idy = g.idx[1][p[1]];
    double R[5];
#pragma unroll
    for (int m = 0; m < 4; ++m) {
      const double *fx = fl + 2 * NF * m + ty * (T + 1) + tx;
      const double *fy = fl + 2 * NF * m + NF + ty * T + tx;
      double r = 0.0;
      r -= (fx[1] - fx[0]) * idx;
      r -= (fy[T] - fy[0]) * idy;
      R[m == 3 ? 4 : m] = r;
    }
    R[3] = 0.0;
    sig = update_state<2>(g, A, p, dt, R, A.dtpart != nullptr);
  }
  if (A.dtpart) {
    const double m = block_max<NT>(sig, shx);
    if (tid == 0) A.dtpart[tile] = m;
  }
}

template <bool VISC, int SCH>
__global__ void __launch_bounds__(576) __attribute__((amdgpu_waves_per_eu(SCH == SCHEME_WENO5 ? 5 : 1)))
k_stage2(Dev g, StageArgs A, unsigned nbx) {
  __shared__ double lds[Tile2<VISC, SCH>::SIZE];
  const unsigned tile = xcd_remap(blockIdx.x, gridDim.x);
  stage2_tile<VISC, SCH>(g, A, tile, nbx, lds);
}

static unsigned stage2_nbx(const Dev &g) { return (unsigned)(g.n[0] + 15) / 16; }
static unsigned stage2_tiles(const Dev &g) {
  return stage2_nbx(g) * (unsigned)((g.n[1] + 15) / 16);
}

bool stage_fused(const Dev &g) { return g.ndim == 2; }
unsigned stage_tiles(const Dev &g) { return stage2_tiles(g); }

template <bool VISC>
static void launch_stage2(const Dev &g, const StageArgs &A, hipStream_t st) {
  const unsigned n = stage2_tiles(g), nbx = stage2_nbx(g);
  if (g.scheme == SCHEME_TENO6A)
    k_stage2<VISC, SCHEME_TENO6A><<<n, 576, 0, st>>>(g, A, nbx);
  else
    k_stage2<VISC, SCHEME_WENO5><<<n, 576, 0, st>>>(g, A, nbx);
}

hipError_t launch_stage(const Dev &g, const StageArgs &A, hipStream_t st) {
  if (g.ndim != 2) return hipErrorInvalidValue;
  if (g.visc != VISC_NONE) launch_stage2<true>(g, A, st);
  else launch_stage2<false>(g, A, st);
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

template <bool VISC>
__global__ void __launch_bounds__(576) __attribute__((amdgpu_waves_per_eu(5)))
kb_stage2(const BatchEntry *tab, int stage, double cfl) {
  __shared__ double lds[Tile2<VISC, SCHEME_WENO5>::SIZE];
  const BatchEntry &e = tab[blockIdx.y];
  if (blockIdx.x >= e.st_tiles) return;
  const StageArgs A = batch_args(e, stage, cfl);
  stage2_tile<VISC, SCHEME_WENO5>(e.g, A, blockIdx.x, e.st_nbx, lds);
}

void stage_entry_sizes(BatchEntry &e) {
  e.st_tiles = e.st_nbx = 0;
  if (!stage_fused(e.g)) return;
  e.st_tiles = stage_tiles(e.g);
  e.st_nbx = stage2_nbx(e.g);
}

hipError_t launch_batch_stages(const BatchEntry *tab, const BatchEntry *h, int n, double cfl,
                               hipStream_t st) {
  unsigned nt = 0;
  for (int i = 0; i < n; ++i) nt = std::max(nt, h[i].st_tiles);
  const dim3 grid(nt, (unsigned)n);
  const bool v = h[0].g.visc != VISC_NONE;
  for (int stage = 0; stage < 3; ++stage) {
    if (v) kb_stage2<true><<<grid, 576, 0, st>>>(tab, stage, cfl);
    else kb_stage2<false><<<grid, 576, 0, st>>>(tab, stage, cfl);
  }
  return hipGetLastError();
}

}  // namespace dcf
