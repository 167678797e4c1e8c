// dcf_stage.hip -- one launch per Runge-Kutta stage: a tile's cells and ghost
// cells are converted to primitives while they are loaded, every face flux of
// the tile is computed from LDS, and the stage update writes the new state.
#include <algorithm>

#include "dcf_stage.hpp"

namespace dcf {

// ---------------------------------------------------------------------------
// 2D: tiles of TX x TY cells.
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
    frame_flux<2, VISC, SCH>(g, P, Dv, mf, G);
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

// Both schemes at 4 waves per SIMD: a face's flux takes ~125 VGPRs and the
// stage waits on its dependent chains; at 5 waves (96 VGPRs) it is slower by
// a quarter (1024 x 256: 29.3 against 23.2 us).
template <bool VISC, int SCH, bool SMALL>
__global__ void __launch_bounds__(SMALL ? 256 : 512)
__attribute__((amdgpu_waves_per_eu(SCH == SCHEME_WENO5 ? 4 : 1)))
k_stage2(Dev g, StageArgs A, unsigned nbx) {
  __shared__ double lds[Tile2<VISC, SCH, SMALL>::SIZE];
  const unsigned tile = xcd_remap(blockIdx.x, gridDim.x);
  stage2_tile<VISC, SCH, SMALL>(g, A, tile, nbx, lds);
}

// Small tiles up to 2^16 cells: there 16 x 16 tiles leave CUs without one, and
// a tile's second round of faces (32 of 544) waits alone; above, their extra
// halo conversions and idle lanes cost more (256 x 64: 7.9 against 9.8 us per
// stage, 300 x 200: 10.5 against 10.8, 1024 x 256: 23.2 against 22.6).
static bool stage2_small(const Dev &g) { return g.ncell <= 65536; }

static unsigned tiles_along(int n, int t) { return (unsigned)((n + t - 1) / t); }
template <bool SMALL> static unsigned stage2_nbx_t(const Dev &g) {
  return tiles_along(g.n[0], Tile2<true, SCHEME_WENO5, SMALL>::TX);
}
template <bool SMALL> static unsigned stage2_tiles_t(const Dev &g) {
  return stage2_nbx_t<SMALL>(g) * tiles_along(g.n[1], Tile2<true, SCHEME_WENO5, SMALL>::TY);
}

bool stage_fused(const Dev &g) { return g.ndim == 2; }
unsigned stage_tiles(const Dev &g) {
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

hipError_t launch_stage(const Dev &g, const StageArgs &A, hipStream_t st) {
  if (g.ndim != 2) return hipErrorInvalidValue;
  if (g.visc != VISC_NONE) launch_stage_v<true>(g, A, st);
  else launch_stage_v<false>(g, A, st);
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

// The batch takes 16 x 16 tiles for every member (8 boundary layers of 256 x 64
// to 384 x 96: 79.8 us per step, 81.7 with 12 x 8): its members fill the chip
// together.
template <bool VISC>
__global__ void __launch_bounds__(512) __attribute__((amdgpu_waves_per_eu(4)))
kb_stage2(const BatchEntry *tab, int stage, double cfl) {
  __shared__ double lds[Tile2<VISC, SCHEME_WENO5, false>::SIZE];
  const BatchEntry &e = tab[blockIdx.y];
  if (blockIdx.x >= e.st_tiles) return;
  const StageArgs A = batch_args(e, stage, cfl);
  stage2_tile<VISC, SCHEME_WENO5, false>(e.g, A, blockIdx.x, e.st_nbx, lds);
}

void stage_entry_sizes(BatchEntry &e) {
  e.st_tiles = e.st_nbx = 0;
  if (!stage_fused(e.g)) return;
  e.st_tiles = stage2_tiles_t<false>(e.g);
  e.st_nbx = stage2_nbx_t<false>(e.g);
}

hipError_t launch_batch_stages(const BatchEntry *tab, const BatchEntry *h, int n, double cfl,
                               hipStream_t st) {
  unsigned nt = 0;
  for (int i = 0; i < n; ++i) nt = std::max(nt, h[i].st_tiles);
  const dim3 grid(nt, (unsigned)n);
  const bool v = h[0].g.visc != VISC_NONE;
  for (int stage = 0; stage < 3; ++stage) {
    if (v) kb_stage2<true><<<grid, 512, 0, st>>>(tab, stage, cfl);
    else kb_stage2<false><<<grid, 512, 0, st>>>(tab, stage, cfl);
  }
  return hipGetLastError();
}

}  // namespace dcf
