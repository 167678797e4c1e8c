"""The one-launch stage kernels at the sizes where their tiles end: right-hand
sides and chained CFL steps against the oracle, and gradients whose stage boxes
are kept against gradients that rebuild them."""
import ctypes as C

import numpy as np
import pytest
import torch

from oracle.pyoracle import Oracle
from paper_2406_19494_amd import binding as B
from paper_2406_19494_amd import workloads as W
from paper_2406_19494_amd.solver import Solver
from tests.helpers import flux_scale, rel_err_per_var

pytestmark = pytest.mark.gpu

RHS_TOL = 1e-11   # of the flux scale, as for every right-hand side
# three CFL steps (nine stages) move a state by at most nine CFL numbers of its
# flux scale, each within RHS_TOL
STEP_TOL = 9 * RHS_TOL

P2, W2, Z2 = ("periodic",) * 2, ("wall",) * 2, ("zerograd",) * 2


def _case(n, bc, law="power", scheme="weno5", source="none", T_wall=1.1):
    ndim = 3 if n[2] > 1 else 2 if n[1] > 1 else 1
    bc = sum(bc, ()) + P2 * (3 - len(bc))
    # cells of about the same width, metrics that vary along the second axis
    hi = tuple(m / 16.0 if d < ndim else 1.0 for d, m in enumerate(n))
    stretch = ("uniform", "tanh2" if ndim > 1 else "uniform", "uniform")
    return W.Case(name="edge", ndim=ndim, n=n, hi=hi, stretch=stretch, beta=(0.0, 1.2, 0.0), R=1.3,
                  Pr=0.7, visc_law=law, mu_ref=0.0 if law == "none" else 0.01, T_ref=1.0,
                  visc_param=0.7, bc=bc, T_wall=(T_wall,) * 6, scheme=scheme, source=source)


EDGES = {
    # one workgroup for the line: fewest cells, its three widths' ends, then tiles of 255
    "1d_3": ((3, 1, 1), (P2,)),
    "1d_255": ((255, 1, 1), (W2,), "sutherland"),
    "1d_256_teno": ((256, 1, 1), (P2,), "power", "teno6a"),
    "1d_511": ((511, 1, 1), (Z2,), "none"),
    "1d_512": ((512, 1, 1), (P2,), "none", "teno6a"),
    "1d_1023": ((1023, 1, 1), (W2,)),
    "1d_1024": ((1024, 1, 1), (W2,)),
    "1d_1276_teno": ((1276, 1, 1), (Z2,), "none", "teno6a"),
    "1d_300_force": ((300, 1, 1), (P2,), "power", "weno5", "massflux"),
    # 12 x 8 tiles, and 16 x 16 above 2^16 cells
    "2d_3x3": ((3, 3, 1), (P2, W2)),
    "2d_12x8": ((12, 8, 1), (W2, P2), "none"),
    "2d_13x17_teno": ((13, 17, 1), (Z2, W2), "power", "teno6a"),
    "2d_25x9_force": ((25, 9, 1), (P2, W2), "power", "weno5", "massflux"),
    "2d_241x273": ((241, 273, 1), (P2, W2)),
    "2d_273x256_teno": ((273, 256, 1), (Z2, W2), "none", "teno6a"),
    # columns of 15 x 16 cells: chunks of a tile's planes, ranges over tiles
    "3d_3x3x3": ((3, 3, 3), (P2, P2, P2)),
    "3d_15x16x5": ((15, 16, 5), (P2, W2, Z2), "sutherland"),
    "3d_16x17x4": ((16, 17, 4), (W2, Z2, P2), "none"),
    "3d_31x15x9_force": ((31, 15, 9), (P2, W2, P2), "power", "weno5", "massflux"),
    "3d_47x33x40": ((47, 33, 40), (Z2, P2, W2)),
    "3d_92x97x19_force": ((92, 97, 19), (P2, W2, W2), "sutherland", "weno5", "massflux"),
}


@pytest.mark.parametrize("which", list(EDGES))
def test_stage_kernels_at_tile_edges(which):
    case = _case(*EDGES[which])
    print(f"[stage] {which}", flush=True)
    o, s = Oracle(case), Solver(case)
    U0 = o.cons(W.random_smooth(case, seed=5, amp=0.1))
    U = torch.as_tensor(U0, device="cuda")
    err = rel_err_per_var(s.rhs(U).cpu().numpy(), o.rhs(U0), flux_scale(case, U0))
    # uniform stretches let TENO6-A's cut-off fall either way on rounding
    rhs_tol = RHS_TOL if case.scheme == "weno5" else 1e-10
    assert np.all(err <= rhs_tol), err
    dt = s.compute_dt(U, cfl=0.5)
    s.steps_cfl(U, dt, 3, cfl=0.5)
    ref, dt_ref = U0, o.dt(U0, 0.5)
    for _ in range(3):
        ref, _, _ = o.run(ref, 1, dt_fixed=dt_ref)
        dt_ref = o.dt(ref, 0.5)
    assert s.flags() == 0
    vmax = np.abs(ref).max()  # a component may be zero but for rounding
    err = rel_err_per_var(U.cpu().numpy(), ref, np.full(case.nv, vmax))
    assert np.all(err <= STEP_TOL * (rhs_tol / RHS_TOL)), err
    assert abs(dt.item() - dt_ref) <= STEP_TOL * (rhs_tol / RHS_TOL) * dt_ref


@pytest.mark.parametrize("which", ["1d_1024", "2d_13x17_teno", "2d_25x9_force",
                                   "3d_31x15x9_force", "3d_47x33x40"])
def test_rhs_in_place(which):
    case = _case(*EDGES[which])
    o, s = Oracle(case), Solver(case)
    U0 = o.cons(W.random_smooth(case, seed=5, amp=0.1))
    U = torch.as_tensor(U0, device="cuda")
    p = C.c_void_p(U.data_ptr())
    B.call("dcf_rhs", s.ctx, p, p, C.c_void_p(torch.cuda.current_stream().cuda_stream))
    err = rel_err_per_var(U.cpu().numpy(), o.rhs(U0), flux_scale(case, U0))
    assert np.all(err <= (RHS_TOL if case.scheme == "weno5" else 1e-10)), err


@pytest.mark.parametrize("which", ["1d_255", "1d_1024", "2d_25x9", "3d_16x17x4", "3d_15x16x5"])
def test_kept_stage_boxes_give_the_rebuilt_boxes_gradient(which):
    n = {"2d_25x9": (25, 9, 1)}.get(which) or EDGES[which][0]
    case = _case(n, (P2, W2, P2)[:3 if n[2] > 1 else 2 if n[1] > 1 else 1])
    case.cost_face = 2 if case.ndim > 1 else 0
    U0 = torch.as_tensor(Oracle(case).cons(W.random_smooth(case, seed=6, amp=0.1)), device="cuda")
    dt = Solver(case).compute_dt(U0, cfl=0.3)
    out = [Solver(case, mode=mode, nsteps=5, seg_len=2).gradient(U0, dt) for mode in (2, 3)]
    assert torch.any(out[0][2] != 0.0)
    for a, b in zip(*out):
        assert torch.equal(a, b)


# Chained calls at the limits of their launches: more partial maxima than a stage's
# workgroups reduce themselves (more than 2048 tiles), and more steps of a short
# line than one launch takes (2048).
@pytest.mark.parametrize("n,nsteps", [((720, 736, 1), 3), ((40, 1, 1), 2051)],
                         ids=["2070_tiles", "2051_steps"])
def test_long_chains_equal_single_steps(n, nsteps):
    print(f"[stage] chain {n} {nsteps}", flush=True)
    case = _case(n, (P2, W2)[:2 if n[1] > 1 else 1])
    s = Solver(case)
    U = s.init_state(W.random_smooth(case, seed=5, amp=0.1))
    dt = s.compute_dt(U, cfl=0.4)
    V, dv = U.clone(), dt.clone()
    s.steps_cfl(U, dt, nsteps, cfl=0.4)
    for _ in range(nsteps):
        s.step_cfl(V, dv, cfl=0.4)
    assert s.flags() == 0
    assert torch.equal(U, V) and torch.equal(dt, dv)


# Grids whose stages (and right-hand sides) take the split launches though the
# one-launch kernels could: thin or ragged tiles, the body force on a small box;
# and neighbours of theirs that do not.
ROUTES = {
    "3d_thin": ((128, 3, 128), (P2, W2, Z2)),
    "3d_thin_inviscid": ((130, 4, 127), (P2, P2, W2), "none"),
    "3d_ragged": ((33, 17, 129), (Z2, W2, P2), "sutherland"),
    "3d_full_tiles": ((30, 32, 129), (P2, W2, P2)),
    "3d_force": ((16, 16, 16), (P2, W2, P2), "power", "weno5", "massflux"),
    "3d_force_walls": ((16, 15, 17), (W2, W2, W2), "power", "weno5", "massflux"),
    "3d_force_column": ((24, 24, 24), (P2, W2, P2), "power", "weno5", "massflux"),
}


@pytest.mark.parametrize("which", list(ROUTES))
def test_both_routes_of_a_stage(which):
    case = _case(*ROUTES[which])
    print(f"[stage] route {which}", flush=True)
    o, s = Oracle(case), Solver(case)
    U0 = o.cons(W.random_smooth(case, seed=5, amp=0.1))
    U = torch.as_tensor(U0, device="cuda")
    err = rel_err_per_var(s.rhs(U).cpu().numpy(), o.rhs(U0), flux_scale(case, U0))
    assert np.all(err <= RHS_TOL), err
    dt = s.compute_dt(U, cfl=0.5)
    V, dv = U.clone(), dt.clone()
    s.steps_cfl(U, dt, 2, cfl=0.5)
    s.step_cfl(V, dv, cfl=0.5)
    ref, _, _ = o.run(U0, 1, dt_fixed=o.dt(U0, 0.5))
    err = rel_err_per_var(V.cpu().numpy(), ref, np.full(case.nv, np.abs(ref).max()))
    assert np.all(err <= STEP_TOL / 3), err  # three stages, not nine
    s.step_cfl(V, dv, cfl=0.5)
    assert s.flags() == 0
    assert torch.equal(U, V) and torch.equal(dt, dv)


# Large 2D grids with TENO6-A take the split launches.  (Against the oracle the
# scheme's cut-off would fall either way on rounding somewhere in so many faces.)
# A field that repeats along x takes the same cut-offs in both routes: its
# right-hand side and step are its period's, which one launch computes, to
# rounding.
@pytest.mark.parametrize("period,repeats,law,source", [
    ((30, 520, 1), 20, "power", "none"), ((24, 520, 1), 25, "none", "none"),
    ((30, 520, 1), 20, "power", "massflux"), ((31, 896, 1), 29, "power", "none")],
    ids=["viscous", "inviscid", "force", "rhs"])
def test_large_teno_grids_repeat_their_period(period, repeats, law, source):
    print(f"[stage] teno {period} x {repeats}", flush=True)
    small = _case(period, (P2, W2), law, "teno6a", source)
    large = _case((period[0] * repeats, *period[1:]), (P2, W2), law, "teno6a", source)
    a, b = Solver(small), Solver(large)
    U = a.init_state(W.random_smooth(small, seed=5, amp=0.1))
    V = U.repeat(1, 1, 1, repeats)
    scale = flux_scale(small, U.cpu().numpy())
    err = rel_err_per_var(b.rhs(V).cpu().numpy(), a.rhs(U).repeat(1, 1, 1, repeats).cpu().numpy(),
                          scale)
    assert np.all(err <= RHS_TOL), err
    dt = a.compute_dt(U, cfl=0.5)
    a.step(U, dt)
    b.step(V, dt)
    ref = U.repeat(1, 1, 1, repeats).cpu().numpy()
    err = rel_err_per_var(V.cpu().numpy(), ref, np.full(small.nv, np.abs(ref).max()))
    assert np.all(err <= STEP_TOL / 3), err
    assert a.flags() == 0 and b.flags() == 0
