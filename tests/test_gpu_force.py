"""The mass-flux body force where a periodic axis meets walls with parameters or a
Dirichlet profile on a later axis: the ghosts at the edges carry these only inside
the axis, so the axis' two boundary fluxes differ and are part of the force."""
import numpy as np
import pytest
import torch

from oracle.pyoracle import Oracle
from paper_2406_19494_amd import workloads as W
from paper_2406_19494_amd.solver import Solver
from tests.helpers import flux_scale, rel_err_per_var

pytestmark = pytest.mark.gpu

RHS_TOL = 1e-11           # of the flux scale, as for every right-hand side
VJP_TOL = 1e-10           # as for every reverse step against the oracle
P2, W2, Z2, D2 = ("periodic",) * 2, ("wall",) * 2, ("zerograd",) * 2, ("disturb",) * 2

CASES = {
    "disturb_2d": ((25, 8, 1), (P2, ("zerograd", "disturb"))),
    "porous_2d": ((12, 7, 1), (P2, ("porous", "wall"))),
    "dirichlet_2d": ((12, 9, 1), (P2, ("wall", "dirichlet"))),
    "teno_2d": ((17, 9, 1), (P2, D2), "teno6a"),
    # the last axis periodic: its stage update is one launch with its fluxes
    "disturb_y_3d": ((9, 7, 6), (P2, D2, P2)),
    "disturb_z_3d": ((7, 5, 9), (P2, P2, ("wall", "disturb"))),
    "porous_z_3d": ((6, 5, 7), (P2, W2, ("porous", "wall"))),
    "dirichlet_z_3d": ((6, 5, 7), (P2, Z2, ("wall", "dirichlet"))),
    # an earlier axis with such walls: the fluxes are equal
    "disturb_x_3d": ((7, 6, 5), (D2, P2, P2)),
}


def _case(n, bc, scheme="weno5"):
    ndim = 3 if n[2] > 1 else 2
    bc = sum(bc, ()) + P2 * (3 - ndim)
    c = W.Case(name="force", ndim=ndim, n=n, hi=tuple(m / 8.0 if m > 1 else 1.0 for m in n),
               stretch=("uniform", "tanh2", "uniform"), beta=(0.0, 1.2, 0.0), R=1.3, Pr=0.7,
               visc_law="power", mu_ref=0.01, T_ref=1.0, visc_param=0.7, bc=bc,
               T_wall=(1.1, 0.0, 1.2, 1.1, 1.1, 0.0), dist_amp=(0.05,) * 6,
               dist_kappa=(0.7,) * 6, source="massflux", scheme=scheme)
    K = None
    for f, kind in enumerate(bc):
        t1, t2 = ((1, 2), (0, 2), (0, 1))[f // 2]
        if kind == "porous":
            c.porous_face, c.porous_begin, c.porous_end, c.p_inf = f, 0, n[t1] - 1, 1.1
            K = np.random.default_rng(7).uniform(0.1, 0.5, (n[t1] - 1) * n[t2])
        if kind == "dirichlet":
            P = np.random.default_rng(8).uniform(-0.1, 0.1, (5, n[t2], n[t1]))
            P[0] += 1.0
            P[1 + ndim:4] = 0.0  # a 2D flow has no w
            P[4] += 1.3
            c.dirichlet[f] = P
    return c, K


@pytest.mark.parametrize("which", list(CASES))
def test_force_has_the_boundary_fluxes_of_periodic_axes(which):
    print(f"[force] {which}", flush=True)
    case, K = _case(*CASES[which])
    o, s = Oracle(case, K=K), Solver(case, K=K, mode=1)
    U = o.cons(W.random_smooth(case, seed=5, amp=0.1))
    Ud = torch.as_tensor(U, device="cuda")
    scale = flux_scale(case, U)
    err = rel_err_per_var(s.rhs(Ud).cpu().numpy(), o.rhs(U), scale)
    tol = RHS_TOL if case.scheme == "weno5" else 10 * RHS_TOL
    assert np.all(err <= tol), err
    dt = s.compute_dt(Ud, cfl=0.3)
    V = Ud.clone()
    s.step(V, dt)
    ref, _, _ = o.run(U, 1, dt_fixed=dt.item())
    err = np.abs(V.cpu().numpy() - ref).max(axis=(1, 2, 3)) / (dt.item() * scale)
    assert np.all(err <= 9 * tol), err  # three stages, each carries the errors before it
    if case.scheme != "weno5":
        return
    lam = np.random.default_rng(11).normal(size=U.shape)
    lu_or, lk_or = o.vjp_step(U, lam, dt.item())
    gK = torch.zeros(max(s.nk, 1), dtype=torch.float64, device="cuda")
    lu = s.vjp_step(Ud, dt, torch.as_tensor(lam, device="cuda"),
                    dJdK=gK if s.nk else None).cpu().numpy()
    err = np.abs(lu - lu_or).max(axis=(1, 2, 3)) / np.abs(lu_or).max(axis=(1, 2, 3))
    assert np.all(err <= VJP_TOL), err
    if s.nk:
        assert np.abs(gK.cpu().numpy() - lk_or).max() <= VJP_TOL * np.abs(lk_or).max()
