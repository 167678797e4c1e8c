"""The reverse step's ghost collection and its two 3D forms: short axes whose
two sides copy the same cells, every boundary kind on the later axes, the walls'
parameters on edge columns, and grids on both sides of the size up to which the
flux adjoints of all directions run in one launch."""
import numpy as np
import pytest
import torch

from oracle.pyoracle import Oracle
from paper_2406_19494_amd import workloads as W
from paper_2406_19494_amd.solver import Solver

pytestmark = pytest.mark.gpu

VJP_TOL = 1e-10  # as for every reverse step against the oracle
P2, W2, Z2, D2 = ("periodic",) * 2, ("wall",) * 2, ("zerograd",) * 2, ("disturb",) * 2


def _case(n, bc, law="power", source="none", porous=None):
    ndim = 3 if n[2] > 1 else 2 if n[1] > 1 else 1
    c = W.Case(name="faces", ndim=ndim, n=n, hi=tuple(m / 8.0 if m > 1 else 1.0 for m in n),
               stretch=("uniform", "tanh2" if ndim > 1 else "uniform", "uniform"),
               beta=(0.0, 1.2, 0.0), R=1.3, Pr=0.7, visc_law=law,
               mu_ref=0.0 if law == "none" else 0.01, T_ref=1.0, visc_param=0.7,
               bc=sum(bc, ()) + P2 * (3 - len(bc)), T_wall=(1.1, 0.0, 1.2, 1.1, 1.1, 0.0),
               dist_amp=(0.02,) * 6, dist_kappa=(1.5,) * 6, source=source)
    if porous:
        c.porous_face, c.porous_begin, c.porous_end, c.p_inf = *porous, 1.1
    return c


FACES = {
    "short_walls_1d": _case((3, 1, 1), (W2,)),
    "short_zerograd_1d": _case((4, 1, 1), (Z2,), "none"),
    "short_2d": _case((3, 5, 1), (W2, P2), "sutherland"),
    "zerograd_corner_2d": _case((7, 6, 1), (Z2, Z2)),
    "inviscid_2d": _case((6, 7, 1), (P2, W2), "none"),
    "porous_x_2d": _case((6, 7, 1), (("porous", "wall"), Z2), porous=(0, 2, 5)),
    "short_3d": _case((3, 4, 5), (P2, W2, P2)),
    "zerograd_3d": _case((5, 4, 6), (W2, Z2, Z2)),
    "disturb_z_3d": _case((5, 6, 5), (P2, W2, D2), "sutherland"),
    "disturb_x_3d": _case((6, 5, 4), (D2, P2, W2)),
    "disturb_z_inviscid_3d": _case((4, 5, 6), (Z2, P2, D2), "none"),
    # tiles of 8 wavefronts (59 cells and their ghosts), the last that fill one
    "long_y_2d": _case((4, 49, 1), (P2, W2)),
    "long_y_full_2d": _case((3, 53, 1), (Z2, W2), "none"),
    # more cells along the wall's normal than columns along the wall
    "disturb_narrow_2d": _case((5, 21, 1), (Z2, ("disturb", "zerograd"))),
    "porous_y_3d": _case((6, 6, 4), (Z2, ("porous", "zerograd"), W2), porous=(2, 1, 5)),
}


def _params(n, seed=7):
    """Porous coefficients of the case's layout (the rest follows the case)."""
    return np.random.default_rng(seed).uniform(0.1, 0.5, n)


@pytest.mark.parametrize("which", list(FACES))
def test_faces_match_dense_oracle_adjoint(which):
    case = FACES[which]
    print(f"[faces] {which}", flush=True)
    K = None
    if case.porous_face >= 0:
        nt2 = case.n[1 if case.porous_face >= 4 else 2]
        K = _params((case.porous_end - case.porous_begin) * nt2)
    o, s = Oracle(case, K=K), Solver(case, K=K, mode=1)
    U = o.cons(W.random_smooth(case, seed=5, amp=0.1))
    lam = np.random.default_rng(11).normal(size=U.shape)
    dt = 1e-3
    lu_or, lk_or = o.vjp_step(U, lam, dt)
    gK = torch.zeros(max(s.nk, 1), dtype=torch.float64, device="cuda")
    lu = s.vjp_step(torch.as_tensor(U, device="cuda"),
                    torch.full((1,), dt, dtype=torch.float64, device="cuda"),
                    torch.as_tensor(lam, device="cuda"), dJdK=gK if s.nk else None).cpu().numpy()
    err = np.abs(lu - lu_or).max(axis=(1, 2, 3)) / np.abs(lu_or).max(axis=(1, 2, 3))
    assert np.all(err <= VJP_TOL), err
    if s.nk:
        gk = gK.cpu().numpy()[: s.nk]
        assert np.abs(gk - lk_or).max() <= VJP_TOL * np.abs(lk_or).max(), (gk, lk_or)


@pytest.mark.parametrize("n", [(64, 64, 64), (64, 65, 64), (19, 50, 49), (110, 49, 51)],
                         ids=["one_launch", "per_direction", "one_launch_long_tiles",
                              "per_direction_long_tiles"])
@pytest.mark.parametrize("which", ["force", "disturb"])
def test_both_3d_forms_dot_product(n, which):
    print(f"[3d forms] {n} {which}", flush=True)
    case = (_case(n, (P2, W2, P2), source="massflux") if which == "force"
            else _case(n, (Z2, W2, D2), "sutherland"))
    o, s = Oracle(case), Solver(case, mode=1)
    U = o.cons(W.random_smooth(case, seed=5, amp=0.1))
    rng = np.random.default_rng(12)
    v = rng.normal(size=U.shape) * np.abs(U).max(axis=(1, 2, 3), keepdims=True)
    vk = rng.normal(size=o.nk)
    lam = rng.normal(size=U.shape)
    dt = 1e-3
    _, jv = o.jvp_step(U, v, dt, vk)
    gK = torch.zeros(max(s.nk, 1), dtype=torch.float64, device="cuda")
    lu = s.vjp_step(torch.as_tensor(U, device="cuda"),
                    torch.full((1,), dt, dtype=torch.float64, device="cuda"),
                    torch.as_tensor(lam, device="cuda"), dJdK=gK if s.nk else None).cpu().numpy()
    lhs = np.sum(lam * jv)
    rhs = np.sum(lu * v) + (np.sum(gK.cpu().numpy()[: s.nk] * vk) if s.nk else 0.0)
    assert abs(lhs - rhs) <= VJP_TOL * max(abs(lhs), np.sum(np.abs(lam * jv))), (lhs, rhs)


# disturbance walls along two or three axes at once, each face with parameters of
# its own: the faces of one side of every axis are reduced in the same launch
SEVERAL = {
    "xy_low_2d": ((7, 6, 1), (("disturb", "zerograd"), ("disturb", "wall"))),
    "xy_2d": ((5, 9, 1), (D2, D2)),
    "yz_low_3d": ((5, 6, 4), (P2, ("disturb", "wall"), ("disturb", "zerograd"))),
    "yz_3d": ((4, 5, 6), (Z2, D2, D2)),
    "xz_3d": ((6, 4, 5), (D2, W2, D2)),
    "xyz_inviscid_3d": ((5, 4, 6), (D2, D2, D2), "none"),
}


def _several(n, bc, law="power"):
    case = _case(n, bc, law)
    case.dist_amp = (0.02, -0.03, 0.04, 0.05, -0.06, 0.07)
    case.dist_kappa = (1.5, 0.7, 1.1, 2.3, 0.9, 1.9)
    return case


@pytest.mark.parametrize("which", list(SEVERAL))
def test_disturbance_walls_on_several_axes(which):
    print(f"[faces] {which}", flush=True)
    case = _several(*SEVERAL[which])
    o, s = Oracle(case), Solver(case, mode=1)
    U = o.cons(W.random_smooth(case, seed=5, amp=0.1))
    lam = np.random.default_rng(11).normal(size=U.shape)
    dt = 1e-3
    lu_or, lk_or = o.vjp_step(U, lam, dt)
    gK = torch.zeros(s.nk, dtype=torch.float64, device="cuda")
    lu = s.vjp_step(torch.as_tensor(U, device="cuda"),
                    torch.full((1,), dt, dtype=torch.float64, device="cuda"),
                    torch.as_tensor(lam, device="cuda"), dJdK=gK).cpu().numpy()
    err = np.abs(lu - lu_or).max(axis=(1, 2, 3)) / np.abs(lu_or).max(axis=(1, 2, 3))
    assert np.all(err <= VJP_TOL), err
    gk = gK.cpu().numpy()
    assert np.abs(gk - lk_or).max() <= VJP_TOL * np.abs(lk_or).max(), (gk, lk_or)


def test_disturbance_walls_on_several_axes_per_direction_launches():
    case = _several((64, 65, 64), (P2, D2, D2), "sutherland")
    print(f"[3d forms] {case.n} disturb yz", flush=True)
    o, s = Oracle(case), Solver(case, mode=1)
    U = o.cons(W.random_smooth(case, seed=5, amp=0.1))
    rng = np.random.default_rng(12)
    lam = rng.normal(size=U.shape)
    gK = torch.zeros(s.nk, dtype=torch.float64, device="cuda")
    dt = 1e-3
    s.vjp_step(torch.as_tensor(U, device="cuda"),
               torch.full((1,), dt, dtype=torch.float64, device="cuda"),
               torch.as_tensor(lam, device="cuda"), dJdK=gK)
    gk = gK.cpu().numpy()
    for i in range(s.nk):  # each parameter's derivative by itself
        vk = np.zeros(s.nk)
        vk[i] = 1.0
        _, jv = o.jvp_step(U, np.zeros_like(U), dt, vk)
        lhs = np.sum(lam * jv)
        assert abs(lhs - gk[i]) <= VJP_TOL * np.sum(np.abs(lam * jv)), (i, lhs, gk[i])
