"""3D stages in split launches (porous, disturbance and Dirichlet faces): chained
and batched steps are bitwise the single steps, also in batches that mix them with
one-launch stages of several viscosity laws."""
import numpy as np
import pytest
import torch

from paper_2406_19494_amd import workloads as W
from paper_2406_19494_amd.solver import BatchStepper, Solver

pytestmark = pytest.mark.gpu

P2, W2, Z2, D2 = ("periodic",) * 2, ("wall",) * 2, ("zerograd",) * 2, ("disturb",) * 2


def _case(n, bc, law="power"):
    return W.Case(name="split", ndim=3, n=n, hi=tuple(m / 8.0 for m in n),
                  stretch=("uniform", "tanh2", "uniform"), beta=(0.0, 1.2, 0.0), R=1.3, Pr=0.7,
                  visc_law=law, mu_ref=0.0 if law == "none" else 0.01, T_ref=1.0, visc_param=0.7,
                  bc=sum(bc, ()), T_wall=(0.0, 1.1, 1.1, 1.2, 1.1, 0.0), dist_amp=(0.02,) * 6,
                  dist_kappa=(1.5,) * 6)


# isothermal walls without viscosity: a ghost's temperature is made from the
# source's state or from its box; ghosts fill 30 and 70 % of the box
CHAINED = {
    "inviscid": _case((16, 30, 30), (("wall", "zerograd"), D2, D2), "none"),
    "inviscid_small": _case((5, 7, 6), (P2, W2, D2), "none"),
    "viscous": _case((16, 30, 30), (P2, D2, W2), "sutherland"),
}


@pytest.mark.parametrize("which", list(CHAINED))
def test_chained_steps_equal_single_steps(which):
    print(f"[split] {which}", flush=True)
    case = CHAINED[which]
    s = Solver(case)
    U = s.init_state(W.random_smooth(case, seed=4, amp=0.1))
    dt = s.compute_dt(U, cfl=0.3)
    V, dv = U.clone(), dt.clone()
    s.steps_cfl(U, dt, 3, cfl=0.3)
    for _ in range(3):
        s.step_cfl(V, dv, cfl=0.3)
    assert s.flags() == 0
    assert torch.equal(U, V) and torch.equal(dt, dv)


# one batch of one-launch members under two viscosity laws and of members with
# split launches; the order decides where the packed stage launch finds members
# without workgroups of their own
def _member(kind, k):
    return {"power": lambda: _case((7 + k, 9, 5), (P2, W2, Z2)),
            "suth": lambda: _case((16, 5 + k, 8), (W2, P2, P2), "sutherland"),
            "disturb": lambda: _case((6 + k, 8, 7), (P2, W2, D2)),
            "dirichlet": lambda: _dirichlet((9, 6 + k, 5)),
            # beyond 2^17 cells: in launches of its own
            "large": lambda: _case((52, 51 + k, 50), (P2, D2, W2)),
            # few cells per tile: split although its faces are plain
            "thin": lambda: _case((128, 3, 128 + k), (W2, P2, Z2))}[kind]()


def _dirichlet(n):
    case = _case(n, (("dirichlet", "zerograd"), W2, P2), "sutherland")
    P = np.zeros((5, n[2], n[1]))
    P[0], P[1], P[4] = 1.0, 0.1, 1.3
    case.dirichlet[0] = P
    return case


ORDERS = {
    "split_first": ("disturb", "power", "suth", "power"),
    "split_middle": ("suth", "power", "dirichlet", "disturb", "suth"),
    "split_last": ("power", "suth", "disturb", "dirichlet"),
    "split_around": ("dirichlet", "power", "disturb"),
    "split_alone": ("disturb", "dirichlet"),
    "two_laws": ("suth", "power", "suth"),
    "large": ("large", "power", "disturb", "large", "dirichlet", "thin", "suth"),
}


@pytest.mark.parametrize("cfl", [0.3, None], ids=["cfl", "fixed"])
@pytest.mark.parametrize("order", list(ORDERS))
def test_mixed_batch_equals_single_steps(order, cfl):
    print(f"[split] batch {order} {cfl}", flush=True)
    cases = [_member(kind, k) for k, kind in enumerate(ORDERS[order])]
    one, many = [Solver(c) for c in cases], [Solver(c) for c in cases]
    Us = [s.init_state(W.random_smooth(c, seed=8, amp=0.1)) for s, c in zip(one, cases)]
    dts = [s.compute_dt(U, cfl=0.3) for s, U in zip(one, Us)]
    Vs, dvs = [U.clone() for U in Us], [d.clone() for d in dts]
    bs = BatchStepper()
    for _ in range(3):
        for s, U, d in zip(one, Us, dts):
            if cfl:
                s.compute_dt(U, cfl=cfl, out=d)
            s.step(U, d)
        bs.step(many, Vs, dvs, cfl=cfl)
    torch.cuda.synchronize()
    for k, (U, V, d, e, s) in enumerate(zip(Us, Vs, dts, dvs, many)):
        assert torch.equal(U, V) and torch.equal(d, e), (order, k)
        assert s.flags() == 0
