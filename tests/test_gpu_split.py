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
