"""The power law's (T/T_ref)^omega to within an ulp, read off the CFL step of a
uniform state whose viscous rate is all there is."""
import numpy as np
import pytest

from paper_2406_19494_amd import workloads as W
from paper_2406_19494_amd.solver import Solver

pytestmark = pytest.mark.gpu

EPS = 2.0 ** -52


@pytest.mark.parametrize("omega", [0.5, 0.7, 0.76, 1.0, 1.5])
def test_power_law_to_an_ulp(omega):
    # rho = p = R = 1 and gamma - 1 = 1/2: T = 1 exactly, x = T / T_ref = 1 / T_ref
    # rounded; mu_ref = 1e40 leaves the acoustic rate below a rounding of the
    # viscous one, which is mu times a constant of the state
    print(f"[viscosity] omega {omega}", flush=True)
    T_ref = np.concatenate([[1.0], np.geomspace(0.05, 20.0, 41), np.geomspace(1e-6, 1e6, 13),
                            np.random.default_rng(1).uniform(0.5, 2.0, 20)])
    P = np.zeros((5, 1, 1, 3))
    P[0] = P[4] = 1.0
    dt = []
    for t in T_ref:
        case = W.Case(name="uniform", ndim=1, n=(3, 1, 1), gamma=1.5, R=1.0, Pr=1.0,
                      visc_law="power", mu_ref=1e40, T_ref=float(t), visc_param=omega)
        s = Solver(case)
        dt.append(s.compute_dt(s.init_state(P), cfl=0.5).item())
    x = (1.0 / T_ref).astype(np.longdouble)
    got = np.longdouble(dt[0]) / np.array(dt, dtype=np.longdouble)
    err = np.abs(got / x ** np.longdouble(omega) - 1)
    # the power within an ulp, and the roundings of mu, of three products and of
    # the quotient, half an ulp each, here and at T_ref = 1
    assert np.all(err <= (1 + 2 * 5 * 0.5) * EPS), err.max() / EPS
