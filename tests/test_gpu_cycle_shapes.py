"""V-cycle shapes and fixed cycle counts on contexts coarsened by axis and on those solved in one workgroup:
cycles without sweeps before or after a correction converge to the same potential, and enough fixed cycles take the
steps of the solves to a tolerance."""
import numpy as np
import pytest

from paper_1712_08494_amd import ek
from paper_1712_08494_amd import workloads as wl
from tests.parity import phi_err

pytestmark = pytest.mark.gpu

BOXES = [(22, 18, 31), (4, 40, 40), (50, 11, 9), (16, 16, 16), (10, 7, 5), (16, 8, 8)]


@pytest.fixture(scope="module", autouse=True)
def gpu():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU visible")
    ek.load()
    torch.cuda.init()
    yield


# Both potentials meet a residual of 1e-11: the smoothest mode can carry sqrt(sites) of it, below 1e-8.
@pytest.mark.parametrize("box", BOXES)
@pytest.mark.parametrize("counts,omega", [((0, 2, 0, 1), 1.0), ((2, 0, 1, 0), 1.2), ((0, 1, 2, 0), 1.1), ((3, 3, 0, 0), 1.3)])
def test_shapes_converge_to_the_same_potential(box, counts, omega):
    print(f"V-cycle shape {counts} {omega}, {box}", flush=True)
    cfg, inp = wl.mixture_noise(shape=box, precision="fp64")
    cfg.eps_b = 3.0 * cfg.eps_a
    a, b = ek.EKSim(cfg, inp), ek.EKSim(cfg, inp)
    b.set_multigrid(*counts, omega=omega)
    for sim in (a, b):
        sim.step(2)
        st, it, rel = sim.poisson(1e-11, 400)
        assert st == ek.EK_OK and rel <= 1e-11
    assert phi_err(a.field("phi"), b.field("phi")) < 1e-8
    assert b.observables()["poisson_total"] != a.observables()["poisson_total"]  # the shape is in use
    a.close()
    b.close()


# Twenty cycles take a residual far below 1e-10, so the fields differ by what solves to 1e-10 leave.
@pytest.mark.parametrize("box,precision", [((4, 40, 40), "fp64"), ((4, 40, 40), "fp32"), ((16, 16, 16), "fp64"),
                                           ((8, 8, 16), "fp32")])
def test_fixed_cycles_take_the_converged_steps(box, precision):
    print(f"fixed cycles {box} {precision}", flush=True)
    cfg, inp = wl.mixture_noise(shape=box, precision=precision)
    cfg.eps_b = 3.0 * cfg.eps_a
    a = ek.EKSim(cfg, inp)
    cfg.poisson_cycles = 20
    b = ek.EKSim(cfg, inp)
    for sim in (a, b):
        sim.step(5)
    ob = b.observables()
    assert ob["poisson_iters"] == 20 and 0.0 < ob["poisson_rel_max"] <= cfg.poisson_tol
    assert phi_err(a.field("phi"), b.field("phi")) < 1e-7
    for k in ("rho_a", "rho_b", "n_plus", "n_minus"):
        x, y = a.field(k), b.field(k)
        assert np.max(np.abs(x - y) / np.abs(y)) < (1e-9 if precision == "fp64" else 1e-6), k
    a.close()
    b.close()
