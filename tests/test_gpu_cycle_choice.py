"""Which V-cycle a lattice takes where both cover it: the halving one (as many grids as its axes divide by
two) unless its coarsest grid costs more than the lattice passes that only it has."""
import pytest

from paper_1712_08494_amd import ek
from paper_1712_08494_amd import workloads as wl

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module", autouse=True)
def gpu():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU visible")
    ek.load()
    torch.cuda.init()
    yield


def halving_levels(shape):
    """Grids of the halving cycle, the lattice included."""
    d, n = list(shape), 1
    while all(k % 4 == 0 for k in d) and d[0] * d[1] * d[2] > 512:
        d, n = [k // 2 for k in d], n + 1
    return n


@pytest.mark.parametrize("kind,shape,precision,halving", [
    ("walls", (128, 16, 16), "fp32", True), ("walls", (120, 48, 48), "fp64", True), ("walls", (40, 36, 24), "fp64", False),
    ("walls", (72, 72, 48), "fp32", True), ("walls", (8, 8, 128), "fp32", False), ("walls", (24, 24, 72), "fp64", False),
    ("mixture", (128, 16, 16), "fp64", False), ("mixture", (72, 64, 64), "fp32", True), ("mixture", (8, 128, 128), "fp64", False),
    ("mixture", (16, 144, 144), "fp32", True), ("mixture", (512, 32, 32), "fp64", True),
    ("mixture", (32, 32, 32), "fp64", True)])
def test_cycle_choice(kind, shape, precision, halving):
    print(f"cycle choice, {kind} {shape} {precision}", flush=True)
    cfg, inp = (wl.walls_interface if kind == "walls" else wl.mixture_noise)(shape=shape, precision=precision)
    cfg.eps_b = 3.0 * cfg.eps_a
    sim = ek.EKSim(cfg, inp)
    sim.step(3)
    o = sim.observables()
    assert 0.0 < o["poisson_rel_max"] <= cfg.poisson_tol
    assert (o["poisson_mg_levels"] == halving_levels(shape)) == halving
    sim.close()
