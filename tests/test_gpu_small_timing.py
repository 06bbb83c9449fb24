"""The timers of a lattice solved in one workgroup: cycles and lattice passes inside its one launch."""
import numpy as np
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


@pytest.mark.parametrize("shape,colors", [((16, 16, 16), 2), ((16, 8, 8), 2), ((10, 7, 5), 3)])
def test_cycles_and_passes_are_timed(shape, colors):
    print(f"timers of the single-workgroup solve, {shape}", flush=True)
    cfg, inp = wl.mixture_noise(shape=shape, precision="fp64")
    sim, plain = ek.EKSim(cfg, inp), ek.EKSim(cfg, inp)
    for level in (1, 2):
        sim.set_timing(level)
        before = sim.observables()["poisson_total"]
        sim.step(20)
        cycles = sim.observables()["poisson_total"] - before
        t = sim.timing()
        assert cycles > 0 and t["iter"][1] == cycles
        # inside the launches, and no cycle of three sweeps, each with its barriers, in under a microsecond
        assert 1e-3 * cycles < t["iter"][0] < t["poisson"][0]
        assert t["smooth"][1] == (3 * colors * cycles if level == 2 else 0)
        assert (0.0 < t["smooth"][0] < t["iter"][0]) == (level == 2)
    plain.step(40)
    assert np.array_equal(sim.field("phi"), plain.field("phi"))  # the clock changes nothing else
    for level in (3, 0):
        sim.set_timing(level)
        sim.step(5)
        assert sim.timing()["iter"] == (0.0, 0)
    sim.close()
    plain.close()
