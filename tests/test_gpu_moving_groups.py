"""Moving particles, one and more than 64 (the pair search takes 64 at a time; a box is walked by as
many workgroups as fill the chip): mask, fraction and fields follow the oracle."""
import numpy as np
import pytest

from oracle import oracle as orc
from paper_1712_08494_amd import ek
from paper_1712_08494_amd import workloads as wl
from tests.parity import compare

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module", autouse=True)
def gpu():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU visible")
    ek.load()
    torch.cuda.init()
    yield


@pytest.mark.parametrize("count,radius", [(1, 6.0), (75, 1.7)])
def test_few_and_many_boxes_match_the_oracle(count, radius):
    print(f"{count} moving spheres of radius {radius}", flush=True)
    cfg = wl.EKConfig(40, 40, 24, reproject=True, move_particles=True, precision="fp64", E_ext=(1e-4, 0.0, 2e-4))
    cfg.poisson_tol = 1e-12
    inp = wl.uniform(cfg, 0.6, 0.4, 1e-3, 1e-3)
    r = np.random.Generator(np.random.PCG64(5))
    grid = np.array([(x, y, z) for z in range(3) for y in range(5) for x in range(5)], float)[:count]
    p = np.zeros((count, 8))
    p[:, 0:3] = 8.0 * grid + r.uniform(3.0, 5.0, (count, 3))
    p[:, 3:6] = r.uniform(-0.08, 0.08, (count, 3))
    p[:, 6] = radius
    inp.particles = p
    sim, o = ek.EKSim(cfg, inp), orc.Oracle(cfg, inp)
    changed = 0
    for _ in range(3):
        before = o.field("solid").copy()
        sim.step(4)
        o.step(4)
        changed += int(np.sum(o.field("solid") != before))
        assert np.array_equal(sim.field("solid"), o.field("solid"))
        assert np.array_equal(sim.field("psi_s"), o.field("psi_s"))
    assert changed > 0
    compare(sim, o, "fp64", f"{count} moving spheres")
    pg, po = sim.particles(), o.particles()
    # positions and velocities are sums of a few thousand FP64 terms over 12 steps
    assert np.abs(pg[:, 0:6] - po[:, 0:6]).max() < 1e-10
    sim.close()
    o.close()
