"""Column kernels against the site-order kernels on boxes that do run colour-split: walls with tiles of pairs
and chunks of planes that do not divide the lattice, the shortest rows.  The colour passes, restriction and
interpolation bit for bit; the residual sums against numpy."""
import numpy as np
import pytest

from paper_1712_08494_amd import ek
from paper_1712_08494_amd import workloads as wl
from tests.test_gpu_columns import residual

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module", autouse=True)
def gpu():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU visible")
    ek.load()
    torch.cuda.init()
    yield


# The sums' terms carry rounding errors of 1e-12 of the source or less, against the residual at hand.
@pytest.mark.parametrize("kind,shape,precision", [
    ("walls", (24, 20, 28), "fp64"), ("walls", (4, 48, 32), "fp32"), ("walls", (128, 16, 16), "fp64"),
    ("walls", (72, 72, 48), "fp32"), ("walls", (8, 64, 64), "fp64"), ("mixture", (8, 64, 64), "fp64")])
def test_split_columns_match_site_order(kind, shape, precision, monkeypatch):
    print(f"colour-split column kernels, {kind} {shape} {precision}", flush=True)
    cfg, inp = (wl.walls_interface if kind == "walls" else wl.mixture_noise)(shape=shape, precision=precision)
    cfg.eps_b = 3.0 * cfg.eps_a
    cfg.poisson_tol = 1e-4
    a = ek.EKSim(cfg, inp)
    monkeypatch.setenv("EK_POISSON_SITE_ORDER", "1")
    b = ek.EKSim(cfg, inp)
    monkeypatch.delenv("EK_POISSON_SITE_ORDER")
    assert a.device_bytes() > b.device_bytes()  # the colour-split copies
    for sim in (a, b):
        rel = sim.observables()["poisson_rel"]
        assert 0.0 < rel <= 1e-4 and abs(rel - residual(sim, cfg)) < 1e-12
    a.step(3)
    b.step(3)
    for k in ("phi", "rho_a", "rho_b", "n_plus", "n_minus"):
        assert np.array_equal(a.field(k), b.field(k)), k
    assert a.observables()["poisson_total"] == b.observables()["poisson_total"] > 0
    a.close()
    b.close()
