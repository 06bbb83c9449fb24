"""Column kernels of the Poisson solve (even axes): tiles and chunks of planes that do not divide the
lattice, the shortest axes, walls.  The colour passes, restriction and interpolation against the
site-order kernels bit for bit; the residual sums, which both layouts share, against numpy."""
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


def residual(sim, cfg):
    """|s + A phi| / |s| over the Poisson domain from the fields of the context."""
    phi, eps, q = (sim.field(k) for k in ("phi", "eps", "q"))
    lo, hi = (1, cfg.nz - 1) if cfg.walls_z else (0, cfg.nz)
    s = q.copy()
    if cfg.walls_z:
        s[lo] += cfg.sigma_wall[0]
        s[hi - 1] += cfg.sigma_wall[1]
    s -= s[lo:hi].mean()
    r = s.copy()
    for axis in range(3):
        for d in (1, -1):
            f = 0.5 * (eps + np.roll(eps, d, axis)) * (np.roll(phi, d, axis) - phi)
            if axis == 0 and cfg.walls_z:
                f[lo if d == 1 else hi - 1] = 0.0
            r += f
    return np.linalg.norm(r[lo:hi]) / np.linalg.norm(s[lo:hi])


@pytest.mark.parametrize("kind,shape,precision", [("walls", (40, 36, 24), "fp32"), ("mixture", (24, 20, 28), "fp64"),
                                                  ("mixture", (256, 192, 64), "fp32"), ("walls", (4, 40, 64), "fp64")])
def test_columns_match_site_order(kind, shape, precision, monkeypatch):
    print(f"column kernels, {kind} {shape} {precision}", flush=True)
    cfg, inp = (wl.walls_interface if kind == "walls" else wl.mixture_noise)(shape=shape, precision=precision)
    cfg.eps_b = 3.0 * cfg.eps_a
    cfg.poisson_tol = 1e-4
    cfg.poisson_solver = "mg"
    a = ek.EKSim(cfg, inp)
    monkeypatch.setenv("EK_POISSON_SITE_ORDER", "1")
    b = ek.EKSim(cfg, inp)
    monkeypatch.delenv("EK_POISSON_SITE_ORDER")
    # the sums' terms carry rounding errors of 1e-16 of eps phi, 1e-12 of the source or less,
    # against residuals above 1e-7 of it
    for sim in (a, b):
        rel = sim.observables()["poisson_rel"]
        assert 1e-7 < rel <= 1e-4
        assert abs(rel / residual(sim, cfg) - 1.0) < 1e-5
    a.step(3)
    b.step(3)
    for k in ("phi", "rho_a", "rho_b", "n_plus", "n_minus"):
        assert np.array_equal(a.field(k), b.field(k)), k
    assert a.observables()["poisson_total"] == b.observables()["poisson_total"] > 0
    a.close()
    b.close()
