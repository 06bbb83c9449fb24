"""Fields and populations read from a context on hipStreamPerThread, a handle that names another
stream in every thread: the copy's helper threads take their pieces behind the work that the calling
thread has queued.  Against the same steps of a context on the default stream, byte for byte."""
import ctypes

import numpy as np
import pytest

from paper_1712_08494_amd import ek
from paper_1712_08494_amd import workloads as wl

pytestmark = pytest.mark.gpu

PER_THREAD = ctypes.c_void_p(2)  # hipStreamPerThread


@pytest.fixture(scope="module", autouse=True)
def gpu():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU visible")
    ek.load()
    torch.cuda.init()
    yield


@pytest.mark.parametrize("precision", ["fp32", "fp64"])
def test_reads_follow_the_steps_queued_before_them(precision):
    print(f"field reads on the per-thread stream, 128x128x80 {precision}", flush=True)
    cfg, inp = wl.mixture_noise(shape=(128, 128, 80), precision=precision)
    cfg.poisson_tol = 1e-4
    cfg.poisson_cycles = 3  # steps are only queued: the reads come while they run
    a, b = ek.EKSim(cfg, inp, stream=PER_THREAD), ek.EKSim(cfg, inp)
    for name in ("rho_a", "n_plus", "phi", "uz"):
        a.step(10)
        got = a.field(name)
        b.step(10)
        assert np.array_equal(got, b.field(name)), name
    a.step(10)
    got = a.populations(1)
    b.step(10)
    assert np.array_equal(got, b.populations(1))
    a.step(10)
    got = a.observables(("rho_b", "phi"))["fields"]
    b.step(10)
    want = b.observables(("rho_b", "phi"))["fields"]
    assert all(np.array_equal(got[k], want[k]) for k in want)
    a.close()
    b.close()


def test_reads_with_another_device_current():
    import torch
    if torch.cuda.device_count() < 2:
        pytest.skip("needs two GPUs")
    cfg, inp = wl.mixture_noise(shape=(128, 128, 80), precision="fp32")
    cfg.poisson_tol = 1e-4
    with torch.cuda.device(0):
        sim = ek.EKSim(cfg, inp, stream=torch.cuda.Stream(0).cuda_stream)
        sim.step(1)
    with torch.cuda.device(1):
        got = sim.field("phi")
    with torch.cuda.device(0):
        assert np.array_equal(got, sim.field("phi"))
        sim.close()
