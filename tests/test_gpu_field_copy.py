"""Fields read into host memory: sizes around the one from which threads copy pieces, destinations
that start anywhere in a page, contexts read from several threads, against a copy into pinned memory
(the plain path).  The same bytes."""
import ctypes
import threading

import numpy as np
import pytest

from paper_1712_08494_amd import ek
from paper_1712_08494_amd import workloads as wl

pytestmark = pytest.mark.gpu

NAMES = ("rho_a", "n_plus", "phi", "ux")


@pytest.fixture(scope="module", autouse=True)
def gpu():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU visible")
    ek.load()
    torch.cuda.init()
    yield


def read(sim, name, address):
    st = ek.load().ek_get_field(sim._h, ek.FIELDS[name], ctypes.cast(address, ctypes.POINTER(ctypes.c_double)))
    assert st == ek.EK_OK


def pinned(sim, name):
    import torch
    t = torch.empty(sim.N, dtype=torch.float64).pin_memory()
    read(sim, name, t.data_ptr())
    return t.numpy().copy()


@pytest.mark.parametrize("shape,precision", [((128, 128, 63), "fp32"), ((128, 128, 64), "fp64"), ((130, 126, 65), "fp32")])
def test_pieces_give_the_same_bytes(shape, precision):
    print(f"field copies {shape} {precision}", flush=True)
    cfg, inp = wl.mixture_noise(shape=shape, precision=precision)
    cfg.poisson_tol = 1e-4
    sim = ek.EKSim(cfg, inp)
    sim.step(1)
    for name in NAMES:
        want = pinned(sim, name)
        assert np.array_equal(sim.field(name).ravel(), want), name
        for skip in (1, 511, 262143):  # words before the destination, which end untouched
            out = np.full(sim.N + skip + 5, -7.0)
            read(sim, name, out.ctypes.data + 8 * skip)
            assert np.array_equal(out[skip:-5], want) and np.all(out[:skip] == -7.0) and np.all(out[-5:] == -7.0)
    pops = sim.populations(1)
    assert np.allclose(pops.sum(axis=0), sim.field("rho_b"), rtol=1e-5)
    sim.close()


def test_contexts_read_from_several_threads():
    sims = []
    for seed in (1, 2, 3):
        cfg, inp = wl.mixture_noise(128, precision="fp32", seed=seed)
        cfg.poisson_tol = 1e-4
        sims.append(ek.EKSim(cfg, inp))
    want = [[pinned(s, n) for n in NAMES] for s in sims]
    got = [None] * len(sims)

    def run(k):
        got[k] = [sims[k].field(n).ravel() for n in NAMES]

    threads = [threading.Thread(target=run, args=(k,)) for k in range(len(sims))]
    for t in threads:
        t.start()
    for t in threads:
        t.join()
    for g, w in zip(got, want):
        assert all(np.array_equal(a, b) for a, b in zip(g, w))
    for s in sims:
        s.close()
