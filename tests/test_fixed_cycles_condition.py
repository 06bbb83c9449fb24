"""What a fixed V-cycle count asks of a lattice, and that the refusal says so (host only: it comes before any
device call)."""
import ctypes

import pytest

from paper_1712_08494_amd import ek
from paper_1712_08494_amd import workloads as wl


@pytest.mark.parametrize("shape", [(50, 37, 29), (4, 128, 128), (10, 6, 6)])
def test_lattices_coarsened_by_axis_are_refused_with_the_condition(shape):
    cfg = wl.EKConfig(*shape, poisson_cycles=4)
    inp = wl.uniform(cfg)
    h = ctypes.c_void_p()
    p = ek.params_from_config(cfg)
    dp = [a.ctypes.data_as(ctypes.POINTER(ctypes.c_double)) for a in (inp.rho_a, inp.rho_b, inp.n_plus, inp.n_minus)]
    L = ek.load()
    assert L.ek_init(ctypes.byref(p), *dp, None, 0, None, ctypes.byref(h)) == ek.EK_EINVAL
    message = L.ek_last_error(h).decode()
    L.ek_destroy(h)
    assert "divisible by 4" in message and "4608" in message
