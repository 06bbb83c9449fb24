"""A context's device memory holds the grids its Poisson cycles run on and no others (a host computation)."""
import ctypes

import pytest

from paper_1712_08494_amd import ek
from paper_1712_08494_amd import workloads as wl


def workspace(shape, solver):
    b = ctypes.c_size_t(0)
    p = ek.params_from_config(wl.EKConfig(*shape, precision="fp64", poisson_solver=solver))
    assert ek.load().ek_workspace_bytes(ctypes.byref(p), None, 0, ctypes.byref(b)) == ek.EK_OK
    return b.value


# Beyond an SOR context of the box: in one workgroup four axis tables (8 KiB at most, 256-byte pieces); by
# axis also the one launched grid of 8x8x128, 1024 cells of 40 bytes, and the 48-byte rows of the 1168 cells below
# and on it with the inverse of the coarsest (8 KiB).  The halving grids would add 20 and 46 KB.
@pytest.mark.parametrize("shape,most", [((16, 16, 16), 8192), ((8, 8, 128), 8192 + 40 * 1024 + 48 * 1168 + 8192)])
def test_only_the_grids_in_use_are_allocated(shape, most):
    assert 0 < workspace(shape, "auto") - workspace(shape, "sor") <= most
