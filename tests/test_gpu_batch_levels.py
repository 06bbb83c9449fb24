"""Replicas of a batch cycle on the halving grids whatever a context of their box would take by itself:
they report those, and their first solve is on them."""
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


def test_replicas_report_the_grids_they_cycle_on():
    print("batch levels", flush=True)
    # one workgroup by itself; coarsened by axis by itself; the halving cycle either way
    reps = [wl.mixture_noise(shape=s, precision="fp64") for s in ((16, 16, 16), (8, 8, 128), (32, 32, 32))]
    b = ek.EKBatch([c for c, _ in reps], [i for _, i in reps], cycles=8)
    b.step(4)
    b.sync()
    assert [b.replica(r).observables()["poisson_mg_levels"] for r in range(3)] == [2, 3, 3]
    b.close()
