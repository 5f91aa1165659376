"""Schedules that gmres_solve times are kept for the process per size: a second
handle of the same size times nothing, one of another size in the same power of two
does, for the layout of A and for the basis passes."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")

import paper_2104_01196_amd as g  # noqa: E402
from gen import laplace1d  # noqa: E402

pytestmark = pytest.mark.gpu
DEV = "cuda"


# sizes that no other test solves; from 2^20 rows and restart 16 the basis passes are timed too
@pytest.mark.parametrize("sizes,each", [((70_001, 70_002), 1), ((1_100_002, 1_100_004), 2)])
def test_timed_per_size(sizes, each):
    for n in sizes:
        A = g.DeviceCSR.from_host(laplace1d(n))
        b = torch.as_tensor(np.random.default_rng(1).standard_normal(n), device=DEV)
        for timings in (each, 0):
            h = g.gs2_setup(A, variant=g.SYMMETRIC)
            for _ in range(2):
                g.gmres_solve(A, b, torch.zeros_like(b), 16, 1e-8, 5, g.PREC_GS2, h)
                assert g.gs2_paths(h)["timings"] == timings
            assert g.gs2_gmres_schedule(h)["tuned"] == 1


def test_conjugate_gradients_time_nothing():
    """A solve by conjugate gradients takes a layout by rule where none is known: gmres_solve then still
    times the size, and the layout it found serves later solves."""
    n = 70_011
    A = g.DeviceCSR.from_host(laplace1d(n))
    b = torch.as_tensor(np.random.default_rng(1).standard_normal(n), device=DEV)
    h = g.gs2_setup(A, variant=g.SYMMETRIC)
    g.cg_solve(A, b, torch.zeros_like(b), 1e-8, 5, g.PREC_GS2, h)
    g.gmres_solve(A, b, torch.zeros_like(b), 16, 1e-8, 5, g.PREC_GS2, h)
    assert g.gs2_paths(h)["timings"] == 1
    g.cg_solve(A, b, torch.zeros_like(b), 1e-8, 5, g.PREC_GS2, g.gs2_setup(A, variant=g.SYMMETRIC))
