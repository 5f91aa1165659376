"""gs2_graphs(0) launches every kernel one by one, also where a solve would run in
one launch, with the same bits; and restart cycles too large for one launch give
the same bits replayed from a graph and launched one by one: several replays with
unrelated work and synchronisation in between, even and odd row counts (pairs of rows
and single ones in the second basis pass), the closing serial work riding on the
next apply (GS2, JR) or launched by itself."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")

import paper_2104_01196_amd as g  # noqa: E402
from gen import convdiff2d, laplace3d, poisson2d  # noqa: E402

pytestmark = pytest.mark.gpu
DEV = "cuda"


def solve(dA, db, h, kind, maxit, graphs):
    prev = g.gs2_graphs(graphs)
    try:
        x = torch.zeros_like(db)
        info = g.gmres_solve(dA, db, x, 8, 1e-8, maxit, kind, h)
    finally:
        g.gs2_graphs(prev)
    del info["seconds"]
    return str(info), x


@pytest.mark.parametrize("kind", [g.PREC_NONE, g.PREC_GS2, g.PREC_JR])
def test_off_launches_small_systems(kind):
    A = poisson2d(40)
    dA = g.DeviceCSR.from_host(A)
    db = torch.as_tensor(np.random.default_rng(2).standard_normal(A.n), device=DEV)
    h = g.gs2_setup(dA, 2, 1, 0.8, g.FORWARD)
    one = solve(dA, db, h, kind, 100, True)
    assert g.gs2_paths(h)["last_solve"] == 2
    many = solve(dA, db, h, kind, 100, False)
    assert g.gs2_paths(h)["last_solve"] == 1
    assert one[0] == many[0] and torch.equal(one[1], many[1])


@pytest.mark.parametrize("kind", [g.PREC_NONE, g.PREC_GS2, g.PREC_JR])
@pytest.mark.parametrize("mk", [lambda: laplace3d(42), lambda: laplace3d(41), lambda: convdiff2d(301, 20.0, 0.5)],
                         ids=["even", "odd", "plane"])
def test_replays_of_large_cycles(mk, kind):
    A = mk()
    assert A.n > 65536
    dA = g.DeviceCSR.from_host(A)
    db = torch.as_tensor(np.random.default_rng(2).standard_normal(A.n), device=DEV)
    h = g.gs2_setup(dA, 2, 1, 0.8, g.FORWARD)
    want = solve(dA, db, h, kind, 30, False)
    x = torch.zeros_like(db)
    for rep in range(4):
        junk = torch.randn(1 << 20, device=DEV, dtype=torch.float64)
        _ = float((junk * junk).sum())
        x.zero_()
        info = g.gmres_solve(dA, db, x, 8, 1e-8, 30, kind, h)
        torch.cuda.synchronize()
        del info["seconds"]
        assert g.gs2_paths(h)["last_solve"] == 1
        assert str(info) == want[0] and torch.equal(x, want[1]), rep
    assert info["iterations"] > 16  # several cycles
