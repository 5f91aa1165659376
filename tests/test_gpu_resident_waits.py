"""One-launch solves whose waits end before what is waited for is there: the
solve is repeated launch by launch with the same bits, from the x that was passed
in, and the handle does not try again at every solve."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")

import paper_2104_01196_amd as g  # noqa: E402
from gen import laplace1d, laplace3d, poisson2d  # noqa: E402

pytestmark = pytest.mark.gpu
DEV = "cuda"

# one workgroup, several of 256 rows, of 512 and of 1024
MATS = {
    "chain_65": lambda: laplace1d(65),
    "laplace3d_10": lambda: laplace3d(10),
    "poisson2d_150": lambda: poisson2d(150),
    "poisson2d_200": lambda: poisson2d(200),
}


@pytest.mark.parametrize("kind", [g.PREC_NONE, g.PREC_GS2, g.PREC_JR])
@pytest.mark.parametrize("name", MATS)
def test_given_up_and_remembered(name, kind):
    A = MATS[name]()
    dA = g.DeviceCSR.from_host(A)
    h = g.gs2_setup(dA, 2, 1, 0.8, variant=g.SYMMETRIC)
    rng = np.random.default_rng(7)
    b = torch.as_tensor(rng.standard_normal(A.n), device=DEV)
    x0 = torch.as_tensor(rng.standard_normal(A.n), device=DEV)

    def solve():
        x = x0.clone()
        info = g.gmres_solve(dA, b, x, 10, 1e-9, 35, kind, h)
        del info["seconds"]
        return str(info), x.cpu().numpy().tobytes()

    want = solve()
    assert g.gs2_paths(h)["last_solve"] == 2
    g.gs2_wait_looks(h, 0)
    given_up = skip = in_row = 0
    for _ in range(12):
        assert solve() == want
        p = g.gs2_paths(h)
        if skip > 0:  # launched without trying
            skip -= 1
            assert (p["last_solve"], p["given_up"]) == (1, given_up)
        elif p["last_solve"] == 2:  # every first look found what it was for
            in_row = 0
        else:
            given_up, in_row = given_up + 1, in_row + 1
            assert p["given_up"] == given_up
            skip = 8 ** in_row
    if A.n > 256:  # several workgroups
        assert given_up >= 1
    h2 = g.gs2_setup(dA, 2, 1, 0.8, variant=g.SYMMETRIC)
    x = x0.clone()
    g.gmres_solve(dA, b, x, 10, 1e-9, 35, kind, h2)
    assert x.cpu().numpy().tobytes() == want[1] and g.gs2_paths(h2)["last_solve"] == 2
