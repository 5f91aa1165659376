"""Waits within one-launch applies that end before what is waited for is there:
the wavefronts form it themselves, with the same bits as the passes launched
one by one, whatever the limit, for every precision and preconditioner form;
also beside a batched solve that holds most compute units."""
import threading

import numpy as np
import pytest

torch = pytest.importorskip("torch")

import paper_2104_01196_amd as g  # noqa: E402
from gen import convdiff2d, laplace1d, poisson2d, random_sparse  # noqa: E402

pytestmark = pytest.mark.gpu
DEV = "cuda"

MATS = {
    "one_row": lambda: laplace1d(1),
    "chain_65": lambda: laplace1d(65),
    "poisson2d_40": lambda: poisson2d(40),
    "random_3000": lambda: random_sparse(3000, seed=3, avg_offdiag=5),
    "poisson2d_150": lambda: poisson2d(150),
}
FORMS = {
    "forward_1_1": dict(variant=g.FORWARD),
    "backward_2_2": dict(variant=g.BACKWARD, sweeps=2, inner=2, damping=0.9, inner_damping=0.8),
    "symmetric_1_1": dict(variant=g.SYMMETRIC),
    "symmetric_1_4": dict(variant=g.SYMMETRIC, inner=4, damping=0.9, inner_damping=0.7),
    "compact_2_2": dict(variant=g.FORWARD, sweeps=2, inner=2, damping=0.9, compact=True),
    "jacobi_form": dict(variant=g.SYMMETRIC, sweeps=2, inner=0, damping=0.7),
    "lanes_4": dict(variant=g.SYMMETRIC, lanes_per_row=4, format=g.FORMAT_SELL),
}


def launched(f):
    g.gs2_profile(True)
    try:
        f()
        torch.cuda.synchronize()
    finally:
        g.gs2_profile(False)


def bits(t):
    return t.cpu().numpy().tobytes()


@pytest.mark.parametrize("precision", [g.FP64, g.FP32, g.FP16_SCALED])
@pytest.mark.parametrize("form", FORMS)
@pytest.mark.parametrize("name", MATS)
def test_no_wait_same_bits(name, form, precision):
    A = MATS[name]()
    h = g.gs2_setup(g.DeviceCSR.from_host(A), precision=precision, **FORMS[form])
    rng = np.random.default_rng(7)
    for looks in (0, 1, 0, 5, -1, 0):
        g.gs2_wait_looks(h, looks)
        v = torch.as_tensor(rng.standard_normal(A.n), device=DEV)
        z, zj, want, wantj = (torch.full_like(v, float("nan")) for _ in range(4))
        g.gs2_apply(h, v, z)
        g.jr_apply(h, 2, 0.8, v, zj)
        launched(lambda: (g.gs2_apply(h, v, want), g.jr_apply(h, 2, 0.8, v, wantj)))
        assert bits(z) == bits(want), looks
        assert bits(zj) == bits(wantj), looks


@pytest.mark.parametrize("looks", [-1, 4])
def test_beside_a_batched_solve(looks):
    """230 work items of a batched solve, each on a compute unit of its own for
    the whole solve, leave room for some of the apply's 1024 wavefronts only."""
    A = poisson2d(256)
    h = g.gs2_setup(g.DeviceCSR.from_host(A), variant=g.SYMMETRIC, inner=2, damping=0.9)
    g.gs2_wait_looks(h, looks)
    rng = np.random.default_rng(3)
    v = torch.as_tensor(rng.standard_normal(A.n), device=DEV)
    want = torch.empty_like(v)
    launched(lambda: g.gs2_apply(h, v, want))
    B = g.DeviceCSR.from_host(convdiff2d(60, 20.0, 1.0))
    bh = g.gs2_setup_batched([B] * 230, nrhs=4, team_rows=-1, rhs_per_item=4)
    rhs = torch.as_tensor(rng.standard_normal(230 * 4 * B.n), device=DEV)
    x = torch.zeros_like(rhs)
    side = torch.cuda.Stream()
    torch.cuda.synchronize()
    t = threading.Thread(target=lambda: g.gmres_solve_batched(bh, 4, rhs, x, 1e-30, 40, stream=side,
                                                              raise_on_error=False))
    t.start()
    n = 0
    zs = [torch.full_like(v, float("nan")) for _ in range(50)]
    while t.is_alive() or n == 0:
        for z in zs:
            g.gs2_apply(h, v, z)
        torch.cuda.current_stream().synchronize()
        n += 1
        for z in zs:
            assert torch.equal(z, want)
    t.join()
