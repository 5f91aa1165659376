"""Applies of small systems in one launch against the same applies pass by
pass (which per-kernel profiling selects): the same bits, for every precision
and preconditioner form, one row to the most, ragged wavefronts, rows without
entries, long rows, several lanes per row, repeated applies, applies with other
sweeps in between, replays from a graph, and values that are not finite."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")

import paper_2104_01196_amd as g  # noqa: E402
from gen import elasticity_q1, laplace1d, laplace3d, poisson2d, random_sparse, vardiff3d  # noqa: E402

pytestmark = pytest.mark.gpu
DEV = "cuda"

MATS = {
    "one_row": lambda: laplace1d(1),
    "chain_63": lambda: laplace1d(63),
    "chain_65": lambda: laplace1d(65),
    "laplace3d_16": lambda: laplace3d(16),
    "vardiff3d_23": lambda: vardiff3d(23, seed=4),
    "elasticity_7_6_5": lambda: elasticity_q1(7, 6, 5),  # rows of up to 80 others: pass by pass
    "band_16": lambda: banded(1000, 8),                  # 16 others: the most
    "short_rows": lambda: random_sparse(2000, seed=5, avg_offdiag=2),
    "random_3000": lambda: random_sparse(3000, seed=3, avg_offdiag=6, long_rows=3, long_len=60, neg_diag_rows=40),
    "poisson2d_256": lambda: poisson2d(256),  # 65536: the most rows
    "chain_65537": lambda: laplace1d(65537),  # one more: pass by pass
}
FORMS = {
    "forward_1_1": dict(variant=g.FORWARD),
    "backward_2_2": dict(variant=g.BACKWARD, sweeps=2, inner=2, damping=0.9, inner_damping=0.8),
    "symmetric_1_1": dict(variant=g.SYMMETRIC),
    "symmetric_1_4": dict(variant=g.SYMMETRIC, inner=4, damping=0.9),  # 8 exchanged vectors: the most
    "symmetric_2_2": dict(variant=g.SYMMETRIC, sweeps=2, inner=2),     # more: pass by pass
    "compact_2_2": dict(variant=g.FORWARD, sweeps=2, inner=2, damping=0.9, compact=True),
    "jacobi_form": dict(variant=g.SYMMETRIC, sweeps=2, inner=0, damping=0.7),
    "lanes_4": dict(variant=g.SYMMETRIC, lanes_per_row=4, format=g.FORMAT_SELL),
    "lanes_2": dict(variant=g.SYMMETRIC, lanes_per_row=2, format=g.FORMAT_SELL),
    "lanes_8": dict(variant=g.SYMMETRIC, lanes_per_row=8, format=g.FORMAT_SELL),  # pass by pass
}


def banded(n, k):
    """k nonzero diagonals to either side, other values everywhere."""
    from types import SimpleNamespace

    rows = [np.arange(max(0, i - k), min(n, i + k + 1)) for i in range(n)]
    ci = np.concatenate(rows)
    ri = np.repeat(np.arange(n), [len(r) for r in rows])
    val = np.random.default_rng(2).uniform(-1.0, 1.0, ci.size)
    val[ri == ci] = 2.0 * k
    return SimpleNamespace(n=n, rowptr=np.concatenate([[0], np.cumsum([len(r) for r in rows])]).astype(np.int32),
                           colind=ci.astype(np.int32), val=val)


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
def test_same_bits_as_pass_by_pass(name, form, precision):
    A = MATS[name]()
    dA = g.DeviceCSR.from_host(A)
    h = g.gs2_setup(dA, precision=precision, **FORMS[form])
    rng = np.random.default_rng(7)
    for rep in range(3):
        v = torch.as_tensor(rng.standard_normal(A.n), device=DEV)
        z, zj, want, wantj = (torch.empty_like(v) for _ in range(4))
        g.gs2_apply(h, v, z)
        g.jr_apply(h, 2, 0.8, v, zj)
        launched(lambda: (g.gs2_apply(h, v, want), g.jr_apply(h, 2, 0.8, v, wantj)))
        assert bits(z) == bits(want)
        assert bits(zj) == bits(wantj)


def test_replayed_from_a_graph():
    A = poisson2d(50)
    dA = g.DeviceCSR.from_host(A)
    h = g.gs2_setup(dA, variant=g.SYMMETRIC)
    v, z = (torch.zeros(A.n, dtype=torch.float64, device=DEV) for _ in range(2))
    s = torch.cuda.Stream()
    graph = torch.cuda.CUDAGraph()
    g.gs2_apply(h, v, z)
    torch.cuda.synchronize()
    with torch.cuda.graph(graph, stream=s):
        for _ in range(3):
            g.gs2_apply(h, v, z, stream=s)
    rng = np.random.default_rng(1)
    for _ in range(4):
        v.copy_(torch.as_tensor(rng.standard_normal(A.n)))
        graph.replay()
        torch.cuda.synchronize()
        got = z.clone()
        g.gs2_apply(h, v, z)
        torch.cuda.synchronize()
        assert bits(got) == bits(z)
        want = torch.empty_like(z)
        launched(lambda: g.gs2_apply(h, v, want))
        assert bits(got) == bits(want)


def test_values_not_finite():
    A = poisson2d(40)
    dA = g.DeviceCSR.from_host(A)
    h = g.gs2_setup(dA, variant=g.SYMMETRIC)
    v = torch.as_tensor(np.random.default_rng(1).standard_normal(A.n), device=DEV)
    v[70], v[900], v[1300] = float("nan"), float("inf"), -float("inf")
    z, want = torch.empty_like(v), torch.empty_like(v)
    for _ in range(2):
        g.gs2_apply(h, v, z)
        launched(lambda: g.gs2_apply(h, v, want))
        assert np.array_equal(z.cpu().numpy(), want.cpu().numpy(), equal_nan=True)
