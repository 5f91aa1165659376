"""Conjugate gradients on the solver's copy of A: every layout of the copy,
and a copy that no longer fits.  The solver checks its true residual against
rtol before it reports convergence; forming b - A x here differs from that by
rounding only, far below a tenth of rtol."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")

import paper_2104_01196_amd as g  # noqa: E402
from gen import elasticity_q1, laplace1d, laplace3d, poisson2d  # noqa: E402

pytestmark = pytest.mark.gpu
DEV = "cuda"
RTOL = 1e-10


def residual(A, b, x):
    """||b - A x|| / ||b||, repeated columns summed."""
    rows = np.repeat(np.arange(A.n), np.diff(A.rowptr))
    r = b.copy()
    np.subtract.at(r, rows, A.val * x[A.colind])
    return np.linalg.norm(r) / np.linalg.norm(b)


def solve(A, dA, h, kind, seed):
    b = np.random.default_rng(seed).standard_normal(A.n)
    x = torch.zeros(A.n, dtype=torch.float64, device=DEV)
    info = g.cg_solve(dA, torch.as_tensor(b, device=DEV), x, RTOL, 5000, kind, h)
    assert info["converged"]
    assert residual(A, b, x.cpu().numpy()) <= 1.1 * RTOL
    return info["iterations"]


# 1 row, one and several workgroups, a ragged last one, more than the 65536
# rows from which the layout is timed
MATS = {
    "one_row": lambda: laplace1d(1),
    "chain_257": lambda: laplace1d(257),
    "poisson2d_33": lambda: poisson2d(33),
    "laplace3d_17": lambda: laplace3d(17),
    "laplace3d_41": lambda: laplace3d(41),
    "elasticity_7_6_5": lambda: elasticity_q1(7, 6, 5),
    "elasticity_30_30_25": lambda: elasticity_q1(30, 30, 25),
}


@pytest.mark.parametrize("name", MATS)
@pytest.mark.parametrize("fmt", [g.FORMAT_AUTO, g.FORMAT_SELL, g.FORMAT_DIA, g.FORMAT_BLOCK3])
def test_layouts(name, fmt):
    A = MATS[name]()
    dA = g.DeviceCSR.from_host(A)
    h = g.gs2_setup(dA, variant=g.SYMMETRIC, spmv_format=fmt)
    # one undamped inner sweep is no definite preconditioner for elasticity
    prec = g.PREC_NONE if name.startswith("elasticity") else g.PREC_GS2
    its = [solve(A, dA, h, kind, 3) for kind in (prec, g.PREC_NONE, prec)]
    assert its[0] == its[2]
    dA.val.mul_(2.0)  # values changed in place
    A.val = A.val * 2.0
    solve(A, dA, h, g.PREC_NONE, 4)


@pytest.mark.parametrize("fmt", [g.FORMAT_AUTO, g.FORMAT_SELL, g.FORMAT_DIA])
def test_pattern_changed_in_place(fmt):
    """The arrays of one matrix overwritten by those of its mirror image, whose
    rows have other lengths, and by a permuted one whose offsets differ."""
    A = poisson2d(40)
    keep = np.nonzero(np.arange(A.n) >= A.n // 2)[0]
    rows = np.repeat(np.arange(A.n), np.diff(A.rowptr))
    # no couplings among the last half: rows of one entry there
    drop = (rows >= keep[0]) & (A.colind >= keep[0]) & (rows != A.colind)
    from types import SimpleNamespace

    def build(r, c, v):
        o = np.lexsort((c, r))
        rp = np.zeros(A.n + 1, dtype=np.int64)
        np.add.at(rp, r + 1, 1)
        return SimpleNamespace(n=A.n, rowptr=np.cumsum(rp).astype(np.int32), colind=c[o].astype(np.int32), val=v[o])

    r, c, v = rows[~drop], A.colind[~drop], A.val[~drop]
    # the couplings between the halves are one-sided row sums at most 4: SPD
    first = build(r, c, v)
    mirror = build(A.n - 1 - r, A.n - 1 - c, v)
    perm = np.random.default_rng(1).permutation(A.n)
    shuffled = build(perm[r], perm[c], v)
    dA = g.DeviceCSR.from_host(first)
    h = g.gs2_setup(dA, variant=g.SYMMETRIC, spmv_format=fmt)
    for B in (first, mirror, shuffled, first):
        dA.rowptr.copy_(torch.as_tensor(B.rowptr))
        dA.colind.copy_(torch.as_tensor(B.colind))
        dA.val.copy_(torch.as_tensor(B.val))
        solve(B, dA, h, g.PREC_NONE, 5)


@pytest.mark.parametrize("fmt", [g.FORMAT_AUTO, g.FORMAT_DIA])
def test_rows_not_sorted(fmt):
    """A matrix whose rows hold columns in reverse and twice: no layout
    without column indices, the entries summed."""
    A = laplace3d(12)
    dA0 = g.DeviceCSR.from_host(A)
    h = g.gs2_setup(dA0, variant=g.SYMMETRIC, spmv_format=fmt)
    solve(A, dA0, h, g.PREC_GS2, 6)
    from types import SimpleNamespace

    parts = [np.concatenate([A.colind[a:b][::-1], A.colind[a:b]]) for a, b in zip(A.rowptr[:-1], A.rowptr[1:])]
    vals = [np.concatenate([A.val[a:b][::-1], A.val[a:b]]) * 0.5 for a, b in zip(A.rowptr[:-1], A.rowptr[1:])]
    B = SimpleNamespace(n=A.n, rowptr=(2 * A.rowptr.astype(np.int64)).astype(np.int32), colind=np.concatenate(parts),
                        val=np.concatenate(vals))
    dB = g.DeviceCSR.from_host(B)
    for _ in range(2):
        solve(B, dB, h, g.PREC_GS2, 7)
    solve(A, dA0, h, g.PREC_GS2, 8)
