"""GMRES on a matrix whose rows hold their columns in descending order, or
every entry in two halves (columns down, then up): every entry counts, in
every layout request, with the preconditioner of the sorted matrix and without
a handle, below and above the 65536 rows from which the layout of the solver's
copy is timed.  The residual is formed on the host from the stored entries; the
solver's own differs from it by rounding only, far below a tenth of rtol."""
from types import SimpleNamespace

import numpy as np
import pytest

torch = pytest.importorskip("torch")

import paper_2104_01196_amd as g  # noqa: E402
from gen import elasticity_q1, laplace3d  # noqa: E402

pytestmark = pytest.mark.gpu
DEV = "cuda"
RTOL = 1e-8
MATS = {
    "laplace3d_12": lambda: laplace3d(12),
    "laplace3d_41": lambda: laplace3d(41),  # 68921 rows: the layout is timed
    "elasticity_12_11_10": lambda: elasticity_q1(12, 11, 10, seed=3),
}


def rows_of(A, halves):
    """A's rows in descending column order; halves: each entry twice, with half its value."""
    spans = list(zip(A.rowptr[:-1], A.rowptr[1:]))
    if halves:
        ci = [np.concatenate([A.colind[a:b][::-1], A.colind[a:b]]) for a, b in spans]
        va = [0.5 * np.concatenate([A.val[a:b][::-1], A.val[a:b]]) for a, b in spans]
    else:
        ci = [A.colind[a:b][::-1] for a, b in spans]
        va = [A.val[a:b][::-1] for a, b in spans]
    rp = A.rowptr.astype(np.int64) * (2 if halves else 1)
    return SimpleNamespace(n=A.n, rowptr=rp.astype(np.int32), colind=np.concatenate(ci), val=np.concatenate(va))


def residual(A, b, x):
    rows = np.repeat(np.arange(A.n), np.diff(A.rowptr))
    r = b.copy()
    np.subtract.at(r, rows, A.val * x[A.colind])
    return np.linalg.norm(r) / np.linalg.norm(b)


@pytest.mark.parametrize("halves", [False, True])
@pytest.mark.parametrize("fmt", [g.FORMAT_AUTO, g.FORMAT_SELL, g.FORMAT_DIA, g.FORMAT_BLOCK3])
@pytest.mark.parametrize("name", MATS)
def test_every_entry_counts(name, fmt, halves):
    A = MATS[name]()
    B = rows_of(A, halves)
    dB = g.DeviceCSR.from_host(B)
    b = np.random.default_rng(5).standard_normal(A.n)
    db = torch.as_tensor(b, device=DEV)
    ela = name.startswith("elasticity")
    h = g.gs2_setup(g.DeviceCSR.from_host(A), 1, 3 if ela else 1, 0.7 if ela else 1.0, g.SYMMETRIC,
                    inner_damping=0.5 if ela else 1.0, spmv_format=fmt)
    its = []
    for M, kind, handle in ((dB, g.PREC_GS2, h), (g.DeviceCSR.from_host(A), g.PREC_GS2, h),
                            (dB, g.PREC_NONE, None)):
        x = torch.zeros(A.n, dtype=torch.float64, device=DEV)
        info = g.gmres_solve(M, db, x, 50, RTOL, 20000, kind, handle)
        assert info["converged"]
        assert residual(B, b, x.cpu().numpy()) <= 1.1 * RTOL
        its.append(info["iterations"])
    assert abs(its[0] - its[1]) <= 1  # the sorted matrix's
