"""The setup's pattern scan: the layouts a matrix qualifies for follow from its
distinct offsets, counted here with numpy, at the limits (32 and 33 offsets
per triangle, 64 in all, more than the scan's tables hold), for short and long
rows and for a last row short of a full group."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")

import oracle  # noqa: E402
import paper_2104_01196_amd as g  # noqa: E402
from gen import elasticity_q1, random_sparse, vardiff3d  # noqa: E402
from gen.problems import CSR  # noqa: E402

pytestmark = pytest.mark.gpu
DEV = "cuda"


def banded(n, offsets, seed=5):
    """Every row holds the given offsets that stay inside the matrix; diagonally dominant."""
    offs = np.array(sorted(set(offsets) | {0}))
    cols = np.arange(n)[:, None] + offs
    mask = (cols >= 0) & (cols < n)
    vals = np.random.default_rng(seed).uniform(-1.0, 1.0, cols.shape)
    vals[:, offs == 0] = (np.abs(vals) * mask).sum(1, keepdims=True) + 1.0
    rp = np.concatenate([[0], np.cumsum(mask.sum(1))]).astype(np.int32)
    return CSR(n, rp, cols[mask].astype(np.int32), vals[mask])


CASES = {
    "32_each": lambda: banded(4111, list(range(-32, 0)) + list(range(1, 33))),
    "33_below": lambda: banded(4111, list(range(-33, 0)) + list(range(1, 5))),
    "33_above": lambda: banded(4111, [-7] + list(range(1, 34))),
    "80_each": lambda: banded(4099, list(range(-80, 0)) + list(range(1, 81))),
    "spread": lambda: banded(5003, [-4800, -70, -1, 2, 90, 4700]),
    "none": lambda: banded(4096, []),
    "one_sided": lambda: banded(4200, [-3, -2, -1]),
    "vardiff_17": lambda: vardiff3d(17, seed=3),
    "elasticity_12": lambda: elasticity_q1(12, 12, 12, seed=3),
    "random": lambda: random_sparse(4500, seed=7, avg_offdiag=5, long_rows=2, long_len=300),
}


@pytest.mark.parametrize("name", list(CASES))
def test_layouts_follow_the_offsets(name):
    A = CASES[name]()
    dA = g.DeviceCSR.from_host(A)
    row = np.repeat(np.arange(A.n, dtype=np.int64), np.diff(A.rowptr))
    d = A.colind - row
    low, up = np.unique(d[d < 0]), np.unique(d[d > 0])
    nl, nu = int((d < 0).sum()), int((d > 0).sum())

    def fits(k, nnz, rows):
        return k <= 32 and rows * k * A.n <= 1.5 * nnz + rows * 64.0 * k

    dia = fits(len(low), nl, 1) and fits(len(up), nu, 1)
    nd = A.colind // 3 - row // 3
    blow, bup = np.unique(nd[d < 0]), np.unique(nd[d > 0])
    b3 = A.n % 3 == 0 and fits(len(blow), nl, 3) and fits(len(bup), nu, 3)
    v = np.random.default_rng(1).standard_normal(A.n)
    want = oracle.gs2_apply(A, v, oracle.SYMMETRIC, 1, 2, 0.9)
    for fmt, ok, k in ((g.FORMAT_SELL, True, None), (g.FORMAT_DIA, dia, (len(low), len(up))),
                       (g.FORMAT_BLOCK3, b3, (len(blow), len(bup)))):
        if not ok:
            with pytest.raises(g.Gs2Error) as e:
                g.gs2_setup(dA, 1, 2, 0.9, g.SYMMETRIC, format=fmt)
            assert e.value.status == -1
            continue
        h = g.gs2_setup(dA, 1, 2, 0.9, g.SYMMETRIC, format=fmt)
        s, q = g.gs2_handle_schedule(h), g.gs2_handle_query(h)
        assert (q["nnz_l"], q["nnz_u"]) == (nl, nu)
        if k is not None:
            assert s["format"] == fmt and (s["ndiag_l"], s["ndiag_u"]) == k
        z = torch.empty(A.n, dtype=torch.float64, device=DEV)
        g.gs2_apply(h, torch.as_tensor(v, device=DEV), z)
        assert np.abs(z.cpu().numpy() - want).max() <= 4e-12 * np.abs(want).max()  # 1e-12 per half sweep
