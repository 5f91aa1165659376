"""Conjugate gradients on a sliced-ELL copy that stays in the last-level cache between
products beside the triangles and vectors (normal loads), and on one that does not
(non-temporal loads): banded matrices well on either side, for few and many lanes per
row, with and without a preconditioner, the true residual formed on the host; the
solver's own differs from it by rounding only, far below a tenth of rtol."""
from types import SimpleNamespace

import numpy as np
import pytest

torch = pytest.importorskip("torch")

import paper_2104_01196_amd as g  # noqa: E402

pytestmark = pytest.mark.gpu
DEV = "cuda"
RTOL = 1e-9


def banded(n, k):
    """Symmetric, k entries to either side, strictly dominant diagonal."""
    import scipy.sparse as sp

    rng = np.random.default_rng(k)
    offs = np.arange(1, k + 1)
    diags = [-rng.uniform(0.5, 1.0, n - d) for d in offs]
    A = sp.diags(diags + diags + [np.full(n, 2.0 * k + 1.0)], list(offs) + list(-offs) + [0]).tocsr()
    A.sort_indices()
    return A


# copies of 39 to 250 MB; triangles of about as much and six vectors beside them, against 230 MB
@pytest.mark.parametrize("kind", [g.PREC_GS2, g.PREC_NONE])
@pytest.mark.parametrize("n,k", [(50_001, 32), (320_001, 32), (300_001, 5), (1_900_001, 5)])
def test_either_side_of_the_limit(n, k, kind):
    A = banded(n, k)
    dA = g.DeviceCSR.from_host(SimpleNamespace(n=n, rowptr=A.indptr, colind=A.indices, val=A.data))
    h = g.gs2_setup(dA, variant=g.SYMMETRIC, spmv_format=g.FORMAT_SELL)
    b = np.random.default_rng(1).standard_normal(n)
    for _ in range(2):
        x = torch.zeros(n, dtype=torch.float64, device=DEV)
        info = g.cg_solve(dA, torch.as_tensor(b, device=DEV), x, RTOL, 1000, kind, h)
        assert info["converged"]
        r = b - A @ x.cpu().numpy()
        assert np.linalg.norm(r) <= 1.1 * RTOL * np.linalg.norm(b)
