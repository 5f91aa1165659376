"""Which small systems without a stencil's few distances take their applies in one
launch: those with few entries far (more than 1024 columns) from the diagonal, more of
them in 32-bit arithmetic, or two entries a row; a single Jacobi sweep, one launch as
it is, never.  Values against the oracle at the precisions' bars (1e-12 per half sweep,
2e-5)."""
from types import SimpleNamespace

import numpy as np
import pytest
import scipy.sparse as sp

torch = pytest.importorskip("torch")

import oracle  # noqa: E402
import paper_2104_01196_amd as g  # noqa: E402

pytestmark = pytest.mark.gpu
DEV = "cuda"


def scattered(n, per, reach, seed=2):
    """Rows of exactly `per` others, at distances below `reach`, both signs, wrapped around."""
    rng = np.random.default_rng(seed)
    i = np.repeat(np.arange(n), per)
    j = (i + rng.integers(1, reach, i.size) * rng.choice([-1, 1], i.size)) % n
    S = sp.coo_matrix((rng.uniform(-1.0, -0.1, i.size), (i, j)), shape=(n, n)).tocsr()
    S.sum_duplicates()
    S = (S + sp.diags(np.asarray(abs(S).sum(1)).ravel() + 0.1)).tocsr()
    S.sort_indices()
    return SimpleNamespace(n=n, rowptr=S.indptr.astype(np.int32), colind=S.indices.astype(np.int32), val=S.data)


def far(A):
    return int((np.abs(A.colind - np.repeat(np.arange(A.n), np.diff(A.rowptr))) > 1024).sum())


# rows, others a row, reach; one launch in float64, in float32
@pytest.mark.parametrize("n,per,reach,one64,one32", [
    (15_000, 5, 14_000, True, True),     # 70,000 far
    (20_000, 5, 19_000, False, True),    # 95,000
    (60_000, 5, 1_000, True, True),      # none
    (60_000, 5, 59_000, False, False),   # 295,000
    (60_000, 2, 59_000, True, True),     # two a row
])
def test_rule_and_values(n, per, reach, one64, one32):
    A = scattered(n, per, reach)
    assert (far(A) > 80_000) == (not one64 or per == 2) and (far(A) > 280_000) == (not one32)
    dA = g.DeviceCSR.from_host(A)
    v_h = np.random.default_rng(1).standard_normal(n)
    v = torch.as_tensor(v_h, device=DEV)
    z = torch.empty_like(v)
    want = oracle.gs2_apply(A, v_h, oracle.SYMMETRIC, 1, 2, 0.9)
    for precision, one, bar in ((g.FP64, one64, 2e-12), (g.FP32, one32, 2e-5)):
        h = g.gs2_setup(dA, 1, 2, 0.9, g.SYMMETRIC, precision=precision, lanes_per_row=1, format=g.FORMAT_SELL)
        g.gs2_apply(h, v, z)
        assert g.gs2_paths(h)["applies"] == (1 if one else 0)
        assert np.abs(z.cpu().numpy() - want).max() <= bar * np.abs(want).max()
        g.jr_apply(h, 1, 0.8, v, z)
        assert g.gs2_paths(h)["applies"] == (1 if one else 0)
        assert torch.allclose(z, 0.8 * v / torch.as_tensor(A.val[A.colind == np.repeat(np.arange(n), np.diff(A.rowptr))],
                                                           device=DEV), rtol=3e-7 if precision == g.FP32 else 2e-15,
                              atol=0.0)
