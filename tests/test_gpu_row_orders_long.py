"""Exact Gauss-Seidel on rows longer than the 8 or 16 entries taken at a time: rows of
9 entries on average with longer ones among them (8 at a time, the chunks' main entries
counted), of more than 12 (16 at a time), one lane short of and past a block, full and
ragged last chunks, first half sweeps (no previous iterate) and later ones, every
precision.  The oracle is the sequential loop in float64.  Bars as for short rows: 1e-11
for float64, 2e-5 for the 32-bit arithmetic forms on scaled values (-1/32) that the 32-
and 16-bit formats hold exactly."""
from types import SimpleNamespace

import numpy as np
import pytest
import scipy.sparse as sp

torch = pytest.importorskip("torch")

import oracle  # noqa: E402
import paper_2104_01196_amd as g  # noqa: E402
from gen import elasticity_q1, random_sparse  # noqa: E402

pytestmark = pytest.mark.gpu
DEV = "cuda"


def banded(n, k):
    """k entries of -1 to either side, diagonal 32."""
    offs = [d for d in range(-k, k + 1) if d]
    A = sp.diags([np.full(n - abs(d), -1.0) for d in offs] + [np.full(n, 32.0)], offs + [0]).tocsr()
    A.sort_indices()
    return SimpleNamespace(n=n, rowptr=A.indptr.astype(np.int32), colind=A.indices.astype(np.int32), val=A.data)


ALL = [g.FP64, g.FP32, g.FP16_SCALED]
MATS = {
    "banded_4": (lambda: banded(700, 4), ALL),    # 8 others: not counted
    "banded_5": (lambda: banded(704, 5), ALL),    # 10: counted, two blocks of 8
    "banded_7": (lambda: banded(1000, 7), ALL),   # 14: blocks of 16
    "banded_8": (lambda: banded(641, 8), ALL),    # 16: one full block
    "banded_12": (lambda: banded(333, 12), ALL),  # 24: a block and a half
    "elasticity": (lambda: elasticity_q1(5, 4, 6, seed=2), [g.FP64]),
    "random_9": (lambda: random_sparse(1500, seed=5, avg_offdiag=9, long_rows=6, long_len=200), [g.FP64]),
    "random_25": (lambda: random_sparse(900, seed=6, avg_offdiag=25, long_rows=2, long_len=400, diag_only_rows=30),
                  [g.FP64]),
}


@pytest.mark.parametrize("name,prec", [(k, p) for k, (_, ps) in MATS.items() for p in ps])
@pytest.mark.parametrize("variant,sweeps,w", [(g.FORWARD, 1, 1.0), (g.BACKWARD, 1, 1.0), (g.SYMMETRIC, 1, 0.9),
                                              (g.FORWARD, 3, 1.1), (g.SYMMETRIC, 2, 1.0)])
def test_long_rows(name, prec, variant, sweeps, w):
    A = MATS[name][0]()
    h = g.gs2_setup(g.DeviceCSR.from_host(A), sweeps, 1, 1.0, g.FORWARD, precision=prec, build_levels=True)
    bar = 1e-11 if prec == g.FP64 else 2e-5
    for seed in (3, 4):
        v = np.random.default_rng(seed).standard_normal(A.n)
        z = torch.full((A.n,), float("nan"), dtype=torch.float64, device=DEV)
        want = oracle.sor_sweep(A, v, np.zeros(A.n), variant, sweeps, w)
        g.gs_trisolve_apply(h, variant, w, torch.as_tensor(v, device=DEV), z)
        assert np.abs(z.cpu().numpy() - want).max() <= bar * np.abs(want).max()
