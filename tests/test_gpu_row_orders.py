"""Exact and multicolor Gauss-Seidel on rows stored by level and by color
(64 rows per chunk, one wavefront each): chains whose rows all depend on their
neighbour inside one wavefront, single rows, full and ragged last chunks, rows
longer than the entries polled at once, every precision.  The oracle is the
sequential loop in float64.  Bars: 1e-11 for float64 (rounding order); for the
32-bit arithmetic forms 2e-5, a few hundred unit roundoffs, on matrices whose
scaled values (-1/4) the 32- and 16-bit formats hold exactly."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")

import oracle  # noqa: E402
import paper_2104_01196_amd as g  # noqa: E402
from gen import laplace1d, poisson2d, random_sparse  # noqa: E402

pytestmark = pytest.mark.gpu
DEV = "cuda"


def ring(n):
    """A chain whose last row is coupled to the first: columns up to n - 1 rows
    away, so that 16-bit offsets hold them up to n = 32768 only."""
    from gen import CSR

    i = np.arange(n)
    cols = np.sort(np.stack([(i - 1) % n, i, (i + 1) % n], 1), 1)
    val = np.where(cols == i[:, None], 4.0, -1.0)
    return CSR(n, np.arange(0, 3 * n + 1, 3).astype(np.int32), cols.ravel().astype(np.int32), val.ravel())


MATS = {
    "one_row": (lambda: laplace1d(1), [g.FP64]),
    "chain_63": (lambda: laplace1d(63), [g.FP64]),
    "chain_64": (lambda: laplace1d(64), [g.FP64]),
    "chain_1001": (lambda: laplace1d(1001), [g.FP64]),
    "plane_8": (lambda: poisson2d(8), [g.FP64, g.FP32, g.FP16_SCALED]),
    "plane_23": (lambda: poisson2d(23), [g.FP64, g.FP32, g.FP16_SCALED]),
    "ragged_515": (lambda: random_sparse(515, seed=31, avg_offdiag=5, long_rows=3, long_len=90, diag_only_rows=20),
                   [g.FP64]),
    "ring_32768": (lambda: ring(32768), [g.FP64, g.FP32]),
    "ring_32769": (lambda: ring(32769), [g.FP64, g.FP32]),
}


@pytest.mark.parametrize("name,prec", [(k, p) for k, (_, ps) in MATS.items() for p in ps])
@pytest.mark.parametrize("variant,sweeps,w", [(g.FORWARD, 1, 1.0), (g.BACKWARD, 2, 0.9), (g.SYMMETRIC, 2, 1.1)])
def test_level_and_color_order(name, prec, variant, sweeps, w):
    A = MATS[name][0]()
    dA = g.DeviceCSR.from_host(A)
    h = g.gs2_setup(dA, sweeps, 1, 1.0, g.FORWARD, precision=prec, build_levels=True)
    bar = 1e-11 if prec == g.FP64 else 2e-5
    for seed in (3, 4):  # the second call starts from the first one's buffers
        v = np.random.default_rng(seed).standard_normal(A.n)
        z = torch.empty(A.n, dtype=torch.float64, device=DEV)
        for call, ref in ((g.gs_trisolve_apply, oracle.sor_sweep), (g.mtgs_apply, oracle.mtgs_sweep)):
            want = ref(A, v, np.zeros(A.n), variant, sweeps, w)
            z.fill_(float("nan"))
            call(h, variant, w, torch.as_tensor(v, device=DEV), z)
            err = np.abs(z.cpu().numpy() - want).max()
            assert err <= bar * np.abs(want).max(), (call.__name__, seed, err)


def test_level_order_passes_nan_on():
    """A NaN in the input reaches the rows that depend on it, and only those."""
    A = laplace1d(200)
    h = g.gs2_setup(g.DeviceCSR.from_host(A), 1, 1, 1.0, g.FORWARD, build_levels=True)
    v = torch.ones(A.n, dtype=torch.float64, device=DEV)
    v[120] = float("nan")
    z = torch.empty_like(v)
    g.gs_trisolve_apply(h, g.FORWARD, 1.0, v, z)
    bad = torch.isnan(z).cpu().numpy()
    assert not bad[:120].any() and bad[120:].all()
