"""The second basis pass of delayed reorthogonalisation loads pairs of rows on even
row counts above the 65536 of one-launch solves, single rows on others, and either
form has the widths of loads that basis_loads asks for, with the same bits.  Residuals formed on the host, iteration counts within one of the
oracle's."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")

import oracle  # noqa: E402
import paper_2104_01196_amd as g  # noqa: E402
from gen import elasticity_q1, laplace3d, poisson2d, vardiff3d  # noqa: E402

pytestmark = pytest.mark.gpu
DEV = "cuda"
RTOL = 1e-8

# name: matrix, setup options, restart, kind, (last_solve, paired)
SOLVES = {
    "one_launch": (lambda: laplace3d(20), {}, 30, g.PREC_GS2, (2, None)),
    "odd": (lambda: vardiff3d(23, seed=4), dict(basis_loads=2), 30, g.PREC_GS2, (1, 0)),
    "several_lanes": (lambda: elasticity_q1(12, 11, 10, seed=3), dict(inner=3, damping=0.7, inner_damping=0.5), 30,
                      g.PREC_GS2, (1, 0)),
    "several_lanes_wide": (lambda: elasticity_q1(12, 11, 10, seed=3),
                           dict(inner=3, damping=0.7, inner_damping=0.5, basis_loads=1), 30, g.PREC_GS2, (1, 0)),
    "diagonal_copy": (lambda: laplace3d(20), dict(spmv_format=g.FORMAT_DIA), 30, g.PREC_GS2, (1, 0)),
    "diagonal_copy_narrow": (lambda: laplace3d(20), dict(spmv_format=g.FORMAT_DIA, basis_loads=2), 30, g.PREC_GS2,
                             (1, 0)),
    "narrow_loads": (lambda: laplace3d(20), dict(basis_loads=2), 30, g.PREC_GS2, (1, 0)),
    "long_restart": (lambda: laplace3d(20), {}, 65, g.PREC_GS2, (1, 0)),
    "multicolor": (lambda: laplace3d(20), dict(build_levels=True), 30, g.PREC_MTGS, (1, 0)),
    "exact": (lambda: poisson2d(48), dict(build_levels=True), 30, g.PREC_GS_TRISOLVE, (1, 0)),
    "large": (lambda: laplace3d(42), {}, 30, g.PREC_GS2, (1, 1)),
    "large_odd": (lambda: laplace3d(41), {}, 30, g.PREC_GS2, (1, 0)),
}


@pytest.mark.parametrize("name", SOLVES)
def test_pairs(name):
    mk, kw, m, kind, (last, paired) = SOLVES[name]
    A = mk()
    dA = g.DeviceCSR.from_host(A)
    b = np.random.default_rng(3).standard_normal(A.n)
    db = torch.as_tensor(b, device=DEV)
    kw = {"variant": g.SYMMETRIC, **kw}
    h = g.gs2_setup(dA, **kw)
    x = torch.zeros(A.n, dtype=torch.float64, device=DEV)
    info = g.gmres_solve(dA, db, x, m, RTOL, 5000, kind, h)
    p = g.gs2_paths(h)
    assert p["last_solve"] == last and (paired is None or p["paired"] == paired), p
    assert info["converged"]
    if kind != g.PREC_MTGS:  # the oracle's solver has no multicolor preconditioner
        _, io = oracle.gmres(A, b, restart=m, rtol=RTOL, prec="gs2" if kind == g.PREC_GS2 else "sor",
                             variant=oracle.SYMMETRIC, inner=kw.get("inner", 1), omega=kw.get("damping", 1.0),
                             gamma=kw.get("inner_damping", 1.0))
        assert abs(info["iterations"] - io["iterations"]) <= 1
    r = b - A.to_scipy() @ x.cpu().numpy()
    assert np.linalg.norm(r) <= 1.1 * RTOL * np.linalg.norm(b)


@pytest.mark.parametrize("fmt", [g.FORMAT_AUTO, g.FORMAT_DIA])
@pytest.mark.parametrize("side", [20, 26, 38, 42])
def test_widths_have_the_same_bits(side, fmt):
    """Both passes wide or narrow, or as chosen (below 65536 rows and with no format
    asked for in one launch): 256, 512 and 1024 rows per workgroup, and pairs."""
    A = laplace3d(side)
    dA = g.DeviceCSR.from_host(A)
    b = torch.as_tensor(np.random.default_rng(4).standard_normal(A.n), device=DEV)
    xs = []
    for mode in (0, 1, 2):
        h = g.gs2_setup(dA, variant=g.SYMMETRIC, spmv_format=fmt, basis_loads=mode)
        x = torch.zeros_like(b)
        info = g.gmres_solve(dA, b, x, 40, RTOL, 60, g.PREC_GS2, h)
        bs = g.gs2_gmres_basis_schedule(h)
        assert (bs["dot_narrow_from"], bs["update_narrow_from"]) == ((8, 12) if mode == 2 else (-1, -1))
        p = g.gs2_paths(h)
        one = mode == 0 and fmt == g.FORMAT_AUTO and A.n <= 65536
        assert info["iterations"] > 12 and p["last_solve"] == (2 if one else 1)
        if not one:
            assert p["paired"] == (1 if A.n > 65536 else 0)
        xs.append((info["iterations"], x))
    if fmt == g.FORMAT_DIA or A.n <= 65536:  # above, the layout of the copy is timed for each handle's request alike
        assert xs[0][0] == xs[1][0] and torch.equal(xs[0][1], xs[1][1])
    assert xs[1][0] == xs[2][0] and torch.equal(xs[1][1], xs[2][1])
