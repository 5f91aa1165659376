"""Solves of small systems in one launch against the same solves launch by
launch (which per-kernel profiling selects): the same bits, iteration counts
and records, for every precision and preconditioner form, one workgroup to
the most, full and ragged last workgroups and wavefronts, several lanes per
row, restarts, exhausted budgets, nonzero initial guesses, b = 0 and
non-finite input; the oracle's iteration counts within the usual one."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")

import oracle  # noqa: E402
import paper_2104_01196_amd as g  # noqa: E402
from gen import convdiff2d, laplace1d, laplace3d, poisson2d, random_sparse, vardiff3d  # noqa: E402

pytestmark = pytest.mark.gpu
DEV = "cuda"

MATS = {
    "one_row": lambda: laplace1d(1),
    "chain_65": lambda: laplace1d(65),
    "laplace3d_10": lambda: laplace3d(10),      # 1000 rows: a ragged wavefront
    "chain_257": lambda: laplace1d(257),        # a second workgroup with one row
    "poisson2d_32": lambda: poisson2d(32),      # 1024
    "poisson2d_33": lambda: poisson2d(33),      # 1089
    "poisson2d_128": lambda: poisson2d(128),    # 16384: the most rows at 256 per workgroup
    "chain_16385": lambda: laplace1d(16385),    # at 512
    "chain_32769": lambda: laplace1d(32769),    # at 1024, a last workgroup of one row
    "vardiff3d_23": lambda: vardiff3d(23, seed=4),
    "convdiff_101": lambda: convdiff2d(101, 30.0, 1.0),
    "random_3000": lambda: random_sparse(3000, seed=3, avg_offdiag=6, long_rows=3, long_len=60, neg_diag_rows=40),
    "poisson2d_256": lambda: poisson2d(256),    # 65536: the most rows
}
FORMS = {
    "none": (g.PREC_NONE, {}),
    "jr_2": (g.PREC_JR, dict(sweeps=2, damping=0.8)),
    "forward_1_1": (g.PREC_GS2, dict(variant=g.FORWARD)),
    "backward_2_2": (g.PREC_GS2, dict(variant=g.BACKWARD, sweeps=2, inner=2, damping=0.9)),
    "symmetric_1_1": (g.PREC_GS2, dict(variant=g.SYMMETRIC)),
    "compact_2_2": (g.PREC_GS2, dict(variant=g.FORWARD, sweeps=2, inner=2, damping=0.9, compact=True)),
    "jacobi_form": (g.PREC_GS2, dict(variant=g.SYMMETRIC, sweeps=2, inner=0, damping=0.7)),
}


def both(dA, b, x0, h, m, rtol, maxit, kind):
    """The solve in one launch, and launch by launch."""
    out = []
    for launches in (False, True):
        x = x0.clone()
        if launches:
            g.gs2_profile(True)
        try:
            info = g.gmres_solve(dA, b, x, m, rtol, maxit, kind, h, raise_on_error=False)
        finally:
            g.gs2_profile(False)
        del info["seconds"]
        out.append((info, x))
    return out


def same(a, b):
    return str(a[0]) == str(b[0]) and a[1].cpu().numpy().tobytes() == b[1].cpu().numpy().tobytes()


@pytest.mark.parametrize("prec", [g.FP64, g.FP32, g.FP16_SCALED])
@pytest.mark.parametrize("form", list(FORMS))
@pytest.mark.parametrize("name", list(MATS))
def test_same_bits_as_the_launches(name, form, prec):
    A = MATS[name]()
    dA = g.DeviceCSR.from_host(A)
    kind, kw = FORMS[form]
    h = g.gs2_setup(dA, **{"variant": g.FORWARD, **kw}, precision=prec)
    rng = np.random.default_rng(7)
    b = torch.as_tensor(rng.standard_normal(A.n), device=DEV)
    x0 = torch.as_tensor(rng.standard_normal(A.n), device=DEV)
    for m, maxit, guess in ((20, 47, torch.zeros_like(b)), (7, 16, x0)):
        one, many = both(dA, b, guess, h, m, 1e-8, maxit, kind)
        assert same(one, many), (one[0], many[0], float((one[1] - many[1]).abs().max()))


@pytest.mark.parametrize("lanes", [1, 2, 4, 8])
def test_lanes_per_row(lanes):
    A = MATS["random_3000"]()
    dA = g.DeviceCSR.from_host(A)
    b = torch.as_tensor(np.random.default_rng(8).standard_normal(A.n), device=DEV)
    h = g.gs2_setup(dA, 1, 2, 0.9, g.SYMMETRIC, lanes_per_row=lanes)
    one, many = both(dA, b, torch.zeros_like(b), h, 30, 1e-10, 200, g.PREC_GS2)
    assert same(one, many) and one[0]["converged"]


def test_edges_and_oracle():
    A = MATS["vardiff3d_23"]()
    dA = g.DeviceCSR.from_host(A)
    h = g.gs2_setup(dA, 1, 1, 1.0, g.SYMMETRIC, stagnation_cycles=2)
    b_h = np.random.default_rng(9).standard_normal(A.n)
    b, zero = torch.as_tensor(b_h, device=DEV), torch.zeros(A.n, dtype=torch.float64, device=DEV)
    _, io = oracle.gmres(A, b_h, restart=30, rtol=1e-8, prec="gs2", variant=oracle.SYMMETRIC)
    one, many = both(dA, b, zero, h, 30, 1e-8, 2000, g.PREC_GS2)
    assert same(one, many) and one[0]["converged"] and abs(one[0]["iterations"] - io["iterations"]) <= 1
    # already solved, no budget, b = 0 with a nonzero guess, non-finite b, stagnation (restart 1)
    for rhs, x0, m, rtol, maxit in ((b, one[1], 30, 1e-6, 100), (b, zero, 30, 1e-8, 0), (zero, b, 30, 1e-8, 100),
                                    (b * float("inf"), zero, 30, 1e-8, 100), (b, zero, 1, 1e-12, 4000),
                                    (b, zero, 64, 1e-10, 500), (b, zero, 65, 1e-10, 500)):
        o, l = both(dA, rhs, x0, h, m, rtol, maxit, g.PREC_GS2)
        if not torch.isfinite(rhs).all():
            assert o[0]["status"] == l[0]["status"] == -4
        else:
            assert same(o, l), (m, o[0], l[0])
