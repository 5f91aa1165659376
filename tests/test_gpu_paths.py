"""Which calls run in one launch: the systems and forms that the one-launch tests
compare with the launches do run in one where the rules say so, up to and with
65536 rows (from 65537 on the layout of the solver's copy is timed), and no others."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")

import paper_2104_01196_amd as g  # noqa: E402
import test_gpu_resident as solves  # noqa: E402
import test_gpu_small_apply as applies  # noqa: E402

pytestmark = pytest.mark.gpu
DEV = "cuda"


def exchanged(jr, sweeps, inner, variant):
    halves = sweeps * (2 if not jr and variant == g.SYMMETRIC else 1)
    return (halves if jr or inner == 0 else halves * inner + halves - 1) - 1


def lanes(h):
    s = g.gs2_handle_schedule(h)
    return 1 if s["format"] != g.FORMAT_SELL else s["lanes_per_row"]


@pytest.mark.parametrize("form", solves.FORMS)
@pytest.mark.parametrize("name", solves.MATS)
def test_solves(name, form):
    A = solves.MATS[name]()
    dA = g.DeviceCSR.from_host(A)
    kind, kw = solves.FORMS[form]
    h = g.gs2_setup(dA, **{"variant": g.FORWARD, **kw})
    b = torch.as_tensor(np.random.default_rng(7).standard_normal(A.n), device=DEV)
    g.gmres_solve(dA, b, torch.zeros_like(b), 20, 1e-8, 5, kind, h)
    s = g.gs2_gmres_schedule(h)
    assert s["format"] == g.FORMAT_SELL and s["tuned"] == 0
    one = s["lanes_per_row"] == 1 and lanes(h) <= (4 if A.n <= 32768 else 2)
    if name != "random_3000":
        assert s["lanes_per_row"] == 1
    assert g.gs2_paths(h)["last_solve"] == (2 if one else 1), (s, lanes(h))


@pytest.mark.parametrize("form", applies.FORMS)
@pytest.mark.parametrize("name", applies.MATS)
def test_applies(name, form):
    A = applies.MATS[name]()
    kw = applies.FORMS[form]
    h = g.gs2_setup(g.DeviceCSR.from_host(A), **kw)
    v = torch.as_tensor(np.random.default_rng(7).standard_normal(A.n), device=DEV)
    z = torch.empty_like(v)
    ne = exchanged(False, kw.get("sweeps", 1), kw.get("inner", 1), kw["variant"])
    one = A.n <= 65536 and np.diff(A.rowptr).max() <= 17 and ne <= 8 and lanes(h) <= 4
    g.gs2_apply(h, v, z)
    assert g.gs2_paths(h)["applies"] == (1 if one else 0)
    g.jr_apply(h, 2, 0.8, v, z)
    # a Jacobi sweep exchanges one vector, for which the handle's own applies left room or not
    assert g.gs2_paths(h)["applies"] == (2 if one and ne >= 1 else 1 if one else 0)


def test_one_row_more_is_launched():
    from gen import laplace1d

    for n, one in ((65536, True), (65537, False)):
        A = laplace1d(n)
        dA = g.DeviceCSR.from_host(A)
        h = g.gs2_setup(dA, variant=g.FORWARD, lanes_per_row=1, format=g.FORMAT_SELL)
        b = torch.as_tensor(np.random.default_rng(7).standard_normal(n), device=DEV)
        g.gmres_solve(dA, b, torch.zeros_like(b), 20, 1e-8, 5, g.PREC_GS2, h)
        assert g.gs2_paths(h)["last_solve"] == (2 if one else 1)
        assert g.gs2_gmres_schedule(h)["tuned"] == (0 if one else 1)
        before = g.gs2_paths(h)["applies"]
        g.gs2_apply(h, b, torch.empty_like(b))
        assert g.gs2_paths(h)["applies"] - before == (1 if one else 0)
