"""Triangles of a hybrid handle hold 16-bit column offsets where the entries
inside the row blocks allow them, whatever the couplings between the blocks
span: the stored bytes are those of the same matrix without these couplings."""
from types import SimpleNamespace

import numpy as np
import pytest

torch = pytest.importorskip("torch")

import oracle  # noqa: E402
import paper_2104_01196_amd as g  # noqa: E402

pytestmark = pytest.mark.gpu
DEV = "cuda"
BLOCKS = 2


def matrix(bs, near, far):
    """BLOCKS blocks of bs rows: couplings of +-near inside, of +-far between them."""
    n = BLOCKS * bs
    i = np.arange(n)
    r, c = [i], [i]
    for d in (1, near):
        j = i[:-d]
        keep = j // bs == (j + d) // bs
        r += [j[keep], j[keep] + d]
        c += [j[keep] + d, j[keep]]
    if far:
        j = i[: n - far]
        r += [j, j + far]
        c += [j + far, j]
    r, c = np.concatenate(r), np.concatenate(c)
    o = np.lexsort((c, r))
    r, c = r[o], c[o]
    rng = np.random.default_rng(3)
    v = np.where(r == c, 8.0, rng.uniform(-1.0, 1.0, r.size))
    rp = np.concatenate([[0], np.cumsum(np.bincount(r, minlength=n))])
    return SimpleNamespace(n=n, rowptr=rp.astype(np.int32), colind=c.astype(np.int32), val=v)


def stored(A):
    h = g.gs2_setup(g.DeviceCSR.from_host(A), 1, 1, 0.9, g.FORWARD, blocks=BLOCKS, autotune=False)
    return h, g.gs2_handle_query(h)["bytes_stored"]


# 180002 rows leave 30 past the last one in a slice of 64, whose padding lies up to 30 below the diagonal: 65505 is the
# widest coupling that fits beside it
@pytest.mark.parametrize("bs,near", [(40_000, 300), (90_001, 300), (90_001, 65_505), (90_001, 65_506)])
def test_stored_bytes_and_values(bs, near):
    (_, want), (h, got) = stored(matrix(bs, near, 0)), stored(matrix(bs, near, bs))
    assert got == want
    A = matrix(bs, near, bs)
    v = np.random.default_rng(1).standard_normal(A.n)
    z = torch.empty(A.n, dtype=torch.float64, device=DEV)
    g.gs2_apply(h, torch.as_tensor(v, device=DEV), z)
    want = oracle.gs2_block_sweep(A, v, np.zeros(A.n), BLOCKS, g.FORWARD, 1, 1, 1, 0.9)
    assert np.abs(z.cpu().numpy() - want).max() <= 1e-12 * np.abs(want).max()


def test_widest():
    """The offsets are held beside the columns: at the limit there are more bytes than past it."""
    assert stored(matrix(90_001, 65_505, 90_001))[1] > stored(matrix(90_001, 65_506, 90_001))[1]
