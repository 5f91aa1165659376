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


# blocks whose own span fits 16 bits and ones whose own span does not; near = 65535 - 63: the widest that fits
# beside the padding of rows past the last one
@pytest.mark.parametrize("bs,near", [(40_000, 300), (90_001, 300), (90_001, 65_472), (90_001, 65_600)])
def test_stored_bytes_and_values(bs, near):
    byts = []
    for far in (0, bs):
        A = matrix(bs, near, far)
        h = g.gs2_setup(g.DeviceCSR.from_host(A), 1, 1, 0.9, g.FORWARD, blocks=BLOCKS, autotune=False)
        byts.append(g.gs2_handle_query(h)["bytes_stored"])
    assert byts[0] == byts[1]
    v = np.random.default_rng(1).standard_normal(A.n)
    z = torch.empty(A.n, dtype=torch.float64, device=DEV)
    g.gs2_apply(h, torch.as_tensor(v, device=DEV), z)
    want = oracle.gs2_block_sweep(A, v, np.zeros(A.n), BLOCKS, g.FORWARD, 1, 1, 1, 0.9)
    assert np.abs(z.cpu().numpy() - want).max() <= 1e-12 * np.abs(want).max()
