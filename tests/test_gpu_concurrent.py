"""One-launch applies and solves on several streams at once, a thread and a handle
each: more workgroups that wait for each other than the card holds, and the bits of
the same calls made alone."""
import threading

import numpy as np
import pytest

torch = pytest.importorskip("torch")

import paper_2104_01196_amd as g  # noqa: E402
from gen import convdiff2d, poisson2d  # noqa: E402

pytestmark = pytest.mark.gpu
DEV = "cuda"


def test_streams_and_threads():
    jobs = []
    for k in range(6):
        # up to 64 workgroups of 1024 threads, or 1024 wavefronts, each
        A = poisson2d(240 + k) if k % 2 else convdiff2d(256 - k, 20.0, 0.3 * k)
        dA = g.DeviceCSR.from_host(A)
        h = g.gs2_setup(dA, 1, 2, 0.9, g.SYMMETRIC)
        v = torch.as_tensor(np.random.default_rng(k).standard_normal(A.n), device=DEV)
        jobs.append((dA, h, v))

    def work(job, stream):
        dA, h, v = job
        z, x = torch.empty_like(v), torch.zeros_like(v)
        with torch.cuda.stream(stream):
            z.zero_()
            x.zero_()
            g.gs2_apply(h, v, z, stream=stream)
            info = g.gmres_solve(dA, v, x, 20, 1e-12, 45, g.PREC_GS2, h, stream=stream)
        stream.synchronize()
        return z, x, info["iterations"]

    torch.cuda.synchronize()
    want = [work(j, torch.cuda.Stream()) for j in jobs]
    wrong = []

    def run(k):
        s = torch.cuda.Stream()
        for rep in range(8):
            z, x, its = work(jobs[k], s)
            if not (torch.equal(z, want[k][0]) and torch.equal(x, want[k][1]) and its == want[k][2]):
                wrong.append((k, rep))

    threads = [threading.Thread(target=run, args=(k,)) for k in range(len(jobs))]
    for t in threads:
        t.start()
    for t in threads:
        t.join()
    torch.cuda.synchronize()
    print("solves given up:", [g.gs2_paths(h)["given_up"] for _, h, _ in jobs])
    assert not wrong
