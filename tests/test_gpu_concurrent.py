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
        # everything on the job's own stream: a fill left to the default stream, which
        # nothing orders with it, could land in the middle of the solve
        dA, h, v = job
        with torch.cuda.stream(stream):
            z, x = torch.full_like(v, float("nan")), torch.zeros_like(v)
            g.gs2_apply(h, v, z, stream=stream)
            info = g.gmres_solve(dA, v, x, 20, 1e-12, 45, g.PREC_GS2, h, stream=stream)
            return z.cpu().numpy(), x.cpu().numpy(), info["iterations"]

    torch.cuda.synchronize()
    want = [work(j, torch.cuda.Stream()) for j in jobs]
    wrong = []

    def run(k):
        s = torch.cuda.Stream()
        for rep in range(8):
            z, x, its = work(jobs[k], s)
            dz, dx = (z != want[k][0]).sum(), (x != want[k][1]).sum()
            if dz or dx or its != want[k][2]:
                wrong.append((k, rep, int(dz), int(dx), its, float(np.nanmax(np.abs(x)))))

    threads = [threading.Thread(target=run, args=(k,)) for k in range(len(jobs))]
    for t in threads:
        t.start()
    for t in threads:
        t.join()
    torch.cuda.synchronize()
    print("solves given up:", [g.gs2_paths(h)["given_up"] for _, h, _ in jobs])
    assert not wrong
