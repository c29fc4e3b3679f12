"""The CG's two-launch form on systems of many blocks: a stop at a check while
the launches enqueued ahead of its result still run, beside other solves, and
the iterate it leaves (that of the same number of iterations, bit for bit)."""
import ctypes
import threading

import numpy as np
import pytest

torch = pytest.importorskip("torch")

from paper_2505_02438_amd import _lib, api
from paper_2505_02438_amd import inputs as I

from gpu_util import dev, host

pytestmark = pytest.mark.gpu
MAT = api.Material()


def _system(elem, dims, seed=51):
    pr = I.small_problem(elem, seed=seed, dims=dims)
    pat = api.Pattern.from_mesh(pr.mesh)
    K = pat.assemble(MAT, dev(pr.rho), dev(pr.mask))
    f = np.random.default_rng(seed + 1).standard_normal(pr.mesh.ndof)
    f[pr.mask != 0] = 0.0
    return pat, K, dev(f)


def test_stops_beside_other_solves():
    pat, K, f = _system(I.HEX8, (30, 20, 20))
    # a different stop per stream, each at the first check that reaches its residual
    rels = {n: pat.pcg(K, f, rtol=0.0, max_iter=n)[2] for n in range(8, 200, 8)}
    stops = [n for n in rels if all(rels[n] < rels[k] for k in rels if k < n)][:4]
    want = {n: pat.pcg(K, f, rtol=0.0, max_iter=n) for n in stops}
    torch.cuda.synchronize()
    bad = []

    def work(n):
        st = torch.cuda.Stream()
        for _ in range(10):
            u, it, rel = pat.pcg(K, f, rtol=rels[n], max_iter=1000, stream=st)
            if it != n or rel != want[n][2] or not torch.equal(u.cpu(), ref[n]):
                bad.append((n, it, rel))
    ref = {n: want[n][0].cpu() for n in stops}
    th = [threading.Thread(target=work, args=(n,)) for n in stops]
    [t.start() for t in th]
    [t.join() for t in th]
    assert len(stops) >= 1 and not bad
