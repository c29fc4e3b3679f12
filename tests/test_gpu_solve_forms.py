"""The CG's two-launch form on systems of many blocks: a stop at a check while
the launches enqueued ahead of its result still run, beside other solves, and
the iterate it leaves (that of the same number of iterations, bit for bit); and
the same bits from the five launches of larger systems."""
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


def _separate(fn):
    L = _lib.lib()
    assert L.soptx_debug_set_pcg_variant(0) == 0
    try:
        return fn()
    finally:
        L.soptx_debug_set_pcg_variant(-1)


# one block; a few; more than 1,024 and more than 4,096 blocks of partials of
# the product (16 nodes each in 3D, 32 in 2D), where a thread's share of the sum
# takes several rounds
@pytest.mark.parametrize("elem,dims", [(I.QUAD4, (3, 2)), (I.QUAD4, (150, 50)), (I.QUAD4, (300, 260)),
                                       (I.TRI3, (77, 31)), (I.HEX8, (2, 1, 1)), (I.HEX8, (14, 13, 11)),
                                       (I.HEX8, (40, 30, 20)), (I.HEX8, (66, 40, 26)), (I.TET10, (5, 4, 3))])
def test_two_launches_are_the_five(elem, dims):
    """u, the iterations and the residual bit for bit, at a cap within and at
    the end of a check's eight and at a stop."""
    pat, K, f = _system(elem, dims)
    for rtol, cap in ((0.0, 1), (0.0, 13), (0.0, 24), (1e-3, 400)):
        u, it, rel = pat.pcg(K, f, rtol=rtol, max_iter=cap)
        v, it5, rel5 = _separate(lambda: pat.pcg(K, f, rtol=rtol, max_iter=cap))
        assert it == it5 and torch.equal(u, v)
        assert rel == rel5 or (np.isnan(rel) and np.isnan(rel5))


@pytest.mark.parametrize("skip", [0, 1])
def test_without_memory_for_the_two_launches(skip):
    """No second direction vector, or no stop record: the five launches run."""
    pat, K, f = _system(I.HEX8, (9, 8, 7))
    want = pat.pcg(K, f, rtol=1e-6)
    L = _lib.lib()
    assert L.soptx_debug_fail_optional(skip, 1) == 0
    try:
        got = pat.pcg(K, f, rtol=1e-6)
    finally:
        L.soptx_debug_fail_optional(0, 0)
    assert got[1:] == want[1:] and torch.equal(got[0], want[0])
    assert pat.pcg(K, f, rtol=1e-6)[1:] == want[1:]
