"""The two-launch CG iteration of small systems: caps on the iterations at
every place within a check's eight, a stop at the first check that holds, the
same recurrences in numpy, several streams at once, and a breakdown (NaN).

The numpy iteration rounds differently; over the at most 40 steps compared the
difference stays far below 1e-9 of the solution (unit roundoff times the
steps, times the growth of a recurrence that is not yet converged)."""
import threading

import numpy as np
import pytest

torch = pytest.importorskip("torch")

from oracle import oracle as O
from paper_2505_02438_amd import api
from paper_2505_02438_amd import inputs as I

from gpu_util import dev, host

pytestmark = pytest.mark.gpu
MAT = api.Material()


def _system(elem, dims, seed=81):
    pr = I.small_problem(elem, seed=seed, dims=dims)
    m = pr.mesh
    pat = api.Pattern.from_mesh(m)
    K = pat.assemble(MAT, dev(pr.rho), dev(pr.mask))
    rp, ci = O.pattern(m.elem, m.n_nodes, m.cells)
    f = np.random.default_rng(seed + 1).standard_normal(m.ndof)
    f[pr.mask != 0] = 0.0
    return m, pat, K, rp, ci, f


def _numpy_cg(m, rp, ci, K, f, steps):
    """u and ||r|| / ||f|| after 0 .. steps iterations."""
    d = m.dim
    mul = lambda x: O.spmv(rp, ci, K, x)
    diag = np.zeros((m.n_nodes, d, d))
    rows = np.repeat(np.arange(m.ndof), np.diff(rp))
    own = rows // d == ci // d
    diag[rows[own] // d, rows[own] % d, ci[own] % d] = K[own]
    inv = np.linalg.inv(diag)
    prec = lambda r: np.einsum("nij,nj->ni", inv, r.reshape(-1, d)).ravel()
    u = np.zeros(m.ndof)
    r = f.copy()
    z = prec(r)
    p = z.copy()
    rz = r @ z
    out = [(u.copy(), 1.0)]
    for _ in range(steps):
        q = mul(p)
        al = rz / (p @ q)
        u = u + al * p
        r = r - al * q
        z = prec(r)
        rz, old = r @ z, rz
        p = z + (rz / old) * p
        out.append((u.copy(), np.linalg.norm(r) / np.linalg.norm(f)))
    return out


# one node group up to several blocks of nodes in both launches; rows of 7 to 65 neighbours
SYSTEMS = [(I.QUAD4, (1, 1)), (I.QUAD4, (33, 31)), (I.TRI3, (20, 17)), (I.HEX8, (1, 1, 1)), (I.HEX8, (9, 8, 7)),
           (I.TET10, (3, 3, 3))]


@pytest.mark.parametrize("elem,dims", SYSTEMS)
def test_iteration_caps_match_numpy(elem, dims):
    m, pat, K, rp, ci, f = _system(elem, dims)
    free = int(np.count_nonzero(f))
    cap = min(40, max(1, free // 2))
    ref = _numpy_cg(m, rp, ci, host(K), f, cap)
    for n in sorted({k for k in (0, 1, 2, 7, 8, 9, 11, 12, 13, 16, 17, 20, 21, 40) if k <= cap}):
        u, it, rel = pat.pcg(K, dev(f), rtol=0.0, max_iter=n)
        assert it == n
        err = np.linalg.norm(host(u) - ref[n][0]) / max(np.linalg.norm(ref[n][0]), 1e-300)
        assert err <= 1e-9 and abs(rel - ref[n][1]) <= 1e-9 * max(ref[n][1], 1.0), (n, err, rel, ref[n][1])


@pytest.mark.parametrize("elem,dims", [(I.QUAD4, (33, 31)), (I.HEX8, (9, 8, 7))])
def test_stops_at_the_first_check_that_holds(elem, dims):
    m, pat, K, rp, ci, f = _system(elem, dims)
    rels = {n: pat.pcg(K, dev(f), rtol=0.0, max_iter=n)[2] for n in range(8, 73, 8)}
    for n in range(8, 73, 8):
        if all(rels[n] < rels[k] for k in rels if k < n):
            u, it, rel = pat.pcg(K, dev(f), rtol=rels[n], max_iter=5000)
            v, it2, rel2 = pat.pcg(K, dev(f), rtol=0.0, max_iter=n)
            assert it == n and rel == rels[n] and np.array_equal(host(u), host(v))
            # the next tighter tolerance needs more
            assert pat.pcg(K, dev(f), rtol=rels[n] * (1 - 1e-12), max_iter=5000)[1] > n


def test_solves_on_several_threads_and_streams():
    m, pat, K, rp, ci, f = _system(I.HEX8, (9, 8, 7))
    fs = [dev(f * (k + 1)) for k in range(4)]
    want = [pat.pcg(K, x, rtol=1e-9) for x in fs]
    torch.cuda.synchronize()
    got, errors = [None] * 4, []

    def work(k):
        try:
            st = torch.cuda.Stream()
            for _ in range(3):
                got[k] = pat.pcg(K, fs[k], rtol=1e-9, stream=st)
        except Exception as e:  # pragma: no cover
            errors.append(e)
    th = [threading.Thread(target=work, args=(k,)) for k in range(4)]
    [t.start() for t in th]
    [t.join() for t in th]
    assert not errors
    for a, b in zip(got, want):
        assert a[1:] == b[1:] and np.array_equal(host(a[0]), host(b[0]))


def test_breakdown_stops():
    """K = 0 gives z = 0 and alpha = 0 / 0: the first check stops.  A NaN in K is
    in the first residual already (it = 0) or in the first check's."""
    m, pat, K, rp, ci, f = _system(I.QUAD4, (7, 5))
    u, it, rel = pat.pcg(torch.zeros_like(K), dev(f), rtol=1e-8, max_iter=100)
    assert it == 8 and np.isnan(rel)
    bad = K.clone()
    bad[5] = float("nan")
    u, it, rel = pat.pcg(bad, dev(f), rtol=1e-8, max_iter=100)
    assert it in (0, 8) and np.isnan(rel)
