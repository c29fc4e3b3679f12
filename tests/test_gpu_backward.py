"""The assembly backward on the plan's node groups against the oracle's reverse
assembly: every element type, plans in the given and in canonical order,
groups of a few nodes up to full ones, both precision forms, with and without
Dirichlet rows; and under graph capture, where a first call on a stream has no
workspace yet and runs the element-by-element kernel instead.

Bounds: |drho - ref| is compared with the same sum over absolute values, where
a form's error is its unit roundoff times the terms of an element's sum (at
most 100 blocks of 9): 1e-12 in FP64, 1e-5 in FP32.
"""
import numpy as np
import pytest

torch = pytest.importorskip("torch")

from oracle import oracle as O
from paper_2505_02438_amd import api
from paper_2505_02438_amd import inputs as I

from gpu_util import dev, host

pytestmark = pytest.mark.gpu
MAT = api.Material()

# (element, mesh sizes): one cell; a few groups with remainders; nodes of full
# groups on every side; 2D meshes on either side of 20,000 cells, up to which
# the element-by-element kernel runs
SIZES = [(I.QUAD4, (1, 1)), (I.QUAD4, (35, 33)), (I.QUAD4, (201, 100)), (I.TRI3, (1, 1)), (I.TRI3, (100, 100)),
         (I.TRI3, (97, 107)), (I.HEX8, (1, 1, 1)),
         (I.HEX8, (2, 2, 35)), (I.HEX8, (7, 5, 9)), (I.TET10, (1, 1, 1)), (I.TET10, (3, 4, 5))]


def _reference(pr, pat, Kbar, mask):
    m = pr.mesh
    rp, ci = pat.pattern()
    Kb = Kbar.copy()
    if mask is not None:
        rows = np.repeat(np.arange(m.ndof), np.diff(rp))
        Kb[(mask[rows] != 0) | (mask[ci] != 0)] = 0.0
    rho = pr.rho.astype(np.float64)
    ref = O.assemble_backward(m.elem, m.coords, m.cells, rho, rp, ci, Kb)
    scale = O.assemble_backward(m.elem, m.coords, m.cells, rho, rp, ci, np.abs(Kb))
    return ref, np.maximum(np.abs(scale), np.abs(ref).max())


@pytest.mark.parametrize("prec,tol", [(api.FP64, 1e-12), (api.FP32, 1e-5)])
@pytest.mark.parametrize("order", ["given", "renumbered", "sheared"])
@pytest.mark.parametrize("elem,dims", SIZES)
def test_backward_matches_oracle(elem, dims, order, prec, tol):
    if order == "sheared" and elem not in (I.QUAD4, I.HEX8):
        pytest.skip("shears are for Q1 meshes")
    pr = I.small_problem(elem, seed=61, dims=dims, skew="kink" if order == "sheared" else None)
    if order == "renumbered":
        pr = I.renumber(pr, 62)
    if prec == api.FP32:
        pr.rho = pr.rho.astype(np.float32)
    pat = api.Pattern.from_mesh(pr.mesh)
    rng = np.random.default_rng(63)
    Kbar = rng.standard_normal(pat.nnz)
    for mask in (None, pr.mask, np.zeros_like(pr.mask)):
        got = host(pat.backward(MAT, dev(pr.rho), dev(Kbar), None if mask is None else dev(mask), prec=prec))
        again = host(pat.backward(MAT, dev(pr.rho), dev(Kbar), None if mask is None else dev(mask), prec=prec))
        ref, scale = _reference(pr, pat, Kbar, mask)
        err = np.max(np.abs(got.astype(np.float64) - ref) / scale)
        assert err <= tol, (elem, dims, order, prec, err)
        assert np.array_equal(got, again)


def test_backward_captured_without_and_with_workspace():
    """On a new stream the first backward is captured (no workspace can be
    allocated then), a second one after an eager call; both replays give the
    oracle's values for the inputs in place at the replay."""
    pr = I.small_problem(I.HEX8, seed=64, dims=(6, 5, 7))
    pat = api.Pattern.from_mesh(pr.mesh)
    rng = np.random.default_rng(65)
    kb = [rng.standard_normal(pat.nnz) for _ in range(2)]
    Kbar, rho = dev(kb[0]), dev(pr.rho)
    st = torch.cuda.Stream()
    outs, graphs = [], []
    for _ in range(2):
        out = torch.zeros(pr.mesh.n_cells, dtype=torch.float64, device="cuda")
        torch.cuda.synchronize()
        g = torch.cuda.CUDAGraph()
        with torch.cuda.graph(g, stream=st):
            pat.backward(MAT, rho, Kbar, out=out, stream=st)
        outs.append(out)
        graphs.append(g)
        with torch.cuda.stream(st):
            pat.backward(MAT, rho, Kbar, stream=st)
        torch.cuda.synchronize()
    for k in (0, 1, 0):
        Kbar.copy_(dev(kb[k]))
        torch.cuda.synchronize()
        ref, scale = _reference(pr, pat, kb[k], None)
        for g, out in zip(graphs, outs):
            out.zero_()
            torch.cuda.synchronize()
            g.replay()
            torch.cuda.synchronize()
            assert np.max(np.abs(host(out) - ref) / scale) <= 1e-12
