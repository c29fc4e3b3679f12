"""The assembly backward's scratch belongs to the call: host threads on one
stream, and replays of graphs captured on one stream beside each other and
beside eager calls, give the bits of the same calls one after the other; a
capture on a stream without an earlier call runs the same kernels as an eager
call.  The C entry point refuses scratch that is missing, misaligned or small,
and without memory for it the form without scratch runs (against the oracle to
1e-12 of the sum over absolute values, as every FP64 form)."""
import ctypes
import threading

import numpy as np
import pytest

torch = pytest.importorskip("torch")

from oracle import oracle as O
from paper_2505_02438_amd import _lib, api
from paper_2505_02438_amd import inputs as I

from gpu_util import dev, host

pytestmark = pytest.mark.gpu
MAT = api.Material()


def _setup(n_bar, dims=(24, 16, 12)):
    pr = I.small_problem(I.HEX8, seed=31, dims=dims)
    pat = api.Pattern.from_mesh(pr.mesh)
    rng = np.random.default_rng(32)
    rho, mask = dev(pr.rho), dev(pr.mask)
    bars = [dev(rng.standard_normal(pat.nnz)) for _ in range(n_bar)]
    want = [pat.backward(MAT, rho, b, mask) for b in bars]
    torch.cuda.synchronize()
    return pr, pat, rho, mask, bars, want


def test_threads_on_one_stream():
    _, pat, rho, mask, bars, want = _setup(4)
    st = torch.cuda.Stream()
    start = threading.Barrier(len(bars))
    bad = []

    def work(k):
        start.wait()
        for _ in range(40):
            if not torch.equal(pat.backward(MAT, rho, bars[k], mask, stream=st).cpu(), ref[k]):
                bad.append(k)
    ref = [w.cpu() for w in want]

    def run(k):
        with torch.cuda.stream(st):
            work(k)
    th = [threading.Thread(target=run, args=(k,)) for k in range(len(bars))]
    [t.start() for t in th]
    [t.join() for t in th]
    assert not bad


def test_graphs_of_one_stream_beside_eager_calls():
    _, pat, rho, mask, bars, want = _setup(4)
    cap = torch.cuda.Stream()
    with torch.cuda.stream(cap):
        pat.backward(MAT, rho, bars[3], mask, stream=cap)
    graphs, outs = [], []
    for k in range(3):
        out = torch.empty_like(want[0])
        torch.cuda.synchronize()
        g = torch.cuda.CUDAGraph()
        with torch.cuda.graph(g, stream=cap):
            pat.backward(MAT, rho, bars[k], mask, out=out, stream=cap)
        graphs.append(g)
        outs.append(out)
    on = [torch.cuda.Stream() for _ in graphs]
    for _ in range(10):
        for o in outs:
            o.fill_(float("nan"))
        torch.cuda.synchronize()
        for s, g in zip(on, graphs):
            with torch.cuda.stream(s):
                g.replay()
        with torch.cuda.stream(cap):
            eager = pat.backward(MAT, rho, bars[3], mask, stream=cap)
        torch.cuda.synchronize()
        assert all(torch.equal(o, w) for o, w in zip(outs, want[:3])) and torch.equal(eager, want[3])


@pytest.mark.parametrize("elem,dims", [(I.HEX8, (6, 5, 7)), (I.TET10, (3, 4, 5)), (I.TRI3, (97, 107)),
                                       (I.QUAD4, (201, 100)), (I.QUAD4, (35, 33))])
def test_captured_first_is_the_eager_form(elem, dims):
    pr = I.small_problem(elem, seed=33, dims=dims)
    pat = api.Pattern.from_mesh(pr.mesh)
    rng = np.random.default_rng(34)
    rho, mask, Kbar = dev(pr.rho), dev(pr.mask), dev(rng.standard_normal(pat.nnz))
    out = torch.empty(pr.mesh.n_cells, dtype=torch.float64, device="cuda")
    st = torch.cuda.Stream()
    torch.cuda.synchronize()
    g = torch.cuda.CUDAGraph()
    with torch.cuda.graph(g, stream=st):
        pat.backward(MAT, rho, Kbar, mask, out=out, stream=st)
    for _ in range(3):
        Kbar.copy_(dev(rng.standard_normal(pat.nnz)))
        want = pat.backward(MAT, rho, Kbar, mask)
        out.fill_(float("nan"))
        torch.cuda.synchronize()
        g.replay()
        torch.cuda.synchronize()
        assert torch.equal(out, want)


def test_scratch_arguments():
    pr, pat, rho, mask, bars, want = _setup(1, (6, 5, 7))
    L = _lib.lib()
    mc = MAT._c()
    size = ctypes.c_int64()
    assert L.soptx_backward_scratch_size(pat._h, ctypes.byref(size)) == 0 and size.value > 0
    out = torch.full((pr.mesh.n_cells,), -7.0, dtype=torch.float64, device="cuda")
    buf = torch.empty(size.value + 8, dtype=torch.uint8, device="cuda")

    def call(p, n):
        return L.soptx_assemble_backward_scratch(pat._h, ctypes.byref(mc), rho.data_ptr(), mask.data_ptr(),
                                                 bars[0].data_ptr(), out.data_ptr(), api.FP64, p, n,
                                                 torch.cuda.current_stream().cuda_stream)
    for p, n in ((None, size.value), (buf.data_ptr() + 4, size.value), (buf.data_ptr(), size.value - 1)):
        assert call(p, n) == -1
    torch.cuda.synchronize()
    assert bool((out == -7.0).all())
    assert call(buf.data_ptr(), size.value) == 0
    assert torch.equal(out, want[0])
    # small 2D meshes take no scratch
    quad = api.Pattern.from_mesh(I.quad_grid(35, 33))
    assert L.soptx_backward_scratch_size(quad._h, ctypes.byref(size)) == 0 and size.value == 0


def test_without_memory_for_the_scratch(monkeypatch):
    pr, pat, rho, mask, bars, _ = _setup(1, (6, 5, 7))
    def full(*a, **kw):
        raise torch.cuda.OutOfMemoryError("full")
    monkeypatch.setattr(torch.Tensor, "new_empty", full)
    got = host(pat.backward(MAT, rho, bars[0], mask))
    monkeypatch.undo()
    plain = torch.empty_like(rho)
    mc = MAT._c()
    assert _lib.lib().soptx_assemble_backward(pat._h, ctypes.byref(mc), rho.data_ptr(), mask.data_ptr(),
                                              bars[0].data_ptr(), plain.data_ptr(), api.FP64,
                                              torch.cuda.current_stream().cuda_stream) == 0
    assert np.array_equal(got, host(plain))
    m = pr.mesh
    rp, ci = pat.pattern()
    Kb = host(bars[0]).copy()
    rows = np.repeat(np.arange(m.ndof), np.diff(rp))
    Kb[(pr.mask[rows] != 0) | (pr.mask[ci] != 0)] = 0.0
    ref = O.assemble_backward(m.elem, m.coords, m.cells, pr.rho, rp, ci, Kb)
    scale = O.assemble_backward(m.elem, m.coords, m.cells, pr.rho, rp, ci, np.abs(Kb))
    assert np.max(np.abs(got - ref) / np.maximum(np.abs(scale), np.abs(ref).max())) <= 1e-12
