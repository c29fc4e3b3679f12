"""Which 2D meshes run the assembly backward on node groups (those with a
scratch size): by element and numbering, on either side of the sizes where both
forms take the same time.  Both forms of every mesh against the oracle, to
1e-12 of the sum over absolute values (at most 16 blocks of 4 per element)."""
import ctypes

import numpy as np
import pytest

torch = pytest.importorskip("torch")

from oracle import oracle as O
from paper_2505_02438_amd import _lib, api
from paper_2505_02438_amd import inputs as I

from gpu_util import dev, host

pytestmark = pytest.mark.gpu
MAT = api.Material()


@pytest.mark.parametrize("elem,dims,renumbered,grouped", [
    (I.QUAD4, (100, 50), False, False), (I.QUAD4, (61, 82), False, True),
    (I.QUAD4, (20, 20), True, False), (I.QUAD4, (21, 20), True, True),
    (I.TRI3, (250, 200), False, False), (I.TRI3, (230, 218), False, True),
    (I.TRI3, (70, 50), True, False), (I.TRI3, (67, 53), True, True)])
def test_form_by_element_and_numbering(elem, dims, renumbered, grouped):
    pr = I.small_problem(elem, seed=41, dims=dims)
    if renumbered:
        pr = I.renumber(pr, 42)
    m = pr.mesh
    pat = api.Pattern.from_mesh(m)
    L = _lib.lib()
    size = ctypes.c_int64()
    assert L.soptx_backward_scratch_size(pat._h, ctypes.byref(size)) == 0
    assert (size.value > 0) == grouped
    Kbar = np.random.default_rng(43).standard_normal(pat.nnz)
    rho, K = dev(pr.rho), dev(Kbar)
    got = host(pat.backward(MAT, rho, K))
    plain = torch.empty(m.n_cells, dtype=torch.float64, device="cuda")
    mc = MAT._c()
    assert L.soptx_assemble_backward(pat._h, ctypes.byref(mc), rho.data_ptr(), None, K.data_ptr(), plain.data_ptr(),
                                     api.FP64, torch.cuda.current_stream().cuda_stream) == 0
    rp, ci = pat.pattern()
    ref = O.assemble_backward(elem, m.coords, m.cells, pr.rho, rp, ci, Kbar)
    scale = O.assemble_backward(elem, m.coords, m.cells, pr.rho, rp, ci, np.abs(Kbar))
    scale = np.maximum(np.abs(scale), np.abs(ref).max())
    for x in (got, host(plain)):
        assert np.max(np.abs(x - ref) / scale) <= 1e-12
    if not grouped:
        assert np.array_equal(got, host(plain))
