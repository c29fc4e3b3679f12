"""Q2 hexahedra assembled by row groups (k_assemble_hex27) against the oracle
and against the element-matrix form: boxes of every small size (groups of few
nodes, missing neighbours, rows at the far faces), curved cells, renumbered
meshes, three or four cells around an edge of an unstructured mesh; and a mesh
whose nodes have more elements than a group takes, which stays with the element
matrices.  Bound: 1e-12 row-scaled, the FP64 gate of the assembly; the sums of
at most 8 x 27 terms differ by a few units of roundoff."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")

from oracle import oracle as O
from paper_2505_02438_amd import _lib, api
from paper_2505_02438_amd import inputs as I

from gpu_util import dev, host, row_scaled_err

pytestmark = pytest.mark.gpu
MAT = api.Material()


def _form(pat):
    import ctypes
    f = ctypes.c_int32()
    assert _lib.lib().soptx_debug_general_path(pat._h, ctypes.byref(f)) == 0
    return f.value


def _fan(k, layers, twist=0.2):
    """k quadrilaterals around a vertical axis, `layers` high, as Q2 hexahedra."""
    hexes = []
    for z in range(layers):
        for s in range(k):
            a0, a1 = 2 * np.pi * s / k + twist, 2 * np.pi * (s + 1) / k + twist
            p0, p1 = np.array([np.cos(a0), np.sin(a0)]), np.array([np.cos(a1), np.sin(a1)])
            quad = [np.zeros(2), p0, 0.8 * (p0 + p1), p1]
            hexes.append([np.append(q, z) for q in quad] + [np.append(q, z + 1.0) for q in quad])
    key, coords, cells = {}, [], []
    for h in hexes:
        h = np.array(h)
        cell = []
        for lat in I._HEX27_LATTICE:
            t = np.array(lat) / 2.0
            w = [((t[0] if c in (1, 2, 5, 6) else 1 - t[0]) * (t[1] if c in (2, 3, 6, 7) else 1 - t[1])
                  * (t[2] if c >= 4 else 1 - t[2])) for c in range(8)]
            x = np.array(w) @ h
            r = tuple(np.round(x, 7))
            if r not in key:
                key[r] = len(coords)
                coords.append(x)
            cell.append(key[r])
        cells.append(cell)
    return I.Mesh(I.HEX27, np.array(coords), np.array(cells, dtype=np.int32))


def _mesh(name):
    rng = np.random.default_rng(91)
    if name.startswith("fan"):
        return _fan(int(name[3:]), 3)
    dims = tuple(int(x) for x in name.split("_")[0].split("x"))
    m = I.hex27_grid(*dims, 2.0)
    if "curved" in name:
        m = I.jitter_interior(m, 0.15, rng)
    if "renumbered" in name:
        pr = I.Problem("m", m, np.ones(m.n_cells), np.zeros(m.ndof, np.uint8), np.zeros(m.ndof), None)
        m = I.renumber(pr, 92).mesh
    return m


@pytest.mark.parametrize("name", ["1x1x1", "2x1x1", "1x2x3_curved", "3x3x3_curved", "4x3x5_curved_renumbered",
                                  "9x2x2_curved", "fan3", "fan4", "fan5"])
def test_row_groups_match_oracle_and_element_matrices(name):
    m = _mesh(name)
    rng = np.random.default_rng(93)
    rho = rng.uniform(1e-3, 1.0, m.n_cells)
    mask = (rng.uniform(size=m.ndof) < 0.1).astype(np.uint8)
    pat = api.Pattern(m.elem, m.coords, m.cells, general=True)
    # ten elements meet at the inner nodes of five quadrilaterals' axis
    assert _form(pat) == (0 if name == "fan5" else 3)
    rp, ci = O.pattern(m.elem, m.n_nodes, m.cells)
    for p in (3.0, 2.5):
        mat = api.Material(p=p)
        for mk in (None, mask):
            K = torch.full((pat.nnz,), float("nan"), dtype=torch.float64, device="cuda")
            pat.assemble_general(mat, dev(rho), None if mk is None else dev(mk), out=K)
            ref = O.assemble(m.elem, m.coords, m.cells, rho, rp, ci, mask=mk, p=p)
            assert row_scaled_err(rp, host(K), ref) <= 1e-12
            again = pat.assemble_general(mat, dev(rho), None if mk is None else dev(mk))
            assert torch.equal(K, again)
    L = _lib.lib()
    assert L.soptx_debug_set_general_variant(0) == 0
    try:
        K0 = pat.assemble_general(mat, dev(rho), dev(mask))
    finally:
        L.soptx_debug_set_general_variant(-1)
    assert row_scaled_err(rp, host(K), host(K0)) <= 1e-12


def test_row_groups_captured():
    """Captured without a warm-up (no workspace is needed): every replay is the eager result."""
    m = _mesh("3x3x3_curved")
    pat = api.Pattern(m.elem, m.coords, m.cells, general=True)
    rho = dev(np.random.default_rng(94).uniform(0.01, 1.0, m.n_cells))
    K = torch.empty(pat.nnz, dtype=torch.float64, device="cuda")
    st = torch.cuda.Stream()
    torch.cuda.synchronize()
    g = torch.cuda.CUDAGraph()
    with torch.cuda.graph(g, stream=st):
        pat.assemble_general(MAT, rho, out=K, stream=st)
    for k in range(3):
        rho.mul_(0.9)
        ref = pat.assemble_general(MAT, rho)
        K.fill_(float("nan"))
        torch.cuda.synchronize()
        g.replay()
        torch.cuda.synchronize()
        assert torch.equal(K, ref), k
