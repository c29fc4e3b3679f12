"""Canonical orders of sheared Q1 meshes: nodes and elements are ranked in the
coordinates of the mesh's vertex lattice, so a sheared mesh in any numbering
gets the plan of the same mesh numbered along its grid.  Meshes without one
lattice (half of the cells sheared, elements of mixed local orientation) keep
the order along the axes.  Every plan's walk gives the oracle's K (row-scaled
error at most 1e-13, as for the plans of the given numbering)."""

import numpy as np
import pytest

from oracle import oracle as O
from paper_2505_02438_amd import api
from paper_2505_02438_amd import inputs as I
from test_host_library import _renumbered, row_scaled_err, walk_plan


def _mesh(elem, form):
    m = I.quad_grid(13, 9) if elem == I.QUAD4 else I.hex_grid(8, 6, 5)
    if form == "kink":
        return I.skew_mesh(m, "kink")
    m = I.skew_mesh(m, "global")
    if form == "mixed":
        # every second element starts at its opposite corner: its edges from
        # local vertex 0 point the other way along the first two axes
        c = m.cells.copy()
        turn = [2, 3, 0, 1] if elem == I.QUAD4 else [2, 3, 0, 1, 6, 7, 4, 5]
        c[::2] = c[::2][:, turn]
        return I.Mesh(elem, m.coords, c)
    return m


@pytest.mark.parametrize("elem", [I.QUAD4, I.HEX8])
@pytest.mark.parametrize("form", ["sheared", "kink", "mixed"])
def test_sheared_plans(elem, form):
    m0 = _mesh(elem, form)
    m, _, _ = _renumbered(m0, 19)
    hp = api.host_plan(elem, m.coords, m.cells)
    if form == "sheared":
        hp0 = api.host_plan(elem, m0.coords, m0.cells)
        assert hp["elem_by_rank"].size == m.n_cells and hp0["elem_by_rank"].size == 0
        assert hp["n_signatures"] == hp0["n_signatures"]
        sizes = lambda h: sorted(h["grp_info"].reshape(-1, 6)[:, 1].tolist())
        assert sizes(hp) == sizes(hp0)
    rho = np.random.default_rng(5).uniform(0.05, 1.0, m.n_cells)
    K = walk_plan(hp, m, rho, api.reference_tensor(elem))
    rp, ci = O.pattern(elem, m.n_nodes, m.cells)
    Kref = O.assemble(elem, m.coords, m.cells, rho, rp, ci)
    assert row_scaled_err(rp, K, Kref) <= 1e-13
