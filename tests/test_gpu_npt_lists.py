"""The lists of an NPT system whose box shrinks through several cell grids:
cells and rows are those of the last build's grid, whatever the box is when
they are copied out."""
import numpy as np
import pytest

import oracle
from paper_1607_02427_amd import inputs as I

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("dim,precision", [(2, "fp64"), (3, "fp32")])
def test_lists_follow_the_grid_of_the_last_build(dim, precision):
    from paper_1607_02427_amd import dem
    s = I.replica_system(I.square() if dim == 2 else I.cube(), 500, 0.06, 9, ensemble="npt", dt=1e-3 if dim == 2 else 4e-4)
    s.P, s.tau_P, s.tau_T = (2.0 if dim == 2 else 1.0), 0.5, 0.5
    grids = []
    with dem.DemSystem(s, precision) as g:
        for k in range(24):
            g.step(150)
            print(f"[npt lists] {dim}D {precision} step {150 * (k + 1)}", flush=True)
            L = g.lists()
            cells = int(np.prod(L["dims"]))
            grids.append(tuple(L["dims"]))
            assert len(L["cell_start"]) == cells + 1 <= g.list_info()[1] + 1
            assert L["cell_start"][0] == 0 and L["cell_start"][-1] == s.n and np.all(np.diff(L["cell_start"]) >= 0)
            assert np.array_equal(np.sort(L["cell_particles"]), np.arange(s.n))
        assert len(set(grids)) >= 3  # the box has shrunk through several grids
        g.build_lists()
        now, L = g.state(), g.lists()
        assert tuple(L["dims"][:dim]) == tuple(np.floor(now.box[:dim] / L["r_list"]).astype(int))
        want, n_want, _ = oracle.nbr_list(now, L["r_list"], L["capacity"])
    assert np.array_equal(L["n_nbr"], n_want)
    for i in range(s.n):
        assert np.array_equal(L["nbr"][: n_want[i], i], want[: n_want[i], i]), i
    # every particle in the cell its position falls in
    cell = np.floor(now.x[:, :dim] / (now.box[:dim] / L["dims"][:dim])).astype(int)
    at = np.repeat(np.arange(len(L["cell_start"]) - 1), np.diff(L["cell_start"]))
    lin = cell[:, 0] + L["dims"][0] * (cell[:, 1] + (L["dims"][1] * cell[:, 2] if dim == 3 else 0))
    assert np.array_equal(lin[L["cell_particles"]], at)
