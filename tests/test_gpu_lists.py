"""Neighbour rows and pair entries of a list build against the oracle's rows:
whole numbers, so equal."""
import numpy as np
import pytest

import oracle
from paper_1607_02427_amd import inputs as I

pytestmark = pytest.mark.gpu


def _points(n, skin, dim=3, jitter=0.0, gap=1.08):
    s = I.contact_lattice(I.sphere(0.5) if dim == 3 else I.disk(0.5), n, 3, gap=gap, max_deg=1.0)
    rng = np.random.default_rng(11)
    d = min(s.dim, 3)
    s.x[:, :d] = (s.x[:, :d] + jitter * rng.uniform(-1, 1, (n, d))) % np.asarray(s.box[:d])
    s.skin = skin
    return s


# groups of four and chunks that end early, without cells and with, rows of
# nearly the longest kind (120) and cells nearly full (62), 2D
CASES = [(30, 0.3, 3, 1.08), (63, 0.3, 3, 1.08), (130, 0.4, 3, 1.08), (1029, 2.2, 3, 1.08), (1531, 1.5, 3, 1.08),
         (4099, 0.35, 3, 1.3), (20003, 0.4, 3, 1.08), (70, 0.3, 2, 1.08), (1027, 3.0, 2, 1.08), (9001, 0.3, 2, 1.08)]


def _check_forces(s, F):
    # FP64 sums of a few terms in another order, on a force whose slope is
    # some 1e3 of its size: 1e3 * 2^-52 * a few ulp, with room
    ref = oracle.forces(s)
    assert np.max(np.abs(F - ref["F"]) / np.maximum(ref["scale"][:, :1], 1.0)) <= 1e-10


@pytest.mark.parametrize("n,skin,dim,gap", CASES)
def test_a_build_gives_the_oracles_rows(n, skin, dim, gap):
    from paper_1607_02427_amd import dem
    s = _points(n, skin, dim, jitter=0.02, gap=gap)
    print(f"[lists] {n} {dim}D skin {skin}", flush=True)
    with dem.DemSystem(s, "fp64") as g:
        L = g.lists()
        want, n_want, longest = oracle.nbr_list(s, L["r_list"], L["capacity"])
        assert longest <= L["capacity"]
        assert np.array_equal(L["n_nbr"], n_want)
        for i in range(n):
            assert np.array_equal(L["nbr"][: n_want[i], i], want[: n_want[i], i]), i
        _check_forces(s, g.outputs()["F"])  # every pair has its entry and its two row slots


@pytest.mark.parametrize("n,skin,dim,gap", [(130, 0.12, 3, 1.2), (1531, 0.12, 3, 1.2), (5003, 0.12, 3, 1.2), (2051, 0.12, 2, 1.2)])
def test_builds_within_steps_give_the_oracles_forces(n, skin, dim, gap):
    from paper_1607_02427_amd import dem
    s = _points(n, skin, dim, jitter=0.02, gap=gap)
    rng = np.random.default_rng(7)
    s.v[:, :dim] = rng.normal(0, 1.0, (n, dim))
    s.dt = 1e-3
    print(f"[lists in steps] {n} {dim}D", flush=True)
    with dem.DemSystem(s, "fp64") as g:
        g.step(400)
        assert g.energy()["n_rebuilds"] >= 3
        _check_forces(g.state(), g.outputs()["F"])
