"""Folded steps (the kick-drift carries the replica tail of the step before)
against steps with a tail kernel of their own: the same numbers, bit for bit,
also when a run changes from one form to the other between calls."""
import numpy as np
import pytest

from paper_1607_02427_amd import inputs as I

pytestmark = pytest.mark.gpu


def _cubes(n_side, ensemble, seed=2):
    s = I.lattice_system(I.cube(1.0, 0.15), n_side, 0.8, seed, orient="small", max_deg=3.0)
    s.ensemble, s.dt, s.kT = ensemble, 5e-4, 1.5
    s.P, s.tau_P = 1.0, 0.5
    return s


def _same(a, b):
    (sa, oa), (sb, ob) = a, b
    for k in ("x", "q", "v", "L", "image"):
        assert np.array_equal(getattr(sa, k), getattr(sb, k)), k
    for k in oa:
        assert np.array_equal(oa[k], ob[k]), k


# 5^3 = 125 bodies end in a partly filled chunk; 64 fill one chunk exactly
@pytest.mark.parametrize("n_side,ensemble,precision", [(5, "nvt", "fp32"), (4, "nvt", "fp64"), (5, "nve", "fp64")])
def test_folded_and_unfolded_steps_agree(n_side, ensemble, precision):
    from paper_1607_02427_amd import dem
    s, npt = _cubes(n_side, ensemble), _cubes(5, "npt", seed=3)
    calls = (7, 1, 40, 200, 3, 16)  # list rebuilds fall in the long ones
    with dem.DemBatch(3, precision, max_replicas=2, max_particles=1024) as B:
        rid = B.add(s)
        for n in calls:
            B.step(n)
        want, e0 = B.read(rid), B.energy(rid)
    assert e0["n_rebuilds"] >= 2  # the build of the start, and one in a step at least
    with dem.DemBatch(3, precision, max_replicas=2, max_particles=1024) as B:
        rid = B.add(s)
        for k, n in enumerate(calls):  # a barostat replica in every other call: those steps are not folded
            other = B.add(npt) if k % 2 else None
            print(f"[fold] {ensemble} {precision} call of {n} steps, folded {other is None}", flush=True)
            B.step(n)
            if other is not None:
                B.remove(other)
        got, e1 = B.read(rid), B.energy(rid)
    _same(want, got)
    for k in ("U", "K_trans", "K_rot", "H", "xi", "eta", "step", "n_rebuilds"):
        assert e0[k] == e1[k], k


def test_a_replica_whose_budget_ends_mid_call_closes_its_step():
    from paper_1607_02427_amd import dem
    a, b = _cubes(5, "nvt"), _cubes(4, "nvt", seed=4)
    with dem.DemBatch(3, "fp32", max_replicas=1, max_particles=256) as B:
        rid = B.add(a)
        B.step(13)
        want, e0 = B.read(rid), B.energy(rid)
    with dem.DemBatch(3, "fp32", max_replicas=2, max_particles=512) as B:
        ra, rb = B.add(a, steps=13), B.add(b)
        B.step(30)
        got, e1 = B.read(ra), B.energy(ra)
        assert list(B.progress(2)[1]) == [13, 30]
    _same(want, got)
    for k in ("H", "xi", "eta", "step"):
        assert e0[k] == e1[k], k
