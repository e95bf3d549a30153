"""Folded steps where a replica has more chunks than a wavefront has lanes
(every lane of the kinetic sum adds more than one, the last chunk ragged), and
where the only replica left does not begin at the first chunk: the same
numbers, bit for bit, as in the unfolded form and alone."""
import numpy as np
import pytest

from paper_1607_02427_amd import inputs as I

pytestmark = pytest.mark.gpu


def _cubes(n, ensemble="nvt", seed=2):
    s = I.replica_system(I.cube(1.0, 0.15), n, 0.3, seed, kT=1.5, max_deg=3.0, ensemble=ensemble)
    s.P, s.tau_P = 1.0, 0.5
    return s


def _same(a, b):
    (sa, oa), (sb, ob) = a, b
    for k in ("x", "q", "v", "L", "image"):
        assert np.array_equal(getattr(sa, k), getattr(sb, k)), k
    for k in oa:
        assert np.array_equal(oa[k], ob[k]), k


def _run(B, rid, calls, between=None):
    for k, n in enumerate(calls):
        other = between(k)
        B.step(n)
        if other is not None:
            B.remove(other)
    return B.read(rid), B.energy(rid)


# 4161 = 65 chunks and one body, 8320 = 130 chunks
@pytest.mark.parametrize("n,precision", [(4161, "fp32"), (8320, "fp32"), (4161, "fp64")])
def test_kinetic_sums_over_many_chunks(n, precision):
    from paper_1607_02427_amd import dem
    s, npt = _cubes(n), _cubes(125, "npt", seed=3)
    calls = (5, 1, 120, 9, 3, 16)
    got = []
    for fold in (True, False):
        print(f"[fold] {n} {precision} folded throughout: {fold}", flush=True)
        with dem.DemBatch(3, precision, max_replicas=2, max_particles=n + 512) as B:
            rid = B.add(s)
            got.append(_run(B, rid, calls, lambda k: B.add(npt) if not fold and k % 2 == 0 else None))
    _same(got[0][0], got[1][0])
    assert got[0][1]["n_rebuilds"] >= 2
    for k in ("U", "K_trans", "K_rot", "H", "xi", "eta", "step", "n_rebuilds"):
        assert got[0][1][k] == got[1][1][k], k


@pytest.mark.parametrize("ensemble,precision", [("nvt", "fp32"), ("nve", "fp32"), ("nvt", "fp64")])
def test_a_lone_replica_behind_free_chunks(ensemble, precision):
    from paper_1607_02427_amd import dem
    a, b, c = _cubes(64, seed=5), _cubes(125, seed=6), _cubes(201, ensemble, seed=7)
    calls = (7, 1, 200, 16)
    with dem.DemBatch(3, precision, max_replicas=1, max_particles=512) as B:
        want, e0 = _run(B, B.add(c), calls, lambda k: None)
    assert e0["n_rebuilds"] >= 2
    with dem.DemBatch(3, precision, max_replicas=2, max_particles=1024) as B:
        ra, rb = B.add(a), B.add(b)
        B.step(12)
        B.remove(ra)
        rc = B.add(c)  # slot 0 again, but too large for the first chunk
        assert rc == ra == 0
        B.remove(rb)   # the first three chunks are free now
        info = B.info()
        assert info["live"] == 1 and info["largest_free_run"] < info["free_particles"]
        print(f"[fold] lone replica behind free chunks, {ensemble} {precision}", flush=True)
        got, e1 = _run(B, rc, calls, lambda k: None)
    _same(want, got)
    for k in ("U", "K_trans", "K_rot", "H", "xi", "eta", "step", "n_rebuilds"):
        assert e0[k] == e1[k], k
