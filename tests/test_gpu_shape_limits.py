"""Which pair-kernel shape the library picks by itself: either side of each
limit of the rule, the side shown from the sizes, and the bits of every other
shape on both."""
import ctypes as C

import numpy as np
import pytest

from paper_1607_02427_amd import inputs as I

pytestmark = pytest.mark.gpu

FEW = {"fp32": 40960, "fp64": 32768}  # pair slots up to which a system is small


def _in_use(g):
    """(lanes, separation lanes) of the handle's pair kernel."""
    from paper_1607_02427_amd import dem
    s = (C.c_int32 * 5)()
    f = dem.lib().dem_pair_shape_in_use
    f.argtypes, f.restype = [C.c_void_p, C.POINTER(C.c_int32)], None
    f(g.h, s)
    assert (s[1], s[4]) == (1, 0)
    return s[0], s[3]


def _gas(shape, n, seed=5):
    return I.contact_lattice(shape, n, seed, gap=1.08, max_deg=1.0)


def _slots(n, cap):
    return (n + 63) // 64 * 64 * cap // 2


# bodies of few and of many features on either side of the small-system limit
@pytest.mark.parametrize("make,n,precision,few,want", [
    (lambda: I.cube(), 1024, "fp32", True, (16, 16)), (lambda: I.cube(), 2000, "fp32", False, (8, 4)),
    (lambda: I.cube(), 768, "fp64", True, (16, 16)), (lambda: I.cube(), 1500, "fp64", False, (8, 4)),
    (lambda: I.lprism(), 900, "fp64", True, (16, 16)), (lambda: I.lprism(), 1500, "fp64", False, (16, 4)),
    (lambda: I.lprism(), 2500, "fp32", False, (8, 4)),
    (lambda: I.icosahedron(), 2000, "fp32", True, (16, 16)), (lambda: I.icosahedron(), 4000, "fp32", False, (16, 4)),
    (lambda: I.square(), 1500, "fp32", True, (16, 16)), (lambda: I.square(), 4500, "fp64", False, (8, 4)),
    (lambda: I.hexadecagon(), 4500, "fp64", False, (8, 4)), (lambda: I.hexadecagon(), 4500, "fp32", False, (8, 4)),
    (lambda: I.regular_polygon(9, 0.6), 4500, "fp64", False, (8, 4))])
def test_either_side_of_a_limit(make, n, precision, few, want):
    from paper_1607_02427_amd import dem
    s = _gas(make(), n)
    with dem.DemSystem(s, precision) as g:
        slots = _slots(n, g.list_info()[2])
        print(f"[limits] {s.shapes[0].name} {n} {precision}: {slots} slots, {_in_use(g)}", flush=True)
        assert (slots <= FEW[precision]) == few
        assert _in_use(g) == want
        out = g.outputs()
        for shape in ((16, 1, 2, 16), (8, 1, 2, 4), (16, 1, 2, 4)):
            g.set_pair_shape(*shape)
            assert _in_use(g) == (shape[0], shape[3])
            g.compute_forces()
            got = g.outputs()
            for k in out:
                assert np.array_equal(out[k], got[k]), (k, shape)


# the limits are of pairs: a row capacity that the caller sets moves none
@pytest.mark.parametrize("make,n,capacity", [(lambda: I.cube(), 1000, 128), (lambda: I.cube(), 2000, 32),
                                             (lambda: I.sphere(0.5), 20000, 64), (lambda: I.square(), 1500, 96)])
def test_row_capacity_leaves_the_shape_alone(make, n, capacity):
    from paper_1607_02427_amd import dem
    s = _gas(make(), n)
    with dem.DemSystem(s, "fp32") as g:
        want, auto = _in_use(g), g.list_info()[2]
    assert auto != capacity
    with dem.DemSystem(s, "fp32", nbr_capacity=capacity) as g:
        assert g.list_info()[2] == capacity
        print(f"[limits] {s.shapes[0].name} {n} rows of {capacity} ({auto}): {_in_use(g)}", flush=True)
        assert _in_use(g) == want
    with dem.DemBatch(s.dim, "fp32", max_replicas=1, max_particles=s.n + 64, nbr_capacity=capacity) as B:
        B.add(s)
        assert _in_use(B) == want


# a lane per pair from 500,000 slots of bodies of one vertex on
@pytest.mark.parametrize("n,want", [(20000, (8, 4)), (30011, (8, 1))])
def test_a_lane_per_pair_from_its_limit_on(n, want):
    from paper_1607_02427_amd import dem
    s = _gas(I.sphere(0.5), n)
    with dem.DemSystem(s, "fp32") as g:
        assert (_slots(n, g.list_info()[2]) >= 500000) == (want[1] == 1)
        assert _in_use(g) == want


# bodies of many features hold most of the slots, or not
@pytest.mark.parametrize("shapes,precision,want", [(((I.lprism, 1500), (I.cube, 700)), "fp64", (16, 4)),
                                                   (((I.lprism, 700), (I.cube, 2000)), "fp64", (8, 4)),
                                                   (((I.icosahedron, 3000), (I.cube, 700)), "fp32", (16, 4)),
                                                   (((I.icosahedron, 1000), (I.cube, 2500)), "fp32", (8, 4))])
def test_a_batch_goes_by_what_holds_most_of_its_slots(shapes, precision, want):
    from paper_1607_02427_amd import dem
    systems = [_gas(make(), n) for make, n in shapes]
    own, solo = [], []
    for s in systems:
        with dem.DemSystem(s, precision) as g:
            own.append(_slots(s.n, g.list_info()[2]))
            g.step(10)
            solo.append((g.state(), g.outputs()))
    assert sum(own) > FEW[precision] and (2 * own[0] > sum(own)) == (want[0] == 16)
    with dem.DemBatch(3, precision, max_replicas=2, max_particles=8192) as B:
        rids = [B.add(s) for s in systems]
        print(f"[limits] batch of {own} slots, {precision}: {_in_use(B)}", flush=True)
        assert _in_use(B) == want
        B.step(10)
        for rid, (st, out) in zip(rids, solo):
            got, gout = B.read(rid)
            for k in ("x", "q", "v", "L"):
                assert np.array_equal(getattr(st, k), getattr(got, k)), k
            for k in out:
                assert np.array_equal(out[k], gout[k]), k
