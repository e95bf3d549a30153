"""The admission charge (no GPU): a replica's footprint is its share of a
batch's memory, so what a handle holds once is not in it, and it does not
move with the layout of the library's own structures: a batch of a fixed
budget admits the replicas it always admitted."""
import os

import pytest

from paper_1607_02427_amd import dem, inputs as I

pytestmark = pytest.mark.skipif(not os.path.exists(dem.LIB_PATH), reason="libdem.so is not built")


def _four_shapes(n):
    s = I.contact_lattice(I.lprism(), n, 5)
    s.shapes = [s.shapes[0], I.sphere(0.5), I.cube(), I.octahedron()]
    return s


# bytes as admission budgets have been set by: one chunk, few, many, planar
# with a fixed row capacity, four shapes, the largest cubes of Table I
@pytest.mark.parametrize("make,precision,capacity,want", [
    (lambda: I.cubes_3d(n_side=4), "fp32", 0, 305056),
    (lambda: I.cubes_3d(n_side=6), "fp32", 0, 823820),
    (lambda: I.cubes_3d(n_side=16), "fp64", 0, 18315208),
    (lambda: I.squares_2d(), "fp64", 40, 1419292),
    (lambda: _four_shapes(700), "fp32", 0, 4683944),
    (lambda: I.cubes_3d(n_side=40), "fp32", 0, 174544048)])
def test_charge_of_a_replica(make, precision, capacity, want):
    assert dem.footprint_bytes(make(), precision, capacity) == want
