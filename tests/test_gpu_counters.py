"""Work counters of counted force evaluations: they add up over workgroups
and launches, whatever the launch shape, and clear when asked to."""
import numpy as np
import pytest

from paper_1607_02427_amd import inputs as I

pytestmark = pytest.mark.gpu


def _pairs_within_bound(s):
    shp = s.shapes[0]
    bound = 2.0 * shp.circumradius + 2.0 ** (1.0 / 6.0) * 2.0 * shp.r
    d = s.x[:, None, :] - s.x[None, :, :]
    d -= s.box * np.rint(d / s.box)
    r2 = np.sum(d[..., :s.dim] ** 2, axis=-1)
    return int(np.count_nonzero(np.triu(r2 < bound * bound, 1)))


# a system of fewer tiles than workgroups, one of many, a planar one
@pytest.mark.parametrize("make,precision", [(lambda: I.cubes_3d_contact(n_side=4), "fp32"),
                                            (lambda: I.cubes_3d_contact(n_side=11), "fp64"),
                                            (lambda: I.squares_2d_contact(), "fp32")])
def test_counters_sum_over_workgroups_and_launches(make, precision):
    from paper_1607_02427_amd import dem
    s = make()
    want = _pairs_within_bound(s)
    seen = []
    for shape in ((16, 1, 2, 4, 0), (8, 2, 2, 4, 0), (16, 1, 2, 16, 0), (8, 1, 2, 4, 1)):
        print(f"[counters] {s.name} {precision} {shape}", flush=True)
        with dem.DemSystem(s, precision) as g:
            g.set_pair_shape(*shape)
            g.force_stats(reset=True)
            g.compute_forces()
            one = g.force_stats()
            g.compute_forces()
            g.compute_forces()
            three = g.force_stats(reset=True)
            assert all(v == 0 for v in g.force_stats().values())
        if shape[4] == 0:  # (the split form's second kernel does not see the separated pairs)
            assert one["pairs"] == want
            assert one["launches"] == 1 and three["launches"] == 3
        assert one["in_cutoff"] > 0
        for k in one:
            assert three[k] == 3 * one[k], k
        seen.append({k: one[k] for k in ("pairs", "features", "in_cutoff", "vf_near", "ee_near", "refined", "separated")})
    assert all(c == seen[0] for c in seen[1:])
