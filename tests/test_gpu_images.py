"""dem_compute_forces on positions that the caller has shifted by whole boxes
since the lists were built: the same forces, whatever images they are."""
import numpy as np
import pytest

from paper_1607_02427_amd import inputs as I

pytestmark = pytest.mark.gpu

# positions of up to three boxes are rounded to 1e-14, on a force whose slope
# is some 1e3 of its size: 1e-11, with room; in FP32 the pair offsets round
# anew to 24 bits, 6e-8 of a box-independent offset of order one, 1e-4, with room
TOL = {"fp64": 1e-9, "fp32": 1e-3}


@pytest.mark.parametrize("make,precision", [(lambda: I.cubes_3d_contact(n_side=6), "fp64"),
                                            (lambda: I.cubes_3d_contact(n_side=6), "fp32"),
                                            (lambda: I.squares_2d_contact(), "fp64"),
                                            (lambda: I.contact_lattice(I.sphere(0.5), 500, 3), "fp32")])
def test_forces_of_other_images(make, precision):
    import torch
    from paper_1607_02427_amd import dem
    s = make()
    rng = np.random.default_rng(4)
    with dem.DemSystem(s, precision) as g:
        g.compute_forces()
        want = g.outputs()
        for a, k in enumerate("xyz"[: s.dim]):
            g.t[k] += torch.tensor(rng.integers(-2, 3, s.n) * float(s.box[a]), device=g.t[k].device)
        torch.cuda.synchronize()
        print(f"[images] {s.name} {s.shapes[0].name} {precision}", flush=True)
        g.compute_forces()
        got = g.outputs()
    for k in ("F", "T", "U", "W"):
        scale = np.max(np.abs(want[k]))
        assert (k == "T" and s.shapes[0].edges.shape[0] == 0) or scale > 0
        assert np.max(np.abs(got[k] - want[k])) <= TOL[precision] * max(scale, 1e-300), k
