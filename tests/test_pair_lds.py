"""LDS of the pair kernel's forms (no GPU): for replicas of one shape a CU
holds as many workgroups as the form is compiled for, three in FP32 and two
in FP64 or with the feature cells, in granules of 1280 of its 163,840 bytes."""
import ctypes as C
import os

import pytest

from paper_1607_02427_amd import dem

pytestmark = pytest.mark.skipif(not os.path.exists(dem.LIB_PATH), reason="libdem.so is not built")

FUSED, FORCES = 0, 2


# (a lane per pair in the separation stage: 3D without the feature cells)
FORMS = [(dim, cells, *form) for dim in (2, 3) for cells in (0, 1)
         for form in ((16, 4, FUSED), (8, 4, FUSED), (16, 16, FUSED), (8, 1, FUSED), (16, 4, FORCES), (8, 4, FORCES))
         if form[1] != 1 or (dim == 3 and not cells)]


@pytest.mark.parametrize("precision", [dem.DEM_FP32, dem.DEM_FP64])
@pytest.mark.parametrize("dim,cells,lanes,sep,stage", FORMS)
def test_workgroups_per_cu(precision, dim, cells, lanes, sep, stage):
    f = dem.lib()["_ZN3dem15pair_kernel_ldsEiiiiiii"]  # dem::pair_kernel_lds
    f.restype = C.c_size_t
    lds = f(precision, dim, 1, lanes, sep, stage, cells)
    held = 163840 // (-(-lds // 1280) * 1280)
    assert held >= (2 if precision == dem.DEM_FP64 or cells else 3), lds
