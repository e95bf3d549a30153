"""dem_batch_read into arrays outside the device's memory: each takes a copy
command, and the values are those a read into device arrays gives.  The
virial, whose rows are copied by one strided command, is refused there when
its memory is pageable."""
import ctypes as C

import numpy as np
import pytest

from paper_1607_02427_amd import inputs as I

pytestmark = pytest.mark.gpu


def _host_arrays(n, pinned):
    import torch
    f = lambda m: torch.zeros(m, dtype=torch.float64, pin_memory=pinned)
    g = lambda m: torch.zeros(m, dtype=torch.int32, pin_memory=pinned)
    from paper_1607_02427_amd import dem
    t = {k: f(n) for k in dem.STATE}
    t["shape_id"], t["image"] = g(n), g(3 * n)
    o = {k: f(n) for k in dem.OUT}
    o["W"] = f(9 * n)
    return t, o


@pytest.mark.parametrize("pinned", [False, True])
def test_read_into_host_arrays(pinned):
    from paper_1607_02427_amd import dem
    a, b = I.cubes_3d(n_side=5), I.cubes_3d_contact(n_side=6)
    with dem.DemBatch(3, "fp32", max_replicas=2, max_particles=1024) as B:
        B.add(a)
        rid = B.add(b)  # (not at slot 0)
        B.step(5)
        s, out = B.read(rid)
        t, o = _host_arrays(b.n, pinned)
        # some of the arrays in device memory, so that both ways are taken in one call
        t["y"], o["U"], host_w = t["y"].cuda(), o["U"].cuda(), o["W"]
        o["W"] = o["W"].cuda()
        import torch
        torch.cuda.synchronize()
        print(f"[read] host arrays, pinned {pinned}", flush=True)
        B._check(dem.lib().dem_batch_read(B.h, rid, C.byref(dem._state_ptrs(t)), C.byref(dem._out_ptrs(o))), "dem_batch_read")
        B.sync()
        hs, hout = dem._state_np(t, b), dem._outputs_np(o, b.n)
        st = dem.lib().dem_batch_read(B.h, rid, None, C.byref(dem.OutPtrs(W=host_w.data_ptr())))
        assert st == (0 if pinned else 4)  # DEM_E_HIP
        if not pinned:
            dem.lib().dem_sync(B.h)  # (takes the runtime's own record of the error with it)
        else:
            B.sync()
            assert np.array_equal(host_w.numpy().reshape(9, b.n).T, out["W"])
    for k in ("x", "q", "v", "L", "image"):
        assert np.array_equal(getattr(s, k), getattr(hs, k)), k
    assert np.array_equal(t["shape_id"].numpy(), b.shape_id)
    for k in out:
        assert np.array_equal(out[k], hout[k]), k
