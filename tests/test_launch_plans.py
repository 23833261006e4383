"""The launch planners on the host, for a device of 256 compute units."""
import ctypes
import time

from paper_1312_0195_amd import lbm as L


def _plan3(nx, ny, nz, dtype, walls=0):
    """(steps per launch, tile x, tile y, planes per run)"""
    out = (ctypes.c_int32 * 4)()
    p = L.make_params3(nx, ny, nz, 0.8, 0.4, 0.1, 1.0, (1e-6, 0.0, 0.0), walls, dtype)
    assert L.lib().lbm3d_plan_of(ctypes.byref(p), 256, out) == L.LBM_OK
    return tuple(out)


def test_a_column_of_many_planes_is_planned_at_once():
    """Each number of runs is tried once, so the longest column that a solver
    takes (2^30 planes) costs tens of thousands of trials, not 10^9."""
    _plan3(8, 8, 8, L.LBM_F32_SHIFTED)  # loads the library
    t = time.perf_counter()
    assert _plan3(1, 1, (1 << 30) - 65537, L.LBM_F32_SHIFTED)[0] in (1, 2)
    assert time.perf_counter() - t < 0.2
