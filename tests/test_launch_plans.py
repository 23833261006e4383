"""The launch planners on the host, for a device of 256 compute units."""
import ctypes
import time

import pytest

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


def _plan(nx, ny, dtype, steps, walls=0, force=0, perm=1, scheme=0, gy=3e-7):
    """((steps, kernel, tile x, tile y), predicted us) of the first launch"""
    out, us = (ctypes.c_int32 * 4)(), ctypes.c_double()
    p = L.make_params(nx, ny, 0.8, 0.4, 0.1, 1.0, 1e-6, gy, walls, dtype, perm, scheme)
    assert L.lib().lbm_plan_of(ctypes.byref(p), force, 256, ctypes.c_int64(steps), out, ctypes.byref(us)) == L.LBM_OK
    return tuple(out), us.value


def _run_us(n, steps, **kw):
    t = 0.0
    while steps > 0:
        (d, *_), us = _plan(n, n, L.LBM_F32_SHIFTED, steps, **kw)
        t += us
        steps -= d
    return t


@pytest.mark.parametrize("n,measured", [(700, 3.5), (1000, 6.3), (1400, 11.6), (2048, 26.8)])
def test_tensor_rows_are_planned_as_one_workgroup_per_cu(n, measured):
    """FP32 state with a tensor in FP64 arithmetic: the registers allow one
    workgroup of the row kernel per CU. us per step as measured on the planned
    launches, to 15%."""
    t = _run_us(n, 600, perm=L.LBM_PERM_TENSOR) / 600
    assert abs(t / measured - 1) < 0.15, t


# grids that test_gpu_planned_kernels.py steps, with the tile that each plans:
# narrower than a tile and its halo, runs of two planes, last runs of one, and
# several ragged columns
D3Q19_GRIDS = {L.LBM_F32_SHIFTED: [((63, 33, 101), (64, 8, 2)), ((61, 2001, 2), (64, 8, 2)),
                                   ((130, 90, 75), (64, 8, 11)), ((15, 501, 31), (16, 8, 3)),
                                   ((31, 131, 67), (16, 8, 3)), ((130, 129, 130), (16, 8, 33))],
               L.LBM_F64: [((63, 501, 5), (64, 4, 3)), ((703, 699, 2), (64, 4, 2)), ((191, 9, 131), (64, 4, 5)),
                           ((128, 128, 128), (64, 4, 32)), ((15, 1001, 5), (16, 8, 2)), ((9, 2001, 4), (16, 8, 2)),
                           ((130, 7, 101), (16, 8, 2))]}


def test_the_d3q19_grids_reach_every_tile():
    for dtype, grids in D3Q19_GRIDS.items():
        for n, tile in grids:
            assert _plan3(*n, dtype) == (2, *tile), n


# stretches over which a 1030 x 777 grid with a drive along x only and FP32
# arithmetic takes the row kernels: 64 x 36 and 64 x 32 halo tiles
ROW_GRID, ROW_STRETCHES = (1030, 777), (2, 3, 4, 5, 6, 7, 8, 13)


def test_the_row_grid_reaches_both_row_kernels():
    kernels = [_plan(*ROW_GRID, L.LBM_F32_FAST, n, gy=0.0)[0][1] for n in ROW_STRETCHES]
    assert {4, 5} <= set(kernels)


# thin grids that take two steps per launch, with walls in z or without
THIN_GRIDS = {(L.LBM_F32_SHIFTED, 0): [(1500, 700, 2), (301, 299, 2)],
              (L.LBM_F32_SHIFTED, 1): [(61, 67, 1), (255, 130, 1), (1999, 1001, 1), (301, 299, 2), (1500, 700, 2),
                                       (1201, 401, 3)],
              (L.LBM_F64, 0): [(703, 699, 2), (500, 501, 3)],
              (L.LBM_F64, 1): [(61, 67, 1), (255, 130, 1), (703, 1001, 1), (301, 299, 2), (500, 301, 4)]}


def test_thin_grids_take_two_steps_per_launch():
    for (dtype, walls), grids in THIN_GRIDS.items():
        for n in grids:
            steps, _, _, zc = _plan3(*n, dtype, walls)
            assert (steps, zc) == (2, n[2]), (n, dtype, walls)


FORMS = [(0, 0, 1, 0), (0, 1, 1, 0), (0, 0, 4, 0), (0, 1, 4, 0), (0, 0, 1, 1), (0, 1, 1, 1), (1, 0, 1, 0), (1, 1, 4, 0),
         (1, 0, 1, 1), (2, 0, 1, 0), (2, 1, 1, 0), (2, 0, 4, 0), (2, 1, 4, 0)]  # type, force, perm, scheme


def test_few_steps_do_not_run_on_slivers():
    """Rows of a few cells read partial cache lines: a two-step launch of 512^2
    cells on tiles of 4 x 256 took twice the time of one on 30 x 14."""
    for dtype, force, perm, scheme in FORMS:
        for n in (200, 256, 300, 400, 512, 600, 700, 850, 1024, 1400, 2048, 4096):
            for stretch in (2, 3, 4, 5):
                (steps, kernel, tx, _), _ = _plan(n, n, dtype, stretch, 0, force, perm, scheme)
                assert steps == 1 or tx >= 16, (n, dtype, force, perm, scheme, stretch, kernel, tx)


# grids in and beyond the caches whose launches of two (and, with a tensor, three
# and four) steps have their tiles from few_steps
FEW_GRIDS = [(523, 401), (1030, 777), (1337, 1411), (1901, 1803)]


def test_the_few_step_grids_reach_each_tile():
    reached = {_plan(nx, ny, dtype, d, 1, force, perm, scheme)[0][:2]
               for nx, ny in FEW_GRIDS for dtype, force, perm, scheme in FORMS for d in (2, 3, 4)}
    assert {(2, 0), (2, 1), (3, 1), (4, 1)} <= reached
