"""GPU: the local problems' two plane layouts and two drives.

Launches on 1024 threads hold an item's planes at a fixed distance, smaller
ones pack them by the item's own cells; a drive along x and one along y run
code of their own. The layouts only move values, so an item gives the same
steps and tensor (to the FP64 summation order of its mean) in both; a patch and
its transpose exchange the drives, with the same steps up to a check.
"""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")


@pytest.fixture(scope="module")
def L():
    from paper_1312_0195_amd import lbm
    assert torch.cuda.is_available(), "GPU tests need a GPU"
    lbm.lib()
    return lbm


def _run(L, field, x0, y0, side, **kw):
    return L.local_keff(field, x0, y0, side, 0.8, 0.4, 0.1, 1e-6, tol=1e-7, check_every=100, max_steps=50000,
                        use_tuned=False, **kw)


@pytest.mark.parametrize("block", [256, 512])
def test_fixed_and_packed_planes_agree(L, block):
    from paper_1312_0195_amd import inputs as I
    field = I.lognormal_kappa(96, 96, 1.0, 8.0, seed=9)
    side = np.array([1, 2, 5, 8, 15, 16, 17, 20, 23, 29, 31, 32], np.int32)
    x0 = (np.arange(len(side)) * 7).astype(np.int32)
    y0 = (np.arange(len(side)) * 5).astype(np.int32)
    if block == 256:  # at most four cells per thread
        side, x0, y0 = side[side * side <= 1024], x0[:len(side)], y0[:len(side)]
    a = _run(L, field, x0, y0, side, block_threads=1024)
    b = _run(L, field, x0, y0, side, block_threads=block)
    assert (a.flags == 0).all() and np.array_equal(a.steps, b.steps)
    scale = np.maximum(np.abs(a.keff[:, 0]), np.abs(a.keff[:, 3]))[:, None]
    # the state is the same; the FP64 sum of up to 1024 cells may be ordered otherwise
    assert (np.abs(a.keff - b.keff) <= 1e-12 * scale).all()


@pytest.mark.parametrize("dtype", ["f32", "f64"])
def test_transposed_patch_exchanges_the_drives(L, dtype):
    from paper_1312_0195_amd import inputs as I
    field = I.lognormal_kappa(64, 64, 1.0, 6.0, seed=10)
    pd = L.LBM_F32_SHIFTED if dtype == "f32" else L.LBM_F64
    side = np.array([3, 11, 16, 27, 32, 40, 44] + ([48, 64] if dtype == "f32" else []), np.int32)
    o = (np.arange(len(side)) * 9 % 64).astype(np.int32)
    a = _run(L, field, o, o[::-1].copy(), side, pop_dtype=pd)
    b = _run(L, np.ascontiguousarray(field.T), o[::-1].copy(), o, side, pop_dtype=pd)
    assert (a.flags == 0).all() and (b.flags == 0).all()
    assert (np.abs(a.steps - b.steps[:, ::-1]) <= 100).all()
    scale = np.maximum(np.abs(a.keff[:, 0]), np.abs(a.keff[:, 3]))[:, None]
    # both within the convergence tolerance's distance of the same fixed point (1e-4 of the larger diagonal)
    assert (np.abs(a.keff - b.keff[:, [3, 2, 1, 0]]) <= 1e-4 * scale).all()
