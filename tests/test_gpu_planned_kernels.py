"""GPU: the multi-step kernels that only some grids plan, against single steps,
bit for bit. test_launch_plans.py checks on the host that these grids plan
them."""
import numpy as np
import pytest

from test_launch_plans import D3Q19_GRIDS, FEW_GRIDS, FORMS, ROW_GRID, ROW_STRETCHES, THIN_GRIDS

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")


@pytest.fixture(scope="module")
def L():
    from paper_1312_0195_amd import lbm
    assert torch.cuda.is_available(), "GPU tests need a GPU"
    lbm.lib()
    return lbm


@pytest.mark.parametrize("walls", [0, 1])
@pytest.mark.parametrize("dtype,n", [(d, n) for d, grids in D3Q19_GRIDS.items() for n, _ in grids])
def test_d3q19_two_step_tiles_equal_single_steps(L, dtype, n, walls):
    k = np.exp(np.random.default_rng(sum(n)).standard_normal(n[::-1]))
    p = L.make_params3(*n, 0.8, 0.4, 0.1, 1.0, (1e-6, 2e-7, -3e-7), walls, dtype)
    a, b = L.Solver3D(p, k), L.Solver3D(p, k)
    a.step(9)
    for _ in range(9):
        b.step(1)
    fa = a.populations()
    assert torch.equal(fa, b.populations())
    assert float((fa[1] - fa[2]).abs().max()) > 0
    a.close()
    b.close()


@pytest.mark.parametrize("dtype,walls,n", [(d, w, n) for (d, w), grids in THIN_GRIDS.items() for n in grids])
def test_d3q19_thin_grids_equal_single_steps(L, dtype, walls, n):
    test_d3q19_two_step_tiles_equal_single_steps(L, dtype, n, walls)


@pytest.mark.parametrize("walls", [0, 1])
def test_rows_with_a_drive_along_x_only_equal_single_steps(L, walls):
    nx, ny = ROW_GRID
    k = np.exp(np.random.default_rng(7).standard_normal((ny, nx)))
    p = L.make_params(nx, ny, 0.8, 0.4, 0.1, 1.0, 1e-6, 0.0, walls, L.LBM_F32_FAST)
    a, b = L.FineSolver(p, k), L.FineSolver(p, k)
    for n in ROW_STRETCHES:
        a.step(n, mean=False)
        for _ in range(n):
            b.step(1, mean=False)
        assert torch.equal(a.populations(), b.populations()), n
    f = a.populations()
    assert float((f[2] - f[4]).abs().max()) > 0  # the heterogeneity drives a flow along y
    a.close()
    b.close()


def _equal_single_steps(L, nx, ny, walls, stretches, dtype, force, perm, scheme):
    rng = np.random.default_rng(8)
    k = np.exp(rng.standard_normal((ny, nx)))
    if perm == L.LBM_PERM_TENSOR:
        off = 0.2 * np.minimum(k, k[::-1])
        k = np.stack([k, off, 0.5 * off, k[::-1]], axis=-1)
    g = 1e-6 * rng.standard_normal((ny, nx, 2)) if force else None
    p = L.make_params(nx, ny, 0.8, 0.4, 0.1, 1.0, 1e-6, 3e-7, walls, dtype, perm, scheme)
    a, b = L.FineSolver(p, k, g), L.FineSolver(p, k, g)
    for n in stretches:
        a.step(n, mean=False)
    for _ in range(sum(stretches)):
        b.step(1, mean=False)
    assert torch.equal(a.populations(), b.populations())
    a.close()
    b.close()


@pytest.mark.parametrize("dtype,force,perm,scheme", FORMS)
def test_large_walled_grids_equal_single_steps(L, dtype, force, perm, scheme):
    """The kernels of large grids between walls, where the edge tiles bounce
    back in LDS."""
    _equal_single_steps(L, *ROW_GRID, 1, ROW_STRETCHES, dtype, force, perm, scheme)


@pytest.mark.parametrize("nx,ny", FEW_GRIDS)
@pytest.mark.parametrize("dtype,force,perm,scheme", FORMS)
def test_few_steps_equal_single_steps(L, nx, ny, dtype, force, perm, scheme):
    _equal_single_steps(L, nx, ny, (nx + dtype) % 2, (2, 3, 4), dtype, force, perm, scheme)
