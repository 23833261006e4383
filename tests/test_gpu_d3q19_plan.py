"""GPU: D3Q19 two-step launches and planned single steps against single steps,
bit for bit, on grids that reach each tile with ragged edges, runs of planes
that do not divide the grid, walls, and grids smaller than a tile."""
# FP64 state on 64 x 4 tiles and FP32 state on 16 x 8 tiles: test_gpu_planned_kernels.py
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


@pytest.mark.parametrize("walls", [0, 1])
@pytest.mark.parametrize("dtype", [0, 1])
@pytest.mark.parametrize("n", [(1, 1, 1), (5, 3, 2), (33, 20, 7), (30, 190, 40), (65, 70, 67), (111, 90, 75),
                               (130, 129, 61), (191, 120, 100)])
def test_launches_equal_single_steps(L, n, dtype, walls):
    rng = np.random.default_rng(sum(n))
    k = np.exp(rng.standard_normal(n[::-1]))
    p = L.make_params3(*n, 0.8, 0.4, 0.1, 1.0, (1e-6, 2e-7, -3e-7), walls, dtype)
    a, b = L.Solver3D(p, k), L.Solver3D(p, k)
    a.step(9)
    for _ in range(9):
        b.step(1)
    assert torch.equal(a.populations(), b.populations())
    a.close()
    b.close()
