"""GPU: launches of several time steps against single steps, bit for bit.

The planner picks a depth, a kernel and a tile per grid; the grids here reach
each kernel with ragged last tiles, grids narrower than a halo, walls, and
rounds of more tiles than the device holds. Every value is rounded where a
single step's store rounds it, so nothing but equality is right.
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


def _solver(L, nx, ny, dtype, walls, force, perm, scheme):
    rng = np.random.default_rng(nx * 1000 + ny)
    k = np.exp(rng.standard_normal((ny, nx)))
    if perm == L.LBM_PERM_TENSOR:
        off = 0.2 * np.minimum(k, k[::-1])
        k = np.stack([k, off, 0.5 * off, k[::-1]], axis=-1)
    g = 1e-6 * rng.standard_normal((ny, nx, 2)) if force else None
    p = L.make_params(nx, ny, 0.8, 0.4, 0.1, 1.0, 1e-6, 3e-7, walls, dtype, perm, scheme)
    return L.FineSolver(p, k, g)


@pytest.mark.parametrize("dtype,force,perm,scheme", [(0, 0, 1, 0), (0, 1, 4, 0), (0, 0, 1, 1), (1, 0, 1, 0),
                                                     (1, 1, 4, 0), (1, 1, 1, 1), (2, 0, 1, 0), (2, 1, 4, 0)])
@pytest.mark.parametrize("nx,ny,walls", [(1, 1, 0), (3, 17, 1), (19, 5, 0), (67, 131, 1), (131, 67, 0),
                                         (401, 390, 1), (1030, 777, 0)])
def test_launches_equal_single_steps(L, nx, ny, walls, dtype, force, perm, scheme):
    a = _solver(L, nx, ny, dtype, walls, force, perm, scheme)
    b = _solver(L, nx, ny, dtype, walls, force, perm, scheme)
    total = 0
    # every depth on its own (a call's steps are covered by one plan), then a
    # stretch longer than the planned ones
    for n in (2, 3, 4, 5, 6, 7, 8, 9, 10, 11, 12, 13, 77):
        if n == 77 and nx * ny > 200_000:
            break
        a.step(n, mean=False)
        total += n
    for _ in range(total):
        b.step(1, mean=False)
    assert a.steps_total == b.steps_total == total
    assert torch.equal(a.populations(), b.populations())
    a.close()
    b.close()
