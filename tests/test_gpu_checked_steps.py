"""The launch that is queued behind a check counts only if the run goes on:
after convergence, a non-finite mean or the last step the state is that of
plain steps, bit for bit (every split of a run into launches is)."""
import numpy as np
import pytest

from paper_1312_0195_amd import lbm as L

pytestmark = pytest.mark.gpu


def _solver(nx, ny, dtype):
    k = np.exp(np.random.default_rng(3).standard_normal((ny, nx)))
    return L.FineSolver(L.make_params(nx, ny, .8, .4, .1, 1., 1e-6, 0., 1, dtype, 1, 0), k, None)


def _plain(nx, ny, dtype, steps, state=None):
    s = _solver(nx, ny, dtype)
    if state is not None:
        s.set_populations(state)
    s.step(steps, 0., 0, mean=False)
    f, u = s.populations(), s.fields()[0]
    s.close()
    return f, u


@pytest.mark.parametrize("nx,ny,dtype,every", [(64, 64, L.LBM_F32_SHIFTED, 100), (33, 20, L.LBM_F64, 7),
                                               (600, 500, L.LBM_F32_FAST, 1), (300, 700, L.LBM_F64, 16)])
def test_state_after_a_check(nx, ny, dtype, every):
    # ends on a check without converging, then converges at the next one
    s = _solver(nx, ny, dtype)
    st, done, _ = s.step(3 * every, 1e-300, every)
    assert (st, done) == (L.LBM_ENOTCONV, 3 * every)
    st, done, mean = s.step(50 * every, 0.9, every)
    assert (st, done, s.steps_total) == (L.LBM_OK, every, 4 * every)
    f, u = _plain(nx, ny, dtype, 4 * every)
    assert (s.populations() == f).all() and (s.fields()[0] == u).all()
    m = u.reshape(2, -1).mean(1).cpu().numpy()
    assert np.allclose(mean, m, rtol=1e-9, atol=1e-13 * u.abs().max().item())
    s.step(5, 0., 0, mean=False)
    assert (s.populations() == _plain(nx, ny, dtype, 4 * every + 5)[0]).all()
    s.close()


@pytest.mark.parametrize("nx,ny,dtype", [(64, 64, L.LBM_F32_SHIFTED), (128, 300, L.LBM_F64)])
def test_state_after_a_non_finite_mean(nx, ny, dtype):
    s = _solver(nx, ny, dtype)
    f = s.populations()
    f[1, 5, 7] = float("nan")
    s.set_populations(f)
    st, done, _ = s.step(100, 0., 10)
    assert (st, done, s.steps_total) == (L.LBM_ENONFINITE, 10, 10)
    want = _plain(nx, ny, dtype, 10, f)[0].cpu().numpy()
    assert np.array_equal(s.populations().cpu().numpy(), want, equal_nan=True)
    s.close()


@pytest.mark.parametrize("nx,ny,dtype", [(2048, 1024, L.LBM_F32_SHIFTED), (1024, 1024, L.LBM_F64)])
def test_a_converged_run_takes_no_step_beyond_its_last(nx, ny, dtype):
    """A launch of a large grid costs far more than the idle time it would
    fill: a run that converges at its second check leaves both population
    buffers as a run of exactly those steps does."""
    el, n = (8, nx * ny) if dtype == L.LBM_F64 else (4, nx * ny)
    stride = (n + 63) // 64 * 64 * el + 16384
    second = (9 * stride + 255) // 256 * 256

    def buffers(s):
        return [s.ws[o:o + 9 * stride].reshape(9, stride)[:, :n * el].clone() for o in (0, second)]

    a, b = _solver(nx, ny, dtype), _solver(nx, ny, dtype)
    st, done, _ = a.step(50, 0.9, 1)  # from rest the velocity doubles in the second step
    assert (st, done) == (L.LBM_OK, 2)
    for _ in range(2):
        b.step(1, 0., 0, mean=False)
    for x, y in zip(buffers(a), buffers(b)):
        assert (x == y).all()
    a.close()
    b.close()
