"""GPU: a coarse solve beside other work. The middle range of sizes reads its
status from pinned host memory that a thread keeps."""
import threading

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


class _Problem:
    def __init__(self, L, n, dtype, seed):
        self.L, self.n = L, n
        self.fine = L.make_params(8 * n, 8 * n, 0.8, 0.4, 0.1, 1.0, 1e-6, 0.0, 0, dtype)
        k = np.exp(0.5 * np.random.default_rng(seed).standard_normal((n, n)))
        self.K = torch.as_tensor(np.stack([k, 0.1 * k, 0.1 * k, 0.5 + k[::-1, ::-1]], axis=-1)).cuda()
        self.nb = L.lbm_coarse_workspace_bytes(n, n)
        self.ws = torch.empty(self.nb, dtype=torch.uint8, device="cuda")
        self.u = torch.empty((2, n, n), dtype=torch.float64, device="cuda")
        torch.cuda.synchronize()

    def solve(self, stream):
        st, steps = self.L.lbm_coarse_solve(self.fine, 8, self.K, self.L.LBM_KEFF_TENSOR, None, 4000, 1e-6, 50, self.u,
                                            None, self.ws, self.nb, stream=stream.cuda_stream)
        assert st == self.L.LBM_OK
        return steps


def _sleep_cycles(seconds):
    a, b = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
    a.record()
    torch.cuda._sleep(1_000_000)
    b.record()
    torch.cuda.synchronize()
    return int(1_000_000 * seconds * 1e3 / max(a.elapsed_time(b), 1e-3))


def test_a_solve_waits_for_its_own_stream_only(L):
    p = _Problem(L, 50, L.LBM_F32_SHIFTED, 1)
    other = torch.cuda.Stream()
    cycles = _sleep_cycles(0.5)
    streams = [torch.cuda.Stream() for _ in range(6)]
    for s in streams:
        p.solve(s)
    # a stream that does not share a hardware queue with the sleeping one
    x = torch.zeros(1, device="cuda")
    with torch.cuda.stream(other):
        torch.cuda._sleep(cycles)
    awake = torch.cuda.Event()
    awake.record(other)
    free = None
    for s in streams:
        with torch.cuda.stream(s):
            x += 1
        done = torch.cuda.Event()
        done.record(s)
        for _ in range(2000):
            if done.query() or awake.query():
                break
        if done.query() and not awake.query():
            free = s
            break
    torch.cuda.synchronize()
    if free is None:
        pytest.skip("every stream tried shares a hardware queue with the sleeping one")
    with torch.cuda.stream(other):
        torch.cuda._sleep(cycles)
    awake.record(other)
    p.solve(free)
    assert not awake.query()
    torch.cuda.synchronize()


def test_solves_in_several_threads(L):
    """Threads that solve at the same time on streams of their own find the
    fields and step counts of solves alone."""
    ps = [_Problem(L, n, dt, seed) for seed, (n, dt) in enumerate([(50, 0), (64, 0), (45, 1), (41, 1)])]
    alone = []
    for p in ps:
        steps = p.solve(torch.cuda.current_stream())
        alone.append((steps, p.u.clone()))
        p.u.zero_()
    torch.cuda.synchronize()
    got = [[] for _ in ps]

    def work(i):
        torch.cuda.set_device(0)
        s = torch.cuda.Stream()
        for _ in range(3):
            got[i].append((ps[i].solve(s), ps[i].u.clone()))
            s.synchronize()

    ts = [threading.Thread(target=work, args=(i,)) for i in range(len(ps))]
    for t in ts:
        t.start()
    for t in ts:
        t.join(60)
        assert not t.is_alive()
    torch.cuda.synchronize()
    for (steps, u), runs in zip(alone, got):
        assert len(runs) == 3
        for st, v in runs:
            assert st == steps and torch.equal(u, v)
