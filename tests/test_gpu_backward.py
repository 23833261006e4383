"""GPU: the surrogate's backward pass at the edges of its work split.

One workgroup takes a patch, at most 256 workgroups run, and a workgroup with
several patches goes on from the sums of its earlier ones.
"""
import numpy as np
import pytest

from oracle import cnn_oracle as C
from test_gpu_surrogate import NAMES, _flat, _params, _patches, _unflat

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")


@pytest.fixture(scope="module")
def L():
    from paper_1312_0195_amd import lbm
    assert torch.cuda.is_available(), "GPU tests need a GPU"
    lbm.lib()
    return lbm


def _gradients(L, prm, x, sym, t):
    n = len(x)
    grad = torch.empty_like(prm)
    loss = torch.empty(1, dtype=torch.float32, device="cuda")
    pred = torch.empty((n, 2), dtype=torch.float32, device="cuda")
    nb = L.lbm_cnn_workspace_bytes(n, True)
    ws = torch.empty(nb, dtype=torch.uint8, device="cuda")
    L.lbm_cnn_gradients(prm, n, x, sym, t, grad, loss, pred, ws, nb)
    torch.cuda.synchronize()
    return grad.cpu().numpy().astype(np.float64), float(loss.item())


def test_two_patches_match_oracle(L):
    """BF16 roundings of 2^-9 in four layers forward and three back: about 1%
    of a gradient tensor, within the 3e-2 the larger batches are held to."""
    p = _params(11)
    x = _patches(2, 12)
    t = x.mean(axis=(1, 2))[:, None] + np.array([[0.4, -0.3], [0.7, 0.2]])
    sym = np.array([5, 0], np.int8)
    xo = np.stack([C.transform(x[i:i + 1], int(sym[i]))[0] for i in range(2)])
    to = np.where((sym & 1)[:, None] == 1, t[:, ::-1], t)
    y, cache = C.forward(p, xo)
    ref = C.backward(p, cache, y, to - cache["m"][:, None])
    prm = torch.tensor(_flat(p), device="cuda")
    g, _ = _gradients(L, prm, torch.tensor(x.astype(np.float32), device="cuda"), torch.tensor(sym, device="cuda"),
                      torch.tensor(t.astype(np.float32), device="cuda"))
    got = _unflat(g, p)
    for k in NAMES:
        rel = np.linalg.norm(got[k] - ref[k]) / (np.linalg.norm(ref[k]) + 1e-300)
        assert rel < 3e-2, (k, rel)


@pytest.mark.parametrize("n", [1, 129, 256, 300])
def test_repeated_batch_has_the_same_gradients(L, n):
    """A batch taken twice: every patch's gradient is exactly half of the
    single batch's (the factor 1 / batch is a power of two smaller, BF16 keeps
    it), so the sums agree up to FP32 summation order: at most 1024 products
    per pixel sum and 2 patches per workgroup, 2^-24 sqrt(2048) = 3e-6 of the
    norm."""
    prm = torch.tensor(_flat(_params(13)), device="cuda")
    x = torch.tensor(_patches(n, 14).astype(np.float32), device="cuda")
    t = x.mean((1, 2))[:, None].repeat(1, 2).contiguous() + 0.3
    sym = (torch.arange(n, device="cuda") % 8).to(torch.int8)
    g1, l1 = _gradients(L, prm, x, sym, t)
    g2, l2 = _gradients(L, prm, x.repeat(2, 1, 1).contiguous(), sym.repeat(2).contiguous(),
                        t.repeat(2, 1).contiguous())
    assert abs(l1 - l2) <= 3e-6 * l1
    for k, (a, b) in {k: (_unflat(g1, _params(13))[k], _unflat(g2, _params(13))[k]) for k in NAMES}.items():
        assert np.linalg.norm(a - b) <= 1e-5 * np.linalg.norm(a), k
