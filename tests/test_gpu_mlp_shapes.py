"""The closure network's gradient and training kernels at the edges of their
tiling: a pass is 4 to 16 tiles of 16 rows, a gradient spreads its passes over
up to 256 workgroups (65,536 rows) and then loops, a training batch is one pass
up to 256 rows and several above.

Gates: those of test_gpu_mlp.py against the oracle at the same FP16 rounding
points (2e-3 relative in L2 norm for gradients, 1e-4 for the loss); Adam's
own arithmetic to a few FP32 roundings.
"""
import ctypes

import numpy as np
import pytest

from oracle import mlp as omlp
from paper_1105_2904_amd import lbm
from paper_1105_2904_amd import workloads as wl


def _params(seed):
    rng = np.random.Generator(np.random.PCG64(seed + 100))
    b = omlp.unpack(wl.mlp_init(seed))
    b["b1"], b["b2"], b["b3"] = rng.uniform(-0.3, 0.3, 64), rng.uniform(-0.3, 0.3, 64), rng.uniform(-0.1, 0.1, 2)
    return omlp.pack(b).astype(np.float32).astype(np.float64)


def _data(n, seed):
    rng = np.random.Generator(np.random.PCG64(seed))
    X = rng.uniform(-1.5, 1.5, size=(n, 8)).astype(np.float32).astype(np.float64)
    T = np.stack([np.sin(X[:, 0] * X[:, 1]) + 0.3 * X[:, 2], np.tanh(X[:, 3] - X[:, 4] * X[:, 5])], axis=1)
    return X, T.astype(np.float32).astype(np.float64)


def _t(a):
    import torch
    return torch.tensor(np.asarray(a, dtype=np.float32), device="cuda").contiguous()


def _close(a, b, tol):
    return np.linalg.norm(a - b) <= tol * np.linalg.norm(b)


@pytest.mark.gpu
@pytest.mark.parametrize("n", [1, 15, 16, 255, 256, 257, 4101, 15360, 15361, 30721, 46081, 65536, 65537, 70003])
def test_gradient_of_every_split(n):
    theta = _params(3)
    X, T = _data(n, 4)
    lo, go = omlp.loss_and_grad(theta, X, T, quantize=True, scale=1024.0)
    loss, g = lbm.mlp_gradient(_t(theta), _t(X), _t(T))
    assert abs(float(loss.item()) - lo) <= 1e-4 * lo
    assert _close(g.cpu().numpy().astype(np.float64), go, 2e-3)
    again = lbm.mlp_gradient(_t(theta), _t(X), _t(T))
    assert np.array_equal(again[1].cpu().numpy(), g.cpu().numpy())  # sums in a fixed order
    # the C entry without a workspace runs the same rows on one workgroup
    p, x, t = _t(theta), _t(X), _t(T)
    g1, l1 = _t(np.zeros(theta.size)), _t(np.zeros(1))
    vp = ctypes.c_void_p
    assert lbm.lib().lbm_mlp_gradient(vp(p.data_ptr()), vp(x.data_ptr()), vp(t.data_ptr()), n, 1024.0,
                                      vp(g1.data_ptr()), vp(l1.data_ptr()), lbm._stream(None)) == lbm.LBM_OK
    assert _close(g1.cpu().numpy().astype(np.float64), go, 2e-3) and abs(float(l1.item()) - lo) <= 1e-4 * lo


@pytest.mark.gpu
@pytest.mark.parametrize("n,batch,step0", [(1000, 64, 0), (100, 192, 3), (5000, 256, 7), (777, 320, 2), (5000, 1024, 1),
                                           (13, 512, 10 ** 6)])
def test_training_steps(n, batch, step0):
    import torch
    theta = _params(5)
    X, T = _data(n, 6)
    p, m, v = _t(theta), _t(np.zeros(theta.size)), _t(np.zeros(theta.size))
    steps, lr = 3, 1e-9  # the weights stand still: the moments follow the oracle's gradients
    losses = lbm.mlp_train(p, m, v, _t(X), _t(T), batch=batch, steps=steps, step0=step0, lr=lr).cpu().numpy()
    mo, vo = np.zeros(theta.size), np.zeros(theta.size)
    for s in range(steps):
        rows = ((step0 + s) * batch + np.arange(batch)) % n
        lo, go = omlp.loss_and_grad(theta, X[rows], T[rows], quantize=True, scale=1024.0)
        assert abs(losses[s] - lo) <= 1e-4 * lo
        mo, vo = 0.9 * mo + 0.1 * go, 0.999 * vo + 0.001 * go * go
    assert _close(m.cpu().numpy().astype(np.float64), mo, 2e-3)
    assert _close(v.cpu().numpy().astype(np.float64), vo, 4e-3)
    # one more step from these moments: the update itself, from the moments it leaves
    p0 = p.cpu().numpy().astype(np.float64)
    lbm.mlp_train(p, m, v, _t(X), _t(T), batch=batch, steps=1, step0=step0 + steps, lr=1e-2)
    torch.cuda.synchronize()
    m64, v64, t = m.cpu().numpy().astype(np.float64), v.cpu().numpy().astype(np.float64), step0 + steps + 1
    # the kernel's constants are FP32: 1 - 0.9^t, 1 - 0.999^t carry an absolute error of about 2^-23
    c1, c2 = 1.0 - 0.9 ** t, 1.0 - 0.999 ** t
    step = 1e-2 * (m64 / c1) / (np.sqrt(v64 / c2) + 1e-8)
    tol = 2.0 ** -24 * np.abs(p0) + np.abs(step) * (8 * 2.0 ** -24 + 2.0 ** -22 / c1 + 2.0 ** -22 / c2)
    assert np.all(np.abs(p.cpu().numpy() - (p0 - step)) <= tol)


@pytest.mark.gpu
@pytest.mark.parametrize("n", [5, 16, 33, 70003, (1 << 21) + 5])
def test_forward_rows_are_independent(n):
    """Every split of the rows over workgroups gives a row the same value."""
    import torch
    g = torch.Generator(device="cuda").manual_seed(n)
    x = 3.0 * torch.rand((n, 8), device="cuda", generator=g) - 1.5
    p = _t(_params(9))
    y = lbm.mlp_forward(p, x)
    parts = torch.cat([lbm.mlp_forward(p, c.contiguous()) for c in x.split(37 if n < 100 else 30011)])
    assert torch.equal(y, parts)
    yo, _ = omlp.forward(_params(9), x[-20:].cpu().numpy().astype(np.float64), quantize=True)
    assert np.abs(y[-20:].cpu().numpy() - yo).max() <= 2e-3 * max(1.0, np.abs(yo).max())


def test_gradient_workspace_is_checked_on_the_host():
    need = ctypes.c_size_t(1)
    fn, vp = lbm.lib().lbm_mlp_gradient_in, ctypes.c_void_p
    for n, some in ((1, False), (256, False), (257, True), (2 ** 31 - 1, True)):
        assert lbm.lib().lbm_mlp_gradient_work_size(n, ctypes.byref(need)) == lbm.LBM_OK
        assert (need.value > 0) == some and need.value <= 256 * 4 * 4868
    assert lbm.lib().lbm_mlp_gradient_work_size(0, ctypes.byref(need)) == lbm.LBM_EINVAL
    ptr = vp(4096)  # refused before any use
    assert fn(ptr, ptr, ptr, 257, 1.0, ptr, ptr, None, 1 << 30, None) == lbm.LBM_EWORKSPACE
    assert fn(ptr, ptr, ptr, 257, 1.0, ptr, ptr, ptr, 16, None) == lbm.LBM_EWORKSPACE
    assert fn(ptr, ptr, ptr, 257, 1.0, ptr, ptr, vp(4098), 1 << 30, None) == lbm.LBM_EWORKSPACE
    assert fn(ptr, ptr, ptr, 0, 1.0, ptr, ptr, ptr, 1 << 30, None) == lbm.LBM_EINVAL
    assert fn(ptr, ptr, ptr, 16, 0.0, ptr, ptr, ptr, 1 << 30, None) == lbm.LBM_EINVAL
