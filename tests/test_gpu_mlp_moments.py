"""One Adam step from moments at and past the ends of the FP32 range, against the
same step in plain torch FP32: an infinite second moment leaves a finite weight
where it is, an infinite first moment does not."""
import numpy as np
import pytest

from paper_1105_2904_amd import lbm
from paper_1105_2904_amd import workloads as wl

INF = float("inf")
CASES = [(0.5, INF), (-3.0, INF), (0.0, INF), (INF, 1.0), (-INF, 4.0), (INF, INF), (2.0, 1e36), (-1e30, 3e38),
         (3e38, 1.0), (1e37, 1e30), (float("nan"), 1.0), (1.0, float("nan")), (1e-30, 1e-30), (1e-44, 1e-44), (0.0, 0.0)]


@pytest.mark.gpu
@pytest.mark.parametrize("batch,step0", [(64, 0), (512, 3)])
def test_moments_past_the_range(batch, step0):
    import torch
    rng = np.random.Generator(np.random.PCG64(4))
    x = torch.tensor(rng.uniform(-1, 1, size=(batch, 8)).astype(np.float32), device="cuda")
    t = torch.tensor(rng.uniform(-1, 1, size=(batch, 2)).astype(np.float32), device="cuda")
    p0 = torch.tensor(wl.mlp_init(2).astype(np.float32) + np.float32(0.01))
    n = p0.numel()
    k = torch.arange(n) % len(CASES)
    c = torch.tensor(CASES, dtype=torch.float32)
    m0, v0 = c[k, 0].clone(), c[k, 1].clone()
    g = lbm.mlp_gradient(p0.cuda(), x, t)[1].cpu()
    p, m, v = p0.cuda(), m0.cuda(), v0.cuda()
    lbm.mlp_train(p, m, v, x, t, batch=batch, steps=1, step0=step0, lr=1e-2)
    c1 = torch.tensor(1.0 - 0.9 ** (step0 + 1), dtype=torch.float32)
    c2 = torch.tensor(1.0 - 0.999 ** (step0 + 1), dtype=torch.float32)
    m1 = 0.9 * m0 + 0.1 * g
    v1 = 0.999 * v0 + 0.001 * g * g
    u = 1e-2 * (m1 / c1) / (torch.sqrt(v1 / c2) + 1e-8)
    ref, got = p0 - u, p.cpu()
    # which values are finite is exact; the step itself to the error of c2 (an
    # FP32 1 - 0.999^t: 2^-24 of 0.001) and of the gradient's own sum order
    for want, have in ((ref, got), (m1, m.cpu()), (v1, v.cpu())):
        assert torch.equal(torch.isnan(want), torch.isnan(have))
        assert torch.equal(torch.isinf(want), torch.isinf(have)) and torch.equal(want[torch.isinf(want)], have[torch.isinf(have)])
    ok = torch.isfinite(ref)
    assert bool((torch.abs(got - ref)[ok] <= 2.0 ** -23 * torch.abs(p0)[ok] + 2e-3 * torch.abs(u)[ok]).all())
    inf = ok & torch.isinf(v0)
    assert int(inf.sum()) > 900 and torch.equal(got[inf], p0[inf])
