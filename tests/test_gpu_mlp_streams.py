"""The stream argument of the closure network's calls: a torch stream, or any object
with a cuda_stream handle (the null stream's among them), gives what the current
stream gives."""
import numpy as np
import pytest

from paper_1105_2904_amd import lbm
from paper_1105_2904_amd import workloads as wl


class Handle:
    def __init__(self, cuda_stream):
        self.cuda_stream = cuda_stream


@pytest.mark.gpu
@pytest.mark.parametrize("n", [100, 5000])
def test_any_object_with_a_handle(n):
    import torch
    rng = np.random.Generator(np.random.PCG64(n))
    p = torch.tensor(wl.mlp_init(3).astype(np.float32), device="cuda")
    x = torch.tensor(rng.uniform(-1, 1, size=(n, 8)).astype(np.float32), device="cuda")
    t = torch.tensor(rng.uniform(-1, 1, size=(n, 2)).astype(np.float32), device="cuda")

    def calls(stream):
        y = lbm.mlp_forward(p, x, stream=stream)
        loss, g = lbm.mlp_gradient(p, x, t, stream=stream)
        q, m, v = p.clone(), torch.zeros_like(p), torch.zeros_like(p)
        torch.cuda.synchronize()
        losses = lbm.mlp_train(q, m, v, x, t, batch=64, steps=3, stream=stream)
        torch.cuda.synchronize()
        return [a.cpu().numpy() for a in (y, loss, g, q, m, v, losses)]

    torch.cuda.synchronize()
    ref = calls(None)
    side = torch.cuda.Stream()
    for stream in (side, Handle(side.cuda_stream), Handle(0)):
        for a, b in zip(ref, calls(stream)):
            assert np.array_equal(a, b)
