"""Field read-outs of a context on a stream of its own, against one on the null
stream, and (with two GPUs) of a context whose device is not the current one."""
import numpy as np
import pytest

from paper_1105_2904_amd import lbm


def _fields(device, stream, read_on):
    import torch
    with torch.cuda.device(device):
        sim = lbm.Simulation(9, 610, 400, tau=0.8, max_particles=1, max_radius=4.0, storage="fp64", device=device, stream=stream)
        sim.add_particles([[50.3, 40.1, 0.0]], u=[[0.05, 0.03, 0.0]], radius=4.0, mass=200.0, inertia=900.0)
        sim.step(30)
    with torch.cuda.device(read_on):
        out = list(sim.fields())
        assert torch.cuda.current_device() == torch.device(read_on).index
    sim.close()
    return out


@pytest.mark.gpu
def test_fields_on_a_stream_of_its_own():
    import torch
    a = _fields("cuda:0", None, "cuda:0")
    for x, y in zip(a, _fields("cuda:0", torch.cuda.Stream("cuda:0"), "cuda:0")):
        assert np.array_equal(x, y)
    assert np.abs(a[1]).max() > 1e-3


@pytest.mark.gpu
def test_fields_of_a_context_on_another_device():
    import torch
    if torch.cuda.device_count() < 2:
        pytest.skip("needs two GPUs")
    a = _fields("cuda:1", torch.cuda.Stream("cuda:1"), "cuda:1")
    for x, y in zip(a, _fields("cuda:1", torch.cuda.Stream("cuda:1"), "cuda:0")):
        assert np.array_equal(x, y)
