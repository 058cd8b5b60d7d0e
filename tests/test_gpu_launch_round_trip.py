"""A sweep launch read from one context and set in another runs as it did: the
default launch, whose cap on large 3D boxes is the library's own, is the same
launch again when (0, 0, 0) is given back."""
import pytest

from paper_1105_2904_amd import lbm


@pytest.mark.gpu
def test_default_launch_given_back_keeps_its_time():
    """256^3 FP32 with a sphere, the fastest of 6 alternating runs of 20 steps each;
    without the default's cap a step takes 7 % longer, the runs of one side differ by
    under 1."""
    import torch
    sims = [lbm.Simulation(19, 256, 256, 256, tau=0.7, storage="fp32", max_particles=1, max_radius=6.0) for _ in range(2)]
    for sim in sims:
        sim.add_particles([[40.0, 50.0, 60.0]], radius=6.0, mass=float("inf"), inertia=float("inf"))
    sims[1].set_sweep_config(*sims[0].sweep_config())
    best = [1e9, 1e9]
    for sim in sims:
        sim.step(10)
    for _ in range(6):
        for k, sim in enumerate(sims):
            a, b = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
            a.record()
            sim.step(20)
            b.record()
            b.synchronize()
            best[k] = min(best[k], a.elapsed_time(b) / 20)
    print("ms per step: default %.4f, given back %.4f" % tuple(best), flush=True)
    assert sims[1].sweep_config() == (0, 0, 0)
    for sim in sims:
        sim.close()
    assert best[1] <= 1.035 * best[0]
