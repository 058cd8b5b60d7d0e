"""What forces() returns: five arrays that own their memory, so that keeping one of
them keeps no other, and that later read-outs leave alone."""
import numpy as np
import pytest

from paper_1105_2904_amd import lbm
from paper_1105_2904_amd import workloads as wl


@pytest.mark.gpu
@pytest.mark.parametrize("n", [0, 1, 3])
def test_arrays_of_their_own(n):
    p = wl.suspension(9, (64, 48, 1), max(n, 1), 4.0, 1.5, seed=5)
    sim = lbm.Simulation(9, 64, 48, tau=0.8, gravity=(0, -1e-4, 0), max_particles=4, max_radius=4.0)
    if n:
        sim.add_particles(p["x"], u=wl.seeded_velocities(n, 2, 0.02, 3), radius=p["radius"], mass=p["mass"], inertia=p["inertia"])
    sim.step(3)
    out = sim.forces()
    kept = [a.copy() for a in out]
    sim.step(5)
    again = sim.forces()
    for a, b, c in zip(out, kept, again):
        assert a.shape == (n, 3) and a.dtype == np.float64 and a.base is None and a.flags.writeable and a.flags.c_contiguous
        assert np.array_equal(a, b)
    assert n == 0 or not np.array_equal(out[2], again[2])
    sim.close()
