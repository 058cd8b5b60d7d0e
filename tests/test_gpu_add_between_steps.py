"""Particles added to a later box of an ensemble after steps in which two
particles of an earlier box, further apart than any sharing list reaches when
they were added, have come to share sites: every box against its own FP64
oracle after every following step.  The earlier box holds two particles (its
particle work in one workgroup), five (separate kernels), or is stepped
without the workspace's scratch."""
import numpy as np
import pytest

import oracle
from paper_1105_2904_amd import lbm

pytestmark = pytest.mark.gpu


def _approaching(dim, r, extra):
    """Two kinematic balls 5.2 apart that close in at 0.1 a step (after 72 steps
    their site sets overlap by three rows), and `extra` more far from them."""
    x = np.zeros((2 + extra, 3))
    x[:, 1:dim] = 14.1
    x[0, 0] = 8.3
    x[1, 0] = 8.3 + 2 * r + 5.2
    for k in range(extra):
        x[2 + k, :2] = 8.0 + 11.0 * k, 31.0
    u = np.zeros_like(x)
    u[0, 0], u[1, 0] = 0.05, -0.05
    return x, u


@pytest.mark.parametrize("way", ["few", "separate", "noalloc", "noalloc-separate"])
@pytest.mark.parametrize("q", [9, 19])
def test_add_to_a_later_box(q, way):
    dim = 2 if q == 9 else 3
    r = 4.6
    nz = 1 if dim == 2 else 26
    dims = [(44, 42, nz), (30, 28, nz), (26, 27, nz)]
    x, u = _approaching(dim, r, 3 if "separate" in way else 0)
    g = (0.0, -1e-4, 0.0)
    sim = lbm.Simulation(q, 1, 1, 1, tau=0.8, gravity=g, storage="fp64", max_particles=len(x) + 2, max_radius=r, boxes=dims)
    oras = [oracle.Oracle(q, *d, 0.8, gravity=g) for d in dims]
    count = [0, 0, 0]

    def add(box, x, u):
        kw = dict(u=u, radius=np.full(len(x), r), mass=np.full(len(x), np.inf), inertia=np.full(len(x), np.inf))
        sim.add_particles(x, box=box, **kw)
        oras[box].add_particles(x, **kw)
        count[box] += len(x)

    def step(n):
        (sim.step_noalloc if way.startswith("noalloc") else sim.step)(n)
        for o in oras:
            o.step(n)

    def compare(label):
        f, kind, k, F = sim.get_distributions(), sim.site_kind(), sim.shifts(), sim.forces()[0]
        p0 = 0
        for b, o in enumerate(oras):
            s0, N = int(sim.box_start[b]), int(sim.box_sites[b])
            fo = o.get_f().reshape(q, -1)
            assert np.array_equal(kind[s0:s0 + N], o.site_kind().ravel()), (label, b)
            assert np.abs(f[:, s0:s0 + N] - fo).max() <= 1e-12 * np.abs(fo).max(), (label, b)
            n = count[b]
            if n:
                Fo = o.forces()[0]
                assert np.array_equal(k[p0:p0 + n], o.shifts()), (label, b)
                e = np.linalg.norm(F[p0:p0 + n] - Fo, axis=1).max()
                assert e <= 1e-12 * max(np.linalg.norm(Fo, axis=1).max(), 1e-30), (label, b, e)
            p0 += n

    add(0, x, u)
    step(72)
    one = np.array([[12.2, 13.4, 0.0 if dim == 2 else 12.6]])
    for box in (1, 2):
        add(box, one, np.zeros((1, 3)))
        for t in range(7):
            step(1)
            compare((q, way, box, t))
    sim.close()
