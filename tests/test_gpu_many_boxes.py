"""Ensembles on either side of the number of boxes up to which small balls' particle
work runs in one workgroup per box, and of balls large enough to keep that beyond
it: the first and the last box against the same box stepped alone, bit for bit."""
import numpy as np
import pytest

from paper_1105_2904_amd import lbm
from paper_1105_2904_amd import workloads as wl

pytestmark = pytest.mark.gpu


def _run(q, box, boxes, n, r):
    dim = 2 if q == 9 else 3
    k = np.arange(n)
    x = np.stack([1.0 + (k % 2) * (2 * r + 1.2), 1.3 + (k // 2) * (2 * r + 1.2), np.full(n, 2.0 if dim == 3 else 0.0)], axis=1)
    u = wl.seeded_velocities(n, dim, 0.08, 3)
    m, inertia = wl.solid_body(dim, np.full(n, r), 2.0)
    sim = lbm.Simulation(q, 1, 1, 1, tau=0.8, gravity=(1e-4, 0, 0), max_particles=n * boxes, max_radius=r, boxes=[box] * boxes)
    for b in range(boxes):
        sim.add_particles(x, u=u, radius=np.full(n, r), mass=m, inertia=inertia, box=b)
    sim.step(30)
    N, f, kind = int(np.prod(box)), sim.get_distributions().reshape(q, -1), sim.site_kind().reshape(-1)
    arrays = list(sim.forces()) + [sim.shifts()]
    sim.close()
    return [[f[:, s], kind[s]] + [a[p] for a in arrays]
            for s, p in ((slice(0, N), slice(0, n)), (slice(N * (boxes - 1), N * boxes), slice(n * (boxes - 1), n * boxes)))]


@pytest.mark.parametrize("q,box,n,r,counts", [(9, (15, 14, 1), 1, 2.2, (1024, 1025)), (9, (16, 14, 1), 2, 2.2, (512, 513)),
                                              (9, (16, 17, 1), 3, 2.2, (256, 257)), (9, (16, 17, 1), 4, 2.2, (256, 257)),
                                              (19, (14, 13, 12), 1, 1.9, (1024, 1025)), (9, (55, 38, 1), 2, 12.3, (513,))])
def test_boxes_of_a_large_ensemble(q, box, n, r, counts):
    alone = _run(q, box, 1, n, r)[0]
    for boxes in counts:
        for k, one in enumerate(_run(q, box, boxes, n, r)):
            for j, (a, b) in enumerate(zip(alone, one)):
                assert np.array_equal(a, b), (boxes, k, j)
