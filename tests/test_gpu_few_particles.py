"""Boxes of one to four particles, whose particle work runs in one workgroup
per box, against the separate kernels, bit for bit: the same box is stepped
alone and as the first box of an ensemble whose last box holds five particles
(which keeps the separate kernels for all of them).  With collisions, walls,
particles that share sites, shifts of every kind, both layouts, every storage,
the closure, empty boxes in between, balls on either side of the size up to
which the box is fused, and a fifth particle added between steps."""
import numpy as np
import pytest

from paper_1105_2904_amd import lbm
from paper_1105_2904_amd import workloads as wl

pytestmark = pytest.mark.gpu


def _cluster(dim, box, n, r, seed):
    """n balls in a tight cluster about the box's corner (or, with walls, its
    centre), moving into each other."""
    dirs = np.array([[0, 0, 0], [1, 0.1, 0], [0.2, 1, 0.1], [1.25, 1.2, 0.3]])[:n]
    if dim == 2:
        dirs[:, 2] = 0.0
    x = dirs * (2 * r + 0.6) + 0.37
    u = wl.seeded_velocities(n, dim, 0.03, seed)
    u[:, :dim] -= 0.04 * dirs[:, :dim]
    om = np.zeros((n, 3))
    om[:, 2] = 2e-3
    m, inertia = wl.solid_body(dim, np.full(n, r), 2.0)
    return x, u, om, np.full(n, r), m, inertia


def _five(dim, box):
    x = np.zeros((5, 3))
    x[:, 0] = 4.0 + 7.5 * np.arange(5)
    x[:, 1] = 6.0
    x[:, 2] = 0.0 if dim == 2 else 6.0
    m, inertia = wl.solid_body(dim, np.full(5, 2.0), 2.0)
    return x, np.zeros((5, 3)), np.zeros((5, 3)), np.full(5, 2.0), m, inertia


def _add(sim, p, box):
    sim.add_particles(p[0], u=p[1], omega=p[2], radius=p[3], mass=p[4], inertia=p[5], box=box)


def _run(q, dims, parts, closure, steps, **kw):
    n = sum(len(p[0]) for p in parts) + 8
    sim = lbm.Simulation(q, *dims[0], tau=0.8, gravity=(1e-5, -2e-5, 0), max_particles=n,
                         max_radius=max(p[3].max(initial=1.0) for p in parts), boxes=dims if len(dims) > 1 else None, **kw)
    for b, p in enumerate(parts):
        if len(p[0]):
            _add(sim, p, b)
    if closure is not None:
        sim.set_closure(closure, 2.0)
    out = []
    N0, n0 = int(sim.box_sites[0]), len(parts[0][0])
    for _ in range(3):
        sim.step(steps)
        out += [a[:n0] for a in sim.forces()] + [sim.shifts()[:n0], sim.site_kind().reshape(-1)[:N0]]
        out.append(sim.get_distributions().reshape(q, -1)[:, :N0])
    sim.close()
    return out


def _compare(q, box, p, closure=None, steps=13, **kw):
    dim = 2 if q == 9 else 3
    other = (45, 20, 1) if dim == 2 else (45, 20, 18)
    empty = _cluster(dim, box, 0, 3.0, 1)
    a = _run(q, [box], [p], closure, steps, **kw)
    b = _run(q, [box, (12, 11, 1) if dim == 2 else (12, 11, 10), other], [p, empty, _five(dim, other)], closure, steps, **kw)
    c = _run(q, [box, other], [p, empty], closure, steps, **kw)  # fused, an empty box beside it
    for k, (x, y, z) in enumerate(zip(a, b, c)):
        assert np.array_equal(x, y), k
        assert np.array_equal(x, z), k


@pytest.mark.parametrize("storage,aa", [("fp64", False), ("fp32", True), ("fp16", False), ("bf16", True)])
@pytest.mark.parametrize("n", [1, 2, 3, 4])
def test_2d(n, storage, aa):
    _compare(9, (64, 57, 1), _cluster(2, None, n, 5.3, 3), storage=storage, aa=aa)


@pytest.mark.parametrize("storage,aa", [("fp64", True), ("fp32", False), ("bf16", False)])
@pytest.mark.parametrize("n", [1, 2, 4])
def test_3d(n, storage, aa):
    _compare(19, (40, 37, 36), _cluster(3, None, n, 3.2, 4), storage=storage, aa=aa)


def test_walls():
    x, u, om, r, m, inertia = _cluster(2, None, 3, 4.0, 5)
    p = (x + 6.0, u - [0.02, 0.0, 0.0], om, r, m, inertia)
    _compare(9, (48, 50, 1), p, storage="fp64", walls=3)


@pytest.mark.parametrize("n", [2, 3, 4])
def test_closure(n):
    import torch
    params = torch.tensor(wl.mlp_init(5).astype(np.float32) + np.float32(0.05), device="cuda")
    _compare(9, (64, 57, 1), _cluster(2, None, n, 6.1, 6), closure=params, storage="fp32")


@pytest.mark.parametrize("q,box,n,r", [(9, (210, 205, 1), 2, 47.0), (9, (230, 215, 1), 2, 52.0), (9, (120, 110, 1), 4, 17.0),
                                       (19, (40, 41, 39), 1, 8.9), (19, (40, 41, 39), 1, 9.6), (19, (50, 41, 39), 3, 4.6)])
def test_either_side_of_the_size_limit(q, box, n, r):
    _compare(q, box, _cluster(2 if q == 9 else 3, None, n, r, 7), storage="fp64", steps=7)


def test_fifth_particle_added_between_steps():
    import oracle
    p = _cluster(2, None, 4, 4.0, 8)
    m, inertia = wl.solid_body(2, np.array([3.0]), 2.0)
    far = (np.array([[40.0, 30.0, 0.0]]), np.zeros((1, 3)), np.zeros((1, 3)), np.array([3.0]), m, inertia)
    kw = dict(gravity=(1e-5, -2e-5, 0))
    sim = lbm.Simulation(9, 64, 57, tau=0.8, max_particles=5, max_radius=4.0, storage="fp64", **kw)
    ora = oracle.Oracle(9, 64, 57, 1, 0.8, **kw)
    for q in (p, far):
        _add(sim, q, 0)
        ora.add_particles(q[0], u=q[1], omega=q[2], radius=q[3], mass=q[4], inertia=q[5])
        sim.step(18)
        ora.step(18)
        fo = ora.get_f()
        assert np.abs(sim.get_distributions() - fo).max() <= 1e-12 * np.abs(fo).max()
        assert np.array_equal(sim.shifts(), ora.shifts())
    sim.close()
