"""The one-box sweep (width 0) at the edges of its rules against the tile
kernel, bit for bit: boxes below and above the size at which workgroups grow
from 64 to 256 sites, rows that are whole cache lines or not (streaming or
cached loads, neighbours grouped per XCD), rows that 16-bit storage takes with
two sites per lane or with one, a last workgroup that is nearly empty, walls,
a sphere across the seams, and both layouts of the population array."""
import numpy as np
import pytest

from paper_1105_2904_amd import lbm
from paper_1105_2904_amd import workloads as wl

BOXES = [(9, (1, 5, 1)), (9, (3, 7, 1)), (9, (64, 511, 1)), (9, (64, 512, 1)), (9, (65, 505, 1)), (9, (127, 300, 1)),
         (19, (31, 33, 32)), (19, (33, 32, 32)), (19, (64, 24, 24)), (19, (96, 19, 21)), (19, (100, 20, 17)),
         (19, (128, 17, 16)), (19, (192, 14, 13)), (19, (320, 12, 11))]


def _run(q, box, storage, aa, walls, shape, f0):
    r = 3.4
    fits = all(n >= (17 if walls else 2 * 4 + 3) for n in box[:2 if q == 9 else 3])
    sim = lbm.Simulation(q, *box, tau=0.7, body_force=(2e-6, -1e-6, 0.0), storage=storage, max_particles=1, max_radius=r,
                         walls=walls, aa=aa)
    sim.set_distributions(f0)
    if fits:
        dim = 2 if q == 9 else 3
        m, inertia = wl.solid_body(dim, np.array([r]), 3.0)
        x = [[box[0] / 2.0 + 0.3, box[1] / 2.0, box[2] / 2.0]] if walls else [[box[0] - 0.4, 0.3, box[2] - 1.0]]
        sim.add_particles(x, u=[[0.05, 0.03, 0.04 if dim == 3 else 0.0]], radius=r, mass=m, inertia=inertia)
    sim.set_sweep_config(*shape)
    sim.step(24)
    out = [sim.get_distributions()] + list(sim.forces()) + [sim.shifts()]
    sim.close()
    return out


@pytest.mark.gpu
@pytest.mark.parametrize("aa", [False, True])
@pytest.mark.parametrize("storage", ["fp64", "fp32", "fp16", "bf16"])
@pytest.mark.parametrize("q,box", BOXES)
def test_one_box_sweep_equals_tiles(q, box, storage, aa):
    w = [4 / 9] + [1 / 9] * 4 + [1 / 36] * 4 if q == 9 else [1 / 3] + [1 / 18] * 6 + [1 / 36] * 12
    f0 = wl.random_populations(w, (box[2], box[1], box[0]), 5, 0.01)
    for walls in (0, 3) if min(box[:2]) >= 17 else (0,):
        a = _run(q, box, storage, aa, walls, (0, 0, 0), f0)
        for shape in ((64, 0, 0), (256, 8, 4)):
            b = _run(q, box, storage, aa, walls, shape, f0)
            for x, y in zip(a, b):
                assert np.array_equal(x, y), (q, box, storage, aa, walls, shape)


@pytest.mark.gpu
@pytest.mark.parametrize("aa", [False, True])
@pytest.mark.parametrize("storage,box", [("fp32", (32, 32, 32)), ("fp32", (31, 33, 32)), ("fp32", (45, 47, 49)),
                                         ("fp64", (74, 73, 74)), ("fp64", (75, 73, 74))])
def test_launch_never_set_equals_a_set_one(storage, box, aa):
    """The cap that a context picks by itself (below and above the sizes where
    it does) changes no value and no reported shape, also where a shape is set
    after a step graph was captured."""
    w = [1 / 3] + [1 / 18] * 6 + [1 / 36] * 12
    f0 = wl.random_populations(w, (box[2], box[1], box[0]), 6, 0.01)
    m, inertia = wl.solid_body(3, np.array([3.4]), 3.0)
    out = []
    for shapes in ((None, None), ((0, 0, 0), (0, 0, 0)), (None, (0, 0, 0)), (None, (0, 0, 5))):
        sim = lbm.Simulation(19, *box, tau=0.7, storage=storage, max_particles=1, max_radius=3.4, aa=aa)
        sim.set_distributions(f0)
        sim.add_particles([[box[0] - 0.4, 0.3, 5.0]], u=[[0.05, 0.03, 0.04]], radius=3.4, mass=m, inertia=inertia)
        sim.set_graph(2)
        for shape in shapes:
            if shape is None:
                assert sim.sweep_config() == (0, 0, 0)
            else:
                sim.set_sweep_config(*shape)
            sim.step(5)
        out.append([sim.get_distributions()] + list(sim.forces()))
        sim.close()
    for o in out[1:]:
        for x, y in zip(out[0], o):
            assert np.array_equal(x, y), (storage, box, aa)


@pytest.mark.gpu
@pytest.mark.parametrize("box", [(483, 483, 483), (484, 484, 485)])
def test_push_sweep_on_both_sides_of_4_gib(box):
    """BF16 in one array of just below and just above 4 GiB (32-bit offsets,
    64-bit addresses) against the tile kernel: spheres at both ends of the
    array, whose forces and motion depend on every population around them."""
    m, inertia = wl.solid_body(3, np.array([3.4] * 3), 3.0)
    out = []
    for shape in ((0, 0, 0), (256, 0, 0)):
        sim = lbm.Simulation(19, *box, tau=0.7, storage="bf16", max_particles=3, max_radius=3.4, aa=True)
        sim.add_particles([[0.3, 0.2, box[2] - 0.6], [box[0] - 8.2, box[1] - 7.9, box[2] - 9.1], [11.0, 12.0, 10.5]],
                          u=[[0.05, 0.03, 0.04], [-0.04, 0.05, 0.03], [0.03, -0.05, 0.04]], radius=[3.4] * 3, mass=m,
                          inertia=inertia)
        sim.set_sweep_config(*shape)
        sim.step(8)
        out.append(list(sim.forces()) + [sim.shifts()])
        sim.close()
    assert np.abs(out[0][0]).max() > 1e-6
    for x, y in zip(*out):
        assert np.array_equal(x, y), box


def test_division_by_multiplication_is_exact():
    """n / d as (n ceil(2^sh / d)) >> sh, sh = 31 + ceil(log2 d), for
    0 <= n < 2^31: the multiplier fits 32 bits and the quotient is exact."""
    rng = np.random.Generator(np.random.PCG64(1))
    ds = [1, 2, 3, 5, 7, 63, 64, 65, 100, 191, 255, 256, 257, 1001, 65535, 65537, 2 ** 30 - 1, 2 ** 30, 2 ** 31 - 1]
    for d in ds + [int(v) for v in rng.integers(1, 2 ** 31, size=300)]:
        sh = 31 + (d - 1).bit_length()
        m = -(-(1 << sh) // d)
        assert m < 2 ** 32
        ns = {0, 1, d - 1, d, d + 1, 2 ** 31 - 1, 2 ** 31 - 2, (2 ** 31 - 1) // d * d, (2 ** 31 - 1) // d * d - 1}
        for n in list(ns) + [int(v) for v in rng.integers(0, 2 ** 31, size=50)]:
            if 0 <= n < 2 ** 31:
                assert (n * m) >> sh == n // d, (n, d)
