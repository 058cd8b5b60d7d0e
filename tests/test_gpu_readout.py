"""Read-outs through pinned blocks: fields in one and in several chunks (the
chunk is 233,016 sites) that end inside boxes of an ensemble, each of the
three arrays alone and in pairs, both population layouts, particle read-outs
with the context's pinned block and without (above 16,384 particles), and two
contexts read from two threads at once.  References: the moments of the
populations the library returns, and the oracle-checked site kinds."""
import ctypes
import threading

import numpy as np
import pytest

from paper_1105_2904_amd import lbm
from paper_1105_2904_amd import workloads as wl

pytestmark = pytest.mark.gpu

C9 = np.array([(0, 0), (1, 0), (0, 1), (-1, 0), (0, -1), (1, 1), (-1, 1), (-1, -1), (1, -1)], dtype=np.float64)


def _sim(dims, aa=False, capacity=None, **kw):
    parts = [wl.suspension(9, d, 3, 4.0, 1.5, seed=40 + b) for b, d in enumerate(dims)]
    sim = lbm.Simulation(9, *dims[0], tau=0.8, storage="fp64", max_particles=capacity or 3 * len(dims), max_radius=4.0,
                         boxes=dims if len(dims) > 1 else None, aa=aa, **kw)
    for b, p in enumerate(parts):
        sim.add_particles(p["x"], u=wl.seeded_velocities(3, 2, 0.03, 50 + b), radius=p["radius"], mass=p["mass"],
                          inertia=p["inertia"], box=b)
    sim.step(7)
    return sim


def _check(sim):
    rho, u, own = (a.reshape((sim.N,) + a.shape[a.ndim - 1:] if a.ndim > 1 and a.shape[-1] == 3 and a.size == 3 * sim.N
                             else (sim.N,)) for a in sim.fields())
    f = sim.get_distributions().reshape(9, sim.N)
    assert np.allclose(rho, f.sum(axis=0), rtol=1e-14, atol=0)
    j = np.einsum("ia,is->sa", C9, f)
    assert np.abs(u[:, :2] * rho[:, None] - j).max() <= 1e-15 * 9 and np.all(u[:, 2] == 0)
    kind = sim.site_kind().reshape(-1)
    assert np.array_equal(own >= 0, kind > 0) and own.max() == sim.n_particles - 1
    for b, (s0, n) in enumerate(zip(sim.box_start, sim.box_sites)):
        ids = np.unique(own[s0:s0 + n])
        assert set(ids) == {-1, 3 * b, 3 * b + 1, 3 * b + 2}
    # every subset of the arrays gives the same values
    P = lambda a: None if a is None else a.ctypes.data_as(lbm._dp if a.dtype == np.float64 else lbm._ip)
    for mask in range(1, 7):
        r = np.zeros(sim.N) if mask & 1 else None
        v = np.zeros((sim.N, 3)) if mask & 2 else None
        o = np.zeros(sim.N, dtype=np.int32) if mask & 4 else None
        assert lbm.lib().lbm_fields(sim.ctx, P(r), P(v), P(o)) == lbm.LBM_OK
        assert r is None or np.array_equal(r, rho)
        assert v is None or np.array_equal(v, u)
        assert o is None or np.array_equal(o, own)
    assert lbm.lib().lbm_fields(sim.ctx, None, None, None) == lbm.LBM_OK


@pytest.mark.parametrize("aa", [False, True])
@pytest.mark.parametrize("dims", [[(48, 40, 1)], [(365, 319, 1)], [(483, 482, 1)], [(484, 482, 1)], [(700, 801, 1)],
                                  [(61, 53, 1), (300, 301, 1), (200, 190, 1), (400, 400, 1)]])
def test_fields_chunks(dims, aa):
    sim = _sim(dims, aa)
    _check(sim)
    sim.close()


def test_one_site_and_no_particles():
    for aa in (False, True):
        sim = lbm.Simulation(9, 1, 1, 1, tau=0.8, storage="fp64", aa=aa)
        sim.step(3)
        rho, u, own = sim.fields()
        assert rho.ravel().tolist() == [1.0] and not u.any() and own.ravel().tolist() == [-1]
        assert all(a.shape == (0, 3) for a in sim.forces())
        sim.close()


def test_particle_readouts_with_and_without_the_pinned_block():
    a, b = _sim([(64, 56, 1)]), _sim([(64, 56, 1)], capacity=16385)
    for x, y in zip(a.forces(), b.forces()):
        assert x.shape == (3, 3) and x.any() and np.array_equal(x, y)
    buf = np.full((3, 3), 7.0)
    assert lbm.lib().lbm_forces(a.ctx, None, None, ctypes.cast(buf.ctypes.data, lbm._dp), None, None) == lbm.LBM_OK
    assert np.array_equal(buf, b.forces()[2])
    a.close()
    b.close()


def test_two_threads_read_two_contexts():
    import torch
    sims = [_sim([(400, 399, 1)], stream=torch.cuda.Stream()) for _ in range(2)]
    want = [(s.fields(), s.forces()) for s in sims]
    got = [None, None]

    def read(k):
        got[k] = [(sims[k].fields(), sims[k].forces()) for _ in range(5)]

    ts = [threading.Thread(target=read, args=(k,)) for k in range(2)]
    for t in ts:
        t.start()
    for t in ts:
        t.join()
    for k in range(2):
        for fields, forces in got[k]:
            assert all(np.array_equal(x, y) for x, y in zip(fields, want[k][0]))
            assert all(np.array_equal(x, y) for x, y in zip(forces, want[k][1]))
        sims[k].close()
