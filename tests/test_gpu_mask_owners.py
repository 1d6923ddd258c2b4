"""Solid masks of spheres that share nodes or differ in size, after creation, steps and
pushes, exactly as the FP64 oracle has them: nodes that pass from one sphere to another
(the lowest index that holds a node owns it) in both directions, a large sphere beside and
among small ones, more spheres meeting one than the search lists, and boxes on both sides
of the number of particles from which nodes are claimed in memory."""
import numpy as np
import pytest

from oracle.oracle import OracleSim
from paper_2505_10171_amd import workloads as W

pytestmark = pytest.mark.gpu


def _pair(cfg, parts):
    from paper_2505_10171_amd.lbm import Simulation
    return Simulation(cfg, None, parts), OracleSim(cfg, None, parts)


def _same(g, o, label):
    mg, mo = g.phi_mask()[1], o.fields()[3]
    assert np.array_equal(mg, mo), (label, int((mg != mo).sum()), np.argwhere(mg != mo)[:5])
    return mo


def _push(g, o, parts, moves):
    parts = [dict(p, x=tuple(np.array(p["x"]) + m)) for p, m in zip(parts, moves)]
    g.push_particles(parts)
    o.set_particles(parts)
    return parts


@pytest.mark.parametrize("order", [(0, 1, 2), (2, 1, 0), (1, 2, 0)])
def test_overlapping_spheres_change_owners(order):
    """Three spheres through each other and through the periodic boundary; a pushed
    one lands inside another, and leaves it again."""
    cfg = W.config(36, 30, 28, has_wall=0, sigma=0.0)
    ps = [W.particle((16.1, 14.2, 13.7), 4.0, v=(0.08, 0.02, 0.0), kinematic=1),
          W.particle((20.3, 15.4, 14.1), 3.0, v=(-0.07, 0.0, 0.05), kinematic=1),
          W.particle((34.6, 2.3, 26.4), 3.5, v=(0.05, -0.06, 0.08), kinematic=1)]
    ps = [ps[k] for k in order]
    g, o = _pair(cfg, ps)
    m0 = _same(g, o, "created")
    seen = [m0]
    for k in range(4):
        g.step(5)
        o.step(5)
        seen.append(_same(g, o, f"step {5 * (k + 1)}"))
    at = [dict(p, x=tuple(q["x"])) for p, q in zip(ps, g.particles())]
    for k, mv in enumerate(([(4, 1, 0), (0, 0, 0), (-17, 13, -13)],
                            [(-4, -1, 0), (3, 0, 1), (0, 0, 0)],
                            [(0.4, 0, 0), (-0.3, 0.5, 0), (17.2, -13, 13)])):
        mv = [mv[i] for i in order]
        at = _push(g, o, at, mv)
        seen.append(_same(g, o, f"push {k}"))
    passed = set()
    for a, b in zip(seen[:-1], seen[1:]):
        ch = (a != b) & (a > 1) & (b > 1)
        passed |= set(zip(a[ch].tolist(), b[ch].tolist()))
    assert {(x < y) for x, y in passed} == {True, False}, passed  # both ways
    g.close()


@pytest.mark.parametrize("first", [0, 35, 70])
def test_more_neighbours_than_the_search_lists(first):
    """A sphere of radius 9 (index `first`) that 70 of radius 1.2 touch or lie in,
    pushed past them (no step: so many contacts overflow the contact table)."""
    r = W.rng(61)
    cfg = W.config(48, 40, 40, has_wall=0, sigma=0.0)
    d = r.normal(size=(70, 3))
    d *= (r.uniform(2.0, 10.0, 70) / np.linalg.norm(d, axis=1))[:, None]
    ps = [W.particle(tuple((20.2, 19.7, 20.4) + e), 1.2, kinematic=1) for e in d]
    ps.insert(first, W.particle((20.2, 19.7, 20.4), 9.0, kinematic=1))
    g, o = _pair(cfg, ps)
    _same(g, o, "created")
    for k, dx in enumerate(((1.3, -0.6, 0.4), (7.5, 2.0, 0.0), (-9.1, 0.0, -3.0))):
        mv = r.uniform(-0.4, 0.4, (71, 3))
        mv[first] = dx
        ps = _push(g, o, ps, mv)
        _same(g, o, f"push {k}")
    g.close()


@pytest.mark.parametrize("n", [40, 512, 513, 1024, 1025])
def test_many_spheres(n):
    """n spheres of radius 2, 6 nodes apart and jittered, on prescribed paths, then
    pushed so that neighbours overlap; the last two of radius 5 and 14 in a corner of their
    own (14: more nodes than the blocks of a sphere take at once)."""
    r = W.rng(62, n)
    side = 8 if n <= 513 else 11
    cfg = W.config(6 * side, 6 * side, 108, has_wall=0, sigma=0.0)
    sites = [(6 * x + 3, 6 * y + 3, 6 * z + 3)
             for z in range(9) for y in range(side) for x in range(side)]
    ps = [W.particle(tuple(np.array(sites[k]) + r.uniform(-0.4, 0.4, 3)), 2.0,
                     v=tuple(r.uniform(-0.05, 0.05, 3)), kinematic=1) for k in range(n - 2)]
    ps += [W.particle((40.3, 40.1, 64.2), 5.0, v=(0.06, 0.0, 0.0), kinematic=1),
           W.particle((20.2, 22.4, 82.8), 14.0, v=(0.0, 0.05, 0.02), kinematic=1)]
    g, o = _pair(cfg, ps)
    _same(g, o, "created")
    for k in range(2):
        g.step(4)
        o.step(4)
        _same(g, o, f"step {4 * (k + 1)}")
        at = [dict(p, x=tuple(q["x"])) for p, q in zip(ps, g.particles())]
        ps = _push(g, o, at, r.uniform(-1.2, 1.2, (n, 3)))
        _same(g, o, f"push {k}")
    g.close()
