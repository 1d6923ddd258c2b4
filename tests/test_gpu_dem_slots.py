"""A full contact table of the single-workgroup DEM: a sphere with sixteen contacts,
of which one ends in the sub-step in which a seventeenth begins.  The springs of the
one that ends are free for the one that begins if it comes first among the particle's
partners, so the step is carried out, with the oracle's contact forces (bars of
tests/test_gpu_parity.py: 1e-5 of the largest oracle magnitude); the other way round, or
with seventeen contacts at once, the table overflows.
"""
import numpy as np
import pytest

from oracle.oracle import OracleSim
from paper_2505_10171_amd import workloads as W

pytestmark = pytest.mark.gpu


def _shell(n):
    """n points on the unit sphere, well apart (a spiral)."""
    k = np.arange(n) + 0.5
    th, ph = np.arccos(1 - 2 * k / n), np.pi * (1 + 5 ** 0.5) * k
    return np.stack([np.sin(th) * np.cos(ph), np.sin(th) * np.sin(ph), np.cos(th)], 1)


def _parts(cfg, order, move):
    """A sphere of contact radius 7 and seventeen of contact radius 2 about it, all on
    prescribed paths: fifteen touch it throughout, `order` places the one that leaves
    and the one that arrives; they pass the touching distance 1.5 `move` away."""
    c = np.array([20.3, 19.8, 20.1])
    e = _shell(17)
    ps = [W.particle(tuple(c), 6.0, kinematic=1)]
    for k in range(17):
        d, v = 9.0 - 0.05, 0.0
        if k == order[0]:
            d, v = 9.0 - 1.5 * move, SPEED
        elif k == order[1]:
            d, v = 9.0 + 1.5 * move, -SPEED
        ps.append(W.particle(tuple(c + d * e[k]), 1.0, v=tuple(v * e[k]), kinematic=1))
    return ps


SPEED = 0.02


def _case(order):
    from paper_2505_10171_amd.lbm import Simulation
    cfg = W.config(40, 40, 40, has_wall=0, sigma=0.0)
    s = Simulation(cfg, None, _parts(cfg, order, 0.0))
    n_sub = s.dem_substeps()
    s.close()
    assert n_sub >= 4
    parts = _parts(cfg, order, SPEED / n_sub)
    return cfg, parts


@pytest.mark.parametrize("order", [(0, 1), (3, 9), (14, 15), (0, 16)])
def test_a_slot_freed_in_the_same_sub_step(order):
    from paper_2505_10171_amd.lbm import Simulation
    cfg, parts = _case(order)
    g, o = Simulation(cfg, None, parts), OracleSim(cfg, None, parts)
    g.step(2)
    o.step(2)
    g.sync()
    pg, po = g.particles(), o.particles()
    for k in ("F_con", "T_con", "x"):
        a, b = np.array([p[k] for p in pg]), np.array([p[k] for p in po])
        scale = np.abs(b).max() if k != "T_con" else 6.0 * np.abs([p["F_con"] for p in po]).max()
        assert np.abs(a - b).max() <= 1e-5 * scale, (k, np.abs(a - b).max(), scale)
    assert np.linalg.norm(pg[1 + order[1]]["F_con"]) > 0.0  # the one that arrived
    g.close()


@pytest.mark.parametrize("order", [(1, 0), (15, 2), (16, 0)])
def test_a_slot_freed_too_late(order):
    from paper_2505_10171_amd.lbm import LBM_ERANGE, LbmError, Simulation
    cfg, parts = _case(order)
    with pytest.raises(RuntimeError):
        OracleSim(cfg, None, parts).step(2)
    g = Simulation(cfg, None, parts)
    g.step(2)
    with pytest.raises(LbmError) as e:
        g.sync()
    assert e.value.code == LBM_ERANGE
    g.close()


def test_seventeen_contacts_overflow():
    from paper_2505_10171_amd.lbm import LBM_ERANGE, LbmError, Simulation
    cfg, parts = _case((0, 1))
    for k in (1, 2):
        parts[k]["v"] = (0.0, 0.0, 0.0)
        e = np.array(parts[k]["x"]) - np.array(parts[0]["x"])
        parts[k]["x"] = tuple(np.array(parts[0]["x"]) + 8.95 * e / np.linalg.norm(e))
    g = Simulation(cfg, None, parts)
    g.step(1)
    with pytest.raises(LbmError) as e:
        g.sync()
    assert e.value.code == LBM_ERANGE
    g.close()
