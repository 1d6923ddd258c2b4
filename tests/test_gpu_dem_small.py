"""The single-workgroup DEM (16 lanes per particle, boxes of up to 48
particles) at the edges of its range, against the FP64 oracle: one particle,
particles that fill whole waves and one more, the largest box it takes and the
smallest it does not; many DEM sub-steps (past 16, where the orientations are
taken in batches); a sphere touching the plane and several boxes of a textured
wall, whose wall partners and pair candidates take more than one pass of 16.

The records are FP64 but the fluid force that drives them is FP32's, so the bars
are tests/test_gpu_parity.py's: 1e-5 of the largest oracle magnitude.
"""
import numpy as np
import pytest

from oracle.oracle import OracleSim
from paper_2505_10171_amd import workloads as W

pytestmark = pytest.mark.gpu


def _compare(g, o, R):
    pg, po = g.particles(), o.particles()
    assert np.abs(np.array([p["F_con"] for p in po])).max() > 0.05  # the contacts act
    for k in ("F_con", "T_con", "x", "v", "w", "q"):
        a = np.array([p[k] for p in pg])
        b = np.array([p[k] for p in po])
        scale = np.abs(b).max()
        if k == "T_con":
            scale = max(scale, R * np.abs(np.array([p["F_con"] for p in po])).max())
        err = np.abs(a - b).max()
        print(k, f"{err:.2e} of {scale:.2e}", flush=True)
        assert err <= 1e-5 * scale, (k, err, scale)


@pytest.mark.parametrize("n,kn", [(1, 2.5), (4, 2.5), (5, 2.5), (16, 2.5), (17, 3.0), (48, 2.5),
                                  (49, 2.5)])
def test_spheres_on_the_wall(n, kn):
    """n spheres (R = 2, contact radius 3) on the wall in rows, closer than
    their contact diameter, with seeded jitter, velocities and spins."""
    from paper_2505_10171_amd.lbm import Simulation
    g0 = W.rng(91, n)
    side = int(np.ceil(np.sqrt(n)))
    L, sp = 6 * side + 10, 5.95
    cfg = W.config(L, L, 16, kn=kn, gn=0.05, gt=0.02, gr=0.01)
    Rc = 2.0 + cfg["delta_R"]
    parts = [W.particle((5.0 + k % side * sp + g0.uniform(-0.03, 0.03),
                         5.0 + k // side * sp + g0.uniform(-0.03, 0.03),
                         0.5 + Rc - 0.05 + g0.uniform(-0.02, 0.02)), 2.0,
                        v=tuple(g0.uniform(-0.01, 0.01, 3)), w=tuple(g0.uniform(-0.005, 0.005, 3)))
             for k in range(n)]
    phi0 = W.slab_phi0(L, L, 16, 8.0)
    g, o = Simulation(cfg, phi0, parts, history_steps=3), OracleSim(cfg, phi0, parts)
    if kn > 2.5:
        assert g.dem_substeps() > 16
    g.step(3)
    o.step(3)
    _compare(g, o, 2.0)
    _, h = g.particles(history=True)
    last = g.particles()
    assert np.array_equal(h[-1, :, 18:21], np.array([p["x"] for p in last]))
    g.close()


def test_more_partners_than_lanes():
    """A sphere in a pit of four pillars among eight boxes (ten wall partners),
    touching the pillars' edges, with seven neighbours within its candidate
    range (17 partners), some of which rest on the pillars."""
    from paper_2505_10171_amd.lbm import Simulation
    boxes = [(x, y, 1, x + 3, y + 3, 3) for x, y in ((14, 14), (22, 14), (14, 22), (22, 22),
                                                     (2, 2), (34, 2), (2, 34), (34, 34))]
    cfg = W.config(40, 40, 20, has_wall=3, boxes=boxes)
    Rc = 2.0 + cfg["delta_R"]
    parts = [W.particle((19.5, 19.5, 0.5 + Rc - 0.05), 2.0, v=(0.004, 0.002, 0.0),
                        w=(0.001, 0.0, 0.002)),
             W.particle((19.5, 19.5, 0.5 + Rc + 6.95), 2.0)]
    for k in range(6):
        a = np.pi * k / 3
        parts.append(W.particle((19.5 + 6.32 * np.cos(a), 19.5 + 6.32 * np.sin(a), 3.5 + Rc - 0.05),
                                2.0, v=(-0.01 * np.cos(a), -0.01 * np.sin(a), -0.005)))
    phi0 = W.slab_phi0(40, 40, 20, 12.0)
    g, o = Simulation(cfg, phi0, parts), OracleSim(cfg, phi0, parts)
    g.step(4)
    o.step(4)
    _compare(g, o, 2.0)
    g.close()
