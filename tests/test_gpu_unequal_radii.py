"""Spheres of very different radius in one simulation, whose launches the largest sizes:
forces, torques, masks and fields against the FP64 oracle, in both storages; 330 spheres
(so that the blocks of the largest sphere's boxes take several turns) and a few.

Bars of tests/parity_util.py: 1e-5 (FP32; the field bars), for FP16 storage 1e-3 and no
bar at single nodes."""
import numpy as np
import pytest

from oracle.oracle import OracleSim
from parity_util import compare_fields, compare_particles
from paper_2505_10171_amd import workloads as W

pytestmark = pytest.mark.gpu

R = 20.0


def _case(n, storage):
    L = (72, 64, 60)
    cfg = W.config(*L, has_wall=0, storage=storage, theta_wall_deg=80.0)
    c = np.array([35.7, 31.6, 30.2])
    g = W.rng(83, n)
    sites = [np.array([x, y, z], float) for z in np.arange(3.6, 60.0, 7.4)
             for y in np.arange(4.0, 64.0, 8.0) for x in np.arange(4.0, 72.0, 8.0)]
    sites = [s for s in sites if np.linalg.norm(s - c) > R + 6.5]
    # around the interface at z = 30 first
    sites.sort(key=lambda s: (abs(s[2] - 30.0) > 5.0, s[0], s[1], s[2]))
    ps = [W.particle(tuple(s + g.uniform(-0.4, 0.4, 3)), g.uniform(1.0, 2.4),
                     theta_deg=g.uniform(50.0, 120.0), v=tuple(g.uniform(-0.02, 0.02, 3)),
                     w=tuple(g.uniform(-0.002, 0.002, 3)), kinematic=1) for s in sites[:n - 1]]
    ps.insert(2, W.particle(tuple(c), R, theta_deg=70.0, v=(0.01, -0.02, 0.015), kinematic=1))
    assert len(ps) == n
    return cfg, W.slab_phi0(*L, 30.0), ps


@pytest.mark.parametrize("n,storage", [(4, "fp32"), (330, "fp32"), (330, "fp16")])
def test_one_large_sphere_among_small_ones(n, storage):
    from paper_2505_10171_amd.lbm import Simulation
    cfg, phi0, ps = _case(n, storage)
    g, o = Simulation(cfg, phi0, ps), OracleSim(dict(cfg, storage="fp32"), phi0, ps)
    tol = 1e-5 if storage == "fp32" else 1e-3
    g.step(3)
    o.step(3)
    pg, po = g.particles(), o.particles()
    # the large sphere, then the small ones, on their own scales
    for part, r in (([2], R), ([k for k in range(n) if k != 2], 2.4)):
        compare_particles([pg[k] for k in part], [po[k] for k in part],
                          ("F_hyd", "T_hyd", "F_cap", "T_cap", "x"), tol=tol, R=r,
                          label=f"{n} {storage} R={r}")
    assert min(np.abs(p["F_cap"]).max() for p in (po[0], po[2])) > 0.01 * cfg["sigma"]
    compare_fields(g, o, label=f"{n} {storage}", tol=tol,
                   node_tol=1e-4 if storage == "fp32" else None)
    g.close()
