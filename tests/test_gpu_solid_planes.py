"""Tile planes without a fluid node, which the collide and moments passes leave by their
kind: the wall below mixed fluids at every tile width, and the middle of a sphere that
covers whole tiles, which moves and is pushed away (every node there becomes fluid), against
the FP64 oracle; bars of tests/parity_util.py."""
import numpy as np
import pytest

from oracle.oracle import OracleSim
from parity_util import compare_fields, rel_l2
from paper_2505_10171_amd import workloads as W

pytestmark = pytest.mark.gpu


def _tol(storage):
    return dict(tol=1e-3, node_tol=None) if storage == "fp16" else {}


def _rho_phi(g, o, storage):
    (rg, _, pg, mg), (ro, _, po, mo) = g.fields(), o.fields()
    assert np.array_equal(mg, mo)
    fl = mo == 0
    assert max(rel_l2(rg[fl], ro[fl]), rel_l2(pg[fl], po[fl])) <= (1e-5 if storage == "fp32"
                                                                   else 1e-3)


@pytest.mark.parametrize("storage", ["fp32", "fp16"])
@pytest.mark.parametrize("nx,ny,nz", [(64, 9, 5), (33, 17, 7), (48, 33, 12)])
def test_wall_under_an_interface(nx, ny, nz, storage):
    from paper_2505_10171_amd.lbm import Simulation
    cfg = W.config(nx, ny, nz, theta_wall_deg=80.0, body_force=(3e-6, 0.0, 0.0), storage=storage)
    phi0 = W.drop_phi0(nx, ny, nz, (0.4 * nx, 0.5 * ny, 0.5), 0.3 * nx)
    g, o = Simulation(cfg, phi0, []), OracleSim(dict(cfg, storage="fp32"), phi0, [])
    g.step(10)
    o.step(10)
    compare_fields(g, o, label=f"wall {nx}x{ny}x{nz} {storage}", **_tol(storage))
    assert np.all(np.abs(g.mass() - o.mass()) <= (1e-6 if storage == "fp32" else 1e-5) * o.mass())
    g.close()


@pytest.mark.parametrize("storage", ["fp32", "fp16"])
def test_a_sphere_that_covers_tiles(storage):
    """Radius 17 about the middle of a tile of 16 x 16 nodes (20 x 20 grown), in an
    interface; the nodes it uncovers had no fluid neighbour at all.  After the push the
    masks, rho and phi: the force of freshly refilled nodes beside the interface, half of
    which is in u, turns on thresholds of the wetting rotation."""
    from paper_2505_10171_amd.lbm import Simulation
    n = (48, 48, 44)
    cfg = W.config(*n, has_wall=0, storage=storage)
    phi0 = W.slab_phi0(*n, 20.3)
    p = W.particle((23.6, 23.4, 21.7), 17.0, theta_deg=70.0, v=(0.04, -0.02, 0.03), kinematic=1)
    g, o = Simulation(cfg, phi0, [p]), OracleSim(dict(cfg, storage="fp32"), phi0, [p])
    g.step(6)
    o.step(6)
    compare_fields(g, o, label=f"sphere {storage}", **_tol(storage))
    q = dict(p, x=(24.9, 22.6, 23.4))
    g.push_particles([q])
    o.set_particles([q])
    _rho_phi(g, o, storage)
    g.step(4)
    o.step(4)
    _rho_phi(g, o, storage)
    # far away: masks exactly (the refilled nodes start from the mean density)
    q = dict(q, x=(1.3, 45.2, 40.6))
    g.push_particles([q])
    o.set_particles([q])
    assert np.array_equal(g.phi_mask()[1], o.fields()[3])
    g.close()
