"""Tile planes that hold one pure fluid (phi exactly +1 or -1), which the
interface, collide and moments passes treat apart, against the FP64 oracle.

A drop with a sharp edge (phi within rounding of +-1 four nodes from its edge)
and a sphere on a prescribed path through the pure outer fluid, on boxes one node
below, at and above the tile sizes (64 x 4, 32 x 8, 16 x 16) and the march
depths: fields, masks and links after a few steps, after a push between steps
(the refill from the current state) and after further steps, and the masses,
which sum the populations where phi is pure.  The sphere's links and the refill
need densities that the moments pass does not keep there.

Bars as in tests/parity_util.py; masses within 1e-6 relative (the bar of
test_mass_against_oracle).
"""
import numpy as np
import pytest

from oracle.oracle import OracleSim
from paper_2505_10171_amd import workloads as W
from parity_util import compare_fields

pytestmark = pytest.mark.gpu

R = 3.0


def _case(nx, ny, nz, storage, wall, inner):
    cfg = W.config(nx, ny, nz, has_wall=wall, theta_wall_deg=80.0, storage=storage,
                   body_force=(3e-6, 0.0, 0.0))
    if wall == 2:
        cfg["tube_R"] = 0.5 * min(ny, nz) - 1.0
    c = (8.0, 0.5 * (ny - 1), 0.5 * (nz - 1))
    phi0 = W.drop_phi0(nx, ny, nz, c, 3.0, width=0.5)
    if inner:  # the sphere in fluid a, the drop of fluid b
        phi0 = -phi0
    p = W.particle((nx - 9.3, 0.5 * ny + 0.2, 0.5 * nz - 0.4), R, theta_deg=70.0,
                   v=(0.03, 0.01, -0.02), w=(0.0, 0.004, 0.002), kinematic=1)
    return cfg, phi0, p


@pytest.mark.parametrize("nx,ny,nz,storage,wall,inner", [
    (64, 12, 13, "fp32", 1, False), (65, 13, 12, "fp32", 1, True), (63, 11, 12, "fp16", 1, False),
    (32, 16, 25, "fp32", 0, False), (33, 17, 24, "fp32", 2, False), (96, 15, 11, "fp16", 0, True),
    (48, 16, 13, "fp32", 1, False), (130, 20, 20, "fp32", 2, True)])
def test_pure_tile_planes(nx, ny, nz, storage, wall, inner):
    from paper_2505_10171_amd.lbm import Simulation
    cfg, phi0, p = _case(nx, ny, nz, storage, wall, inner)
    g = Simulation(cfg, phi0, [p])
    o = OracleSim(dict(cfg, storage="fp32"), phi0, [p])
    tol = dict(tol=1e-3, node_tol=None) if storage == "fp16" else {}
    pure = -1.0 if not inner else 1.0
    for k in range(3):
        if k:
            q = dict(p, x=tuple(a + k * b for a, b in zip(p["x"], (0.6, -0.5, 0.4))))
            g.push_particles([q])
            o.set_particles([q])
            compare_fields(g, o, label=f"{nx}x{ny}x{nz} pushed", **tol)
        g.step(3)
        o.step(3)
        compare_fields(g, o, label=f"{nx}x{ny}x{nz} after {3 * (k + 1)} steps", **tol)
        phi, mask = g.phi_mask()
        assert np.mean(phi[mask == 0] == pure) > 0.2  # the case holds what it is about
        lg, pid_g = g.links()
        lo, pid_o = o.links()[:2]
        assert np.array_equal(lg, lo) and np.array_equal(pid_g, pid_o)
        mg, mo = g.mass(), o.mass()
        assert np.all(np.abs(mg - mo) <= (1e-6 if storage == "fp32" else 1e-5) * mo), (mg, mo)
        assert np.allclose(g.mass_all_noalloc()[0], mg, rtol=1e-12)
    g.close()


def test_pure_planes_do_not_depend_on_the_march():
    """The same case at march depths 1, 2, 5 and 24 and with x-y tiles in the
    fused kernel: fields identical to the bit."""
    from paper_2505_10171_amd.lbm import Simulation
    cfg, phi0, p = _case(65, 13, 27, "fp32", 1, False)
    ref = None
    for depth, tile in ((1, 0), (2, 64), (5, 16), (24, 256)):
        g = Simulation(cfg, phi0, [p])
        g.set_march(0, depth)
        g.set_tile(0, tile)
        g.step(8)
        f = g.fields()
        g.close()
        ref = ref or f
        for a, b in zip(f, ref):
            assert np.array_equal(a, b), (depth, tile)
