"""The wetting rotation of queued entries at the edges of its queue: a block of the
interface kernel in which every node next to the wall is rotated (an interface
standing across the wall everywhere: more entries than threads), tiles of every
width (boxes of 16, 32, 48 and 64 nodes a side), pillars with their corners, spheres
that share nodes with the wall: the force field of the initial state, which the
kernel alone decides, against the FP64 oracle.

Bar: G is a sum of 18 FP32 terms of phi of order one, 5e-7 off; the unit normal and
the rotation's blend magnify that by at most 1 / EPS = 1e4 where |G| or its tangential
part is near the threshold, on a hundredth of the nodes or fewer: 5e-3 sqrt(0.01)
= 5e-4 of the norm, taken as 1e-3.  One entry in a thousand left unturned or turned
twice gives 3e-2.
"""
import numpy as np
import pytest

from oracle.oracle import OracleSim
from paper_2505_10171_amd import workloads as W

pytestmark = pytest.mark.gpu


def _check(cfg, phi0, parts, label):
    from paper_2505_10171_amd.lbm import Simulation
    g = Simulation(cfg, phi0, parts)
    F = g.force().astype(np.float64)
    Fo = np.asarray(OracleSim(cfg, phi0, parts).grad_force()[1])
    fl = g.fields()[3] == 0
    assert F.shape == Fo.shape
    e = np.linalg.norm(F[fl] - Fo[fl]) / np.linalg.norm(Fo[fl])
    print(label, f"{e:.2e}", flush=True)
    assert e <= 1e-3, (label, e)
    g.close()


@pytest.mark.parametrize("n", [(16, 16, 16), (32, 20, 18), (48, 17, 19), (64, 12, 20)])
def test_every_wall_node_is_rotated(n):
    """phi varies over the whole wall (amplitude below 1: inside the interface
    everywhere), so all entries of the planes next to it are queued."""
    nx, ny, nz = n
    x, y = np.arange(nx), np.arange(ny)
    w = 0.6 * np.sin(2 * np.pi * x / nx)[None, :] * np.cos(2 * np.pi * y / ny)[:, None] + 0.2
    phi0 = np.ascontiguousarray(np.broadcast_to(w, (nz, ny, nx)), np.float32).copy()
    R = 2.5
    ps = [W.particle([0.5 * nx + 0.2, 0.5 * ny - 0.3, 0.5 + R + 0.5], R, theta_deg=70.0)]
    _check(W.config(nx, ny, nz, theta_wall_deg=50.0), phi0, ps, f"{nx}x{ny}x{nz}")


@pytest.mark.parametrize("nx", [24, 64])
def test_pillars(nx):
    boxes = [(5, 4, 1, 10, 9, 5), (nx - 9, 6, 1, nx - 5, 12, 4)]
    cfg = W.config(nx, 20, 24, has_wall=3, boxes=boxes, theta_wall_deg=110.0)
    phi0 = W.drop_phi0(nx, 20, 24, (7.0, 7.0, 6.0), 7.0)
    _check(cfg, phi0, [], f"pillars {nx}")
