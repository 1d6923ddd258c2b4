"""Tubes and open channels that hold two fluids: the force field of the initial state,
which the interface kernel alone decides, against the FP64 oracle, for interfaces across
and along the tube, on tiles of every width, with a sphere in the interface.  Bar: that of
tests/test_gpu_wet_queue.py (1e-3 of the norm)."""
import numpy as np
import pytest

from oracle.oracle import OracleSim
from parity_util import rel_l2
from test_gpu_wet_queue import _check
from paper_2505_10171_amd import workloads as W

pytestmark = pytest.mark.gpu


def _phi(n, kind):
    nx, ny, nz = n
    x = np.arange(nx)[None, None, :]
    z = np.arange(nz)[:, None, None]
    if kind == "plug":
        p = np.tanh((0.25 * nx - np.abs(x - 0.5 * nx)) / 2) + 0.0 * z
    elif kind == "layer":
        p = np.tanh((0.5 * nz - z) / 2) + 0.0 * x
    else:
        return W.drop_phi0(nx, ny, nz, (0.5 * nx, 0.5 * ny, 0.25 * nz), 0.25 * nz)
    return np.ascontiguousarray(np.broadcast_to(p, (nz, ny, nx)), np.float32).copy()


@pytest.mark.parametrize("kind", ["plug", "layer", "drop"])
@pytest.mark.parametrize("n", [(16, 19, 19), (32, 24, 21), (48, 17, 25), (64, 29, 29), (70, 20, 22)])
def test_two_fluids_in_a_tube(n, kind):
    nx, ny, nz = n
    cfg = W.config(nx, ny, nz, has_wall=2, tube_R=0.5 * min(ny, nz) - 1.3, theta_wall_deg=60.0)
    ps = [W.particle((0.5 * nx + 0.3, 0.5 * ny - 0.7, 0.5 * nz + 0.2), 2.5, theta_deg=110.0)]
    _check(cfg, _phi(n, kind), ps, f"tube {nx}x{ny}x{nz} {kind}")


@pytest.mark.parametrize("wall", [0, 1, 2])
def test_two_fluids_between_open_ends(wall):
    n = (48, 21, 23)
    cfg = W.config(*n, has_wall=wall, tube_R=9.0, open_x=1, rho_in=0.0501, rho_out=0.0499,
                   theta_wall_deg=120.0)
    _check(cfg, _phi(n, "layer"), [W.particle((24.2, 10.1, 11.4), 2.5, theta_deg=70.0)],
           f"open {wall}")


def test_batches_of_all_geometries():
    """A plane, a tube without and one with surface tension in one context, which one
    instance of the kernel steps: phi and u after a step, the same bar."""
    from paper_2505_10171_amd.lbm import Context
    n = (33, 20, 22)
    ms = [dict(cfg=W.config(*n, **kw), phi0=_phi(n, kind), particles=[])
          for kw, kind in ((dict(), "drop"), (dict(has_wall=2, tube_R=9.0, sigma=0.0), "plug"),
                           (dict(has_wall=2, tube_R=9.0), "layer"))]
    for members in (ms[:2], ms):
        ens = Context(members)
        ens.step(1)
        for i, m in enumerate(members):
            o = OracleSim(m["cfg"], m["phi0"], [])
            o.step(1)
            _, ug, pg, mg = ens.fields(i)
            _, uo, po, mo = o.fields()
            assert np.array_equal(mg, mo)
            fl = mo == 0
            assert rel_l2(pg[fl], po[fl]) <= 1e-3, i
            if m["cfg"]["sigma"] > 0.0:  # else there is no flow yet
                assert rel_l2(ug[:, fl], uo[:, fl]) <= 1e-3, i
        ens.close()
