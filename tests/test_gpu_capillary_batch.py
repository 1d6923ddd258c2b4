"""Capillary forces of one context whose members have boxes of different size
(radius 2.5, 4 and 7), one of them without surface tension, against each member
alone, in both storages: filling the boxes and summing them are split over blocks
by the largest member, and each member must come out as by itself.

The lattice part of a step is the same per member whatever the batch, so after two
steps only the order of the FP64 sums over a sphere's points may differ: 1e-11 of
sigma R (R for the torque), for about 10^4 terms of at most that size."""
import numpy as np
import pytest

from paper_2505_10171_amd import workloads as W

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("storage", ["fp32", "fp16"])
def test_boxes_of_different_size_in_one_context(storage):
    from paper_2505_10171_amd.lbm import Context, Simulation
    ms = []
    for n, R, sigma in ((24, 2.5, 0.01), (40, 7.0, 0.01), (32, 4.0, 0.01), (32, 4.0, 0.0)):
        cfg = W.config(n, n, n, sigma=sigma, storage=storage)
        ps = [W.particle([0.5 * n + 0.3, 0.5 * n - 0.2, 0.5 * n + 0.4], R, theta_deg=60.0)]
        ms.append(dict(cfg=cfg, phi0=W.slab_phi0(n, n, n, 0.5 * n + 0.3 * R), particles=ps))
    ens = Context(ms)
    ens.step(2)
    for i, m in enumerate(ms):
        one = Simulation(m["cfg"], m["phi0"], m["particles"])
        one.step(2)
        a, b = ens.particles(i)[0], one.particles()[0]
        scale = 0.01 * m["particles"][0]["R"]
        fa, fb = np.array(a["F_cap"]), np.array(b["F_cap"])
        ta, tb = np.array(a["T_cap"]), np.array(b["T_cap"])
        if m["cfg"]["sigma"] == 0.0:
            assert not fa.any() and not fb.any() and not ta.any()
        else:
            assert np.abs(fb).max() > 0.1 * scale, fb  # the interface pulls
        assert np.abs(fa - fb).max() <= 1e-11 * scale, (i, fa, fb)
        assert np.abs(ta - tb).max() <= 1e-11 * scale * m["particles"][0]["R"], (i, ta, tb)
        one.close()
    ens.close()
