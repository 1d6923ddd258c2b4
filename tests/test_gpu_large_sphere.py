"""A sphere so much larger than the 500 beside it that a block per 256 nodes of every
particle's capillary box, sized by the largest, would not fit one dimension of a grid:
the step is carried out, and the large sphere and some small ones come out as in a
context that holds only these (the others are far from them; only the order of the FP64
sums may differ: 1e-11 of sigma R, as in test_gpu_capillary_batch.py)."""
import numpy as np
import pytest

from paper_2505_10171_amd import workloads as W

pytestmark = pytest.mark.gpu

R, L = 102.0, 240


def _particles():
    c = 0.5 * L
    small = []
    for x in np.arange(6.0, L - 6.0, 9.0):
        for y in np.arange(6.0, L - 6.0, 9.0):
            for z in (98.2, 109.1, 119.7, 130.3, 141.2):  # the interface lies at 120
                if (x - c) ** 2 + (y - c) ** 2 + (z - c) ** 2 > (R + 12.0) ** 2:
                    small.append((x, y, z))
    g = W.rng(17)
    small = [small[k] for k in g.permutation(len(small))[:500]]
    return [W.particle((c, c, c), R, theta_deg=70.0, kinematic=1)] + [
        W.particle(p, 3.0, theta_deg=60.0, kinematic=1) for p in small]


def test_capillary_boxes_beyond_one_grid_dimension():
    import torch
    from paper_2505_10171_amd.lbm import Simulation
    if torch.cuda.mem_get_info()[0] < 130 << 30:
        pytest.skip("needs 130 GB of device memory")
    cfg, parts = W.config(L, L, L), _particles()
    assert len(parts) == 501
    phi0 = W.slab_phi0(L, L, L, 0.5 * L)
    few = [0] + [k for k in range(1, 501) if abs(parts[k]["x"][2] - 0.5 * L) < 5.0][:9]
    g = Simulation(cfg, phi0, parts)
    g.step(1)
    a = [g.particles()[k] for k in few]
    g.close()
    del g
    torch.cuda.empty_cache()
    g = Simulation(cfg, phi0, [parts[k] for k in few])
    g.step(1)
    b = g.particles()
    g.close()
    del g
    torch.cuda.empty_cache()
    for p, q in zip(a, b):
        scale = cfg["sigma"] * p["R"]
        assert np.abs(q["F_cap"]).max() > 0.1 * scale, q["F_cap"]  # the interface pulls
        assert np.abs(p["F_cap"] - q["F_cap"]).max() <= 1e-11 * scale
        assert np.abs(p["T_cap"] - q["T_cap"]).max() <= 1e-11 * scale * p["R"]
