"""Fields copied to device pointers (dst_is_device): memory of the context's GPU, which
the kernel writes itself, pinned host memory and, where there is one, another GPU's
memory, which a copy writes: the same bytes as through host arrays."""
import ctypes as C

import numpy as np
import pytest

from paper_2505_10171_amd import workloads as W

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("where", ["own", "pinned", "other"])
def test_fields_to_device_pointers(where):
    import torch
    from paper_2505_10171_amd import lbm
    if where == "other" and torch.cuda.device_count() < 2:
        pytest.skip("needs a second GPU")
    cfg = W.config(24, 20, 16, body_force=(3e-6, 0.0, 0.0))
    s = lbm.Simulation(cfg, W.drop_phi0(24, 20, 16, (10.0, 10.0, 0.5), 7.0),
                       [W.particle((15.3, 9.8, 4.5), 3.0, theta_deg=70.0)])
    s.step(5)
    N = 24 * 20 * 16
    kw = {"own": dict(device="cuda:0"), "pinned": dict(pin_memory=True),
          "other": dict(device="cuda:1")}[where]
    rho, u, phi, F = (torch.empty(n * N, dtype=torch.float32, **kw) for n in (1, 3, 1, 3))
    bits = lbm.LBM_F_RHO | lbm.LBM_F_U | lbm.LBM_F_PHI | lbm.LBM_F_FORCE
    torch.cuda.synchronize()
    s._check(lbm.load_library().lbm_fields2(
        s.h, 0, bits, *(C.c_void_p(t.data_ptr()) for t in (rho, u, phi, F)), None, None, 1))
    hr, hu, hp, _ = s.fields()
    hF = s.force()
    assert np.array_equal(rho.cpu().numpy(), hr.ravel())
    assert np.array_equal(u.cpu().numpy(), hu.ravel())
    assert np.array_equal(phi.cpu().numpy(), hp.ravel())
    assert np.array_equal(F.cpu().numpy().reshape(3, -1), np.moveaxis(hF, -1, 0).reshape(3, -1))
    s.close()
