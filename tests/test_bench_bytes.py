"""The bytes that the benchmark charges its kernels: what they move, also on tile planes of
one pure fluid, so that no kernel's share of the memory's peak can pass one by bytes that
were not moved."""
import os
import sys

import numpy as np
import pytest
import torch

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
sys.path.insert(0, ROOT)
import bench  # noqa: E402


def _plain(phi, mask, open_x):
    """The same node by node."""
    nz, ny, nx = phi.shape
    w = 64 if 100 * -(-nx // 64) * 64 <= 120 * nx else 32 if 100 * -(-nx // 32) * 32 <= 120 * nx else 16
    h = 256 // w
    out = {"mixed": [0, 0], "pure": [0, 0], "pure_solid": [0, 0]}
    for z in range(nz):
        for y0 in range(0, ny, h):
            for x0 in range(0, nx, w):
                seen = set()
                for dz in range(-2, 3):
                    for y in range(y0 - 2, y0 + h + 2):
                        for x in range(x0 - 2, x0 + w + 2):
                            if open_x and not 0 <= x < nx:
                                seen.add("s")
                                continue
                            k = (z + dz) % nz, y % ny, x % nx
                            seen.add("s" if mask[k] else phi[k] if abs(phi[k]) == 1 else "o")
                mixed = "o" in seen or {1.0, -1.0} <= seen
                key = "mixed" if mixed else "pure_solid" if "s" in seen else "pure"
                t = mask[z, y0:y0 + h, x0:x0 + w]
                out[key][0] += int((t == 0).sum())
                out[key][1] += int((t != 0).sum())
    return {k: tuple(v) for k, v in out.items()}


@pytest.mark.parametrize("nx,open_x", [(20, 0), (33, 0), (33, 1), (64, 0), (70, 1)])
def test_plane_classes(nx, open_x):
    g = np.random.default_rng(nx)
    phi = np.ones((13, 21, nx), np.float32)
    phi[:, :, : nx // 3] = -1
    phi[4, 5, nx // 2] = 0.5
    mask = np.zeros(phi.shape, np.uint8)
    mask[9:, 14:, nx - 6:] = 2
    mask[g.integers(0, 13, 3), g.integers(0, 21, 3), g.integers(0, nx, 3)] = 1
    phi[mask != 0] = 0
    got = bench.plane_classes(torch.from_numpy(phi), torch.from_numpy(mask), open_x)
    assert got == _plain(phi, mask, open_x)
    assert sum(sum(v) for v in got.values()) == phi.size


@pytest.mark.parametrize("storage", ["fp32", "fp16"])
def test_bytes_of_mixed_and_pure_planes(storage):
    p = 4 if storage == "fp32" else 2
    none = {"mixed": (0, 0), "pure": (0, 0), "pure_solid": (0, 0)}
    m = bench.kernel_bytes(storage, dict(none, mixed=(1000, 0)))
    assert m["interface"] == 28000 and m["moments"] == (19 * p + 30) * 1000
    assert m["group"] == min(bench.B_ALG[storage], 28 + 38 * p + 24 + (8 if p == 2 else 0)
                             + 19 * p + 30) * 1000
    q = bench.kernel_bytes(storage, dict(none, pure=(1000, 0)))
    if storage == "fp32":
        # populations read and written once, phi read twice and written, the mask
        assert (q["interface"], q["fused"], q["moments"]) == (4000, 152000, 6000)
        assert q["group"] == 162000
    else:
        assert (q["interface"], q["fused"]) == (m["interface"], m["fused"])
        assert q["moments"] == 52000 and q["group"] == 162000
    s = bench.kernel_bytes(storage, dict(none, pure_solid=(0, 1000)))
    assert s["moments"] == 10000 and s["fused"] <= 8000


def test_counter_traffic_is_of_the_same_steps(monkeypatch):
    """The counters' bytes are given with a run of as many steps only."""
    from paper_2505_10171_amd import prof_summary
    path = bench.COUNTERS["fp32"]
    n = prof_summary.counted_launches(path, "k_fused<")
    assert n > 0 and prof_summary.counted_launches(path, "no such kernel") == 0
    monkeypatch.setattr(prof_summary, "kernel_sources_hash",
                        lambda: prof_summary.read_counters(path)[1])
    assert bench.traffic_from_profile("fp32", n) > 1e9
    assert bench.traffic_from_profile("fp32", n + 1) is None
    assert bench.traffic_from_profile("fp16", n) is None
