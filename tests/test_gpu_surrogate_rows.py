"""The surrogate's row counts at the edges of its kernels: inference with 32, 64
and 128 rows per workgroup (and the pinned path of small host batches), and
training batches that are and are not a multiple of 128, each against the FP64
reference on BF16-rounded weights and inputs (the bars of
tests/test_gpu_surrogate.py: outputs 2e-2, gradients 5e-2 relative L2), and the
row groupings against each other: a row's outputs do not depend on how many rows
it comes with, to the bit."""
import numpy as np
import pytest

from oracle import surrogate_oracle as S
from test_gpu_surrogate import _setup, bf16, rel

pytestmark = pytest.mark.gpu


def test_inference_row_groupings():
    import torch
    from paper_2505_10171_amd.surrogate import Surrogate, flatten
    _, ps, ref, *_ = _setup()
    s = Surrogate(max_batch=40960, max_train=64)
    s.set_params(flatten(ps))
    X = np.random.default_rng(5).standard_normal((32900, 6)).astype(np.float32)
    Xd = torch.from_numpy(X).to("cuda")
    full = None
    # 128, 64 and 32 rows per workgroup, whole and ragged last groups
    for n in (32900, 32769, 32768, 8193, 8192, 1025, 1024, 97, 33, 32, 31, 1):
        Yd = torch.full((n + 2, 51), 7.0, device="cuda")
        s.predict_device(Xd[:n], Yd)
        s.sync()
        Y = Yd.cpu().numpy()
        assert np.all(Y[n:] == 7.0), n
        if full is None:
            full = Y[:n]
            assert rel(full[:2000], S.forward(ref, bf16(X[:2000]))[0]) <= 2e-2
        assert np.array_equal(Y[:n], full[:n]), n
    for n in (1, 256, 1024, 1025):  # host arrays: pinned up to 1,024 rows, copied beyond
        assert np.array_equal(s.predict(X[:n]), full[:n]), n
    s.close()


@pytest.mark.parametrize("n", [64, 128, 192, 320, 1024])
def test_gradients_at_batch_sizes(n):
    from paper_2505_10171_amd.surrogate import unflatten
    s, ps, ref, Xr, X, lab, tr = _setup(seed=8, n=n)
    g, L = s.gradients(X, lab, tr, w_traj=0.7)
    go, Lo = S.gradients(ref, Xr, lab, tr, w_traj=0.7)
    assert abs(L - Lo) <= 2e-2 * abs(Lo), (L, Lo)
    for k, (a, b) in enumerate(zip(unflatten(g), go)):
        assert rel(a, b) <= 5e-2, (k, rel(a, b))
    s.close()


@pytest.mark.parametrize("n", [64, 192, 320])
def test_adam_step_at_batch_sizes(n):
    """The first step from zero moments is lr * sign(g) where g is resolved: the
    training set in another order gives the same gradient up to the order of FP32
    sums (n terms, far below 1e-3 of the largest), so every such step has its sign
    and its size to 2e-5."""
    s, ps, ref, Xr, X, lab, tr = _setup(seed=9, n=n)
    g, _ = s.gradients(X, lab, tr)
    p0 = s.get_params().astype(np.float64)
    s.set_train(X, lab, tr)
    s.train(1, batch=n, lr=1e-3, seed=3)
    p1 = s.get_params().astype(np.float64)
    po, _, _ = S.adam_step([p0], [g.astype(np.float64)], [np.zeros_like(p0)],
                           [np.zeros_like(p0)], 1, lr=1e-3)
    big = np.abs(g) > 1e-3 * np.abs(g).max()
    assert np.abs(p1[big] - po[0][big]).max() <= 2e-5
    s.close()
