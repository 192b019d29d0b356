"""Sparse rows of the classifier's backward pass (needs an MI355X).

The gradient enters at the rows of the pooled maxima and the candidate's own
and spreads by one row per layer; the kernels skip all other rows.
"""
import numpy as np
import pytest

from oracle import cnn
from paper_2510_18136_amd import nsfrb
from tests._lib import ensure_built
from tests.test_gpu_cnn import bf16_device, make_case, tensor_slices

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module", autouse=True)
def _lib():
    ensure_built()
    assert torch.cuda.is_available()


def step(c, x, labels):
    xd, yd = bf16_device(x), torch.from_numpy(labels.astype(np.float32)).cuda()
    c.train_step(xd.data_ptr(), yd.data_ptr(), x.shape[0], update=False, stream=torch.cuda.current_stream().cuda_stream)
    return c.grads()


# one row; planes and rows at the edges of the 16-plane, 8-row and 4-row tiles
@pytest.mark.parametrize("n,T,Y", [(1, 1, 1), (2, 17, 9), (1, 33, 12), (3, 20, 5), (1, 64, 32)])
def test_gradients_of_sparse_rows(n, T, Y):
    x, theta, labels = make_case(n + T, n=n, T=T, Y=Y)
    x[:, T // 2, Y // 2, 10:20] += 6.0                 # most maxima in a few rows, as around a pulse
    with nsfrb.Classifier(max_batch=n, n_time=T, ny=Y, lr=0.0) as c:
        c.set_params(theta)
        print(f"[gpu] sparse rows n={n} T={T} Y={Y}", flush=True)
        step(c, np.roll(x, 1, axis=1), 1.0 - labels)   # another step first: nothing of it may be left
        g = step(c, x, labels)
        rows = [np.abs(c.grad_pre(l, n)).max(axis=(3, 4)) > 0 for l in range(1, 5)]
    for l in range(3):                                 # no further than one row per layer
        for i, t, y in np.argwhere(rows[l]):
            assert rows[l + 1][i, max(t - 1, 0):t + 2, max(y - 1, 0):y + 2].any()
    ref = cnn.loss_and_grad(theta, x, labels, bf16_points=True)[1]
    for name, sl in tensor_slices():                   # the bound of the dense check: BF16 flips cascade
        assert np.linalg.norm(g[sl] - ref[sl]) <= 2e-2 * np.linalg.norm(ref[sl]) + 1e-6, name


def test_non_finite_samples_keep_every_row():
    """0 * inf is not 0: a channel with an infinite sample has no finite weight
    gradient in any tap that reaches it, wherever the gradient's rows are."""
    x, theta, labels = make_case(3, n=2, T=24, Y=16)
    x[1, 2, 3, 5, 7] = np.inf
    with nsfrb.Classifier(max_batch=2, n_time=24, ny=16, lr=0.0) as c:
        c.set_params(theta)
        g = step(c, x, labels)
        w1 = g[tensor_slices()[0][1]].reshape(32, 27, 16)
        assert np.isnan(w1[:, :, 7]).all()
        x[1, 2, 3, 5, 7] = 0.0
        assert np.isfinite(step(c, x, labels)).all()   # and the next step is back to normal
