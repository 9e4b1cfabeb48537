"""The network's kernels at the edges of their split: 32-row tiles, batch splits of the
weight gradients that are ragged or empty of a full round of eight steps, and more tiles than
workgroups.  Tolerances: the element-wise bounds of test_gpu_mlp.py, on its problem whose
forward pass is exact in binary32."""
import numpy as np
import pytest

from oracle import mlp as M
from test_gpu_mlp import IN_DIM, flat, gradient_bounds, logit_bound, problem, quantized_problem, unflat

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def P():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2003_04920_amd as P
    P.load()
    return P


@pytest.mark.parametrize("B", [31, 32, 33, 8225])
def test_forward_of_ragged_tiles(P, B):
    """Within the bound, and a row's logit is the same bits wherever it lies in a batch."""
    p, x, _ = problem(70 + B, B)
    net = P.Mlp(IN_DIM, B)
    net.set_params(flat(p))
    z = net.forward(x)
    assert np.all(np.abs(z - M.forward(p, x)[0]) <= logit_bound(p, x))
    for a, b in ((0, 1), (B - 1, B), (B // 2, B // 2 + 7)):
        assert np.array_equal(net.forward(x[a:b]).view(np.uint32), z[a:b].view(np.uint32))


@pytest.mark.parametrize("B", [1, 31, 33, 255, 257, 545, 4129, 8225])
def test_gradients_of_ragged_splits(P, B):
    p, x, y = quantized_problem(90 + B, B)
    net = P.Mlp(IN_DIM, 8225)
    net.set_params(flat(p))
    net.gradients(x[::-1].copy(), y)  # what a larger or other batch leaves behind is not read
    loss, g = net.gradients(x, y)
    want_loss, want, _ = M.loss_and_grads(p, x, y)
    assert abs(loss - want_loss) <= 1e-3 * abs(want_loss) + 1e-5
    gd = unflat(g)
    bounds = gradient_bounds(p, x, y, exact_forward=True)
    for k in M.PARAM_NAMES:
        ref = np.asarray(want[k], np.float64).reshape(gd[k].shape)
        err = np.abs(gd[k].astype(np.float64) - ref)
        assert np.all(err <= 2.0 * bounds[k].reshape(gd[k].shape)), k
