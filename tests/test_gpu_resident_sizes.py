"""The one-launch Replan at every step of its vertices per thread, against the oracle."""
import numpy as np
import pytest

import workloads as W
from test_gpu_pull import free, pair, same

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def P():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2003_04920_amd as P
    P.load()
    return P


@pytest.mark.parametrize("n", [1024 * k + e for k in (1, 2, 3, 4, 5, 6, 8, 10, 12, 15) for e in (0, 1) if k + e < 16])
def test_steps(P, n):
    rng = np.random.default_rng(n)
    pts = rng.random((n, 3))
    pts[0], pts[1] = 0.05, 0.95
    G, R = pair(P, W.build_rows(pts, 0, n, W.radius(n, 3), free(3)))
    h = np.sqrt(((pts - pts[1]) ** 2).sum(1)).astype(np.float32)
    for tag, args in (("prune", (0, 1, h)), ("all", (n - 1, 0, None, False)), ("lookahead", (n // 2, 1, h, True, True))):
        same((n, tag), G, R, *args)
