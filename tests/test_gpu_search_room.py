"""What one crowded place leaves behind for a handle's later radius searches, against the
exploration oracle."""
import numpy as np
import pytest

import workloads as W
from test_gpu_search import check, stream

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def P():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2003_04920_amd as P
    P.load()
    return P


def test_room_comes_and_goes(P):
    """Crowded calls and sparse ones in turn on one handle, also many rows after a crowd."""
    rng = np.random.default_rng(8)
    d = 3
    obs = W.make_obstacles(d, 5, "mixed", 3)
    G = P.Rrg(d, obs, stream=stream())
    pts = np.zeros((0, d))
    for kind, m in (("sparse", 3000), ("crowd", 5000), ("sparse", 200), ("sparse", 4000), ("crowd", 300), ("sparse", 40)):
        new = rng.random((m, d)) if kind == "sparse" else 0.3 + 0.01 * rng.random((m, d))
        n_old, pts = len(pts), np.concatenate([pts, new])
        G.add_points(new)
        check(P, pts, n_old, 0.05, obs, G)
    check(P, pts, 0, 0.05, obs, G)  # sparse, crowded and sparse slabs in one call
    check(P, pts, len(pts) - 40, 0.05, obs, G)
