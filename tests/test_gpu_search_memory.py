"""A radius search that finds no memory for its candidate lists: the all-pairs search answers."""
import numpy as np
import pytest

import workloads as W
from oracle import rrg as R
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


def test_without_memory_for_the_lists(P, monkeypatch):
    import torch
    pts = np.random.default_rng(11).random((2500, 3))
    obs = W.make_obstacles(3, 5, "mixed", 3)
    for n_old in (0, 2400):
        monkeypatch.setenv("PIRRT_FAULT_INJECT", "search")
        G = P.Rrg(3, obs, stream=stream())
        monkeypatch.delenv("PIRRT_FAULT_INJECT")
        G.add_points(pts)
        check(P, pts, n_old, 0.15, obs, G)
        check(P, pts, n_old, 0.15, obs, G)
    monkeypatch.setenv("PIRRT_FAULT_INJECT", "search")
    G = P.Rrg(3, obs, stream=stream())
    monkeypatch.delenv("PIRRT_FAULT_INJECT")
    G.add_points(pts)
    rp, col, cost = (a.cpu().numpy() for a in G.rows(1000, 0.15, device=torch.device("cuda", 0)))
    orp, ocol, ocost = R.build_rows(pts, 1000, 0.15, obs)
    assert np.array_equal(rp, orp) and np.array_equal(col[:orp[-1]], ocol)
    assert np.array_equal(cost[:orp[-1]].view(np.uint32), ocost.view(np.uint32))
