"""Calls whose result is a few words that a kernel writes to host memory: samples over one
round, several rounds and past the workgroups whose counts are added up directly, the replan
test's count at both of its kernels, and a device heuristic that is refused."""
import numpy as np
import pytest

import workloads as W
from oracle import rrg as R

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def P():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2003_04920_amd as P
    P.load()
    return P


@pytest.mark.parametrize("d,count,filled", [(2, 1, False), (1, 255, False), (3, 256, True), (2, 5000, True),
                                            (2, 346_000, False), (6, 360_000, True)])
def test_samples(P, d, count, filled):
    """filled: a box leaves about a seventh of the cube, so the first round falls short."""
    obs = W.make_obstacles(d, 3, "mixed", d)
    if filled:
        obs = W.Obstacles(d, np.ones(1, np.int32), np.full((1, d), 0.5), np.full((1, d), 0.5 * 0.85 ** (1 / d)))
    G = P.Rrg(d, obs)
    k = G.sample(seed=5, stream=3, counter=7, count=count)
    want, wk = R.sample(d, 5, 3, 7, count, obs)
    assert k == wk
    assert np.array_equal(G.points(), want)


@pytest.mark.parametrize("n,first,count", [(20, 0, 20), (20, 3, 1), (40_000, 0, 16384), (40_000, 100, 16385),
                                           (40_000, 0, 40_000)])
def test_promising_counts(P, n, first, count):
    import torch
    rng = np.random.default_rng(count)
    b = W.path_graph(n, rng.random(n - 1).astype(np.float32))
    G = P.Graph()
    G.insert_rows(b)
    g = G.get_policy()[0]
    goal = n // 2
    for h in (None, rng.random(n).astype(np.float32) * 3):
        val = g + (0 if h is None else h)
        want = int(np.sum(val.astype(np.float32)[first:first + count] < g[goal]))
        assert G.promising_count(goal, h, first, count) == want
        if h is not None:
            assert G.promising_count(goal, torch.from_numpy(h).cuda(), first, count) == want


@pytest.mark.parametrize("n", [600, 20_000])
@pytest.mark.parametrize("bad", [float("nan"), -1.0])
def test_refused_heuristic_leaves_the_policy(P, n, bad):
    import torch
    G = P.Graph()
    G.insert_rows(W.path_graph(n, np.ones(n - 1, np.float32)))
    before = [x.copy() for x in G.get_policy()]
    h = torch.zeros(n, device="cuda")
    h[n - 1] = bad
    with pytest.raises(P.PirrtError):
        G.replan(0, n - 1, h)
    assert all(np.array_equal(a, b) for a, b in zip(before, G.get_policy()))
    h[n - 1] = 0.0
    g, _, _ = G.replan(0, n - 1, h)
    assert float(g[n - 1]) == n - 1
