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


@pytest.mark.parametrize("kw", [dict(timing=True), dict(truncated=True), dict(lookahead=True), dict()])
@pytest.mark.parametrize("n", [600, 20_000])
def test_refused_in_every_mode(P, monkeypatch, n, kw):
    """A device heuristic is checked while the Replan is enqueued: a refused one changes neither
    the policy, nor the roots, nor the caller's arrays, and the next call is as if it had not been."""
    import torch
    rng = np.random.default_rng(n)
    e = [(int(rng.integers(max(0, v - 50), v)), v, float(np.float32(rng.random()))) for v in range(1, n) for _ in range(3)]
    b = W.from_edges(n, e)
    G, H = P.Graph(), P.Graph()
    for X in (G, H):
        X.insert_rows(b)
    good = torch.from_numpy((rng.random(n) * 0.1).astype(np.float32)).cuda()
    bad = good.clone()
    bad[n // 2] = -1.0
    g_out = torch.full((n,), 7.0, device="cuda")
    p_out = torch.full((n,), 7, dtype=torch.int32, device="cuda")
    for root in (0, n // 3, 0):
        before = [x.copy() for x in G.get_policy()]
        with pytest.raises(P.PirrtError):
            G.replan(n - 1, root, bad, True, g_out=g_out.fill_(7.0), parent_out=p_out.fill_(7), **kw)
        assert bool((g_out == 7.0).all()) and bool((p_out == 7).all())
        assert all(np.array_equal(x, y) for x, y in zip(before, G.get_policy()))
        a = G.replan(root, n - 1, good, True, **kw)
        c = H.replan(root, n - 1, good, True, **kw)
        assert all(np.array_equal(x.cpu().numpy() if x.is_cuda else x, y.cpu().numpy()) for x, y in zip(a[:2], c[:2]))
        assert a[2]["iterations"] == c[2]["iterations"] and a[2]["sum_P"] == c[2]["sum_P"]


@pytest.mark.parametrize("count", [4095, 4096, 4097])
def test_promising_counts_host_heuristic(P, count):
    """Where a heuristic copied from host memory leaves the one workgroup for the counter."""
    n, first = 9000, 77
    rng = np.random.default_rng(count)
    G = P.Graph()
    G.insert_rows(W.path_graph(n, rng.random(n - 1).astype(np.float32)))
    g = G.get_policy()[0]
    h = rng.random(n).astype(np.float32) * 3
    want = int(np.sum((g + h).astype(np.float32)[first:first + count] < g[n // 2]))
    for _ in range(2):
        assert G.promising_count(n // 2, h, first, count) == want
