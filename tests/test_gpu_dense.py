"""Improve that takes pull form only in the iterations whose promising set is dense
(PIRRT_PULL=2 forces the rule of large graphs at any size), against the oracle: both forms in
one Replan, the marks' byte that wraps while the set is dense, all row splits, both domains."""
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


@pytest.fixture(autouse=True)
def loop(monkeypatch):
    monkeypatch.setenv("PIRRT_SMALL", "0")
    monkeypatch.setenv("PIRRT_HOST_MAX", "0")
    monkeypatch.setenv("PIRRT_PULL", "2")


@pytest.mark.parametrize("variant", [0, 1, 2, 3])
@pytest.mark.parametrize("d,n", [(2, 1), (2, 3), (2, 1027), (3, 5000), (6, 4099), (6, 20_000)])
def test_forms(P, monkeypatch, variant, d, n):
    monkeypatch.setenv("PIRRT_ROW_VARIANT", str(variant))
    rng = np.random.default_rng(n + d)
    pts = rng.random((n, d))
    pts[0] = 0.05
    pts[min(1, n - 1)] = 0.95 if n > 1 else 0.05
    G, R = pair(P, W.build_rows(pts, 0, n, W.radius(max(n, 3), d), free(d)))
    goal = min(1, n - 1)
    h = np.sqrt(((pts - pts[goal]) ** 2).sum(1)).astype(np.float32)
    for tag, args in (("prune", (0, goal, h)), ("no h", (0, goal, None)), ("moved", (n // 2, 0, None)),
                      ("lookahead", (0, goal, h, True, True)), ("lookahead, no h", (n // 3, goal, None, True, True)),
                      ("all", (0, goal, None, False)), ("again", (0, goal, h))):
        same(tag, G, R, *args)


@pytest.mark.parametrize("share", [0.3, 0.36, 0.9])
def test_many_iterations(P, share):
    """600 iterations with about this share of the vertices promising throughout."""
    n = 1300
    edges = [(i, i + 1, 1.0) for i in range(n - 1)] + [(0, n - 1, 3000.0)]
    G, R = pair(P, W.from_edges(n, edges))
    par = np.arange(1, n + 1, dtype=np.int32)
    par[0] = par[n - 1] = -1
    pc = np.ones(n, np.float32)
    par[n - 1], pc[n - 1] = 0, 3000.0
    g = np.zeros(n, np.float32)
    G.set_policy(g, par, pc)
    assert R.set_state(g, par, pc) == 0
    h = np.full(n, 0.0, np.float32)
    h[int(share * n):n - 1] = np.inf  # never promising
    st = same("chain", G, R, 0, n - 1, h)
    assert st["iterations"] > min(255, int(share * n) - 5)


def test_without_pruning(P):
    """Promising sets that grow from a few vertices to all of them (a root far below the one
    the policy was built for), and one that stays at a component of two."""
    n = 6000
    rng = np.random.default_rng(3)
    b = W.build_rows(rng.random((n, 2)), 0, n, W.radius(n, 2), free(2))
    rows = (np.concatenate([b.row_ptr, b.row_ptr[-1] + np.array([0, 1])]), np.append(b.col, np.int32(n)),
            np.append(b.cost, np.float32(0.5)))
    G, R = pair(P, W.Batch(0, n + 2, *rows, 0.0))
    seen = []
    for root, goal in ((n - 1, 0), (n, n + 1), (0, n - 1), (n // 2, 5)):
        st = same(root, G, R, root, goal, None, False)
        seen.append(st["sum_P"] / st["iterations"])
    assert min(seen) < 3 and max(seen) > n / 3
