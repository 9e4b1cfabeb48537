"""The two forms of a single graph's Improve, marks and domain list (PIRRT_PULL=0) and
every row finding the domain by itself (PIRRT_PULL=1), against the oracle in the
multi-kernel loop: every row split, both domains, no pruning, more than 255 iterations
(the marks' byte wraps), long rows, empty rows and the level-synchronous Evaluate."""
import numpy as np
import pytest

import oracle as O
import workloads as W

pytestmark = pytest.mark.gpu

COUNTERS = ("iterations", "edges_examined", "sum_P", "sum_D", "changed_total", "mark_edges")


@pytest.fixture(scope="module")
def P():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2003_04920_amd as P
    P.load()
    return P


@pytest.fixture(params=["0", "1"], ids=["marks", "pull"])
def loop(request, monkeypatch):
    monkeypatch.setenv("PIRRT_SMALL", "0")
    monkeypatch.setenv("PIRRT_HOST_MAX", "0")
    monkeypatch.setenv("PIRRT_PULL", request.param)
    return request.param


def same(tag, G, R, root, goal, h, prune=True, lookahead=False):
    g, p, st = G.replan(root, goal, h, prune, lookahead=lookahead)
    rc, so = R.replan(root, goal, h, prune, lookahead=lookahead)
    assert rc == 0
    ref = R.state()
    assert np.array_equal(g.view(np.uint32), ref.g.view(np.uint32)), tag
    assert np.array_equal(p, ref.parent), tag
    for k in COUNTERS:
        assert st[k] == so[k], (tag, k)
    return st


def pair(P, b):
    G, R = P.Graph(), O.Graph()
    G.insert_rows(b)
    assert R.insert_batch(b) == 0
    return G, R


def free(d):
    return W.Obstacles(d, np.zeros(0, np.int32), np.zeros((0, d)), np.zeros((0, d)))


@pytest.mark.parametrize("variant", [0, 1, 2, 3])
@pytest.mark.parametrize("d,n", [(2, 1), (2, 3), (2, 33), (2, 1027), (3, 5000), (6, 4099)])
def test_forms(P, loop, monkeypatch, variant, d, n):
    monkeypatch.setenv("PIRRT_ROW_VARIANT", str(variant))
    rng = np.random.default_rng(n + d)
    pts = rng.random((n, d))
    pts[0] = 0.05
    pts[min(1, n - 1)] = 0.95 if n > 1 else 0.05
    G, R = pair(P, W.build_rows(pts, 0, n, W.radius(max(n, 3), d), free(d)))
    goal = min(1, n - 1)
    h = np.sqrt(((pts - pts[goal]) ** 2).sum(1)).astype(np.float32)
    for tag, args in (("prune", (0, goal, h)), ("again", (0, goal, h)), ("all", (n // 2, 0, None, False)),
                      ("lookahead", (0, goal, h, True, True)), ("lookahead, all", (n - 1, 0, h * 0, False, True))):
        same(tag, G, R, *args)


def test_many_iterations(P, loop):
    """A chain of shortcuts that improves one vertex an iteration, 600 iterations."""
    n = 1300
    edges = [(i, i + 1, 1.0) for i in range(n - 1)] + [(0, n - 1, 3000.0)]
    G, R = pair(P, W.from_edges(n, edges))
    par = np.arange(1, n + 1, dtype=np.int32)  # every vertex hangs below the next one
    par[0] = par[n - 1] = -1
    pc = np.ones(n, np.float32)
    par[n - 1], pc[n - 1] = 0, 3000.0
    g = np.zeros(n, np.float32)
    G.set_policy(g, par, pc)
    assert R.set_state(g, par, pc) == 0
    st = same("chain", G, R, 0, n // 2, None, False)
    assert st["iterations"] > 520


def test_long_and_empty_rows(P, loop):
    rng = np.random.default_rng(3)
    edges = []
    for v in range(1, 700):
        if v % 50 == 0:
            continue  # no forward edges; some never get any
        for u in rng.choice(v, min(v, int(rng.choice([1, 3, 64, 200]))), replace=False):
            edges.append((int(u), v, float(rng.choice([0.0, 1.0, 1.0, 2.5]))))
    G, R = pair(P, W.from_edges(700, edges))
    h = (rng.random(700) * 0.5).astype(np.float32)
    h[::7] = np.inf
    h[9] = 0.0
    for lookahead in (False, True):
        same("rows", G, R, 0, 9, h, True, lookahead)
        same("rows, all", G, R, 5, 0, h, False, lookahead)


def test_level_evaluate(P, loop, monkeypatch):
    monkeypatch.setenv("PIRRT_EVALUATE", "levels")
    wl = W.plain_2d(samples=2500, seed=8)
    G, R = pair(P, wl.batches[0])
    same("levels", G, R, 0, 1, wl.heuristic())
    same("levels, all", G, R, 7, 1, None, False)


def test_loop_from_graphs_and_timing(P, loop):
    """The same Replan repeated from a snapshot (captured loops), and the timing pass."""
    wl = W.plain_2d(samples=4000, seed=9)
    G, R = pair(P, wl.batches[0])
    h = wl.heuristic()
    G.snapshot_save()
    st0 = R.state()
    rc, so = R.replan(0, 1, h, True)
    ref = R.state()
    for i in range(4):
        G.snapshot_restore()
        g, p, st = G.replan(0, 1, h, True, timing=i == 3)
        assert np.array_equal(g.view(np.uint32), ref.g.view(np.uint32)) and np.array_equal(p, ref.parent)
        for k in COUNTERS:
            assert st[k] == so[k]
