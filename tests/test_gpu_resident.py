"""The one-launch Replan of graphs of 513 to 15,360 vertices (resident workgroups) against
the oracle: sizes around its blocks, rows longer than its registers hold, ties, parallel
and zero-cost edges, changing roots, starting policies with cycles, the iteration cap, two
handles at once, and the multi-kernel loop taking over when its workgroups cannot meet."""
import threading

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


def same(tag, G, R, root, goal, h, prune=True, lookahead=False, max_iters=0):
    g, p, st = G.replan(root, goal, h, prune, lookahead=lookahead, allow_not_converged=max_iters > 0)
    rc, so = R.replan(root, goal, h, prune, max_iters=max_iters, lookahead=lookahead)
    ref = R.state()
    assert st["on_host"] == 0, tag
    assert (rc == 0) == (st["rc"] == 0), tag
    assert np.array_equal(g.view(np.uint32), ref.g.view(np.uint32)), tag
    assert np.array_equal(p, ref.parent), tag
    for k in COUNTERS:
        assert st[k] == so[k], (tag, k)
    return st


def pair(P, batches, **kw):
    G, R = P.Graph(**kw), O.Graph()
    for b in batches:
        G.insert_rows(b)
        assert R.insert_batch(b) == 0
    return G, R


def grid(n, d, seed, radius):
    rng = np.random.default_rng(seed)
    pts = rng.random((n, d))
    pts[0], pts[1] = 0.05, 0.95
    return pts, W.build_rows(pts, 0, n, radius, W.Obstacles(d, np.zeros(0, np.int32), np.zeros((0, d)), np.zeros((0, d))))


@pytest.mark.parametrize("n", [513, 640, 1024, 1025, 2048, 2049, 4096, 4097, 8192, 8193, 15359, 15360, 15361])
@pytest.mark.parametrize("mode", ["prune", "all", "lookahead"])
def test_sizes(P, n, mode):
    d = 2 + n % 2
    pts, b = grid(n, d, n, W.radius(n, d))
    G, R = pair(P, [b])
    h = np.sqrt(((pts - pts[1]) ** 2).sum(1)).astype(np.float32)
    same("first", G, R, 0, 1, h, mode != "all", mode == "lookahead")
    same("again", G, R, 0, 1, h, mode != "all", mode == "lookahead")
    same("other root", G, R, n - 1, 0, None, mode != "all", mode == "lookahead")
    same("back", G, R, 0, n // 2, None, mode != "all", mode == "lookahead")


def test_growth_past_the_limit(P):
    """Batches inserted between Replans, from the one-launch sizes into the loop's."""
    n = 16_000
    rng = np.random.default_rng(2)
    pts = rng.random((n, 2))
    pts[0], pts[1] = 0.05, 0.95
    free = W.Obstacles(2, np.zeros(0, np.int32), np.zeros((0, 2)), np.zeros((0, 2)))
    h = np.sqrt(((pts - pts[1]) ** 2).sum(1)).astype(np.float32)
    G, R = P.Graph(), O.Graph()
    at = 0
    for to in (700, 750, 3000, 3010, 9000, 15_000, 15_360, 15_361, 16_000):
        b = W.build_rows(pts, at, to - at, W.radius(to, 2), free)
        G.insert_rows(b)
        assert R.insert_batch(b) == 0
        same("n=%d" % to, G, R, 0, 1, h[:to])
        at = to


@pytest.mark.parametrize("lookahead", [False, True])
def test_long_rows(P, lookahead):
    """Rows of 63 to several hundred entries: the first 64 sit in registers, aligned to
    quads, the rest come from memory."""
    rng = np.random.default_rng(11)
    edges = []
    for v in range(1, 900):
        k = int(rng.choice([1, 2, 30, 61, 62, 63, 64, 65, 66, 67, 68, 130, 400]))
        for u in rng.choice(v, min(k, v), replace=False):
            edges.append((int(u), v, float(np.float32(rng.choice([0.5, 1.0, 1.5, rng.random()])))))
    G, R = pair(P, [W.from_edges(900, edges)])
    h = (rng.random(900) * 0.2).astype(np.float32)
    h[7] = 0.0
    same("long", G, R, 0, 7, h, True, lookahead)
    same("long, all", G, R, 3, 0, None, False, lookahead)


def test_ties_parallel_and_zero_edges(P):
    """Unit costs, parallel edges of equal and different cost, zero-cost edges."""
    rng = np.random.default_rng(5)
    edges = []
    for v in range(1, 1500):
        for u in rng.choice(v, min(v, 6), replace=False):
            c = float(rng.choice([0.0, 1.0, 1.0, 1.0, 2.0]))
            edges.append((int(u), v, c))
            if rng.random() < 0.3:
                edges.append((int(u), v, c if rng.random() < 0.5 else c + 1.0))
    G, R = pair(P, [W.from_edges(1500, edges)])
    for root, goal, prune in ((0, 1, True), (1400, 3, False), (9, 1499, True), (0, 700, False)):
        same("root %d" % root, G, R, root, goal, None, prune)


def test_starting_policies(P):
    """Orphans, wrong g, and parents that form cycles away from the root."""
    n = 1300
    pts, b = grid(n, 2, 8, W.radius(n, 2))
    rng = np.random.default_rng(1)
    row = b.row_ptr
    for kind in ("orphans", "random", "cycles"):
        G, R = pair(P, [b])
        g = (rng.random(n) * 3).astype(np.float32)
        par, pc = np.full(n, -1, np.int32), np.zeros(n, np.float32)
        if kind != "orphans":
            for v in range(2, n):
                k = row[v] + rng.integers(0, max(1, row[v + 1] - row[v]))
                if k < row[v + 1]:
                    u, c = int(b.col[k]), b.cost[k]
                    if kind == "cycles" and v % 3 == 0:
                        par[u], pc[u] = v, c  # the lower vertex hangs below the higher one
                        if u:
                            par[v], pc[v] = u, c
                    else:
                        par[v], pc[v] = u, c
        par[0] = -1
        G.set_policy(g, par, pc)
        assert R.set_state(g, par, pc) == 0
        same(kind, G, R, 0, 1, None)
        same(kind + ", second", G, R, 5, 1, None, False)


@pytest.mark.parametrize("cap", [1, 2, 5])
def test_iteration_cap(P, cap):
    pts, b = grid(3000, 2, 4, W.radius(3000, 2))
    G, R = pair(P, [b], max_iters=cap)
    same("cap", G, R, 0, 1, np.sqrt(((pts - pts[1]) ** 2).sum(1)).astype(np.float32), True, False, cap)


def test_snapshot_and_unreachable_goal(P):
    n = 2000
    pts, b = grid(n, 3, 9, 0.6 * W.radius(n, 3))  # many components
    G, R = pair(P, [b])
    G.snapshot_save()
    st0 = R.state()
    for _ in range(3):
        G.snapshot_restore()
        assert R.set_state(st0.g, st0.parent, st0.pcost) == 0
        same("restored", G, R, 0, 1, None)
        same("restored, other root", G, R, 17, 3, None)


def test_closed_gate(P, monkeypatch):
    """The gate found closed: nothing is changed and the multi-kernel loop replans."""
    pts, b = grid(2500, 2, 6, W.radius(2500, 2))
    h = np.sqrt(((pts - pts[1]) ** 2).sum(1)).astype(np.float32)
    monkeypatch.setenv("PIRRT_FAULT_INJECT", "gate")
    G, R = pair(P, [b])
    same("closed", G, R, 0, 1, h)
    same("open again", G, R, 4, 1, h)


def test_two_handles_at_once(P):
    """Two threads, each replanning its own graph on its own stream."""
    import torch
    n = 12_000
    errs = []
    jobs = []
    for i in range(2):
        pts, b = grid(n + 500 * i, 2, 20 + i, W.radius(n, 2))
        R = O.Graph()
        assert R.insert_batch(b) == 0
        h = np.sqrt(((pts - pts[1]) ** 2).sum(1)).astype(np.float32)
        assert R.replan(0, 1, h, True)[0] == 0
        jobs.append((b, h, R.state()))

    def work(b, h, ref):
        try:
            s = torch.cuda.Stream()
            G = P.Graph(stream=s.cuda_stream)
            G.insert_rows(b)
            G.snapshot_save()
            for _ in range(10):
                G.snapshot_restore()
                g, p, _ = G.replan(0, 1, h)
                assert np.array_equal(g.view(np.uint32), ref.g.view(np.uint32)) and np.array_equal(p, ref.parent)
        except BaseException as e:
            errs.append(e)

    ts = [threading.Thread(target=work, args=j) for j in jobs]
    for t in ts:
        t.start()
    for t in ts:
        t.join()
    assert not errs, errs
