"""The four-launch insert of small batches against the oracle: adjacency and insertion-time
policy after batches of 1 to 2,048 vertices (and just past that) onto graphs around its
tiles, with unsorted rows, parallel edges, orphans, edges inside the batch up to and past
what it keeps in LDS, from host and device rows, and from the device's own search."""
import numpy as np
import pytest

import oracle as O
import workloads as W
from oracle import rrg as RR

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def P():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2003_04920_amd as P
    P.load()
    return P


def rows(rng, n_old, n_new, deg, shuffle=True, inner=0.5):
    """Random forward rows: about deg entries each, a share of them inside the batch."""
    rp, col, cost = [0], [], []
    for v in range(n_old, n_old + n_new):
        k = int(rng.integers(0, 2 * deg + 1)) if v else 0
        us = []
        for _ in range(k):
            if v > n_old and (n_old == 0 or rng.random() < inner):
                us.append(int(rng.integers(n_old, v)))
            elif n_old:
                us.append(int(rng.integers(0, n_old)))
        if us and rng.random() < 0.2:
            us.append(us[0])  # a parallel edge
        us = us if shuffle else sorted(us)
        col += us
        cost += [float(rng.choice([0.0, 0.5, 1.0, rng.random()])) for _ in us]
        rp.append(len(col))
    return W.Batch(n_old, n_new, np.array(rp, np.int64), np.array(col, np.int32), np.array(cost, np.float32), 0.0)


def canonical(ptr, nbr, cst):
    at = np.repeat(np.arange(len(ptr) - 1), np.diff(ptr))
    order = np.lexsort((cst, nbr, at))
    return at[order], nbr[order], cst[order]


def check(tag, G, R):
    g, p, c = G.get_policy()
    ref = R.state()
    assert np.array_equal(g.view(np.uint32), ref.g.view(np.uint32)), tag
    assert np.array_equal(p, ref.parent), tag
    assert np.array_equal(c.view(np.uint32), ref.pcost.view(np.uint32)), tag
    a, b = canonical(*G.adjacency()), canonical(*R.adjacency())
    for x, y in zip(a, b):
        assert np.array_equal(x, y), tag


@pytest.mark.parametrize("device", [False, True])
@pytest.mark.parametrize("sizes", [(1, 1, 1, 30, 33), (2048, 2049, 2047, 1), (4095, 1, 1, 63, 64, 65), (4090, 100, 2000),
                                   (7, 900, 5000, 1500, 3)])
def test_batches(P, sizes, device):
    import torch
    rng = np.random.default_rng(sum(sizes))
    G, R = P.Graph(), O.Graph()
    n = 0
    for k, m in enumerate(sizes):
        b = rows(rng, n, m, 4 if m > 1500 else 9)
        if device and len(b.col):
            G.insert_batch(torch.from_numpy(b.row_ptr).cuda(), torch.from_numpy(b.col).cuda(),
                           torch.from_numpy(b.cost).cuda())
        else:
            G.insert_rows(b)
        assert R.insert_batch(b) == 0
        n += m
        check((sizes, k), G, R)
    G.replan(0, n - 1, None, False)
    assert R.replan(0, n - 1, None, False)[0] == 0
    check("after Replan", G, R)
    b = rows(rng, n, 50, 6)
    G.insert_rows(b)
    assert R.insert_batch(b) == 0
    check("after Replan and one more", G, R)


@pytest.mark.parametrize("deg", [6, 8, 20])
def test_inner_edges_in_and_past_lds(P, deg):
    """About 12k, 16k and 40k edges inside one batch of 2,000 (16,384 fit)."""
    rng = np.random.default_rng(deg)
    G, R = P.Graph(), O.Graph()
    for n_old, m in ((0, 2000), (2000, 2000)):
        b = rows(rng, n_old, m, deg, inner=0.97)
        G.insert_rows(b)
        assert R.insert_batch(b) == 0
        check((deg, n_old), G, R)


def test_chain_inside_a_batch(P):
    """The longest dependency: every vertex hangs below the one before it."""
    n = 2048
    b = W.path_graph(n, np.linspace(0.1, 1.0, n - 1).astype(np.float32))
    G, R = P.Graph(), O.Graph()
    G.insert_rows(b)
    assert R.insert_batch(b) == 0
    check("chain", G, R)


def test_bad_rows_leave_the_graph(P):
    rng = np.random.default_rng(4)
    G, R = P.Graph(), O.Graph()
    b = rows(rng, 0, 500, 6)
    G.insert_rows(b)
    assert R.insert_batch(b) == 0
    good = rows(rng, 500, 40, 5)
    for what in ("col", "cost"):
        bad = W.Batch(500, 40, good.row_ptr, good.col.copy(), good.cost.copy(), 0.0)
        if what == "col":
            bad.col[-1] = 600
        else:
            bad.cost[0] = -1.0
        with pytest.raises(P.PirrtError):
            G.insert_rows(bad)
        check(what, G, R)
    G.insert_rows(good)
    assert R.insert_batch(good) == 0
    check("good", G, R)


def test_connect_in_batches(P):
    """The search's rows go in without validation; points outside the cube go the long way."""
    d = 3
    rng = np.random.default_rng(9)
    obs = W.make_obstacles(d, 6, "mixed", 3)
    X = P.Rrg(d, obs)
    G, R = P.Graph(), O.Graph()
    pts = np.zeros((0, d))
    for k, m in enumerate((2, 300, 1, 1500, 64, 40)):
        new = rng.random((m, d))
        if k == 5:
            new[3] = 1.5
        X.add_points(new)
        pts = np.concatenate([pts, new])
        r = W.radius(len(pts), d)
        X.connect(len(pts) - m, r, G)
        rp, col, cost = RR.build_rows(pts, len(pts) - m, r, obs)
        assert R.insert_batch(W.Batch(len(pts) - m, m, rp, col, cost, r)) == 0
        check(k, G, R)
