"""Evaluate by jumps against the oracle: paths of a length around one record, around the ring
of recorded steps and far past it, many exact ties, components without the root, roots that
move (the old policy then hangs below another vertex), single graphs past the size of the
one-launch Replan, small ones through the loop, and batches."""
import numpy as np
import pytest

import workloads as W
from test_gpu_batch import Problem, build, check_problem, lattice
from test_gpu_parity import assert_same_policy, assert_same_stats, gpu_graph

import oracle as O

pytestmark = pytest.mark.gpu

BIG = 15_500  # past the one-launch Replan


@pytest.fixture(scope="module")
def P():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2003_04920_amd as P
    P.load()
    return P


def broom(n, lengths):
    """Chains of the given lengths from vertex 0, over and over, then a component of its own
    (a chain) that no path from 0 reaches; costs differ, so left folds round differently."""
    rng = np.random.default_rng(n)
    e, v, k = [], 1, 0
    while v < n - 50:
        m = min(lengths[k % len(lengths)], n - 50 - v)
        k += 1
        ids = [0] + list(range(v, v + m))
        e += [(a, b, float(np.float32(rng.random()))) for a, b in zip(ids, ids[1:])]
        v += m
    e += [(u, u + 1, 0.5) for u in range(v, n - 1)]
    return W.from_edges(n, e)


CASES = {
    "chain": (lambda: W.path_graph(BIG, np.linspace(0.1, 1.0, BIG - 1).astype(np.float32)), BIG),
    "records": (lambda: broom(BIG, [1, 7, 8, 9, 15, 16, 17]), BIG),
    "ring": (lambda: broom(BIG, [126, 127, 128, 129, 135, 136, 137, 300]), BIG),
    "ties": (lambda: W.Batch(0, 126 * 126, *lattice(126, 3).rows, 0.0), 126 * 126),
}


@pytest.mark.parametrize("case", list(CASES))
@pytest.mark.parametrize("prune", [False, True])
def test_single(P, case, prune):
    make, n = CASES[case]
    b = make()
    G, R = gpu_graph(P), O.Graph()
    G.insert_rows(b)
    assert R.insert_batch(b) == 0
    for root, goal in ((0, n - 60), (n // 2, 0), (n // 2, 0), (0, n // 3)):
        g, p, st = G.replan(root, goal, None, prune)
        rc, so = R.replan(root, goal, None, prune)
        assert rc == 0 and st["rc"] == 0
        want = R.state()
        assert_same_policy((case, root), g, p, want.g, want.parent)
        assert_same_stats((case, root), st, so)


def test_small_graph_through_the_loop(P):
    """Timed Replans take the loop whatever the size."""
    b = broom(700, [8, 40, 129])
    G, R = gpu_graph(P), O.Graph()
    G.insert_rows(b)
    assert R.insert_batch(b) == 0
    for root in (0, 600, 3):
        g, p, st = G.replan(root, 699, None, False, timing=True)
        assert R.replan(root, 699, None, False)[0] == 0
        want = R.state()
        assert_same_policy(root, g, p, want.g, want.parent)


def test_batch(P):
    rows = lambda b: (b.row_ptr, b.col, b.cost)  # noqa: E731
    probs = [lattice(70, 5),
             Problem("ring", rows(broom(3000, [127, 128, 129])), 0, 900, np.zeros(3000, np.float32), prune=False),
             Problem("chain", rows(W.path_graph(2100, np.ones(2099, np.float32))), 0, 2099, None),
             Problem("records", rows(broom(1237, [7, 8, 9])), 0, 5, None),
             lattice(45, 6)]
    B = build(P, probs)
    off = B.offsets
    for roots in ([p.root for p in probs], [p.n // 2 for p in probs]):
        R = []
        for pr, root in zip(probs, roots):
            r = O.Graph()
            assert r.insert_batch(W.Batch(0, pr.n, *pr.rows, 0.0)) == 0
            for q in ([pr.root], [pr.root, root])[roots[0] != probs[0].root]:
                assert r.replan(q, pr.goal, None, False)[0] == 0
            R.append(r.state())
        g, p, st = B.replan(roots, [pr.goal for pr in probs], None, False)
        assert all(s["rc"] == 0 for s in st)
        for i, pr in enumerate(probs):
            check_problem("batch", g, p, int(off[i]), pr, R[i].g, R[i].parent)
