"""Batches that stop at the iteration cap: every problem ends with the oracle's policy and the g
of that policy, also where the workgroups of a launch loop over several units of slots, where
other problems converge before the cap, where the cap falls on the first iteration that climbs
by jumps, and when a second call goes on from the capped state."""
import numpy as np
import pytest

import oracle as O
import workloads as W
from test_gpu_batch import STAT_KEYS, Problem, build, check_problem, lattice
from test_gpu_jumps import broom

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def P():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2003_04920_amd as P
    P.load()
    return P


def grid(side, seed, root, goal):
    """side x side vertices, row by row, with edge costs U(0.5, 1)."""
    n = side * side
    v = np.arange(n)
    up, left = v >= side, v % side > 0
    ptr = np.concatenate([[0], np.cumsum(up.astype(np.int64) + left)])
    at = np.repeat(v, np.diff(ptr))
    second = np.arange(len(at)) > ptr[at]
    col = np.where(up[at] & ~second, at - side, at - 1).astype(np.int32)
    cost = np.random.default_rng(seed).uniform(0.5, 1.0, len(col)).astype(np.float32)
    return Problem("grid-%d" % side, (ptr.astype(np.int64), col, cost), root, goal, None, prune=False)


def check(P, probs, cap, calls=2):
    roots, goals = [p.root for p in probs], [p.goal for p in probs]
    B = build(P, probs, max_iters=cap)
    off = B.offsets
    R = []
    for pr in probs:
        r = O.Graph()
        assert r.insert_batch(W.Batch(0, pr.n, *pr.rows, 0.0)) == 0
        R.append(r)
    capped = 0
    for call in range(calls):
        g, parent, stats = B.replan(roots, goals, None, False, allow_not_converged=True)
        for i, pr in enumerate(probs):
            rc, st = R[i].replan(pr.root, pr.goal, None, False, max_iters=cap)
            want = R[i].state()
            check_problem("cap %d call %d" % (cap, call), g, parent, int(off[i]), pr, want.g, want.parent)
            for k in STAT_KEYS:
                assert stats[i][k] == st[k], (cap, call, pr.name, k)
            capped += rc != 0
    return capped


@pytest.mark.parametrize("cap", [1, 2, 3, 9, 17])
def test_units_past_the_workgroups(P, monkeypatch, cap):
    """Eight workgroups over some 80 units of 256 slots."""
    monkeypatch.setenv("PIRRT_BATCH_BLOCKS", "8")
    rows = lambda b: (b.row_ptr, b.col, b.cost)  # noqa: E731
    probs = [lattice(70, 5),
             Problem("records", rows(broom(3000, [7, 8, 9, 127])), 2900, 5, None),
             Problem("one", (np.zeros(2, np.int64), np.zeros(0, np.int32), np.zeros(0, np.float32)), 0, 0, None),
             grid(110, 1, 110 * 55, 0),
             lattice(12, 6)]
    assert check(P, probs, cap) > 0


@pytest.mark.parametrize("cap", [2, 20])
def test_more_slots_than_the_chip_holds_threads(P, cap):
    """Past 524,288 slots (2,048 workgroups of 256) with the default launch shape."""
    probs = [grid(430, 2, 430 * 215, 0), grid(437, 3, 0, 5), grid(441, 4, 441 * 441 - 1, 7)]
    assert sum(p.n for p in probs) > 2048 * 256
    assert check(P, probs, cap) > 0


@pytest.mark.parametrize("cap", [16, 17, 18])
def test_cap_at_the_first_jumps(P, cap):
    """A problem of more than 2^19 vertices climbs by jumps from its 17th iteration on."""
    pr = grid(725, 5, 725 * 362, 0)
    assert pr.n > 1 << 19
    assert check(P, [pr], cap) > 0
