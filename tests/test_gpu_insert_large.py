"""The insertion-time policy of batches past 2,048 vertices (offers by rounds, not levels)
and the renumbering after them, against the oracle: chains as long as the batch, stars that
overflow a workgroup's list, components no batch edge reaches, ties, and batches onto graphs
whose vertices are renumbered."""
import numpy as np
import pytest

import oracle as O
import workloads as W
from test_gpu_insert import check, rows

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def P():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2003_04920_amd as P
    P.load()
    return P


def chain(n):
    return W.path_graph(n, np.linspace(0.1, 1.0, n - 1).astype(np.float32))


def star(n):
    """One workgroup reaches all: 0 next to every vertex, every third also to its predecessor."""
    e = [(0, v, 1.0) for v in range(1, n)] + [(v - 1, v, 0.0 if v % 2 else 0.25) for v in range(3, n, 3)]
    return W.from_edges(n, e)


def ties(n):
    """Unit costs on a shuffled lattice: every vertex has several equal parents."""
    side = int(n ** 0.5)
    perm = np.random.default_rng(n).permutation(side * side)
    e = [(int(perm[v]), int(perm[w]), 1.0) for v in range(side * side)
         for w in (v + 1 if (v + 1) % side else 0, v + side) if 0 < w < side * side]
    return W.from_edges(side * side, e)


@pytest.mark.parametrize("make,n", [(chain, 2049), (chain, 2500), (star, 2100), (star, 9000), (ties, 70 ** 2)])
def test_one_batch(P, make, n):
    b = make(n)
    G, R = P.Graph(), O.Graph()
    G.insert_rows(b)
    assert R.insert_batch(b) == 0
    check(make.__name__, G, R)
    G.replan(0, n - 1, None, False)
    assert R.replan(0, n - 1, None, False)[0] == 0
    check("after Replan", G, R)


@pytest.mark.parametrize("sizes", [(2049, 2049, 3000), (1, 2100, 16000, 2500), (20000, 5, 5000)])
def test_batches_onto_a_graph(P, sizes):
    rng = np.random.default_rng(sum(sizes))
    G, R = P.Graph(), O.Graph()
    n = 0
    for k, m in enumerate(sizes):
        b = rows(rng, n, m, 5, inner=0.8)
        G.insert_rows(b)
        assert R.insert_batch(b) == 0
        n += m
        check((sizes, k), G, R)
        G.replan(0, n - 1, None, k % 2 == 0)
        assert R.replan(0, n - 1, None, k % 2 == 0)[0] == 0
        check((sizes, k, "after Replan"), G, R)
