"""Device memory of the handles: arrays that grow, shrink out of use and grow again keep their
contents (against the oracle), and destroying the handles gives everything back."""
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


def free_bytes():
    import torch
    torch.cuda.synchronize()
    return torch.cuda.mem_get_info()[0]


@pytest.mark.parametrize("sizes", [(3, 1500, 40, 9000, 1, 30000), (40000, 10, 60000)])
def test_growth_keeps_the_graph(P, sizes):
    rng = np.random.default_rng(sizes[0])
    G, R = P.Graph(vertex_capacity=1), O.Graph()
    n = 0
    for m in sizes:
        b = rows(rng, n, m, 6)
        G.insert_rows(b)
        assert R.insert_batch(b) == 0
        n += m
        check(n, G, R)
        G.replan(0, n - 1, None, False)
        assert R.replan(0, n - 1, None, False)[0] == 0
        check((n, "after Replan"), G, R)


def test_memory_is_given_back(P):
    """Slabs and larger arrays of their own: all returned (2 MiB of slack for
    the runtime's own bookkeeping, after one pass that loads the kernels)."""
    obs = W.make_obstacles(3, 5, "mixed", 1)

    def once():
        X = P.Rrg(3, obs)
        X.sample(seed=1, stream=0, counter=0, count=300_000)
        G = P.Graph()
        X.connect(0, 0.02, G)
        G.replan(0, 1, None, False)
        used = free_bytes()
        X.close()
        G.close()
        return used

    once()
    before = free_bytes()
    inside = once()
    after = free_bytes()
    assert inside < before - (100 << 20)
    assert after >= before - (2 << 20)
