"""The one-launch Replan at every step of its vertices per thread, against the oracle."""
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


@pytest.mark.parametrize("n", [1024 * k + e for k in (1, 2, 3, 4, 5, 6, 8, 10, 12, 15) for e in (0, 1) if k + e < 16])
def test_steps(P, n):
    rng = np.random.default_rng(n)
    pts = rng.random((n, 3))
    pts[0], pts[1] = 0.05, 0.95
    G, R = pair(P, W.build_rows(pts, 0, n, W.radius(n, 3), free(3)))
    h = np.sqrt(((pts - pts[1]) ** 2).sum(1)).astype(np.float32)
    for tag, args in (("prune", (0, 1, h)), ("all", (n - 1, 0, None, False)), ("lookahead", (n // 2, 1, h, True, True))):
        same((n, tag), G, R, *args)


@pytest.mark.parametrize("n", [513, 2002, 15_360])
@pytest.mark.parametrize("device", [False, True])
def test_results_of_a_renumbered_graph(P, n, device):
    """Outputs in caller order where the storage order is another one, each left out in turn,
    with the heuristic from host and device memory; a refused one changes nothing."""
    import torch
    rng = np.random.default_rng(n)
    pts = rng.random((n, 2))
    pts[0], pts[1] = 0.05, 0.95
    G, R = pair(P, W.build_rows(pts, 0, n, W.radius(n, 2), free(2)))
    h = np.sqrt(((pts - pts[1]) ** 2).sum(1)).astype(np.float32)
    G.snapshot_save()  # renumbers
    mem = (lambda x: torch.from_numpy(x).cuda()) if device else (lambda x: x)
    for root, hh in ((0, h), (n // 2, h), (n // 2, None), (3, h)):
        kw = {}
        if device:
            kw = dict(g_out=torch.empty(n, device="cuda"), parent_out=torch.empty(n, dtype=torch.int32, device="cuda"))
        g, p, st = G.replan(root, 1, None if hh is None else mem(hh), True, **kw)
        rc, so = R.replan(root, 1, hh, True)
        ref = R.state()
        if device:
            g, p = g.cpu().numpy(), p.cpu().numpy()
        assert np.array_equal(g.view(np.uint32), ref.g.view(np.uint32)) and np.array_equal(p, ref.parent)
        assert st["sum_P"] == so["sum_P"] and st["edges_examined"] == so["edges_examined"]
        bad = h.copy()
        bad[n - 1] = np.nan
        before = [x.copy() for x in G.get_policy()]
        with pytest.raises(P.PirrtError):
            G.replan(1, 0, mem(bad), True)
        assert all(np.array_equal(x, y) for x, y in zip(before, G.get_policy()))
