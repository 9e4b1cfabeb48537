"""The host Replan's state moves through pinned memory: sizes around the room every handle has,
host and device buffers, outputs left out, a heuristic that is refused, and growth, against
the device's own Replan of the same graph."""
import numpy as np
import pytest

import workloads as W

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def P():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2003_04920_amd as P
    P.load()
    return P


def graph(rng, n):
    e = [(int(rng.integers(0, v)), v, float(np.float32(rng.random()))) for v in range(1, n) for _ in range(3)]
    return W.from_edges(n, e)


@pytest.mark.parametrize("n", [1, 2, 511, 512, 513, 800, 3000])
@pytest.mark.parametrize("device", [False, True])
def test_same_as_the_device(P, monkeypatch, n, device):
    import torch
    rng = np.random.default_rng(n)
    b = graph(rng, n)
    monkeypatch.setenv("PIRRT_HOST_MAX", "100000")
    H = P.Graph()
    monkeypatch.setenv("PIRRT_HOST_MAX", "0")
    D = P.Graph()
    for G in (H, D):
        G.insert_rows(b)
    h = (rng.random(n) * 0.2).astype(np.float32)
    for root, goal, hh, prune in ((0, n - 1, h, True), (n // 2, 0, None, False), (n // 2, 0, h, True)):
        arg = torch.from_numpy(hh).cuda() if device and hh is not None else hh
        out = {}
        if device:
            out = dict(g_out=torch.empty(n, device="cuda"), parent_out=torch.empty(n, dtype=torch.int32, device="cuda"))
        gh, ph, sh = H.replan(root, goal, arg, prune, **out)
        if device:
            gh, ph = gh.cpu().numpy(), ph.cpu().numpy()
        gd, pd, sd = D.replan(root, goal, hh, prune)
        assert sh["on_host"] == 1 and sd["on_host"] == 0
        assert np.array_equal(gh.view(np.uint32), gd.view(np.uint32)) and np.array_equal(ph, pd)
        assert all(np.array_equal(x, y) for x, y in zip(H.get_policy(), D.get_policy()))
        assert sh["iterations"] == sd["iterations"] and sh["edges_examined"] == sd["edges_examined"]
    before = [x.copy() for x in H.get_policy()]
    bad = torch.full((n,), float("nan"), device="cuda") if device else np.full(n, np.nan, np.float32)
    with pytest.raises(P.PirrtError):
        H.replan(0, 0, bad, True)
    assert all(np.array_equal(x, y) for x, y in zip(before, H.get_policy()))
