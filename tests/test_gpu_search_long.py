"""Long rows of pirrt_rrg_rows against the exploration oracle: thousands of neighbours a row, and
ids of several windows of the finish by a workgroup."""
import numpy as np
import pytest

import workloads as W
from test_gpu_search import check, stream

pytestmark = pytest.mark.gpu

WINDOW = 1 << 18  # ids that are ordered together


@pytest.fixture(scope="module")
def P():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2003_04920_amd as P
    P.load()
    return P


@pytest.mark.parametrize("d,n,n_old,r", [(2, 9000, 0, 0.7), (3, 6000, 5990, 2.0), (1, 7000, 6000, 0.9), (8, 5000, 0, 3.0)])
def test_thousands(P, d, n, n_old, r):
    """Up to every earlier point in reach, several slabs of rows."""
    pts = np.random.default_rng(n).random((n, d))
    pts[n // 2:n // 2 + 50] = pts[:50]  # twice the same point: no edge
    check(P, pts, n_old, r, W.make_obstacles(d, 3, "mixed", d))


@pytest.mark.parametrize("n,rows", [(WINDOW - 1, 40), (WINDOW + 1, 40), (WINDOW + 300, 200), (3 * WINDOW + 77, 40)])
def test_windows(P, n, rows):
    """Rows of some 1,000 neighbours spread over one, two and four windows of ids; the last ids
    of the first window and the first ones of the second are neighbours of the last rows."""
    pts = np.random.default_rng(n).random((n, 2))
    pts[WINDOW - 40:WINDOW + 40] = 0.6 + 1e-3 * np.random.default_rng(1).random((len(pts[WINDOW - 40:WINDOW + 40]), 2))
    pts[-rows // 2:] = 0.6 + 1e-3 * np.random.default_rng(2).random((len(pts[-rows // 2:]), 2))
    assert check(P, pts, n - rows, float(np.sqrt(1000 / (np.pi * n))), W.make_obstacles(2, 6, "box", 4)) > 600 * rows // 2
