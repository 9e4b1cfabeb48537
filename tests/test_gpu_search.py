"""The matrix-core radius search of pirrt_rrg_rows against the exploration oracle, entry
for entry: sizes around its tiles, blocks and chunks, points it must get right at the
threshold (lattices, faces of the cube, duplicates, clusters), candidate lists that turn
out too short, and the calls that fall back to the all-pairs search."""
import numpy as np
import pytest

import workloads as W
from oracle import rrg as R

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def P():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2003_04920_amd as P
    P.load()
    return P


def stream():
    import torch
    return torch.cuda.current_stream().cuda_stream


def check(P, pts, n_old, r, obs, G=None):
    if G is None:
        G = P.Rrg(pts.shape[1], obs, stream=stream())
        G.add_points(pts)
    rp, col, cost = G.rows(n_old, r)
    orp, ocol, ocost = R.build_rows(pts, n_old, r, obs)
    assert np.array_equal(rp, orp) and np.array_equal(col, ocol)
    assert np.array_equal(cost.view(np.uint32), ocost.view(np.uint32))
    return int(rp[-1])


@pytest.mark.parametrize("d", range(1, 9))
@pytest.mark.parametrize("n_old,rows", [(0, 1), (1, 31), (7, 33), (255, 128), (256, 129), (1023, 513)])
def test_sizes(P, d, n_old, rows):
    rng = np.random.default_rng(1000 * d + rows)
    obs = W.make_obstacles(d, 6, "mixed", d + rows)
    n = n_old + rows
    # dimension 1 has 2 r n neighbours a point, dimension 8 few inside the cube
    r = min(W.radius(max(n, 3), d), 0.2) if d == 1 else W.radius(max(n, 3), d)
    check(P, rng.random((n, d)), n_old, r, obs)


def test_chunks_many_points_few_rows(P):
    rng = np.random.default_rng(5)
    obs = W.make_obstacles(6, 40, "sphere", 9)
    pts = rng.random((20011, 6))
    G = P.Rrg(6, obs, stream=stream())
    G.add_points(pts)
    for n_old in (20010, 19900, 19000):
        assert check(P, pts, n_old, W.radius(len(pts), 6), obs, G) > 0


@pytest.mark.parametrize("d,step", [(2, 1 / 32), (3, 1 / 8), (6, 1 / 3)])
def test_lattice_at_the_threshold(P, d, step):
    """Every neighbour of a lattice point lies at the radius exactly, or just past it;
    the lattice includes the faces and corners of the cube and every point twice."""
    k = int(round(1 / step)) + 1
    axes = np.meshgrid(*[np.arange(k) * step] * d, indexing="ij")
    pts = np.stack([a.ravel() for a in axes], 1)
    pts = np.concatenate([pts, pts])[np.random.default_rng(d).permutation(2 * k ** d)][:3000]
    for r in (step, np.nextafter(step, 0), np.sqrt(2) * step):
        check(P, pts, 0, float(r), None)


@pytest.mark.parametrize("members", [60, 300, 700])
def test_clusters_outgrow_the_lists(P, members):
    """Clusters denser than the lists' first room: longer lists up to 512 candidates a
    row (60, 300), rows finished by a workgroup each above (700)."""
    rng = np.random.default_rng(members)
    pts = rng.random((2500, 3))
    pts[800:800 + members] = 0.4 + 1e-3 * rng.random((members, 3))  # ids close together: one chunk's list
    obs = W.make_obstacles(3, 5, "sphere", 3)
    G = P.Rrg(3, obs, stream=stream())
    G.add_points(pts)
    for n_old in (0, 2300, 1200):
        check(P, pts, n_old, 0.05, obs, G)


@pytest.mark.parametrize("r", [1e-7, 1e-3, 0.9, 2.0, 1e200])
def test_radii_small_and_large(P, r):
    rng = np.random.default_rng(17)
    pts = rng.random((400, 4))
    pts[200:220] = pts[:20] + 3e-8
    check(P, pts, 0, r, W.make_obstacles(4, 3, "box", 2))


def test_points_outside_the_cube(P):
    """A point outside [0, 1]^d, also one that arrives later, takes the all-pairs search."""
    rng = np.random.default_rng(23)
    pts = rng.random((700, 3))
    obs = W.make_obstacles(3, 5, "mixed", 8)
    G = P.Rrg(3, obs, stream=stream())
    G.add_points(pts)
    check(P, pts, 100, 0.2, obs, G)
    more = 5.0 * rng.random((50, 3)) - 2.0
    G.add_points(more)
    every = np.concatenate([pts, more])
    check(P, every, 600, 0.2, obs, G)
    check(P, 1e6 * rng.random((300, 2)), 0, 1e5, None)


def test_wide_blocks(P):
    """From 65,536 rows on a wave takes four blocks of rows: the first and the last rows
    against the oracle, all of them against the same rows asked for in parts."""
    d, n = 2, 66_003
    obs = W.make_obstacles(d, 8, "box", 1)
    pts = np.random.default_rng(2).random((n, d))
    r = W.radius(n, d)
    G = P.Rrg(d, obs, stream=stream())
    G.add_points(pts)
    rp, col, cost = G.rows(0, r)
    orp, ocol, ocost = R.build_rows(pts[:3000], 0, r, obs)
    assert np.array_equal(rp[:3001], orp) and np.array_equal(col[:orp[-1]], ocol)
    for n_old in (n - 700, n - 5000, 40_000):
        rp2, col2, cost2 = G.rows(n_old, r)
        assert np.array_equal(rp[n_old:] - rp[n_old], rp2) and np.array_equal(col[rp[n_old]:], col2)
        assert np.array_equal(cost[rp[n_old]:].view(np.uint32), cost2.view(np.uint32))
        if n_old == n - 700:
            orp, ocol, ocost = R.build_rows(pts, n_old, r, obs)
            assert np.array_equal(rp2, orp) and np.array_equal(col2, ocol)
            assert np.array_equal(cost2.view(np.uint32), ocost.view(np.uint32))


def test_device_rows_capacity(P):
    """Device buffers are written where they are when the rows fit, and stay untouched
    when they do not."""
    import ctypes
    import torch
    rng = np.random.default_rng(3)
    pts = rng.random((1500, 3))
    G = P.Rrg(3, None, stream=stream())
    G.add_points(pts)
    orp, ocol, ocost = R.build_rows(pts, 1000, 0.15, None)
    m = int(orp[-1])
    rp = torch.full((501,), -7, dtype=torch.int64, device="cuda")
    col = torch.full((m + 5,), -7, dtype=torch.int32, device="cuda")
    nnz = ctypes.c_int64(0)
    lib = P.load()
    args = lambda cap, c, w: lib.pirrt_rrg_rows(G._h, 1000, 0.15, rp.data_ptr(), c, w, cap, ctypes.byref(nnz), 1)
    torch.cuda.synchronize()
    assert args(m - 1, col.data_ptr(), None) == -1 and nnz.value == m
    assert (rp == -7).all() and (col == -7).all()
    assert args(m, col.data_ptr(), None) == 0
    assert np.array_equal(rp.cpu().numpy(), orp) and np.array_equal(col.cpu().numpy()[:m], ocol)
    assert (col[m:] == -7).all()


@pytest.mark.parametrize("d,count", [(2, 64), (3, 65), (2, 129), (5, 200)])
def test_many_obstacles(P, d, count):
    """More obstacles than one mask, and than the bounding spheres kept in LDS, holds;
    some far outside the cube, some huge: sampling and rows as the oracle has them."""
    obs = W.make_obstacles(d, count, "mixed", count)
    obs.size[:] *= 0.3
    obs.centre[-3:] += 7.0
    obs.size[-1] += 6.5
    obs.centre[1] = 60.0
    n = 500
    G = P.Rrg(d, obs, stream=stream())
    G.add_points(np.stack([np.full(d, 0.05), np.full(d, 0.95)]))
    c = G.sample(seed=4, stream=1, counter=0, count=n)
    want, wc = R.sample(d, 4, 1, 0, n, obs)
    pts = G.points()
    assert c == wc and np.array_equal(pts[2:], want)
    check(P, pts, 100, W.radius(n, d), obs, G)


@pytest.mark.parametrize("d", [1, 3, 8])
@pytest.mark.parametrize("members", [513, 514, 769, 1600, 4097, 4098])
def test_rows_of_hundreds(P, d, members):
    """A cluster whose last row has members - 1 candidates: up to 512 by 32 lanes, up to
    4,096 by a workgroup, the all-pairs search above; then rows of few candidates and the
    cluster's again with the same handle."""
    rng = np.random.default_rng(members + d)
    pts = rng.random((members + 600, d))
    pts[:, 0] = 0.5 + 0.5 * pts[:, 0]
    pts[300:300 + members] = 0.3 + 0.02 * rng.random((members, d))
    obs = W.make_obstacles(d, 5, "mixed", 3)
    # the centre is not crossed by chance alone: an obstacle inside the cluster
    obs.centre[0], obs.size[0] = 0.31, 0.002
    G = P.Rrg(d, obs, stream=stream())
    G.add_points(pts)
    n = len(pts)
    for n_old in (300 + members - 40, n - 200, 300 + members - 520):
        check(P, pts, n_old, 0.08, obs, G)


def test_device_rows_in_slabs(P):
    """More rows than one slab holds, into device buffers: the same as on the host."""
    import torch
    pts = np.random.default_rng(4).random((66_003, 2))
    r = W.radius(len(pts), 2)
    G = P.Rrg(2, W.make_obstacles(2, 8, "box", 1), stream=stream())
    G.add_points(pts)
    want = G.rows(0, r)
    got = G.rows(0, r, device=torch.device("cuda", 0))
    torch.cuda.synchronize()
    for a, b in zip(want, got):
        b = b.cpu().numpy()
        assert np.array_equal(a.view(np.uint8), b.view(np.uint8))


def test_slabs_of_long_rows(P):
    """Rows of up to some 900 candidates, several slabs of them, a workgroup a row."""
    pts = np.random.default_rng(6).random((20_000, 2))
    obs = W.make_obstacles(2, 4, "mixed", 5)
    G = P.Rrg(2, obs, stream=stream())
    G.add_points(pts)
    r = 0.12
    rp, col, cost = G.rows(0, r)
    for lo, hi in ((0, 4000), (19_000, 20_000)):
        orp, ocol, ocost = R.build_rows(pts[:hi], lo, r, obs)
        assert np.array_equal(rp[lo:hi + 1] - rp[lo], orp)
        assert np.array_equal(col[rp[lo]:rp[hi]], ocol)
        assert np.array_equal(cost[rp[lo]:rp[hi]].view(np.uint32), ocost.view(np.uint32))
