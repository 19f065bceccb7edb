"""GPU parity of the kNN paths behind the cell directory: the cell select, the wider scan of queries near
the faces of the cloud, and the scans of what both leave open (of every point up to 16,384 points, of a
stream of cells above), at the sizes and clouds where a query changes from one to the next.  Neighbour
lists are exact."""
import numpy as np
import pytest

from paper_2609_24802_amd import synth
from tests.test_gpu_knn import check, cloud, dev

pytestmark = pytest.mark.gpu


def points(kind, n):
    rng = np.random.default_rng(n)
    if kind == "box":         # a long box: the longest axis sets the table, most cells are empty
        return (rng.random((n, 3)) * [40.0, 1.0, 0.02]).astype(np.float32)
    if kind == "outlier":     # one far point: everything else shares a cell
        p = rng.random((n, 3)).astype(np.float32)
        p[17] = [1e4, -3e4, 5.0]
        return p
    if kind == "same":        # coincident points, and a few others
        p = np.full((n, 3), 0.25, np.float32)
        p[:40] = rng.random((40, 3))
        return p
    if kind == "far":         # coordinates whose spacing is a large part of a cell
        return (1000.0 + rng.random((n, 3)) * 0.02).astype(np.float32)
    if kind == "tiny":        # squared distances that underflow
        return (rng.random((n, 3)) * 1e-22).astype(np.float32)
    if kind == "holes":       # non-finite points among the others
        p = rng.random((n, 3)).astype(np.float32)
        p[rng.integers(0, n, 50), rng.integers(0, 3, 50)] = rng.choice([np.nan, np.inf, -np.inf], 50)
        return p
    if kind == "many holes":  # more of them than a block of cells may hold
        p = rng.random((n, 3)).astype(np.float32)
        p[: n // 8, 1] = np.nan
        p[rng.integers(0, n, n // 50)] = np.inf
        return p
    if kind == "clumps":      # clumps of more points than a block may hold, and far points
        p = rng.random((n, 3))
        for a in range(4):
            p[a * 2500: (a + 1) * 2500] = rng.random(3) + 1e-6 * rng.random((2500, 3))
        p[-9:] *= 50.0
        return p.astype(np.float32)
    if kind == "copies":      # more equal keys than a wavefront has lanes, at every query
        return np.repeat(rng.random((n // 90 + 1, 3)), 90, 0)[rng.permutation(n)].astype(np.float32)
    if kind == "lattice":     # more than 64 equal distances at many keys
        return synth.binary_grid_points(n, 3, (98, n), span=20)
    return cloud(kind, n, 3)


@pytest.mark.parametrize("kind", ["uniform", "box", "outlier", "same", "far", "tiny", "holes", "lattice", "line",
                                  "grid", "cluster", "flat"])
@pytest.mark.parametrize("k", [1, 16, 32])
def test_clouds(lib, kind, k):
    check(lib, points(kind, 7300), 1, k)


@pytest.mark.parametrize("kind", ["uniform", "box", "outlier", "same", "far", "tiny", "holes", "lattice", "line",
                                  "grid", "cluster", "flat", "clumps", "many holes", "copies"])
@pytest.mark.parametrize("n,k", [(16385, 1), (16385, 16), (20001, 32)])
def test_clouds_behind_the_streaming_scan(lib, kind, n, k):
    # above 16,384 points the queries that the other scans leave open are streamed
    pos = points(kind, n)
    rng = np.random.default_rng(1)
    pts = np.unique(np.concatenate([np.arange(64), rng.integers(0, n, 4000), np.arange(n // 3 - 40, n // 3 + 40)]))
    check(lib, pos, 1, k, pts=pts)


@pytest.mark.parametrize("kind", ["uniform", "box", "outlier", "same", "far", "tiny", "holes", "lattice", "line",
                                  "grid", "cluster", "flat", "clumps", "many holes", "copies"])
@pytest.mark.parametrize("n,k", [(12501, 1), (11600, 16), (11600, 32)])
def test_clouds_above_the_scan_of_every_point(lib, kind, n, k):
    check(lib, points(kind, n), 1, k)


@pytest.mark.parametrize("n", [200, 2500])
@pytest.mark.parametrize("kind", ["same", "copies", "line", "holes"])
@pytest.mark.parametrize("k", [0, 1, 17, 32])
def test_scan_of_every_point(lib, kind, n, k):
    check(lib, points(kind, n), 1, k)


@pytest.mark.parametrize("n", [11000, 11001, 11004, 12500, 12501, 16384, 23999, 24000])
@pytest.mark.parametrize("k,F", [(0, 1), (5, 0), (8, 2), (9, 1), (17, 9), (31, 3)])
def test_sizes_at_the_bounds(lib, n, k, F):
    check(lib, points("uniform", n), F, k)


@pytest.mark.parametrize("n", [7168, 7169, 7176, 9001])
@pytest.mark.parametrize("k,F", [(0, 1), (5, 0), (17, 9), (31, 3)])
def test_sizes(lib, n, k, F):
    check(lib, points("uniform", n), F, k)


@pytest.mark.parametrize("kind", ["uniform", "cluster", "outlier"])
@pytest.mark.parametrize("n", [7169, 11001, 12000, 17000])
def test_sums_are_added_in_key_order(lib, kind, n):
    # above 7,168 points, whichever scan decides a query; the clump and the outlier reach all of them
    pos, k = points(kind, n), 32
    x = np.random.default_rng(n).standard_normal((n, 2)).astype(np.float32)
    y, nbr = lib.tiga_mp_knn_fwd(dev(pos), dev(x), k, want_nbr=True)
    nbr, want = nbr.cpu().numpy(), np.zeros((n, 2), np.float32)
    for t in range(k):
        want = np.where(nbr[:, t:t + 1] >= 0, want + x[nbr[:, t]], want)
    assert np.array_equal(y.cpu().numpy(), want)


def test_neighbours_across_a_face_closer_than_the_coordinates_round(lib):
    # A box of [-1, 1] in x: x + 1 rounds to multiples of u above the face at 0 and of u / 2 below it.  The query at
    # 4.6 u rounds to 5 u, so the cells left of the face look 5 u away; the source at -0.26 u is 4.86 u away and must
    # come before the one 4.95 u to the right.  3,000 points around them crowd every level of cells.
    n, u = 20000, 2.0 ** -52
    rng = np.random.default_rng(8)
    pos = np.zeros((n, 3))
    pos[:, :2] = rng.uniform(-1, 1, (n, 2))
    pos[0, :2], pos[1, :2] = -1, 1
    pos[100:3100, :2] = rng.uniform(2e-4, 1.9e-3, (3000, 2))
    pos[7:10, 0] = [4.6 * u, -0.26 * u, 9.55 * u]
    pos[7:10, 1] = 1e-3
    check(lib, pos.astype(np.float32), 1, 1, pts=np.arange(7, 300))
