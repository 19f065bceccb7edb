"""GPU parity of the radius kernels on tiles of 16 destinations: row widths around the dispatch's bounds, partial
tiles, tiles that cross rows of cells, more candidates than one pass holds, non-finite rows and denormals."""
import numpy as np
import pytest
import torch

import oracle
from tests.parity import assert_terms_close

pytestmark = pytest.mark.gpu


def dev(a):
    return torch.from_numpy(np.ascontiguousarray(a)).cuda()


def host(t):
    return t.cpu().numpy()


def check(lib, pos, F, r, sigma, seed=0, offset=0):
    n = pos.shape[0]
    rng = np.random.default_rng(seed + F)
    x, dy = (rng.standard_normal((n, F)).astype(np.float32) for _ in range(2))

    def put(a):   # a contiguous copy that starts `offset` floats past an aligned address
        t = torch.empty(a.size + offset, dtype=torch.float32, device="cuda")[offset:].view(a.shape)
        return t.copy_(dev(a))

    y, cnt = lib.tiga_mp_radius_fwd(dev(pos), put(x), r, sigma)
    dx, dp = lib.tiga_mp_radius_bwd(dev(pos), put(x), put(dy), r, sigma)
    dx1, _ = lib.tiga_mp_radius_bwd(dev(pos), put(x), put(dy), r, sigma, want_dpos=False)
    _, dp1 = lib.tiga_mp_radius_bwd(dev(pos), put(x), put(dy), r, sigma, want_dx=False)
    ry, rya, rc = oracle.radius_fwd(pos, x, r, sigma)
    rdx, rdxa, rdp, rdpa = oracle.radius_bwd(pos, x, dy, r, sigma)
    assert np.array_equal(host(cnt), rc)
    assert_terms_close(host(y), ry, rya, what="y")
    for a in (dx, dx1):
        assert_terms_close(host(a), rdx, rdxa, what="dx")
    for a in (dp, dp1):
        assert_terms_close(host(a), rdp, rdpa, what="dpos")


@pytest.mark.parametrize("F", [1, 2, 3, 4, 5, 8, 9, 15, 16, 17, 18, 31, 32, 33, 36, 50, 63, 64, 65])
@pytest.mark.parametrize("offset", [0, 1])
def test_widths(lib, F, offset):
    pos = np.random.default_rng(1).random((700, 3)).astype(np.float32)
    check(lib, pos, F, 0.15, 0.08, offset=offset)


@pytest.mark.parametrize("n", [1, 2, 15, 16, 17, 31, 33, 64, 65, 129])
def test_sizes(lib, n):
    pos = np.random.default_rng(n).random((n, 3)).astype(np.float32)
    for F in (1, 6, 32):
        check(lib, pos, F, 0.4, 0.3)


@pytest.mark.parametrize("kind", ["thin", "dense", "line", "grid", "gaps"])
def test_clouds(lib, kind):
    rng = np.random.default_rng(4)
    pos = rng.random((900, 3)).astype(np.float32)
    r = 0.12
    if kind == "thin":       # one or two points per row of cells: a tile has many segments
        pos *= np.float32([0.2, 3.0, 3.0])
    elif kind == "dense":    # several hundred candidates per tile: more than one pass
        pos[:600] = pos[:600] * np.float32(0.2) + np.float32(0.4)
    elif kind == "line":
        pos[:, 1:] = 0.5
    elif kind == "gaps":     # rows of few points beside a dense one: gaps of every width between a tile's points
        pos[:, 1:] *= np.float32(0.1)
        pos[:, 0] *= 9
        pos[:60, 1] += np.float32(0.13)
        pos[60:75, 1] += np.float32(0.26)
    else:                    # coincident points and distances equal to the radius
        pos = (rng.integers(0, 9, (900, 3)) / 8).astype(np.float32)
        r = 0.125
    for F in (1, 7, 32):
        check(lib, pos, F, r, 0.1)


@pytest.mark.parametrize("F", [1, 8, 32, 64])
def test_non_finite_rows_reach_their_neighbours_only(lib, F):
    rng = np.random.default_rng(5)
    n, r, sigma = 500, 0.15, 0.1
    pos = rng.random((n, 3)).astype(np.float32)
    x, dy = (rng.standard_normal((n, F)).astype(np.float32) for _ in range(2))
    pos[7, 1] = np.nan
    bx, by = x.copy(), dy.copy()
    bx[100], by[200] = np.inf, np.nan
    y, _ = lib.tiga_mp_radius_fwd(dev(pos), dev(bx), r, sigma)
    ry, rya, rc = oracle.radius_fwd(pos, x, r, sigma)
    with np.errstate(all="ignore"):
        near = ((pos[None] - pos[:, None]) ** 2).sum(-1) < np.float32(r) ** 2
    np.fill_diagonal(near, False)
    far = ~near[:, 100]
    assert_terms_close(host(y)[far], ry[far], rya[far], what="y")
    assert np.all(host(y)[near[:, 100]] == np.inf)
    if F > 32:
        return
    dx, dp = lib.tiga_mp_radius_bwd(dev(pos), dev(bx), dev(by), r, sigma)
    rdx, rdxa, rdp, rdpa = oracle.radius_bwd(pos, x, dy, r, sigma)
    far = ~near[:, 200]
    assert_terms_close(host(dx)[far], rdx[far], rdxa[far], what="dx")
    assert np.all(np.isnan(host(dx)[near[:, 200]]))
    far = ~(near[:, 100] | near[:, 200])
    far[[100, 200]] = False
    assert_terms_close(host(dp)[far], rdp[far], rdpa[far], what="dpos")


@pytest.mark.parametrize("F", [1, 16, 32])
def test_denormal_rows(lib, F):
    # sigma so large that every weight is 1: sums of multiples of the smallest float are exact
    rng = np.random.default_rng(6)
    pos = rng.random((400, 3)).astype(np.float32)
    k = rng.integers(-50, 50, (400, F))
    x = (k * 2.0 ** -149).astype(np.float32)
    y, _ = lib.tiga_mp_radius_fwd(dev(pos), dev(x), 0.2, 1e18)
    ry, _, _ = oracle.radius_fwd(pos, x, 0.2, 1e18)
    assert np.array_equal(host(y).astype(np.float64), ry)


@pytest.mark.parametrize("F", [32, 16, 5])
def test_row_arrays_of_4_gib(lib, F):
    # their byte offsets pass 32 bits, so one wavefront per cell with its lists takes them; the same columns in narrower
    # arrays go by tiles
    n = (1 << 30) // F + 3
    g = torch.Generator(device="cuda").manual_seed(F)
    pos = torch.rand(n, 3, generator=g, device="cuda")
    x, dy = (torch.randn(n, F, generator=g, device="cuda") for _ in range(2))
    r = float((5.0 * 3 / (4 * np.pi * n)) ** (1 / 3))
    s = 0.6 * r
    y, cnt = lib.tiga_mp_radius_fwd(pos, x, r, s)
    dx, dp = lib.tiga_mp_radius_bwd(pos, x, dy, r, s)
    dp_sum, dp_mag = (torch.zeros_like(dp) for _ in range(2))
    for cols in (slice(0, F // 2), slice(F // 2, F)):
        xs, dys = x[:, cols].contiguous(), dy[:, cols].contiguous()
        ya, ca = lib.tiga_mp_radius_fwd(pos, xs.abs(), r, s)
        dxa, _ = lib.tiga_mp_radius_fwd(pos, dys.abs(), r, s)
        # |p_j - p_i| < r in the sum of the position gradient's terms
        dp_mag += (2 * r / s ** 2) * ((ya * dys.abs()).sum(1) + (dxa * xs.abs()).sum(1))[:, None]
        yt, ct = lib.tiga_mp_radius_fwd(pos, xs, r, s)
        assert torch.equal(ct, cnt) and torch.equal(ca, cnt)
        assert bool(((y[:, cols] - yt).abs() <= 1e-5 * ya).all())
        dxt, dpt = lib.tiga_mp_radius_bwd(pos, xs, dys, r, s)
        assert bool(((dx[:, cols] - dxt).abs() <= 1e-5 * dxa).all())
        dp_sum += dpt
        del xs, dys, ya, dxa, yt, dxt, dpt
    assert bool(((dp - dp_sum).abs() <= 1e-5 * dp_mag).all())


@pytest.mark.parametrize("F", [1, 4, 8, 15, 16, 31, 32])
def test_distance_from_64_bits(lib, F):
    # 31 neighbours of a point: summed in one run of roundings they end 1.2e-7 (norms of difference and result) from
    # 64 bits and the position gradient 1.5e-7; as trees over lane groups at most 1.1e-7, and 1.0e-7 and 1.4e-7 here
    n = 30000
    rng = np.random.default_rng(F)
    pos = rng.random((n, 3)).astype(np.float32)
    x, dy = (rng.standard_normal((n, F)).astype(np.float32) for _ in range(2))
    r = float(np.float32((31 * 3 / (4 * np.pi * n)) ** (1 / 3)))
    y, _ = lib.tiga_mp_radius_fwd(dev(pos), dev(x), r, 0.5 * r)
    dx, dp = lib.tiga_mp_radius_bwd(dev(pos), dev(x), dev(dy), r, 0.5 * r)
    ry = oracle.radius_fwd(pos, x, r, 0.5 * r)[0]
    rdx, _, rdp, _ = oracle.radius_bwd(pos, x, dy, r, 0.5 * r)
    for name, a, b, most in (("y", y, ry, 1.1e-7), ("dx", dx, rdx, 1.1e-7), ("dpos", dp, rdp, 1.45e-7)):
        assert np.linalg.norm(host(a).astype(np.float64) - b) < most * np.linalg.norm(b), name
