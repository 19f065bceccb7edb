"""GPU parity of the CSR traversals on rows that are no multiple of 16 bytes, or not aligned to them (the last
unit of such a row repeats floats of the one before it).  Integer-valued inputs: every comparison is exact."""
import numpy as np
import pytest
import torch

import oracle
from tests.test_gpu_csr import dev, host, make_graph, mixed_degrees

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("F", [4, 5, 6, 7, 9, 16, 17, 31, 33, 65, 129, 255, 257, 258])
@pytest.mark.parametrize("reducer", ["sum", "max"])
@pytest.mark.parametrize("offset", [0, 1, 3])
def test_ragged_rows(lib, F, reducer, offset):
    n = 300 if offset else 900   # at most 2^16 edges, or more
    rp, col, x, w, dy = make_graph(mixed_degrees(n, F, big=(3000,)), 500, F, F + offset, integer=True)

    def put(a):   # a contiguous copy that starts `offset` floats past an aligned address
        t = torch.empty(a.size + offset, dtype=torch.float32, device="cuda")[offset:].view(a.shape)
        return t.copy_(dev(a))

    rel = lib.Csr(dev(rp), dev(col), 500)
    rev = lib.tiga_csr_transpose(rel)
    red = lib.REDUCE_MAX if reducer == "max" else lib.REDUCE_SUM
    y, arg = lib.tiga_mp_csr_fwd(rel, put(x), dev(w), reducer=red, y=put(np.full((n, F), 7.0, np.float32)))
    dx, dw = lib.tiga_mp_csr_bwd(rel, put(dy), put(x), dev(w), reducer=red, argmax=arg, rev=rev)
    if reducer == "max":
        ry, rarg = oracle.csr_max_fwd(rp, col, x, w)
        assert np.array_equal(host(arg), rarg)
        rdx, _, rdw, _ = oracle.csr_max_bwd(rp, col, x, w, rarg, dy, 500)
    else:
        ry = oracle.csr_sum_fwd(rp, col, x, w)[0]
        rdx, _, rdw, _ = oracle.csr_sum_bwd(rp, col, x, w, dy, 500)
    assert np.array_equal(host(y), ry)
    assert np.array_equal(host(dx), rdx)
    assert np.array_equal(host(dw), rdw)


@pytest.mark.parametrize("F", [5, 7, 17, 18, 33, 64, 255])
@pytest.mark.parametrize("reducer", ["sum", "max"])
@pytest.mark.parametrize("n", [300, 900])   # at most 2^16 edges, or more
def test_non_finite_values(lib, F, reducer, n):
    # one infinite or NaN cotangent in most rows, one such source value in some: at the repeated floats of the last
    # unit (F - 4 .. F - 1 for these widths) and before them.  Integers otherwise, so everything else is exact.
    rp, col, x, w, dy = make_graph(mixed_degrees(n, F, big=(3000,)), 500, F, F, integer=True)
    w += 1
    rng = np.random.default_rng(F)
    vals = np.array([np.inf, -np.inf, np.nan], np.float32)
    at = np.arange(0, n, 3)
    dy[at, F - 1 - rng.integers(0, min(F, 9), at.size)] = vals[rng.integers(0, 3, at.size)]
    x[::50, F - 1 - rng.integers(0, min(F, 9), 10)] = vals[rng.integers(0, 2, 10)]
    x[x == 0] = 1                                      # 0 x inf stays out of the sources that count
    rel = lib.Csr(dev(rp), dev(col), 500)
    rev = lib.tiga_csr_transpose(rel)
    red = lib.REDUCE_MAX if reducer == "max" else lib.REDUCE_SUM
    y, arg = lib.tiga_mp_csr_fwd(rel, dev(x), dev(w), reducer=red)
    dx, dw = lib.tiga_mp_csr_bwd(rel, dev(dy), dev(x), dev(w), reducer=red, argmax=arg, rev=rev)
    with np.errstate(all="ignore"):
        if reducer == "max":
            ry, rarg = oracle.csr_max_fwd(rp, col, x, w)
            assert np.array_equal(host(arg), rarg)
            rdx, _, rdw, _ = oracle.csr_max_bwd(rp, col, x, w, rarg, dy, 500)
        else:
            ry = oracle.csr_sum_fwd(rp, col, x, w)[0]
            rdx, _, rdw, _ = oracle.csr_sum_bwd(rp, col, x, w, dy, 500)
    assert np.isinf(rdw).any() and np.isfinite(rdw).any()
    for got, ref in ((y, ry), (dx, rdx), (dw, rdw)):
        assert np.array_equal(host(got), ref, equal_nan=True)
