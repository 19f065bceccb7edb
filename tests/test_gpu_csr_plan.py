"""GPU parity of the CSR plan, the split-row merge and the edge records where their paths change:
hub rows around the cooperative bounds, runs of empty rows longer than a staged window, and
relations past the large plan tile.  Integer-valued inputs, so every comparison is exact."""
import numpy as np
import pytest
import torch

import oracle
from tests.test_gpu_csr import dev, host, make_graph

pytestmark = pytest.mark.gpu


def check(lib, deg, num_src, F, reducer, seed):
    rp, col, x, w, dy = make_graph(deg, num_src, F, seed, integer=True)
    rel = lib.Csr(dev(rp), dev(col), num_src)
    rev = lib.tiga_csr_transpose(rel)
    red = lib.REDUCE_MAX if reducer == "max" else lib.REDUCE_SUM
    y, arg = lib.tiga_mp_csr_fwd(rel, dev(x), dev(w), reducer=red)
    dx, dw = lib.tiga_mp_csr_bwd(rel, dev(dy), dev(x), dev(w), reducer=red, argmax=arg, rev=rev)
    if reducer == "max":
        ry, rarg = oracle.csr_max_fwd(rp, col, x, w)[:2]
        assert np.array_equal(host(arg), rarg)
        rdx, _, rdw, _ = oracle.csr_max_bwd(rp, col, x, w, rarg, dy, num_src)
    else:
        ry = oracle.csr_sum_fwd(rp, col, x, w)[0]
        rdx, _, rdw, _ = oracle.csr_sum_bwd(rp, col, x, w, dy, num_src)
    assert np.array_equal(host(y), ry)
    assert np.array_equal(host(dx), rdx)
    assert np.array_equal(host(dw), rdw)


@pytest.mark.parametrize("F", [16, 17, 64, 100])
@pytest.mark.parametrize("reducer", ["sum", "max"])
def test_hub_rows(lib, F, reducer):
    # chunk lengths are 64 to 1,024 edges: rows of 16 and 17 chunks, and rows past the merge's block bound
    deg = np.full(5000, 3)
    deg[1000:4300] = 0                                  # longer than two staged windows of row pointers
    for k, c in enumerate([64, 128, 256, 1024]):
        deg[[k, 600 + k, 700 + k, 4400 + k, 4500 + k]] = [16 * c, 16 * c + 1, 17 * c, 17 * c + 1, 1025]
    deg[[10, 990, 4990, 4999]] = [70_000, 40_000, 2049, 0]
    check(lib, deg, 3001, F, reducer, 5)


@pytest.mark.parametrize("rows", [(1 << 22) - 1, (1 << 22) + 8195])
def test_large_plan_tile(lib, rows):
    deg = np.zeros(rows, np.int64)
    rng = np.random.default_rng(3)
    deg[rng.integers(0, rows, 40_000)] = rng.choice([1, 8, 9, 40, 300, 2000], size=40_000,
                                                     p=[.3, .3, .2, .15, .045, .005])
    deg[[0, 8191, 8192, rows - 1]] = [30_000, 17, 2049, 33]
    check(lib, deg, 1000, 4, "sum", 7)


@pytest.mark.parametrize("rows", [1, 700, 1024, 1025, 1090, 5000])
@pytest.mark.parametrize("edges", [1, 255, 257, 2049, 9000, 2048 * 511, 2048 * 511 + 1, 2048 * 600 + 7])
def test_edge_records(lib, rows, edges):
    # one and eight edges per thread (the latter from 512 blocks of 2,048 edges on), whole and windowed row pointers,
    # empty rows before, between and after the others
    rng = np.random.default_rng(rows + edges)
    deg = np.bincount(rng.choice(rng.permutation(rows)[: max(1, rows // 3)], edges), minlength=rows)
    check(lib, deg, 50, 4, "sum", 11)
