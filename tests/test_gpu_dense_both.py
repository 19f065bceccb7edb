"""GPU parity of the dense relation where a pair is evaluated once for both directions: the bounds of that path,
ragged last row blocks, and every block of rows and points."""
import numpy as np
import pytest

import oracle
from paper_2609_24802_amd import synth
from tests.parity import assert_terms_close
from tests.test_gpu_radius_dense import dev, host

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n", [12287, 12288, 12289, 14001, 40959, 40960, 43011])
def test_all_outputs(lib, n):
    g = synth.config4(n=n)
    y = host(lib.tiga_mp_dense_fwd(dev(g["pos"]), dev(g["q"]), g["eps"]))
    rng = np.random.default_rng(n)
    pts = np.unique(np.concatenate([np.arange(0, n, 1023), np.arange(n - 70, n), rng.integers(0, n, 2000)]))
    ry, rya = oracle.dense_fwd(g["pos"], g["q"], g["eps"], pts=pts)
    assert_terms_close(y[pts], ry, rya, what=f"dense n={n}")
    # Newton's third law over all outputs: sum_i q_i y_i vanishes up to rounding
    f = g["q"].astype(np.float64)[:, None] * y
    assert np.all(np.abs(f.sum(0)) <= 1e-6 * np.abs(f).sum(0))
    again = host(lib.tiga_mp_dense_fwd(dev(g["pos"]), dev(g["q"]), g["eps"]))
    assert np.array_equal(y, again)


def test_above_the_bound(lib):
    n = (1 << 18) + 1
    g = synth.config4(n=n)
    y = host(lib.tiga_mp_dense_fwd(dev(g["pos"]), dev(g["q"]), g["eps"]))
    pts = np.array([0, 1, 2048, n // 2, n - 2, n - 1])
    ry, rya = oracle.dense_fwd(g["pos"], g["q"], g["eps"], pts=pts)
    assert_terms_close(y[pts], ry, rya, what="dense")
