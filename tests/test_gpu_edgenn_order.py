"""Edge MLP: the order and the rounding of its fp32 sums, bit for bit.  Where the sum of the cotangents cancels, a
different order of the same pairs moves the parameter gradients by more than any tolerance on them could allow."""
import numpy as np
import pytest
import torch

from tests.test_gpu_edgenn import dev

pytestmark = pytest.mark.gpu
f32 = np.float32


def butterfly(v, axis):
    """Sum over an axis of a power of two in the order of lane exchanges at distances 1, 2, 4, ..."""
    v = np.moveaxis(v, axis, 0)
    while v.shape[0] > 1:
        v = v[0::2] + v[1::2]
    return v[0]


def replay(pos, x, r, W1, b1, W2, b2, dy):
    """One output; all points in one cell, so candidates come in id order; every wavefront has one point.  The
    64 / HP neighbour slots of a point each take every (64 / HP)-th candidate."""
    n, F = x.shape
    H = W1.shape[0]
    SL = 64 // (16 if H <= 16 else 32 if H <= 32 else 64)
    w2 = W2[0][None, :]
    dhk = w2 * dy                                                    # [n, H]
    acc, g2, g1b = (np.zeros((SL, n, H), f32) for _ in range(3))
    g1 = np.zeros((SL, 3 + F, n, H), f32)
    deg = np.zeros(n, np.int64)
    for j in range(n):
        s = j % SL
        d = pos[j] - pos
        q = d * d
        near = ((q[:, 0] + q[:, 1]) + q[:, 2] < f32(r) * f32(r))
        near[j] = False
        deg += near
        t = [W1[None, :, c] * d[:, c:c + 1] for c in range(3)]
        fwd = ((b1[None, :] + t[0]) + t[1]) + t[2]
        a = b1[None, :] + ((t[0] + t[1]) + t[2])
        for c in range(F):
            p = W1[None, :, 3 + c] * x[j, c]
            fwd, a = fwd + p, a + p
        m = near[:, None]
        acc[s] = np.where(m, acc[s] + w2 * np.maximum(fwd, f32(0)), acc[s])
        g2[s] = np.where(m, g2[s] + dy * np.maximum(a, f32(0)), g2[s])
        da = np.where(a > 0, dhk, f32(0))
        g1b[s] = np.where(m, g1b[s] + da, g1b[s])
        for c in range(3 + F):
            v = d[:, c:c + 1] if c < 3 else x[j, c - 3]
            g1[s, c] = np.where(m, g1[s, c] + da * v, g1[s, c])
    lanes = np.zeros((n, SL * (64 // SL)), f32)
    for s in range(SL):
        lanes[:, s * (64 // SL): s * (64 // SL) + H] = acc[s]
    y = (deg * np.float64(b2[0]) + butterfly(lanes, 1)).astype(f32)   # exact before its rounding: b2 = 0.5
    waves = (n + 3) // 4 * 4
    per = (waves + 63) // 64

    def total(part):   # [n, ...]: wavefronts in order within 64 groups, then the groups
        z = np.zeros((64 * per,) + part.shape[1:], f32)
        z[:n] = part
        z = z.reshape((64, per) + part.shape[1:])
        g = np.zeros((64,) + part.shape[1:], f32)
        for k in range(per):
            g = g + z[:, k]
        out = np.zeros(part.shape[1:], f32)
        for k in range(64):
            out = out + g[k]
        return out

    return dict(y=y[:, None], db1=total(butterfly(g1b, 0)), dW2=total(butterfly(g2, 0))[None],
                dW1=np.stack([total(butterfly(g1[:, c], 0)) for c in range(3 + F)], 1))


@pytest.mark.parametrize("n,F,H", [(301, 0, 32), (190, 3, 16), (230, 8, 24), (150, 1, 64), (200, 20, 7)])
def test_orders(lib, n, F, H):
    rng = np.random.default_rng(n)
    pos = rng.random((n, 3)).astype(f32)
    x = rng.standard_normal((n, F)).astype(f32)
    W1, b1, W2 = (rng.uniform(-0.6, 0.6, s).astype(f32) for s in ((H, 3 + F), H, (1, H)))
    b2 = np.array([0.5], f32)
    dy = rng.standard_normal((n, 1)).astype(f32)
    r = 1.01                                  # one cell: wider than the cloud
    a = [dev(pos), dev(x) if F else None, r] + [dev(v) for v in (W1, b1, W2, b2)]
    want = replay(pos, x, r, W1, b1, W2, b2, dy)
    got = dict(lib.tiga_mp_edgenn_bwd(*a, dev(dy)), y=lib.tiga_mp_edgenn_fwd(*a))
    torch.cuda.synchronize()
    for k, v in want.items():
        assert np.array_equal(got[k].cpu().numpy(), v), k


def test_activity_is_decided_on_rounded_products(lib):
    # w x = 1 + 2^-24 rounds to 1, and 1 + b1 = 0: inactive; unrounded, the unit would be active
    pos = np.array([[0, 0, 0], [0.25, 0, 0]], f32)
    x = np.full((2, 1), 1 + 2.0 ** -12, f32)
    W1 = np.array([[0, 0, 0, (1 + 2.0 ** -23) / (1 + 2.0 ** -12)]], f32)
    b1 = -(W1[:, 3] * x[0])
    assert np.float64(W1[0, 3]) * np.float64(x[0, 0]) + np.float64(b1[0]) > 0
    one = np.ones((1, 1), f32)
    a = [dev(pos), dev(x), 0.5, dev(W1), dev(b1), dev(one), dev(np.zeros(1, f32))]
    g = lib.tiga_mp_edgenn_bwd(*a, dev(np.ones((2, 1), f32)))
    assert torch.count_nonzero(lib.tiga_mp_edgenn_fwd(*a)) == 0
    assert all(torch.count_nonzero(g[k]) == 0 for k in ("dW1", "db1", "dW2"))


def test_an_infinite_weight_meets_real_pairs_only(lib):
    # one pair per point: places past a list's end take no part (0 x inf)
    pos = np.array([[0, 0, 0], [0.25, 0, 0]], f32)
    x = np.ones((2, 1), f32)
    W1 = np.array([[0, 0, 0, 1], [0, 0, 0, 1]], f32)
    W2 = np.array([[np.inf, 1]], f32)
    y = lib.tiga_mp_edgenn_fwd(dev(pos), dev(x), 0.5, dev(W1), dev(np.zeros(2, f32)), dev(W2), dev(np.zeros(1, f32)))
    assert np.all(y.cpu().numpy() == np.inf)
