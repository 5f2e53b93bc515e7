"""Plain FP32 assignment: the form that certifies its candidates on the matrix
cores against the direct form of every codeword (bit for bit: one more codeword
of a huge norm, which never wins, sends every row down the direct form), and
both against FP64.  Sizes at the edges of the 32 / 64-row, 256-codeword and
32-column tiles; data with offsets, duplicate and near-duplicate codewords, rows
on codewords, and numbers that are not finite."""
import numpy as np
import pytest
import torch

from gpu_util import np_, require_gpu

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def xgs():
    return require_gpu()


def assign(xgs, X, E):
    X, E = torch.from_numpy(X).cuda(), torch.from_numpy(E).cuda()
    Eb, en = xgs.xgs_vq_prepare(E)
    idx, dist = xgs.xgs_vq_assign(X, E, Eb, en, xgs.VQ_FP32)
    torch.cuda.synchronize()
    return np_(idx).astype(np.int64), np_(dist)


def data(kind, n, k, d, seed):
    rng = np.random.default_rng(seed)
    E = rng.standard_normal((k, d))
    X = E[rng.integers(0, k, n)] + 0.5 * rng.standard_normal((n, d))
    if kind == "offset":
        X, E = X + 100.0, E + 100.0
    elif kind == "duplicates":
        E = E[rng.integers(0, max(1, k // 8), k)]
    elif kind == "near":        # codewords a few ulp apart: candidates that only the direct form can order
        E = E[rng.integers(0, max(1, k // 2), k)] * (1 + 1e-7 * rng.integers(-3, 4, (k, 1)))
    elif kind == "on":
        X = E[rng.integers(0, k, n)]
    elif kind == "tiny":
        X, E = X * 1e-20, E * 1e-20
    return X.astype(np.float32), E.astype(np.float32)


@pytest.mark.parametrize("n,k,d", [(1, 1, 1), (31, 255, 33), (32, 256, 32), (33, 257, 36), (1200, 700, 64),
                                   (32769, 300, 48), (97, 4096, 8)])
@pytest.mark.parametrize("kind", ["plain", "offset", "duplicates", "near", "on", "tiny"])
def test_same_bits_as_the_direct_form(xgs, n, k, d, kind):
    X, E = data(kind, n, k, d, 7 * n + k + d)
    idx, dist = assign(xgs, X, E)
    ref_idx, ref_dist = assign(xgs, X, np.concatenate([E, np.full((1, d), 1e19, np.float32)]))
    np.testing.assert_array_equal(idx, ref_idx)
    np.testing.assert_array_equal(dist.view(np.int32), ref_dist.view(np.int32))
    rows = np.arange(n) if n <= 1200 else np.random.default_rng(1).choice(n, 1200, replace=False)
    x, e = X[rows].astype(np.float64), E.astype(np.float64)
    # a sum of d squares in FP32: within (d + 2) 2^-24 of its value (and underflow's absolute share)
    g, tiny = (d + 2) * 2.0 ** -24, d * 2.0 ** -126
    own = ((x - e[idx[rows]]) ** 2).sum(1)
    best = np.array([((xi - e) ** 2).sum(1).min() for xi in x])
    assert np.all(np.abs(dist[rows] - own) <= g * own + tiny)
    assert np.all(own <= best * (1 + g) / (1 - g) + 2 * tiny)


@pytest.mark.parametrize("n,k,d", [(70, 300, 40), (33000, 40, 7)])
def test_numbers_that_are_not_finite(xgs, n, k, d):
    """A NaN codeword never wins, an infinite one only at an infinite distance; a
    row with NaN has no codeword, one with infinity the first."""
    X, E = data("plain", n, k, d, 5)
    X[3, 0], X[5, d - 1] = np.nan, np.inf
    clean_idx, clean_dist = assign(xgs, X, E)
    assert clean_idx[3] == 0x7FFFFFFF and np.isinf(clean_dist[3])
    assert clean_idx[5] == 0 and np.isinf(clean_dist[5])
    E2 = np.concatenate([E, E[:2]])
    E2[k, 1], E2[k + 1, 2] = np.nan, -np.inf
    idx, dist = assign(xgs, X, E2)
    np.testing.assert_array_equal(idx, clean_idx)
    np.testing.assert_array_equal(dist, clean_dist)


def test_unaligned_rows(xgs):
    """Views at a 4-byte offset take scalar loads, with the same bits."""
    X, E = data("plain", 100, 270, 64, 3)
    idx, dist = assign(xgs, X, E)
    buf = torch.zeros(X.size + 1, device="cuda")
    buf[1:] = torch.from_numpy(X.reshape(-1)).cuda()
    Eg = torch.from_numpy(E).cuda()
    Eb, en = xgs.xgs_vq_prepare(Eg)
    i2, d2 = xgs.xgs_vq_assign(buf[1:].view(X.shape), Eg, Eb, en, xgs.VQ_FP32)
    torch.cuda.synchronize()
    np.testing.assert_array_equal(np_(i2), idx)
    np.testing.assert_array_equal(np_(d2), dist)
