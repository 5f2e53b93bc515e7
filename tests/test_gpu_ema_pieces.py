"""The sum over a code's pieces of 128 rows, with none, one and several of them."""
import numpy as np
import pytest
import torch

from gpu_util import np_, require_gpu

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("d", [1, 8, 255, 256, 257, 1025])
@pytest.mark.parametrize("few", [False, True])
def test_pieces_of_a_code(d, few):
    """Whole numbers and a decay of one half: every product and sum is exact, so the
    result is NumPy's bit for bit, in both forms of the grouping by code."""
    xgs = require_gpu()
    counts = [0, 1, 2, 127, 128, 129, 0, 256, 257] + ([1000] if few else [1000, 1025, 2049])
    K, rng = len(counts), np.random.default_rng(d)
    idx = rng.permutation(np.repeat(np.arange(K), counts)).astype(np.int32)
    N = len(idx)
    assert (N <= 2048) == few
    X = rng.integers(-8, 9, (N, d)).astype(np.float32)
    M, n = rng.integers(-100, 101, (K, d)).astype(np.float32), rng.integers(1, 100, K).astype(np.float32)
    want = 0.5 * M
    np.add.at(want, idx, 0.5 * X)
    g = lambda a: torch.from_numpy(a).cuda()
    E, Me, Ne = g(M.copy()), g(M.copy()), g(n.copy())
    Eb, en = xgs.xgs_vq_prepare(E)
    got = xgs.xgs_vq_ema_update(g(X), g(idx), Ne, Me, E, Eb, en, 0.5, 1e-5, xgs.EMA_LAPLACE)
    torch.cuda.synchronize()
    np.testing.assert_array_equal(np_(Me), want)
    np.testing.assert_array_equal(np_(Ne), 0.5 * n + 0.5 * np.array(counts, np.float32))
    np.testing.assert_array_equal(np_(got), np.array(counts, np.float32))
