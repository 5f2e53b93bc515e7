"""Plain FP32 assignment of few codewords or few columns, which takes the direct
form in tiles: the same bits as with further codewords that never win and that
send the call down the certified form, on both sides of the rule that picks."""
import numpy as np
import pytest
import torch

from gpu_util import np_, require_gpu
from test_gpu_vq_fp32 import assign, data

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def xgs():
    return require_gpu()


@pytest.mark.parametrize("n", [1, 63, 64, 65, 8192, 8193, 16385, 32768])
@pytest.mark.parametrize("k,d", [(1, 1), (2, 768), (63, 31), (64, 32), (64, 33), (65, 4), (128, 30), (192, 8), (256, 31),
                                 (320, 16), (512, 30)])
@pytest.mark.parametrize("kind", ["plain", "duplicates"])
def test_same_bits_as_the_certified_form(xgs, n, k, d, kind):
    X, E = data(kind, n, k, d, n + 3 * k + d)
    idx, dist = assign(xgs, X, E)
    # 1,800 codewords far from every row and from each other: seven more sweeps
    far = np.float32(1e4) * np.random.default_rng(k).uniform(1, 2, (1800, d)).astype(np.float32)
    ref_idx, ref_dist = assign(xgs, X, np.concatenate([E, far]))
    np.testing.assert_array_equal(idx, ref_idx)
    np.testing.assert_array_equal(dist.view(np.int32), ref_dist.view(np.int32))


@pytest.mark.parametrize("n,k,d", [(70, 40, 12), (33000, 20, 6)])
def test_not_finite_and_unaligned(xgs, n, k, d):
    """As in the certified form: a NaN codeword never wins, an infinite one only at an
    infinite distance; a row with NaN has no codeword, one with infinity the first;
    views at a 4-byte offset are read as they are."""
    X, E = data("plain", n, k, d, 5)
    X[3, 0], X[5, d - 1] = np.nan, np.inf
    E2 = np.concatenate([E, E[:2]])
    E2[k, 1], E2[k + 1, 2] = np.nan, -np.inf
    idx, dist = assign(xgs, X, E)
    idx2, dist2 = assign(xgs, X, E2)
    assert idx[3] == 0x7FFFFFFF and np.isinf(dist[3]) and idx[5] == 0 and np.isinf(dist[5])
    np.testing.assert_array_equal(idx2, idx)
    np.testing.assert_array_equal(dist2, dist)
    buf = torch.zeros(X.size + 1, device="cuda")
    buf[1:] = torch.from_numpy(X.reshape(-1)).cuda()
    Eg = torch.from_numpy(E).cuda()
    i3, d3 = xgs.xgs_vq_assign(buf[1:].view(X.shape), Eg, None, None, xgs.VQ_FP32)
    torch.cuda.synchronize()
    np.testing.assert_array_equal(np_(i3), idx)
    np.testing.assert_array_equal(np_(d3), dist)
