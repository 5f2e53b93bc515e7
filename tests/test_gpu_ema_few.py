"""EMA update of few rows (one workgroup sorts and cuts them into pieces) against
the general sort, bit for bit: one more codeword that no row has sends the same
rows down the general route.  Row counts at the powers of two, at a piece and at
the largest of the route; all rows on one codeword, spread, masked out."""
import numpy as np
import pytest
import torch

from gpu_util import np_, require_gpu

pytestmark = pytest.mark.gpu
K = 1 << 14  # the most codewords of the route


@pytest.fixture(scope="module")
def xgs():
    return require_gpu()


@pytest.mark.parametrize("n", [0, 1, 2, 3, 64, 65, 129, 1200, 2048, 2049, 4096])
@pytest.mark.parametrize("kind", ["spread", "skewed", "one", "masked"])
def test_same_bits_as_the_general_route(xgs, n, kind):
    rng = np.random.default_rng(n)
    D = 8
    X = rng.standard_normal((n, D)).astype(np.float32)
    idx = rng.integers(0, K, n)
    if kind == "skewed":
        idx = np.minimum(rng.zipf(1.3, n), K) - 1
    elif kind == "one":
        idx[:] = K - 1
    conf = rng.random(n).astype(np.float32) if kind != "masked" else np.zeros(n, np.float32)
    if n > 2:
        conf[1] = np.nan
    N0, M0 = rng.random(K + 1).astype(np.float32) + 1, rng.standard_normal((K + 1, D)).astype(np.float32)
    out = []
    for k in (K, K + 1):
        t = lambda a: torch.from_numpy(np.ascontiguousarray(a)).cuda()
        Ng, Mg, Eg = t(N0[:k]), t(M0[:k]), torch.zeros(k, D, device="cuda")
        Xg, ig, cg = t(X), t(idx.astype(np.int32)), t(conf)
        if n == 0:  # tensors of no rows have no address
            Xg, ig, cg = torch.zeros(1, D, device="cuda")[:0], torch.zeros(1, dtype=torch.int32, device="cuda")[:0], \
                torch.zeros(1, device="cuda")[:0]
        res = xgs.xgs_vq_ema_update_robust(Xg, ig, cg, 0.3, Ng, Mg, Eg, None, None, 0.9, 1e-5, xgs.EMA_PAPER, 0.0,
                                           None, 0)
        torch.cuda.synchronize()
        out.append([np_(a)[:K] for a in (res[0], Ng, Mg, Eg)])
    for a, b in zip(*out):
        np.testing.assert_array_equal(a.view(np.int32), b.view(np.int32))
    keep = conf >= 0.3
    np.testing.assert_array_equal(out[0][0], np.bincount(idx[keep], minlength=K).astype(np.float32))
