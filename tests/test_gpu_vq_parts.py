"""BF16 assignment of few rows: the codebook swept in more parts than its size
asks for, against the fewer parts of a smaller workspace: the same codewords and
distances bit for bit, with and without the confidence (whose own sums are added in
another order; its bound against the oracle is tested with the robust update)."""
import numpy as np
import pytest
import torch

from gpu_util import np_, require_gpu

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def xgs():
    return require_gpu()


# parts of one tile and of several, a last part that is short, more than 4 parts by
# size alone; rows split over wavefronts (D >= 384) or not, a last row group that is short
@pytest.mark.parametrize("n,k,d", [(1, 4096, 64), (301, 4096, 384), (1200, 4096, 768), (1199, 5000, 128),
                                   (130, 20000, 64), (2500, 4097, 392)])
def test_more_parts_same_answer(xgs, n, k, d):
    gen = torch.Generator(device="cuda").manual_seed(n + k)
    centres = torch.randn(32, d, device="cuda", generator=gen)
    def rows(m):
        x = centres[torch.randint(0, 32, (m,), device="cuda", generator=gen)]
        return (x + 0.3 * torch.randn(m, d, device="cuda", generator=gen)).contiguous()
    X, E = rows(n), rows(k)
    E[k // 2:k // 2 + 300] = E[:300]          # ties: the lower index wins in any number of parts
    Eb, en = xgs.xgs_vq_prepare(E)
    ws = xgs.vq_assign_workspace(n, d, k)
    out = []
    for w in (ws, ws[:-256]):
        idx, dist = xgs.xgs_vq_assign(X, E, Eb, en, workspace=w)
        i2, d2, conf = xgs.xgs_vq_assign_conf(X, E, Eb, en, 0.7, workspace=w)
        torch.cuda.synchronize()
        out.append([np_(a) for a in (idx, dist, i2, d2)])
    for a, b in zip(*out):
        np.testing.assert_array_equal(a, b)
    assert not np.isin(out[0][0], np.arange(k // 2, k // 2 + 300)).any()


# row counts on either side of the line between one and four rows a wavefront: the
# first rows of a longer call get the same bits as on their own
@pytest.mark.parametrize("n,d", [(65_537, 64), (262_145, 384)])
def test_rescore_forms_same_bits(xgs, n, d):
    gen = torch.Generator(device="cuda").manual_seed(d)
    X, E = torch.randn(n, d, device="cuda", generator=gen), torch.randn(600, d, device="cuda", generator=gen)
    Eb, en = xgs.xgs_vq_prepare(E)
    long = xgs.xgs_vq_assign_conf(X, E, Eb, en, 0.7) + xgs.xgs_vq_assign(X, E, Eb, en)
    few = X[:n - 2].contiguous()
    short = xgs.xgs_vq_assign_conf(few, E, Eb, en, 0.7) + xgs.xgs_vq_assign(few, E, Eb, en)
    torch.cuda.synchronize()
    for a, b in zip(long, short):
        assert torch.equal(a[:n - 2], b)
