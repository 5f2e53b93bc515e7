"""Decode + loss with the targets held in registers: every number of wavefronts,
column and pixel remainders, every alignment of the mask's count, and the
two-pass form beyond 1,024 columns or in a smaller workspace, against the FP64
oracle on the same map."""
import numpy as np
import pytest
import torch

import oracle
from gpu_util import np_, rel_max, require_gpu

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def xgs():
    return require_gpu()


def t(a, dtype=np.float32):
    return torch.from_numpy(np.ascontiguousarray(a, dtype=dtype)).cuda()


# D: one to 16 wavefronts, with whole and partial tiles, then beyond; pixels:
# one, a block less one, a block, odd planes (their rows are not 8-byte aligned)
@pytest.mark.parametrize("L,D,hs,ws", [(4, 4, 1, 1), (8, 60, 1, 31), (64, 68, 4, 8), (16, 132, 3, 43),
                                       (32, 260, 7, 19), (16, 516, 5, 29), (16, 1024, 9, 7), (16, 1028, 9, 7)])
@pytest.mark.parametrize("small_ws", [False, True])
def test_against_oracle(xgs, L, D, hs, ws, small_ws):
    rng = np.random.default_rng(1000 * L + D)
    wmap = rng.random((4 + L, hs, ws)).astype(np.float32)
    E = rng.standard_normal((L, D)).astype(np.float32)
    Gs = rng.standard_normal((D, hs, ws)).astype(np.float32)
    V = (rng.random((hs, ws)) < 0.7).astype(np.uint8) * rng.integers(1, 256, (hs, ws)).astype(np.uint8)
    V.reshape(-1)[0] = 0x80
    a = E.T.astype(np.float64) @ wmap[4:].reshape(L, -1).astype(np.float64)
    b = Gs.reshape(D, -1).astype(np.float64)
    # the L1 derivative jumps at a = b: such pixels are masked on both sides
    V.reshape(-1)[(np.abs(a - b) <= 4e-6 * (np.abs(a) + np.abs(b) + 1.0)).any(0)] = 0
    nbytes = 256 + 4 * (-(-hs * ws // 128)) if small_ws else int(xgs.lib.xgs_semantic_loss_workspace(hs, ws))
    work = torch.empty((nbytes + 255) // 256 * 256, dtype=torch.uint8, device="cuda")
    loss, d_out = xgs.xgs_semantic_loss(t(wmap), t(E), t(Gs), t(V, np.uint8), 0.75, workspace=work)
    torch.cuda.synchronize()
    ref, dref = oracle.semantic_loss(wmap[4:], E, Gs, (V != 0).astype(np.uint8), 0.75)
    d = np_(d_out)
    assert abs(float(np_(loss)[0]) - ref) <= 2e-5 * abs(ref)
    assert np.all(d[:4] == 0) and np.all(d[4:, V == 0] == 0)
    assert rel_max(d[4:], dref) < 1e-4


@pytest.mark.parametrize("offset", [0, 1, 7, 15])
@pytest.mark.parametrize("hs,ws", [(1, 5), (1, 16), (3, 77), (400, 700)])
def test_mask_count_at_any_alignment(xgs, offset, hs, ws):
    """One code, constant map and targets: every valid pixel's gradient is the
    same number over the count, so the count shows in it."""
    rng = np.random.default_rng(hs + offset)
    V = (rng.random((hs, ws)) < 0.5).astype(np.uint8) * 3
    V.reshape(-1)[[0, -1]] = 1
    buf = torch.zeros(offset + hs * ws, dtype=torch.uint8, device="cuda")
    buf[offset:] = t(V.reshape(-1), np.uint8)
    L, D = 4, 4
    wmap, E, Gs = torch.ones(4 + L, hs, ws), torch.ones(L, D), torch.zeros(D, hs, ws)
    loss, d = xgs.xgs_semantic_loss(wmap.cuda(), E.cuda(), Gs.cuda(), buf[offset:].view(hs, ws), 1.0)
    torch.cuda.synchronize()
    # cosine: den = eps, no slope through a zero target; L1: sum of E over D / (n D) = 1 / n
    want = np.where(V != 0, np.float64(1) / np.count_nonzero(V), 0.0)
    np.testing.assert_allclose(np_(d)[4:], np.broadcast_to(want, (L, hs, ws)), rtol=1e-6)
