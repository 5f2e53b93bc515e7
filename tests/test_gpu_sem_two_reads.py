"""Decode + loss without a mask over many pixels, which for some widths reads the
targets twice: the same as under a mask of ones, which holds them in registers."""
import pytest
import torch

from gpu_util import require_gpu

pytestmark = pytest.mark.gpu


# widths at the ends of the rule, below and above its pixel count
@pytest.mark.parametrize("hs,ws", [(256, 383), (256, 384)])
@pytest.mark.parametrize("L,D", [(4, 516), (8, 896), (16, 640), (16, 656), (16, 892), (32, 516), (32, 580), (64, 260),
                                 (64, 292)])
def test_same_as_under_a_mask_of_ones(L, D, hs, ws):
    """Decoded values are the same bits in both forms (one order of products), so are
    the signs of the L1 term; sums of D terms in another order differ by about
    sqrt(D) 2^-24 each, two of them under the cosine: 1e-5 with a factor of two."""
    xgs = require_gpu()
    g = torch.Generator(device="cuda").manual_seed(L * D)
    rand = lambda *s: torch.randn(s, generator=g, device="cuda")
    wmap, E, G = torch.softmax(rand(4 + L, hs, ws), 0), rand(L, D), rand(D, hs, ws)
    loss, d = xgs.xgs_semantic_loss(wmap, E, G, None)
    loss1, d1 = xgs.xgs_semantic_loss(wmap, E, G, torch.ones((hs, ws), dtype=torch.uint8, device="cuda"))
    torch.cuda.synchronize()
    assert not bool(d[:4].any())
    assert abs(float(loss.item()) - float(loss1.item())) <= 1e-5 * abs(float(loss1.item()))
    assert float((d - d1).norm()) <= 1e-5 * float(d1.norm())
