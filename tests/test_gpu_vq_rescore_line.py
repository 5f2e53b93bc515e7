"""The rescore of one and of four rows a wavefront, on both sides of the row counts
where the rule for short rows changes from one to the other."""
import pytest

from gpu_util import require_gpu
from test_gpu_vq_parts import test_rescore_forms_same_bits as same_bits

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n,d", [(45_057, 64), (45_057, 248), (65_537, 256)])
def test_same_bits_at_the_lines(n, d):
    same_bits(require_gpu(), n, d)
