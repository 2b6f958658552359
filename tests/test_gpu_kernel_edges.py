"""Small problems at the edges of the kernels' tiles and of the rules that choose between them, against the oracle.

Tolerances: the ones of tests/parity.py (tiny = toy networks, where fp32 rounding is all there is)."""
import pytest

from dds_inputs.configs import tiny_resnet
from test_gpu_parity import _compare

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("W,B", [(1, 63), (2, 32), (3, 85), (2, 128)])
def test_update_ranges_by_split_count(W, B):
    # 16-channel layers at 16 x 16 pixels have one split per image: 63 / 64 / 255 / 256 of them lie on both sides of the
    # lines between 256-, 64- and 32-element ranges
    _compare(tiny_resnet(K=1, W=W, B=B, hw=16, c=16, precision="bf16"), seed=20, T=2)
