"""The forward at D <= 64 with four waves: either side of the launch sizes and lengths that choose between the
form with the pipelined main loop and the generic one (two or three work-groups per compute unit)."""
import pytest

import test_gpu_rect as base

pytestmark = pytest.mark.gpu

# whole key tiles: two, three; 512 and 514 work-groups; above 896 work-groups, on 300 and 520 keys; more
# work-groups with 1024 rows and more
SHAPES = [(1, 6, 191, 191, 64, True), (1, 6, 192, 192, 64, True), (1, 256, 200, 200, 64, False),
          (1, 257, 200, 200, 64, False), (1, 257, 225, 225, 40, True), (3, 150, 129, 300, 64, False),
          (3, 150, 129, 520, 64, True), (1, 86, 1030, 1030, 64, True), (1, 60, 1100, 1100, 64, True)]

# ... and those that choose between four waves and eight: three and four tiles; 256 and 257 work-groups of four waves and of
# eight, without a mask; narrow tensors; many heads under a mask; more keys than rows
SHAPES += [(1, 40, 255, 255, 64, False), (1, 40, 256, 256, 64, False), (1, 85, 300, 300, 64, False), (1, 86, 300, 300, 64, False),
           (1, 128, 257, 257, 64, False), (1, 129, 257, 257, 64, False), (1, 193, 260, 260, 32, False),
           (1, 513, 300, 300, 64, True), (2, 48, 240, 577, 48, False), (1, 64, 192, 192, 32, False), (1, 256, 195, 195, 24, False),
           (1, 257, 200, 200, 32, False), (1, 64, 191, 191, 32, False)]


@pytest.mark.parametrize("B,H,Sq,Sk,D,causal", SHAPES)
def test_four_waves(B, H, Sq, Sk, D, causal):
    base.test_rect_parity(B, H, H, Sq, Sk, D, causal)
