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


@pytest.mark.parametrize("B,H,Sq,Sk,D,causal", SHAPES)
def test_four_waves(B, H, Sq, Sk, D, causal):
    base.test_rect_parity(B, H, H, Sq, Sk, D, causal)
