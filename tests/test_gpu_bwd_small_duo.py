"""The one-launch backward of short heads with a wave for each part of a block (D <= 64, up to 256 heads),
at the edges of its blocks and either side of the head count that chooses it."""
import pytest

import test_gpu_rect as base

pytestmark = pytest.mark.gpu

SHAPES = [(1, 1, 1, 1, 64, False), (1, 2, 32, 32, 64, True), (2, 3, 33, 65, 64, True), (1, 4, 128, 97, 64, False),
          (1, 2, 96, 128, 32, True), (2, 128, 40, 40, 64, True), (1, 257, 40, 40, 64, True), (4, 64, 127, 128, 48, False)]


@pytest.mark.parametrize("B,H,Sq,Sk,D,causal", SHAPES)
def test_short_heads(B, H, Sq, Sk, D, causal):
    base.test_rect_parity(B, H, H, Sq, Sk, D, causal)
