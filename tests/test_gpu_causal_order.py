"""Causal problems whose head count does not divide over the eight XCDs, and launches of two rounds of
resident work-groups: every tile of every head has to be computed once, whatever the order."""
import pytest

import test_gpu_rect as base

pytestmark = pytest.mark.gpu

# fewer heads than XCDs; one, four and seven heads left over next to whole ones; many tiles per head
# (the heads left over come first); D = 64 launches of at most and just over two rounds
SHAPES = [(1, 3, 3, 700, 700, 64), (1, 5, 5, 513, 513, 128), (3, 3, 3, 400, 400, 64), (4, 3, 3, 300, 300, 128),
          (5, 3, 3, 260, 260, 64), (1, 9, 3, 2100, 2100, 64), (1, 12, 12, 1500, 1500, 64), (8, 8, 8, 1024, 1024, 64),
          (1, 20, 4, 270, 400, 256), (2, 33, 33, 900, 900, 64),
          # three tiles per head: just up to a work-group per unit, two, and more
          (1, 85, 85, 300, 300, 64), (1, 170, 170, 300, 300, 64), (1, 171, 171, 300, 300, 64), (1, 171, 171, 300, 300, 256),
          # D = 64, four waves: more than four work-groups per unit but of few rounds, heads left over or not
          (1, 300, 300, 400, 400, 64), (1, 257, 257, 513, 513, 64), (1, 128, 128, 1100, 1100, 32)]


@pytest.mark.parametrize("B,Hq,Hkv,Sq,Sk,D", SHAPES)
def test_causal_order(B, Hq, Hkv, Sq, Sk, D):
    base.test_rect_parity(B, Hq, Hkv, Sq, Sk, D, True)
