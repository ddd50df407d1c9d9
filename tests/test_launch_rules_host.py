"""Which form of a kernel a launch takes (host only): the rules on the shape, at problems whose forms were timed against
each other."""
import pytest

from parity_util import host_rule


# (heads, rows, keys, at most 32 columns): us with four waves | eight
@pytest.mark.parametrize("BH,S,Sk,narrow,waves", [
    (49, 1967, 1967, False, 8), (53, 1815, 1815, False, 8), (23, 4425, 4425, False, 8), (21, 4904, 4904, False, 8),  # 1.02 .. 1.04
    (26, 4186, 4186, False, 8), (22, 4747, 4747, False, 8), (53, 2028, 3260, False, 8),  # 163 | 157, 116 | 114
    (159, 700, 700, False, 4), (127, 970, 970, False, 4), (388, 254, 254, False, 4),  # 32 | 34, 43 | 44, 16 | 17
    (32, 1957, 1957, False, 8), (65, 817, 817, False, 4), (454, 388, 388, False, 4), (6, 5181, 5181, False, 4),
    (63, 2604, 2604, True, 8), (93, 1772, 1772, True, 8), (102, 5496, 5496, True, 8), (453, 1169, 1169, True, 8),  # 1.05 .. 1.06
    (584, 385, 385, True, 8), (1272, 234, 234, True, 8), (80, 3047, 3047, True, 8),  # 29 | 27, 155 | 145
    (134, 583, 662, True, 4), (250, 291, 291, True, 4), (535, 355, 355, True, 4)])  # 20 | 23, 12 | 13, 27 | 34
def test_waves_of_the_unsplit_forward_at_64_columns(BH, S, Sk, narrow, waves):
    assert host_rule("fwd_waves_unsplit", BH, S, Sk, False, narrow) == waves


@pytest.mark.parametrize("BH,S,narrow,waves", [
    (19, 5250, False, 8), (22, 4595, False, 8), (61, 1763, False, 8), (24, 4624, False, 8),  # 195 | 188, 83 | 81, 200 | 194
    (162, 768, False, 4), (225, 458, False, 4), (9, 5052, False, 8), (316, 318, False, 4)])  # 43 | 46, 31 | 33, 105 | 96
def test_waves_of_the_unsplit_dq_at_64_columns(BH, S, narrow, waves):
    assert host_rule("dq_waves", BH, S, S, 64, False, narrow) == waves
