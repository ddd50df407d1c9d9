"""Which form of a kernel a launch takes (host only): the rules on the shape, at problems whose forms were timed against
each other."""
import ctypes

import pytest

from paper_2601_16238_amd import binding
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


# us split | unsplit where the plan had split as if the unsplit launch had eight waves too: 24 | 17, 22 | 15, 28 | 19, 14 | 10,
# 23 | 16, 27 | 21; splits that pay: 31 | 61, 42 | 48, 84 | 95, 46 | 49, 66 | 70; unsplit eight waves of more than one round:
# 305 | 289, 303 | 290, 486 | 457; of one round: 126 | 133, 124 | 129
@pytest.mark.parametrize("BH,S,Sk,nsplit", [
    (20, 1119, 1119, 1), (16, 1175, 1175, 1), (21, 1353, 1353, 1), (11, 604, 604, 1), (34, 572, 1393, 1), (27, 869, 1886, 1),
    (1, 5740, 5740, 10), (43, 706, 3476, 3), (5, 5391, 8474, 2), (15, 1284, 4319, 2), (83, 463, 3625, 3),
    (16, 6479, 12904, 1), (19, 5197, 13176, 1), (18, 5958, 15230, 1), (17, 2630, 7291, 4), (11, 4259, 7288, 4)])
def test_the_forward_at_64_columns_is_split_where_that_is_quicker(BH, S, Sk, nsplit):
    f = binding.lib()._ZN4attn14fwd_split_planEiiiibbPiiNS_9SplitRuleE
    f.argtypes = [ctypes.c_int] * 4 + [ctypes.c_bool] * 2 + [ctypes.c_void_p, ctypes.c_int, ctypes.c_int]
    assert f(BH, S, Sk, 64, False, False, None, 128, 0) == nsplit


# whole backward, us with eight | sixteen blocks or the latter's time relative to the former's
@pytest.mark.parametrize("heads,S,causal,blocks", [
    (128, 4096, False, 16), (128, 2048, True, 16), (192, 2048, False, 16),  # 1258 | 1228
    (78, 5545, False, 16), (77, 4360, True, 16), (91, 7289, True, 16), (89, 5211, False, 16),  # 0.975, 0.981, 0.968, 0.98
    (120, 2300, False, 16), (100, 3800, False, 16), (100, 3800, True, 8),  # fifteen blocks of 256: a sixteenth only pads
    (442, 935, True, 8), (507, 905, True, 8), (482, 718, True, 8), (482, 718, False, 8),  # 1.037, 1.031, 341 | 347
    (64, 2048, True, 8), (16, 4096, True, 8), (16, 16384, True, 8), (11, 1166, False, 2)])
def test_row_blocks_of_dq_from_the_stored_ds(heads, S, causal, blocks):
    assert host_rule("dq_ds_blocks", heads, S, 128, causal) == blocks
    assert host_rule("dq_ds_blocks", heads, S, 96, causal) == min(blocks, 8)


# us with two work-groups on a unit | three
@pytest.mark.parametrize("BH,S,Sk,nsplit,two", [
    (8, 4471, 4481, 3, True), (8, 4605, 4605, 3, True), (7, 5079, 5079, 3, True), (9, 2375, 2375, 4, True),  # 47 | 54, 39 | 43, 46 | 53, 27 | 29
    (5, 4129, 4129, 4, True), (5, 7688, 7688, 3, True),
    (1, 1000, 1000, 3, True), (22, 2682, 2893, 2, False), (18, 3564, 3832, 2, False), (10, 5626, 5626, 2, False),  # 43 | 37, 57 | 48, 55 | 53
    (15, 6235, 6235, 1, True), (30, 2845, 2845, 1, True), (24, 4096, 4096, 1, True),  # 73 | 77, 45 | 47
    (64, 1024, 1024, 1, False), (60, 1280, 1280, 1, False), (25, 4096, 4096, 1, False)])
def test_work_groups_of_the_causal_forward_on_a_unit(BH, S, Sk, nsplit, two):
    assert host_rule("fwd_takes_two", BH, S, Sk, nsplit, ((Sk + 63) // 64 + nsplit - 1) // nsplit * 64) == two


def test_work_groups_of_one_wave_of_dq_on_a_unit():
    """Two, not three, where both take two rounds."""
    assert [host_rule("dq_takes_two", 1, n) for n in (512, 768, 769, 960, 1024, 1025, 1536)] == [False] * 2 + [True] * 3 + [False] * 2
    assert not host_rule("dq_takes_two", 2, 960) and not host_rule("dq_takes_two", 4, 960)


def test_main_loop_of_four_waves_at_64_columns():
    """Narrow tensors without a mask: from three tiles on where two work-groups share a unit at most (6.1 us, 6.5 without it)."""
    def rule(wgs, Sk, nsplit=1, causal=False, narrow=True):
        return host_rule("fwd_takes_main", wgs, Sk, nsplit, causal, narrow)
    assert rule(128, 192) and rule(512, 255) and not rule(128, 191) and not rule(513, 255)
    assert not rule(128, 255, causal=True) and not rule(128, 255, narrow=False) and rule(2000, 256, causal=True, narrow=False)
    assert rule(128, 100, nsplit=2)


# whole backward, us with dK/dV by pairs of waves | by one wave per SIMD
@pytest.mark.parametrize("heads,group,S,Sk,causal,stored,solo", [
    (22, 4, 583, 2989, True, True, False), (18, 1, 917, 3848, True, True, False), (57, 1, 1528, 1528, True, False, False),  # 235 | 306, 126 | 146, 153 | 178
    (25, 2, 1534, 3086, True, True, False), (83, 4, 1113, 1113, True, True, False), (9, 1, 1166, 7659, True, False, False),  # 254 | 283, 343 | 389, 169 | 193
    (20, 4, 161, 3150, True, True, False), (128, 8, 142, 733, True, True, False),  # 1.18, 1.12
    (128, 1, 4096, 4096, True, True, True), (16, 1, 16384, 16384, True, True, True), (14, 1, 1569, 8812, True, True, True),  # 1625 | 1580, 2835 | 2690, 324 | 286
    (320, 1, 2048, 2048, True, False, True), (320, 1, 2048, 2048, True, True, False),  # 1247 | 1207, 1165 | 1172
    (256, 1, 3000, 3000, True, False, True), (64, 1, 2048, 2048, True, False, True), (512, 1, 1536, 1536, True, False, False),  # 2002 | 1919, 255 | 237, 1214 | 1229
    (128, 1, 4096, 4096, False, True, True), (26, 4, 1156, 1156, False, True, True), (256, 1, 372, 372, True, True, False)])  # 2921 | 2735, 271 | 232, 65 | 77
def test_one_wave_per_simd_for_dkdv(heads, group, S, Sk, causal, stored, solo):
    assert host_rule("dkdv_takes_solo", heads, group, S, Sk, causal, stored) == solo
