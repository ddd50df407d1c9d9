"""Workspace sizes of the split plans (host only): what is asked for with one mask serves the other."""
import ctypes
import time

import pytest

import paper_2601_16238_amd as attn
from paper_2601_16238_amd import binding


@pytest.mark.parametrize("B,Hq,Hkv,Sq,Sk,D", [
    (1, 2, 2, 8192, 8192, 128), (1, 6, 6, 8192, 8192, 64), (1, 3, 1, 8192, 8192, 128), (2, 16, 4, 1537, 1537, 96),
    (1, 32, 8, 512, 4096, 128), (1, 8, 2, 1, 40000, 128), (1, 2, 2, 300, 1500, 256), (4, 8, 8, 40, 9000, 64),
    (1, 2, 1, 12637, 12637, 96), (8, 8, 8, 1024, 1024, 64)])
def test_a_workspace_sized_with_one_mask_serves_the_other(B, Hq, Hkv, Sq, Sk, D):
    assert attn.attn_fwd_rect_workspace_bytes(B, Hq, Hkv, Sq, Sk, D, False) == \
        attn.attn_fwd_rect_workspace_bytes(B, Hq, Hkv, Sq, Sk, D, True)
    size = [int(binding.lib().attn_bwd_rect_workspace_bytes(ctypes.byref(
        binding.make_rect_params(B, Hq, Hkv, Sq, Sk, D, 1.0, c)))) for c in (False, True)]
    assert size[0] == size[1] >= 8 * B * Hq * Sq
    # partial results stay small next to what a GPU holds: at most 256 splits' worth of work-groups
    assert size[0] - 8 * B * Hq * Sq <= 1 << 29


@pytest.mark.parametrize("B,Hq,Hkv,Sq,Sk,D,nsplit", [
    (1, 64, 8, 8, 32000, 128, 32), (8, 64, 8, 16, 4000, 128, 4), (4, 32, 8, 16, 8192, 128, 8), (10, 4, 1, 20, 772, 64, 3),
    (1, 64, 8, 16, 8192, 256, 22), (38, 8, 2, 11, 5537, 256, 3)])
def test_packed_rows_split_as_measured(B, Hq, Hkv, Sq, Sk, D, nsplit):
    """Grouped heads with a few new rows each (33 .. 128 packed rows per key/value head) run in the streaming
    kernel, every row on almost all keys: the number of splits that was measured to be the fastest or
    within 5 % of it (a work-group per compute unit where that divides evenly, never a few more than one)."""
    part = B * Hq * Sq * (max(64, D) + 1) * 4
    for causal in (False, True):
        assert (attn.attn_fwd_rect_workspace_bytes(B, Hq, Hkv, Sq, Sk, D, causal)) // part == nsplit


@pytest.mark.parametrize("H,Sq,Sk,nsplit", [(12, 3358, 13519, 3), (32, 1038, 10654, 3), (24, 1848, 9348, 2)])
def test_dq_is_split_where_the_unsplit_launch_takes_two_rounds(H, Sq, Sk, nsplit):
    """Causal, D = 128, long keys: 288 .. 360 unsplit work-groups of nearly equal length for 256 compute
    units, of which every second waits for a whole other one; measured 5 .. 16 % faster split."""
    part = H * Sq * 128 * 4
    assert (attn.attn_bwd_rect_workspace_bytes(1, H, H, Sq, Sk, 128) - 8 * H * Sq) // part == nsplit


@pytest.mark.parametrize("H,S,D,nsplit", [(3, 7903, 64, 4), (5, 4667, 64, 4), (5, 5787, 64, 4), (5, 9064, 128, 3), (5, 10000, 128, 3),
                                          (4, 13775, 128, 3)])
def test_long_causal_heads_are_split_as_measured(H, S, D, nsplit):
    """160 .. 240 work-groups of more than 4096 rows: 1.1 .. 1.6 times as long unsplit."""
    part = H * S * (D + 1) * 4
    assert attn.attn_fwd_rect_workspace_bytes(1, H, H, S, S, D, True) // part == nsplit


@pytest.mark.parametrize("Hq,Hkv,Sq,Sk,D", [(1, 1, 471, 16714, 64), (8, 1, 225, 19549, 128), (2, 1, 12560, 13659, 256)])
def test_a_plan_takes_a_few_microseconds(Hq, Hkv, Sq, Sk, D):
    """Every backward call makes them (a loop over the key blocks for each cut took 30 .. 53 us here; now at most 4)."""
    p = ctypes.byref(binding.make_rect_params(1, Hq, Hkv, Sq, Sk, D, 1.0, True))
    f, least = binding.lib().attn_bwd_rect_best_workspace_bytes, 1.0
    for _ in range(200):
        t = time.perf_counter()
        f(p)
        least = min(least, time.perf_counter() - t)
    assert least < 12e-6


@pytest.mark.parametrize("Hq,Hkv,Sq,Sk", [(1, 1, 9000, 9007), (2, 1, 5000, 6001), (4, 1, 2000, 2063), (3, 3, 1601, 3000),
                                          (2, 2, 3000, 3001), (16, 2, 225, 3200), (1, 1, 1537, 4096)])
def test_chunks_of_dk_dv_cover_the_key_blocks(Hq, Hkv, Sq, Sk):
    """The chunks that the plan counts in closed form, block by block, D = 256 (where dQ has no partial results)."""
    def chunks(causal):
        group, n_block, n_slot = Hq // Hkv, (Sk + 63) // 64, (Sq + 31) // 32
        slots = [group * (n_slot - max(0, 64 * kt - (Sk - Sq)) // 32 * causal) for kt in range(n_block)]
        if Hkv * n_block >= 256 or slots[0] < 48:
            return 0
        L = max(16, (sum(slots) * Hkv + 255) // 256)
        while 4 * L <= 3 * slots[0]:
            items = sum((s + L - 1) // L for s in slots) * Hkv
            if items <= 256:
                return items
            L += (L + 31) // 32
        return 0
    part = max(chunks(0), chunks(1)) * 2 * 64 * 256 * 4
    assert part > 0
    assert attn.attn_bwd_rect_workspace_bytes(1, Hq, Hkv, Sq, Sk, 256) == (8 * Hq * Sq + 255) // 256 * 256 + part
