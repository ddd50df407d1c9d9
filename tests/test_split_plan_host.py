"""Workspace sizes of the split plans (host only): what is asked for with one mask serves the other."""
import ctypes

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
