"""The forward's workspace at its limits: with less than the plan's partial results, but one work-group per
compute unit's worth (or anything, where that rule does not split), the call is accepted, stays inside the
workspace and gives the unsplit result to rounding."""
import ctypes

import pytest
import torch

import paper_2601_16238_amd as attn
from paper_2601_16238_amd import binding

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("B,Hq,Hkv,Sq,Sk,D,causal,size,refused", [
    (8, 2, 2, 353, 5318, 64, True, 6 * 8 * 2 * 353 * 65 * 4, 256),    # six splits fit of eight
    (1, 8, 1, 2018, 2018, 64, True, 2 * 8 * 2018 * 65 * 4, 256),    # two of three
    (8, 1, 1, 8373, 8373, 128, False, 256, None),                     # fits none: unsplit
    (1, 8, 8, 5748, 5748, 256, False, 256, None)])
def test_smaller_workspace(B, Hq, Hkv, Sq, Sk, D, causal, size, refused):
    size = (size + 255) // 256 * 256
    full = attn.attn_fwd_rect_workspace_bytes(B, Hq, Hkv, Sq, Sk, D, causal)
    assert full > size, "the plan does not split further"
    g = torch.Generator(device="cuda").manual_seed(5)
    Q = torch.randn(B, Hq, Sq, D, device="cuda", generator=g).bfloat16()
    K, V = (torch.randn(B, Hkv, Sk, D, device="cuda", generator=g).bfloat16() for _ in range(2))
    O, LSE = torch.empty_like(Q), torch.empty(B, Hq, Sq, device="cuda")
    ws = torch.full((full + 4096,), 0x5a, dtype=torch.uint8, device="cuda")
    p = binding.make_rect_params(B, Hq, Hkv, Sq, Sk, D, D ** -0.5, causal)
    call = lambda n: binding.lib().attn_fwd_rect(
        *(ctypes.c_void_p(t.data_ptr()) for t in (Q, K, V, O, LSE, ws)), ctypes.c_size_t(n), ctypes.byref(p),
        ctypes.c_void_p(torch.cuda.current_stream().cuda_stream))
    print("case fwd workspace", B, Hq, Hkv, Sq, Sk, D, causal, size, full, flush=True)
    if refused is not None:
        assert call(refused) == binding.ATTN_ERR_WORKSPACE
    assert call(size) == 0
    Oref, Lref = attn.attn_fwd_rect(Q, K, V, D ** -0.5, causal, split=False)
    torch.cuda.synchronize()
    assert bool((ws[size:] == 0x5a).all())
    # Row by row.  Both sides round O to bf16 (a neighbouring value: 2^-7 of it) after fp32 sums over P
    # rounded to bf16 against different reference maxima: independent errors of 2^-9 / sqrt(3) relative per
    # key and side, which over V ~ N(0, 1) add up to sqrt(2) 2^-9 / sqrt(3) of O's own size sqrt(sum P^2),
    # the row's rms; six deviations of that, for 10^5 .. 10^7 values, are below 2^-6 rms
    diff, o = (O.float() - Oref.float()).abs().amax(-1), Oref.float()
    assert (diff <= 2 ** -7 * o.abs().amax(-1) + 2 ** -6 * o.square().mean(-1).sqrt()).all()
    assert (LSE - Lref).abs().max().item() <= 2e-5
