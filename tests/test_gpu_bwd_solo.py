"""dK and dV by work-groups of 256 keys, 64 a wave (attn_bwd_solo.hip), which large launches at D = 65 .. 128 take:
bit for bit those of the producer/consumer kernel, which the oracle tests of smaller calls run (the same products in
the same order), and with dS stored the same dQ as well.  Against the oracle: the large shapes of test_gpu_full_size.py."""
import pytest
import torch

import paper_2601_16238_amd as attn
from parity_util import STORED_DS, backward_form, host_rule, in_layout

pytestmark = pytest.mark.gpu

# last key block with one key and ragged; last slot ragged; offsets off the slots and the key blocks; waves that see no key of a slot, heads of a group one after the other; narrow and padded columns
CASES = [(250, 250, 500, 500, 128, False, False), (128, 32, 545, 1025, 96, False, False), (128, 64, 700, 2311, 128, True, False),
         (90, 45, 1100, 1133, 72, False, True), (96, 48, 2500, 2777, 120, True, True), (64, 64, 3551, 3551, 80, True, False)]


@pytest.mark.parametrize("H,Hkv,Sq,Sk,D,causal,f16", CASES)
def test_keys_by_the_wave(H, Hkv, Sq, Sk, D, causal, f16):
    print("case solo", H, Hkv, Sq, Sk, D, causal, f16, flush=True)
    g = torch.Generator(device="cuda")
    g.manual_seed(Sq + Sk)
    dt = torch.float16 if f16 else torch.bfloat16
    Q = torch.randn((1, H, Sq, D), generator=g, device="cuda").to(dt)
    # (multiples of a quarter and an eighth: delta = rowsum(dO O) is exact in every order in which the kernels that
    # form it may add)
    dO = (torch.randn((1, H, Sq, D), generator=g, device="cuda") * 4).round().div(4).to(dt)
    K, V = (torch.randn((1, Hkv, Sk, D), generator=g, device="cuda").to(dt) for _ in range(2))
    O, LSE = attn.attn_fwd_rect(Q, K, V, D ** -0.5, causal)
    O = (O.float() * 8).round().div(8).to(dt)

    def backward(lo, hi, room):
        """K/V heads lo .. hi - 1, in a workspace of the row statistics and `room` bytes more."""
        G, stats = H // Hkv, 8 * (hi - lo) * (H // Hkv) * Sq
        ws = torch.full(((stats + 255) // 256 * 256 + room,), 0xFF, dtype=torch.uint8, device="cuda")
        q = [x[:, lo * G:hi * G].contiguous() for x in (Q, O, dO, LSE)]
        k = [x[:, lo:hi].contiguous() for x in (K, V)]
        return attn.attn_bwd_rect(q[0], *k, q[1], q[2], q[3], D ** -0.5, causal, workspace=ws)

    assert all(host_rule("dkdv_takes_solo", Hkv, H // Hkv, Sq, Sk, causal, stored) for stored in (False, True))
    whole = backward(0, Hkv, 0)
    n = 255 // ((Sk + 127) // 128)  # fewer than a work-group of 128 keys per compute unit: the pairs
    for lo in range(0, Hkv, n):
        assert not host_rule("dkdv_takes_solo", min(n, Hkv - lo), H // Hkv, Sq, Sk, causal, False)
        part = backward(lo, min(lo + n, Hkv), 0)
        for w, p in zip(whole[1:], part[1:]):
            assert torch.equal(w[:, lo:lo + n].view(torch.int16), p.view(torch.int16))
    best = attn.attn_bwd_rect_best_workspace_bytes(1, H, Hkv, Sq, Sk, D, causal)
    assert backward_form(1, H, Hkv, Sq, Sk, D, causal, best) == STORED_DS
    stored = backward(0, Hkv, best)
    for w, s in zip(whole[1:], stored[1:]):
        assert torch.equal(w.view(torch.int16), s.view(torch.int16))
    # dQ from the stored dS: the recomputed one's products in another order (one rounding step, or the
    # fp32 rounding of the sums where the terms cancel)
    w, s = whole[0].double(), stored[0].double()
    assert bool(((w - s).abs() <= w.abs() * 2.0 ** -7 + 1e-3 * w.abs().max()).all())
    torch.cuda.synchronize()


@pytest.mark.parametrize("B,H,Hkv,Sq,Sk,D,causal", [(2, 64, 32, 700, 2311, 128, True), (2, 64, 16, 545, 1025, 96, False),
                                                    (2, 48, 24, 1100, 1133, 72, False), (4, 32, 16, 420, 650, 128, False)])
@pytest.mark.parametrize("layout", ["BSHD", "padded"])
def test_other_layouts(B, H, Hkv, Sq, Sk, D, causal, layout):
    """[B,S,H,D] storage and rows, heads and batch entries with NaN between them, against contiguous tensors: the same kernels
    on the same values, with dS stored and without.  What lies between the outputs stays as it is."""
    print("case solo layout", B, H, Hkv, Sq, Sk, D, causal, layout, flush=True)
    g = torch.Generator(device="cuda")
    g.manual_seed(Sq + Sk)
    Q, dO = (torch.randn((B, H, Sq, D), generator=g, device="cuda").bfloat16() for _ in range(2))
    K, V = (torch.randn((B, Hkv, Sk, D), generator=g, device="cuda").bfloat16() for _ in range(2))
    O, LSE = attn.attn_fwd_rect(Q, K, V, D ** -0.5, causal)
    assert all(host_rule("dkdv_takes_solo", B * Hkv, H // Hkv, Sq, Sk, causal, stored) for stored in (False, True))
    best = attn.attn_bwd_rect_best_workspace_bytes(B, H, Hkv, Sq, Sk, D, causal)
    assert backward_form(B, H, Hkv, Sq, Sk, D, causal, best) == STORED_DS
    for n in ((8 * B * H * Sq + 255) // 256 * 256, best):
        ws = torch.full((n,), 0xFF, dtype=torch.uint8, device="cuda")
        want = attn.attn_bwd_rect(Q, K, V, O, dO, LSE, D ** -0.5, causal, workspace=ws)
        out = [in_layout(torch.zeros_like(x), layout) for x in (Q, K, V)]
        attn.attn_bwd_rect(*(in_layout(x, layout) for x in (Q, K, V, O, dO)), LSE, D ** -0.5, causal, dQ=out[0], dK=out[1],
                           dV=out[2], workspace=ws.fill_(0xFF))
        torch.cuda.synchronize()
        for o, w in zip(out, want):
            assert torch.equal(o.contiguous().view(torch.int16), w.view(torch.int16))
            if layout == "padded":  # everything else of the storage
                whole = torch.empty(0, dtype=o.dtype, device="cuda").set_(o.untyped_storage())
                assert int(whole.isnan().sum()) == whole.numel() - o.numel()


@pytest.mark.parametrize("H,Hkv,S,D,causal", [(48, 24, 1500, 72, False), (40, 40, 3551, 128, True)])
def test_stage_by_stage(H, Hkv, S, D, causal):
    """The statistics, dK/dV and dQ in calls of their own against one call (delta is exact, as above)."""
    print("case solo stages", H, Hkv, S, D, causal, flush=True)
    g = torch.Generator(device="cuda")
    g.manual_seed(S)
    Q = torch.randn((1, H, S, D), generator=g, device="cuda").bfloat16()
    dO = (torch.randn((1, H, S, D), generator=g, device="cuda") * 4).round().div(4).bfloat16()
    K, V = (torch.randn((1, Hkv, S, D), generator=g, device="cuda").bfloat16() for _ in range(2))
    O, LSE = attn.attn_fwd_gqa(Q, K, V, D ** -0.5, causal)
    O = (O.float() * 8).round().div(8).bfloat16()
    assert host_rule("dkdv_takes_solo", Hkv, H // Hkv, S, S, causal, False)
    ws = torch.full(((8 * H * S + 255) // 256 * 256,), 0xFF, dtype=torch.uint8, device="cuda")
    whole = attn.attn_bwd_gqa(Q, K, V, O, dO, LSE, D ** -0.5, causal, workspace=ws)
    out = [torch.full_like(x, float("nan")) for x in (Q, K, V)]
    ws.fill_(0xFF)
    for stage in (1, 2, 4):
        attn.attn_bwd_gqa(Q, K, V, O, dO, LSE, D ** -0.5, causal, dQ=out[0], dK=out[1], dV=out[2], workspace=ws, stages=stage)
    torch.cuda.synchronize()
    for w, o in zip(whole, out):
        assert torch.equal(w.view(torch.int16), o.view(torch.int16))
