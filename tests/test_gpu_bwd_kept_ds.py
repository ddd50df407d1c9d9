"""dQ from the dS that the dK/dV kernel stores: against the fp64 oracle, against the form that recomputes
dS, and in parts of the heads."""
import numpy as np
import pytest
import torch

import oracle
import paper_2601_16238_amd as attn
from paper_2601_16238_amd import workloads as wl
from parity_util import host_rule, DKDV_CUT, STORED_DS, backward_form, bf16_round, check_grad, f16_round, in_layout, to_f64

pytestmark = pytest.mark.gpu

# (last: dK/dV cut into chunks)  work-groups of 64, 128 and 256 rows; last slot and last key block ragged,
# one row; a causal offset off the 32-key blocks; key blocks that no row of a slot sees; grouped heads; padded head
# dimensions; fp16; four and six pairs
CASES = [(2, 2, 2, 92, 1039, 128, True, False, 0), (1, 33, 33, 1, 900, 128, True, True, 0), (1, 70, 70, 1, 500, 256, False, False, 0),
         (1, 96, 24, 400, 400, 96, True, True, 1), (2, 48, 12, 385, 609, 128, True, False, 1),
         (1, 36, 12, 700, 733, 128, True, False, 1), (1, 72, 9, 290, 321, 200, False, False, 1),
         (1, 56, 14, 400, 433, 256, True, True, 1), (2, 33, 33, 289, 417, 256, False, False, 0),
         (1, 90, 90, 300, 300, 128, False, False, 0), (2, 48, 48, 300, 331, 80, True, False, 0),
         (1, 120, 120, 513, 70, 128, False, False, 0), (2, 256, 256, 40, 161, 128, True, False, 0)]


@pytest.mark.parametrize("B,Hq,Hkv,Sq,Sk,D,causal,f16,cut", CASES)
def test_dq_from_the_stored_ds(B, Hq, Hkv, Sq, Sk, D, causal, f16, cut):
    print("case kept_ds", B, Hq, Hkv, Sq, Sk, D, causal, f16, flush=True)
    draw = wl.random_rect_inputs_f16 if f16 else wl.random_rect_inputs
    x = draw(B, Hq, Hkv, Sq, Sk, D, seed=5200 + Sq + D)
    rnd = f16_round if f16 else bf16_round
    ref = oracle.attn_bwd(x["Q"], x["K"], x["V"], x["dO"], x["scale"], causal, dtype="f16" if f16 else "bf16")
    dt = torch.float16 if f16 else torch.bfloat16
    Q, K, V, dO = (torch.from_numpy(x[k].view(np.int16)).cuda().view(dt) for k in ("Q", "K", "V", "dO"))
    O, LSE = attn.attn_fwd_rect(Q, K, V, x["scale"], causal)
    best = attn.attn_bwd_rect_best_workspace_bytes(B, Hq, Hkv, Sq, Sk, D, causal)
    assert backward_form(B, Hq, Hkv, Sq, Sk, D, causal, best) == STORED_DS + DKDV_CUT * cut
    ws = torch.full((best + 4096,), 0xFF, dtype=torch.uint8, device="cuda")   # NaN: nothing may be relied on
    got = attn.attn_bwd_rect(Q, K, V, O, dO, LSE, x["scale"], causal, workspace=ws[:best])
    again = attn.attn_bwd_rect(Q, K, V, O, dO, LSE, x["scale"], causal)
    torch.cuda.synchronize()
    assert bool((ws[best:] == 0xFF).all()), "written past the workspace"
    for name, g, a, r in zip(("dQ", "dK", "dV"), got, again, ref):
        check_grad(name, to_f64(g), r, rnd=rnd)
        assert torch.equal(g.view(torch.int16), a.view(torch.int16)), name


@pytest.mark.parametrize("H,Hkv,S,D,causal", [(702, 351, 330, 128, True), (400, 400, 333, 256, False)])
def test_ds_of_a_part_of_the_heads_at_a_time(H, Hkv, S, D, causal):
    """A workspace for the dS of some of the heads: bit for bit the result of the whole one.  (The
    recomputed form adds the same products in another order: one rounding step, or the fp32 rounding
    of the sums where the terms cancel.)"""
    print("case kept_ds parts", H, Hkv, S, D, causal, flush=True)
    g = torch.Generator(device="cuda")
    g.manual_seed(S)
    Q, dO = (torch.randn((2, H, S, D), generator=g, device="cuda").bfloat16() for _ in range(2))
    K, V = (torch.randn((2, Hkv, S, D), generator=g, device="cuda").bfloat16() for _ in range(2))
    O, LSE = attn.attn_fwd_rect(Q, K, V, D ** -0.5, causal)
    best = attn.attn_bwd_rect_best_workspace_bytes(2, H, Hkv, S, S, D, causal)
    assert [backward_form(2, H, Hkv, S, S, D, causal, n) for n in (best, int(best * 0.6))] == [STORED_DS] * 2
    ws = torch.full((best,), 0xFF, dtype=torch.uint8, device="cuda")
    whole, part, none = (attn.attn_bwd_rect(Q, K, V, O, dO, LSE, D ** -0.5, causal, workspace=ws[:n])
                         for n in (best, int(best * 0.6), 16 * H * S + 256))
    torch.cuda.synchronize()
    for w, p, n in zip(whole, part, none):
        assert torch.equal(w.view(torch.int16), p.view(torch.int16))
        w, n = w.double(), n.double()
        assert bool(((w - n).abs() <= n.abs() * 2.0 ** -7 + 1e-3 * n.abs().max()).all())
    assert not torch.equal(whole[0].view(torch.int16), none[0].view(torch.int16)), "dS is not kept"


@pytest.mark.parametrize("layout", ["BSHD", "padded"])
@pytest.mark.parametrize("B,Hq,Hkv,Sq,Sk,D,causal,f16,cut", [c for c in CASES if c[:3] in ((2, 48, 12), (1, 96, 24), (2, 33, 33))])
def test_stored_ds_in_other_layouts(B, Hq, Hkv, Sq, Sk, D, causal, f16, cut, layout):
    """[B,S,H,D] storage, and rows and heads with gaps: bit for bit the contiguous result."""
    print("case kept_ds layout", Hq, Hkv, Sq, Sk, D, layout, flush=True)
    g = torch.Generator(device="cuda")
    g.manual_seed(Sq)
    dt = torch.float16 if f16 else torch.bfloat16
    Q, dO = (torch.randn((B, Hq, Sq, D), generator=g, device="cuda").to(dt) for _ in range(2))
    K, V = (torch.randn((B, Hkv, Sk, D), generator=g, device="cuda").to(dt) for _ in range(2))
    O, LSE = attn.attn_fwd_rect(Q, K, V, D ** -0.5, causal)
    want = attn.attn_bwd_rect(Q, K, V, O, dO, LSE, D ** -0.5, causal)
    t = [in_layout(x, layout) for x in (Q, K, V, O, dO)]
    out = [in_layout(torch.full_like(x, float("nan")), layout) for x in (Q, K, V)]
    attn.attn_bwd_rect(*t, LSE, D ** -0.5, causal, dQ=out[0], dK=out[1], dV=out[2])
    torch.cuda.synchronize()
    assert all(torch.equal(a, b) for a, b in zip(out, want))


# two row blocks a wave: the last wave's second block past the end, blocks of unequal length under the mask,
# offsets off the 32-key blocks, grouped heads, more rows than keys
# (blocks: of 32 rows, per work-group of the launch of all heads; that of eight, one a wave, runs the other cases)
@pytest.mark.parametrize("H,Hkv,Sq,Sk,causal,blocks", [
    (520, 520, 385, 385, True, 8), (520, 260, 400, 1100, True, 8), (520, 520, 481, 513, True, 8), (264, 264, 1000, 1031, True, 8),
    (540, 540, 290, 417, False, 16), (518, 518, 512, 403, False, 16)])
def test_two_row_blocks_a_wave(H, Hkv, Sq, Sk, causal, blocks):
    """Work-groups of 512 rows, which a launch of all heads takes, against those of 256, which the parts
    take: a row's sum has the same products in the same order."""
    assert host_rule("dq_ds_blocks", H, Sq, 128, causal) == blocks
    assert host_rule("dq_ds_blocks", (Hkv + 1) // 2 * (H // Hkv), Sq, 128, causal) == 8
    print("case kept_ds two blocks", H, Hkv, Sq, Sk, causal, flush=True)
    g = torch.Generator(device="cuda")
    g.manual_seed(Sq + Sk)
    D = 128
    Q, dO = (torch.randn((1, H, Sq, D), generator=g, device="cuda").bfloat16() for _ in range(2))
    K, V = (torch.randn((1, Hkv, Sk, D), generator=g, device="cuda").bfloat16() for _ in range(2))
    O, LSE = attn.attn_fwd_rect(Q, K, V, D ** -0.5, causal)
    best = attn.attn_bwd_rect_best_workspace_bytes(1, H, Hkv, Sq, Sk, D, causal)
    assert [backward_form(1, H, Hkv, Sq, Sk, D, causal, n) for n in (best, int(best * 0.6))] == [STORED_DS] * 2
    ws = torch.full((best,), 0xFF, dtype=torch.uint8, device="cuda")
    whole, part = (attn.attn_bwd_rect(Q, K, V, O, dO, LSE, D ** -0.5, causal, workspace=ws[:n])
                   for n in (best, int(best * 0.6)))
    torch.cuda.synchronize()
    assert all(torch.equal(w.view(torch.int16), p.view(torch.int16)) for w, p in zip(whole, part))


# the same, and a last work-group of one row and of half its waves
@pytest.mark.parametrize("H,Hkv,Sq,Sk,causal", [(120, 120, 2049, 417, False), (120, 60, 2290, 517, False), (132, 132, 1825, 1825, True),
                                                (132, 66, 2017, 2400, True), (130, 130, 2033, 2065, True), (76, 76, 4130, 4161, True)])
@pytest.mark.parametrize("layout", ["BHSD", "BSHD", "padded"])
def test_two_row_blocks_a_wave_in_longer_calls(H, Hkv, Sq, Sk, causal, layout):
    """All heads at once, in work-groups of 512 rows, against one half and then the other, in those of 256."""
    print("case kept_ds two blocks", H, Hkv, Sq, Sk, causal, layout, flush=True)
    g = torch.Generator(device="cuda")
    g.manual_seed(Sq + Sk)
    D, G = 128, H // Hkv
    Q, dO = (torch.randn((2, H // 2, Sq, D), generator=g, device="cuda").bfloat16() for _ in range(2))
    K, V = (torch.randn((2, Hkv // 2, Sk, D), generator=g, device="cuda").bfloat16() for _ in range(2))
    O, LSE = attn.attn_fwd_rect(Q, K, V, D ** -0.5, causal)

    def backward(t, lse, want):
        B, Hq, Hk = t[0].shape[0], t[0].shape[1], t[1].shape[1]
        best = attn.attn_bwd_rect_best_workspace_bytes(B, Hq, Hk, Sq, Sk, D, causal)
        assert backward_form(B, Hq, Hk, Sq, Sk, D, causal, best) == STORED_DS
        assert host_rule("dq_ds_blocks", B * Hq, Sq, D, causal) == want
        out = [torch.full(x.shape, float("nan"), dtype=x.dtype, device="cuda") for x in t[:3]]
        out = [o if x.is_contiguous() else in_layout(o, layout) for o, x in zip(out, t)]
        attn.attn_bwd_rect(*t, lse, D ** -0.5, causal, dQ=out[0], dK=out[1], dV=out[2],
                           workspace=torch.full((best,), 0xFF, dtype=torch.uint8, device="cuda"))
        return out

    t = (Q, K, V, O, dO)
    whole = backward([x if layout == "BHSD" else in_layout(x, layout) for x in t], LSE, 16)
    for b in range(2):
        half = backward([x[b:b + 1].contiguous() for x in t], LSE[b:b + 1].contiguous(), 8)
        for w, p in zip(whole, half):
            assert torch.equal(w[b:b + 1].contiguous().view(torch.int16), p.view(torch.int16))
