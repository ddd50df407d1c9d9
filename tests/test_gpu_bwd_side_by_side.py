"""dK/dV and dQ in one launch (calls of few work-groups, with a workspace of the best size) against the fp64
oracle and against the kernels one after the other (a workspace of the plain size)."""
import numpy as np
import pytest
import torch

import oracle
import paper_2601_16238_amd as attn
from paper_2601_16238_amd import workloads as wl
from parity_util import (APART, DKDV_CUT, DQ_CUT, SIDE_BY_SIDE, backward_form, bf16_round, check_grad, f16_round, in_layout,
                         to_f64)

pytestmark = pytest.mark.gpu

# (last: dK/dV and dQ cut)  one row over a tile, one block, head counts that eight does not divide; few rows on many
# keys and many on few; grouped heads; padded head dimensions; both element types; D = 256 cut and whole
CASES = [(1, 3, 3, 257, 257, 64, True, False, 0, 0), (1, 1, 1, 1185, 1185, 96, False, False, 1, 1),
         (1, 1, 1, 92, 2100, 128, True, False, 1, 1), (1, 5, 5, 1601, 70, 64, False, False, 1, 0),
         (1, 8, 2, 513, 609, 72, True, True, 1, 1), (1, 4, 1, 321, 321, 128, True, False, 1, 0),
         (3, 1, 1, 65, 129, 256, False, False, 0, 0), (1, 2, 1, 900, 930, 200, True, True, 1, 0),
         (1, 6, 6, 1037, 1037, 32, True, False, 1, 1), (1, 1, 1, 2100, 2133, 128, True, False, 1, 1),
         (1, 1, 1, 1, 300, 64, True, False, 0, 0), (1, 60, 60, 257, 97, 40, False, False, 0, 0),
         (1, 2, 2, 257, 257, 128, True, True, 0, 0), (2, 3, 3, 513, 513, 256, True, False, 0, 0)]


@pytest.mark.parametrize("B,Hq,Hkv,Sq,Sk,D,causal,f16,dkdv_cut,dq_cut", CASES)
def test_dkdv_and_dq_in_one_launch(B, Hq, Hkv, Sq, Sk, D, causal, f16, dkdv_cut, dq_cut):
    print("case side by side", B, Hq, Hkv, Sq, Sk, D, causal, f16, flush=True)
    draw = wl.random_rect_inputs_f16 if f16 else wl.random_rect_inputs
    x = draw(B, Hq, Hkv, Sq, Sk, D, seed=6100 + Sq + D)
    rnd = f16_round if f16 else bf16_round
    ref = oracle.attn_bwd(x["Q"], x["K"], x["V"], x["dO"], x["scale"], causal, dtype="f16" if f16 else "bf16")
    dt = torch.float16 if f16 else torch.bfloat16
    Q, K, V, dO = (torch.from_numpy(x[k].view(np.int16)).cuda().view(dt) for k in ("Q", "K", "V", "dO"))
    O, LSE = attn.attn_fwd_rect(Q, K, V, x["scale"], causal)
    best, plain = (f(B, Hq, Hkv, Sq, Sk, D, *c) for f, c in ((attn.attn_bwd_rect_best_workspace_bytes, (causal,)),
                                                             (attn.attn_bwd_rect_workspace_bytes, ())))
    assert backward_form(B, Hq, Hkv, Sq, Sk, D, causal, best) == SIDE_BY_SIDE + DKDV_CUT * dkdv_cut + DQ_CUT * dq_cut
    assert backward_form(B, Hq, Hkv, Sq, Sk, D, causal, plain) % 16 == APART
    ws = torch.full((best + 4096,), 0xFF, dtype=torch.uint8, device="cuda")   # NaN: nothing may be relied on
    got, again = (attn.attn_bwd_rect(Q, K, V, O, dO, LSE, x["scale"], causal, workspace=ws[:best],
                                     **{k: torch.full_like(t, float("nan")) for k, t in (("dQ", Q), ("dK", K), ("dV", V))})
                  for _ in range(2))
    one = attn.attn_bwd_rect(Q, K, V, O, dO, LSE, x["scale"], causal, workspace=ws[:plain])
    torch.cuda.synchronize()
    assert bool((ws[best:] == 0xFF).all()), "written past the workspace"
    for name, g, a, u, r in zip(("dQ", "dK", "dV"), got, again, one, ref):
        check_grad(name, to_f64(g), r, rnd=rnd)
        assert torch.equal(g.view(torch.int16), a.view(torch.int16)), name
        # the same products in fp32, added in another order: one rounding step of the output, or, where the
        # terms cancel, the fp32 rounding of the partial sums
        g, u = to_f64(g), to_f64(u)
        assert (np.abs(g - u) <= np.abs(u) * 2.0 ** -7 + 1e-3 * np.abs(u).max()).all(), name


def test_few_work_groups_take_one_launch():
    """At D = 64, where dS is not kept, room beyond the plain workspace is for that form alone."""
    for H, S, causal, few in ((6, 1037, True, True), (1, 257, False, True), (64, 1024, True, False), (4, 200, True, False)):
        best = attn.attn_bwd_rect_best_workspace_bytes(1, H, H, S, S, 64, causal)
        assert (best > attn.attn_bwd_rect_workspace_bytes(1, H, H, S, S, 64)) == few, (H, S)
        assert (backward_form(1, H, H, S, S, 64, causal, best) % 16 == SIDE_BY_SIDE) == few, (H, S)


@pytest.mark.parametrize("layout", ["BSHD", "padded"])
@pytest.mark.parametrize("B,Hq,Hkv,Sq,Sk,D,causal", [(1, 8, 2, 513, 609, 72, True), (1, 4, 1, 321, 321, 128, True),
                                                     (2, 3, 3, 513, 513, 256, True), (1, 6, 6, 1037, 1037, 64, False)])
def test_side_by_side_in_other_layouts(B, Hq, Hkv, Sq, Sk, D, causal, layout):
    """[B,S,H,D] storage, and rows and heads with gaps: bit for bit the contiguous result."""
    print("case side by side layout", Hq, Hkv, Sq, Sk, D, layout, flush=True)
    assert backward_form(B, Hq, Hkv, Sq, Sk, D, causal, 1 << 32) % 16 == SIDE_BY_SIDE
    g = torch.Generator(device="cuda")
    g.manual_seed(Sq)
    Q, dO = (torch.randn((B, Hq, Sq, D), generator=g, device="cuda").bfloat16() for _ in range(2))
    K, V = (torch.randn((B, Hkv, Sk, D), generator=g, device="cuda").bfloat16() for _ in range(2))
    O, LSE = attn.attn_fwd_rect(Q, K, V, D ** -0.5, causal)
    want = attn.attn_bwd_rect(Q, K, V, O, dO, LSE, D ** -0.5, causal)
    t = [in_layout(x, layout) for x in (Q, K, V, O, dO)]
    out = [in_layout(torch.full_like(x, float("nan")), layout) for x in (Q, K, V)]
    attn.attn_bwd_rect(*t, LSE, D ** -0.5, causal, dQ=out[0], dK=out[1], dV=out[2])
    torch.cuda.synchronize()
    assert all(torch.equal(a, b) for a, b in zip(out, want))
