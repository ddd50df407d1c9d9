"""The forward at D = 128 with 129 .. 224 rows a head, in one eight-wave work-group a head, against the fp64
oracle: first and last of its row blocks, ragged keys, padded columns, split and whole, both masks."""
import pytest
import torch

import oracle
import paper_2601_16238_amd as attn
from paper_2601_16238_amd import workloads as wl
from parity_util import check_bf16, in_layout, to_dev, to_f64

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("Hq,Hkv,Sq,Sk,D,causal", [(132, 132, 129, 129, 128, True), (130, 65, 224, 225, 96, False),
                                                   (136, 17, 161, 700, 128, True), (48, 12, 193, 2800, 128, True),
                                                   (44, 44, 150, 3001, 80, False)])
def test_five_to_seven_row_blocks(Hq, Hkv, Sq, Sk, D, causal):
    print("case five blocks", Hq, Hkv, Sq, Sk, D, causal, flush=True)
    x = wl.random_rect_inputs(1, Hq, Hkv, Sq, Sk, D, seed=7100 + Sq)
    Q, K, V = (to_dev(x[k]) for k in ("Q", "K", "V"))
    Oref, Lref = oracle.attn_fwd(x["Q"], x["K"], x["V"], x["scale"], causal)
    for split in (True, False):
        O, LSE = attn.attn_fwd_rect(Q, K, V, x["scale"], causal, O=torch.full_like(Q, float("nan")), split=split)
        torch.cuda.synchronize()
        check_bf16("O split=%s" % split, to_f64(O), Oref)
        assert abs(to_f64(LSE) - Lref).max() <= 1e-5


def test_the_workspace_of_four_wave_work_groups_is_accepted():
    """Three splits' partial results, which two work-groups of four waves a head take where one of eight takes seven."""
    H, Sq, Sk, D = 34, 184, 4957, 128
    print("case five blocks, smaller workspace", flush=True)
    part = H * Sq * (D + 1) * 4
    need = (3 * part + 255) // 256 * 256
    assert attn.attn_fwd_rect_workspace_bytes(1, H, H, Sq, Sk, D, True) > need
    g = torch.Generator(device="cuda")
    g.manual_seed(3)
    Q = torch.randn((1, H, Sq, D), generator=g, device="cuda").bfloat16()
    K, V = (torch.randn((1, H, Sk, D), generator=g, device="cuda").bfloat16() for _ in range(2))
    ws = torch.empty(need, dtype=torch.uint8, device="cuda")
    O, LSE = attn.attn_fwd_rect(Q, K, V, D ** -0.5, True, workspace=ws)
    O1, LSE1 = attn.attn_fwd_rect(Q, K, V, D ** -0.5, True, split=False)
    torch.cuda.synchronize()
    assert (LSE - LSE1).abs().max() <= 2e-5   # (each within 1e-5 of the exact one)
    # two roundings of one result, each within the rounding of P of the exact one
    assert (O.double() - O1.double()).norm() <= 5e-3 * O1.double().norm()


@pytest.mark.parametrize("layout", ["BSHD", "padded"])
@pytest.mark.parametrize("Hq,Hkv,Sq,Sk,D,causal", [(130, 65, 224, 225, 96, False), (48, 12, 193, 2800, 128, True)])
def test_five_to_seven_row_blocks_in_other_layouts(Hq, Hkv, Sq, Sk, D, causal, layout):
    """[B,S,H,D] storage, and rows and heads with gaps: bit for bit the contiguous result."""
    print("case five blocks layout", Hq, Hkv, Sq, Sk, D, layout, flush=True)
    g = torch.Generator(device="cuda")
    g.manual_seed(Sq)
    Q = torch.randn((1, Hq, Sq, D), generator=g, device="cuda").bfloat16()
    K, V = (torch.randn((1, Hkv, Sk, D), generator=g, device="cuda").bfloat16() for _ in range(2))
    O, LSE = attn.attn_fwd_rect(Q, K, V, D ** -0.5, causal)
    out = in_layout(torch.full_like(Q, float("nan")), layout)
    _, LSE2 = attn.attn_fwd_rect(*(in_layout(t, layout) for t in (Q, K, V)), D ** -0.5, causal, O=out)
    torch.cuda.synchronize()
    assert torch.equal(out, O) and torch.equal(LSE2, LSE)
