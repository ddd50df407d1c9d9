"""The dK/dV kernel's split over the query slots (few key/value heads whose key blocks would leave
most of the chip idle) against the fp64 oracle and against the unsplit kernel."""
import numpy as np
import pytest
import torch

import oracle
import paper_2601_16238_amd as attn
from paper_2601_16238_amd import workloads as wl
from parity_util import check_grad, f16_round, bf16_round, to_dev, to_f64

pytestmark = pytest.mark.gpu

# grouped heads, ragged blocks, padded head dimension, fp16; every query head of a group in chunks
# that start and end inside a head; more than 64 key blocks (the chunk search goes on past one wave of
# them), some of which few or no rows see; blocks of one chunk next to blocks of several; 64-key blocks
CASES = [(1, 4, 1, 1537, 1537, 96, True, True), (1, 8, 1, 200, 900, 64, False, False),
         (2, 6, 2, 530, 533, 128, False, False), (1, 1, 1, 1600, 8300, 64, True, False),
         (1, 2, 1, 800, 830, 256, True, False), (1, 1, 1, 1540, 4200, 256, True, True),
         (1, 3, 1, 4100, 300, 72, False, False)]


@pytest.mark.parametrize("B,Hq,Hkv,Sq,Sk,D,causal,f16", CASES)
def test_dkdv_split_over_the_query_slots(B, Hq, Hkv, Sq, Sk, D, causal, f16):
    print("case dkdv_split", B, Hq, Hkv, Sq, Sk, D, causal, f16, flush=True)
    draw = wl.random_rect_inputs_f16 if f16 else wl.random_rect_inputs
    x = draw(B, Hq, Hkv, Sq, Sk, D, seed=3100 + Sq + D)
    rnd = f16_round if f16 else bf16_round
    ref = oracle.attn_bwd(x["Q"], x["K"], x["V"], x["dO"], x["scale"], causal, dtype="f16" if f16 else "bf16")
    dt = torch.float16 if f16 else torch.bfloat16
    Q, K, V, dO = (torch.from_numpy(x[k].view(np.int16)).cuda().view(dt) for k in ("Q", "K", "V", "dO"))
    O, LSE = attn.attn_fwd_rect(Q, K, V, x["scale"], causal)
    full, stats = attn.attn_bwd_rect_workspace_bytes(B, Hq, Hkv, Sq, Sk, D), (8 * B * Hq * Sq + 255) // 256 * 256
    assert full > stats, "plan does not split"
    ws = torch.full((full,), 0x7F, dtype=torch.uint8, device="cuda")   # poisoned: nothing may be relied on
    got = attn.attn_bwd_rect(Q, K, V, O, dO, LSE, x["scale"], causal, workspace=ws)
    again = attn.attn_bwd_rect(Q, K, V, O, dO, LSE, x["scale"], causal, workspace=ws)
    one = attn.attn_bwd_rect(Q, K, V, O, dO, LSE, x["scale"], causal, workspace=ws[:stats])
    torch.cuda.synchronize()
    # (the split itself: its other order of the same sums shows in some roundings)
    for g, u in zip(got[1:], one[1:]):
        assert not torch.equal(g.view(torch.int16), u.view(torch.int16)), "dK/dV not split"
    for name, g, a, u, r in zip(("dQ", "dK", "dV"), got, again, one, ref):
        check_grad(name, to_f64(g), r, rnd=rnd)
        check_grad("unsplit " + name, to_f64(u), r, rnd=rnd)
        assert torch.equal(g.view(torch.int16), a.view(torch.int16)), name
        # the same products in fp32, added in another order: one rounding step of the output, or,
        # where the terms cancel, the fp32 rounding of the partial sums
        a, b = to_f64(g), to_f64(u)
        assert (np.abs(a - b) <= np.abs(b) * 2.0 ** -7 + 1e-4 * np.abs(b).max()).all(), name
