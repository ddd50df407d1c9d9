"""The backward in a scratch smaller than its plans ask for: the splits of dQ over the keys and of dK/dV over
the query slots are cut down to what fits (and no further), nothing is written past it, and the gradients are
the oracle's."""
import numpy as np
import pytest
import torch

import oracle
import paper_2601_16238_amd as attn
from paper_2601_16238_amd import binding, workloads as wl
from parity_util import check_grad, to_dev, to_f64

pytestmark = pytest.mark.gpu
STATIC = binding.NOALLOC_SCRATCH_BYTES


def same(a, b):
    return torch.equal(a.view(torch.int16), b.view(torch.int16))


# room: bytes behind the statistics (None: what the static scratch of the call without workspace leaves);
# split: which gradients differ from the unsplit kernels' (other order of the same fp32 sums)
@pytest.mark.parametrize("B,Hq,Hkv,Sq,Sk,D,causal,room,split", [
    (1, 1, 1, 1024, 4096, 128, True, None, (True, False, False)),     # dQ: fewer splits than the plan's
    (1, 1, 1, 1024, 4096, 128, True, 2 * 1024 * 512, (True, False, False)),     # exactly two splits
    (1, 1, 1, 1024, 4096, 128, True, 2 * 1024 * 512 - 256, (False, False, False)),
    (1, 4, 1, 2048, 2048, 64, True, None, (True, True, True)),        # dK/dV: longer chunks than the plan's
    (1, 2, 1, 1537, 3074, 96, False, None, (True, True, True)),
    (1, 1, 1, 1540, 4200, 256, True, 120 << 17, (False, True, True)),
    (1, 1, 1, 1540, 4200, 256, True, 110 << 17, (False, False, False)),         # fewer chunks than halving the long blocks takes
    (1, 1, 1, 1540, 4200, 256, True, 0, (False, False, False))])
def test_splits_are_cut_down_to_the_scratch(B, Hq, Hkv, Sq, Sk, D, causal, room, split):
    print("case bwd scratch", B, Hq, Hkv, Sq, Sk, D, causal, room, flush=True)
    x = wl.random_rect_inputs(B, Hq, Hkv, Sq, Sk, D, seed=4100 + D)
    Q, K, V, dO = (to_dev(x[k]) for k in ("Q", "K", "V", "dO"))
    O, LSE = attn.attn_fwd_rect(Q, K, V, x["scale"], causal)
    stats = (8 * B * Hq * Sq + 255) // 256 * 256
    size = STATIC if room is None else stats + room
    assert attn.attn_bwd_rect_workspace_bytes(B, Hq, Hkv, Sq, Sk, D) > size, "the plan fits whole"
    ws = torch.full((size + (1 << 20),), 0x7F, dtype=torch.uint8, device="cuda")   # poisoned
    got = attn.attn_bwd_rect(Q, K, V, O, dO, LSE, x["scale"], causal, workspace=ws[:size])
    torch.cuda.synchronize()
    assert bool((ws[size:] == 0x7F).all())
    one = attn.attn_bwd_rect(Q, K, V, O, dO, LSE, x["scale"], causal, workspace=ws[:stats])
    if room is None:
        outs = tuple(torch.empty_like(t) for t in got)
        binding.attn_bwd_rect_noalloc(Q, K, V, O, dO, LSE, x["scale"], causal, *outs)
        assert all(same(a, b) for a, b in zip(got, outs))
    assert tuple(not same(a, b) for a, b in zip(got, one)) == split
    ref = oracle.attn_bwd(x["Q"], x["K"], x["V"], x["dO"], x["scale"], causal)
    for name, g, r in zip(("dQ", "dK", "dV"), got, ref):
        assert np.isfinite(to_f64(g)).all(), name
        check_grad(name, to_f64(g), r)
