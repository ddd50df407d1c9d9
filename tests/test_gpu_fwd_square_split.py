"""Square forward calls on few heads, which are split over the keys, against the fp64 oracle and the forward in
one kernel."""
import pytest
import torch

import oracle
import paper_2601_16238_amd as attn
from paper_2601_16238_amd import workloads as wl
from parity_util import check_bf16, to_dev, to_f64

pytestmark = pytest.mark.gpu


# the shortest that is split, ragged ends, padded head dimensions, grouped heads, D = 256
@pytest.mark.parametrize("Hq,Hkv,S,D,causal", [(2, 2, 769, 128, True), (1, 1, 1281, 32, False), (3, 3, 1390, 80, True),
                                               (4, 2, 1030, 64, False), (2, 1, 1100, 256, True)])
def test_square_forward_is_split_over_the_keys(Hq, Hkv, S, D, causal):
    print("case square split", Hq, Hkv, S, D, causal, flush=True)
    assert attn.attn_fwd_rect_workspace_bytes(1, Hq, Hkv, S, S, D, causal) > 0, "the plan does not split"
    x = wl.random_rect_inputs(1, Hq, Hkv, S, S, D, seed=7000 + S)
    Q, K, V = (to_dev(x[k]) for k in ("Q", "K", "V"))
    call = attn.attn_fwd if Hq == Hkv else attn.attn_fwd_gqa
    O, LSE = call(Q, K, V, x["scale"], causal, O=torch.full_like(Q, float("nan")))
    O2, LSE2 = attn.attn_fwd_rect(Q, K, V, x["scale"], causal)
    O1, _ = attn.attn_fwd_rect(Q, K, V, x["scale"], causal, split=False)
    torch.cuda.synchronize()
    Oref, Lref = oracle.attn_fwd(x["Q"], x["K"], x["V"], x["scale"], causal)
    check_bf16("O", to_f64(O), Oref)
    assert abs(to_f64(LSE) - Lref).max() <= 1e-5
    assert torch.equal(O.view(torch.int16), O2.view(torch.int16)) and torch.equal(LSE, LSE2)
    assert not torch.equal(O.view(torch.int16), O1.view(torch.int16)), "not split"  # (other roundings of the same sums)
