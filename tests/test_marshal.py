"""The native marshalling module: what it refuses, and how torch's own machinery sees the calls."""
import pytest
import torch

import paper_2601_16238_amd as attn
from paper_2601_16238_amd import rowops


def half(*shape):
    return torch.zeros(shape, dtype=torch.bfloat16)


@pytest.mark.parametrize("call,error", [
    (lambda: attn.attn_fwd(half(1, 1, 8, 64), half(1, 1, 8, 64), half(1, 1, 8, 64), 0.1, False), ValueError),   # CPU
    (lambda: attn.attn_fwd(half(1, 1, 8, 64), half(1, 1, 9, 64), half(1, 1, 8, 64), 0.1, False), ValueError),   # shapes
    (lambda: attn.attn_fwd_rect(half(8, 64), half(8, 64), half(8, 64), 0.1, False), ValueError),                # 2-d
    (lambda: attn.attn_fwd_rect(half(1, 1, 8, 64), half(1, 1, 8, 32), half(1, 1, 8, 32), 0.1, False), ValueError),
    (lambda: attn.attn_fwd_gqa(half(1, 2, 8, 64), half(1, 1, 9, 64), half(1, 1, 9, 64), 0.1, False), ValueError),
    (lambda: attn.fused_attention(half(8, 64), half(8, 64), half(8, 64)), IndexError),
    (lambda: rowops.rmsnorm_fwd(half(4, 64), torch.zeros(64), 1e-6), ValueError),
    (lambda: rowops.rotary_fwd(half(1, 1, 8, 64), torch.zeros(8, 32), torch.zeros(8, 32)), ValueError),
])
def test_refused_on_the_host(call, error):
    with pytest.raises(error):
        call()


@pytest.mark.gpu
def test_streams_hooks_and_transforms():
    """A call on another stream, saved-tensor hooks around the autograd function, and a transform it
    has no rule for."""
    print("case marshal", flush=True)
    g = torch.Generator(device="cuda"); g.manual_seed(11)
    q, k, v = (torch.randn((2, 3, 70, 64), device="cuda", generator=g).to(torch.bfloat16) for _ in range(3))
    O, LSE = attn.attn_fwd(q, k, v, 0.125, True)
    side = torch.cuda.Stream()
    side.wait_stream(torch.cuda.current_stream())
    O2, LSE2 = attn.attn_fwd(q, k, v, 0.125, True, stream=side)
    side.synchronize()
    assert torch.equal(O, O2) and torch.equal(LSE, LSE2)
    with pytest.raises(attn.AttnError):   # causal with fewer keys than rows
        attn.attn_fwd_rect(q, k[:, :, :8], v[:, :, :8], 0.125, True)
    with pytest.raises(ValueError):
        attn.attn_fwd(q, k, v, 0.125, True, LSE=LSE.double())

    leaves = [t.clone().requires_grad_() for t in (q, k, v)]
    packed = []
    with torch.autograd.graph.saved_tensors_hooks(lambda t: packed.append(t) or t.clone(), lambda t: t):
        out = attn.fused_attention(*leaves, causal=True)
    assert len(packed) == 5 and torch.equal(out, O)
    out.backward(v)
    ref = attn.attn_bwd(q, k, v, O, v, LSE, 0.125, True)
    torch.cuda.synchronize()
    for t, r in zip(leaves, ref):
        assert torch.equal(t.grad, r)
    with pytest.raises(RuntimeError):
        torch.func.vmap(lambda a: attn.fused_attention(a, a, a))(q[None])
