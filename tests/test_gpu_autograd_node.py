"""What a program may do with the autograd node besides one backward: a second one, an in-place change of what
it kept, no gradients asked for, a backward that raises, several threads and a stream of its own, forward mode."""
import threading

import pytest
import torch

import paper_2601_16238_amd as attn

pytestmark = pytest.mark.gpu


def inputs(grad=True):
    g = torch.Generator(device="cuda")
    g.manual_seed(5)
    return [torch.randn((2, 2, 90, 64), device="cuda", generator=g).to(torch.bfloat16).requires_grad_(grad) for _ in range(3)]


def test_graph_rules():
    print("case autograd node", flush=True)
    q, k, v = inputs()
    o = attn.fused_attention(q, k, v, causal=True)
    first = torch.autograd.grad(o, (q, k, v), o.detach(), retain_graph=True)
    again = torch.autograd.grad(o, (q, v), o.detach())
    assert torch.equal(first[0], again[0]) and torch.equal(first[2], again[1])
    with pytest.raises(RuntimeError, match="second time"):
        torch.autograd.grad(o, (q,), o.detach())
    o = attn.fused_attention(q, k, v)
    with torch.no_grad():
        k.mul_(2)
    with pytest.raises(RuntimeError, match="inplace"):
        o.sum().backward()
    with torch.no_grad():
        assert not attn.fused_attention(q, k, v).requires_grad
    assert not attn.fused_attention(*inputs(False)).requires_grad
    with pytest.raises(NotImplementedError):  # forward mode
        with torch.autograd.forward_ad.dual_level():
            attn.fused_attention(torch.autograd.forward_ad.make_dual(q.detach(), q.detach()), k, v)
    with pytest.raises(RuntimeError):
        torch.func.grad(lambda a: attn.fused_attention(a, k, v).sum())(q)


def test_errors_keep_their_type():
    q, k, v = inputs()
    with pytest.raises(attn.AttnError):   # causal with fewer keys than rows
        attn.fused_attention(q, k[:, :, :8], v[:, :, :8], causal=True)
    o = attn.fused_attention(q, k, v)

    def fail(t):
        raise KeyError("unpack")
    with torch.autograd.graph.saved_tensors_hooks(lambda t: t, fail):
        bad = attn.fused_attention(q, k, v)
    with pytest.raises(KeyError):
        bad.sum().backward()
    # tensors that the kernels cannot take: the exception of a direct call with them
    for changed in (lambda t: t.float(), lambda t: t.cpu()):
        with torch.autograd.graph.saved_tensors_hooks(lambda t: t, changed):
            bad = attn.fused_attention(q, k, v)
        with pytest.raises(ValueError, match="on the GPU"):
            bad.sum().backward()
    o.sum().backward()
    torch.cuda.synchronize()
    assert q.grad is not None


@pytest.mark.parametrize("grad", [True, False])
def test_a_traced_call_runs_the_kernels_on_other_inputs(grad):
    print("case traced", grad, flush=True)
    example = [(t * 0.5).detach().requires_grad_(grad) for t in inputs(False)]
    f = torch.jit.trace(lambda q, k, v: attn.fused_attention(q, k, v, causal=True), example, check_trace=False)
    x = inputs(grad)
    want = attn.fused_attention(*x, causal=True)
    for _ in range(2):
        got = f(*x)
        assert torch.equal(got, want) and got.requires_grad == grad
        if grad:
            pairs = zip(torch.autograd.grad(got, x, want.detach()),
                        torch.autograd.grad(want, x, want.detach(), retain_graph=True))
            assert all(torch.equal(a, b) for a, b in pairs)


def test_threads_and_streams():
    q, k, v = inputs(False)
    want = None
    got, errors = {}, []

    def step(i, stream):
        try:
            with torch.cuda.stream(stream):
                for _ in range(5):
                    leaves = [t.clone().requires_grad_() for t in (q, k, v)]
                    o = attn.fused_attention(*leaves, causal=True)
                    got[i] = torch.autograd.grad(o, leaves, v)
            stream.synchronize()
        except BaseException as e:  # noqa: B902 (reported by the test)
            errors.append(e)
    leaves = [t.clone().requires_grad_() for t in (q, k, v)]
    want = torch.autograd.grad(attn.fused_attention(*leaves, causal=True), leaves, v)
    torch.cuda.synchronize()
    threads = [threading.Thread(target=step, args=(i, torch.cuda.Stream())) for i in range(4)]
    for t in threads:
        t.start()
    for t in threads:
        t.join()
    assert not errors and len(got) == 4
    for g in got.values():
        assert all(torch.equal(a, b) for a, b in zip(g, want))
