"""Workspaces that a call takes for speed alone: only where there is memory to spare, without an allocation that
fails for it, and never under torch.use_deterministic_algorithms.  Without them the call is the one with the
plain workspace (backward) or in one kernel (square forward), bit for bit."""
import contextlib
import gc

import pytest
import torch

import paper_2601_16238_amd as attn

pytestmark = pytest.mark.gpu


def inputs(H, S, D):
    g = torch.Generator(device="cuda")
    g.manual_seed(S)
    return [torch.randn((1, H, S, D), generator=g, device="cuda").bfloat16() for _ in range(4)]


@contextlib.contextmanager
def at_most(more):
    """The process may get `more` bytes beyond what its tensors hold."""
    gc.collect()
    torch.cuda.synchronize()
    torch.cuda.empty_cache()
    # idle parts of segments in which a tensor still lies: taken, as they would serve the call
    taken, stream = [], torch.cuda.current_stream().cuda_stream
    for _ in range(8):
        idle = [b["size"] for s in torch.cuda.memory_snapshot() for b in s["blocks"]
                if b["state"] == "inactive" and b["size"] >= 1 << 20 and s["segment_type"] == "large" and s["stream"] == stream]
        taken += [torch.empty(n, dtype=torch.uint8, device="cuda") for n in idle]
    assert not idle
    total = torch.cuda.get_device_properties(0).total_memory
    torch.cuda.set_per_process_memory_fraction((torch.cuda.memory_reserved() + more) / total)
    try:
        yield
    finally:
        torch.cuda.set_per_process_memory_fraction(1.0)
        del taken


@contextlib.contextmanager
def deterministic():
    torch.use_deterministic_algorithms(True)
    try:
        yield
    finally:
        torch.use_deterministic_algorithms(False)


def failures():
    """Allocations that failed, and those that succeeded only after the allocator gave back what it held."""
    s = torch.cuda.memory_stats()
    return s["num_ooms"], s["num_alloc_retries"]


def equal(a, b):
    return all(torch.equal(x.view(torch.int16), y.view(torch.int16)) for x, y in zip(a, b))


# dS of 1 GiB, which is asked about; dS of 18 MB, which is not and fails by the allocation
@pytest.mark.parametrize("H,S,D,limit,fails", [(16, 8192, 128, 600 << 20, False), (36, 700, 128, 8 << 20, True)])
def test_backward_with_little_memory(H, S, D, limit, fails):
    print("case spare backward", H, S, D, flush=True)
    q, k, v, do = inputs(H, S, D)
    o, lse = attn.attn_fwd(q, k, v, D ** -0.5, True)
    size = attn.attn_bwd_workspace_bytes(1, H, S, D)
    assert attn.attn_bwd_rect_best_workspace_bytes(1, H, H, S, S, D, True) > size + limit
    plain = attn.attn_bwd(q, k, v, o, do, lse, D ** -0.5, True, workspace=torch.empty(size, dtype=torch.uint8, device="cuda"))
    free = attn.attn_bwd(q, k, v, o, do, lse, D ** -0.5, True)
    assert not equal(free, plain), "no workspace was taken for speed"
    del free
    out = [torch.empty_like(t) for t in plain]
    with at_most(limit):
        before = failures()
        for _ in range(2):
            attn.attn_bwd(q, k, v, o, do, lse, D ** -0.5, True, dQ=out[0], dK=out[1], dV=out[2])
        torch.cuda.synchronize()
        assert fails or failures() == before
    assert equal(out, plain)
    with deterministic():
        assert equal(attn.attn_bwd(q, k, v, o, do, lse, D ** -0.5, True), plain)
        leaves = [t.detach().clone().requires_grad_() for t in (q, k, v)]
        o2 = attn.fused_attention(*leaves, causal=True)
        assert equal([o2], [o]) and equal(torch.autograd.grad(o2, leaves, do), plain)


def test_square_forward_with_little_memory():
    H, S, D = 8, 8394, 128
    print("case spare forward", H, S, D, flush=True)
    q, k, v, _ = inputs(H, S, D)
    whole = attn.attn_fwd_rect(q, k, v, D ** -0.5, True, split=False)
    need = attn.attn_fwd_rect_workspace_bytes(1, H, H, S, S, D, True)
    assert need > 64 << 20
    assert not equal(attn.attn_fwd(q, k, v, D ** -0.5, True)[:1], whole[:1]), "not split"
    out = torch.empty_like(q), torch.empty_like(whole[1])
    with at_most(need - (16 << 20)):
        before = failures()
        attn.attn_fwd(q, k, v, D ** -0.5, True, O=out[0], LSE=out[1])
        torch.cuda.synchronize()
        assert failures() == before
    assert equal(out[:1], whole[:1]) and torch.equal(out[1], whole[1])
    with deterministic():
        got = attn.attn_fwd(q, k, v, D ** -0.5, True)
    assert equal(got[:1], whole[:1]) and torch.equal(got[1], whole[1])


def test_captured_backward_takes_the_same_form():
    """In a captured graph the call is the eager one, also above the size that is asked about."""
    H, S, D = 16, 4096, 128
    print("case spare capture", flush=True)
    q, k, v, do = inputs(H, S, D)
    o, lse = attn.attn_fwd(q, k, v, D ** -0.5, True)
    want = attn.attn_bwd(q, k, v, o, do, lse, D ** -0.5, True)
    torch.cuda.synchronize()
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph):
        got = attn.attn_bwd(q, k, v, o, do, lse, D ** -0.5, True)
    for _ in range(3):
        for t in got:
            t.zero_()
        graph.replay()
        torch.cuda.synchronize()
        assert equal(got, want)
