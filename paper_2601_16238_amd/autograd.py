"""torch.autograd wrapper around the fused attention entry points, so that the operator can
stand where a framework's scaled-dot-product attention stands in a training step (the paper
trains its ViT and miniGPT examples through its fused attention this way).

Marshalling only, in native code (csrc/marshal.cpp): the forward calls attn_fwd_rect and keeps
(Q, K, V, O, LSE) for the backward, which calls attn_bwd_rect.  No arithmetic happens here, and
there is no fallback: tensors the kernels cannot take (wrong device or type) raise.
"""
import torch

from . import binding


class _RecordedAttention(torch.autograd.Function):
    """The same two calls as a Python function, which a tracer records as one operation and calls again: of
    the native node it would record only the allocations, and replay those without the kernels."""

    @staticmethod
    def forward(ctx, q, k, v, scale, causal):
        q, k, v, O, LSE = binding.marshal().fused_forward(q, k, v, scale, causal)
        ctx.save_for_backward(q, k, v, O, LSE)
        ctx.scale, ctx.causal = scale, causal
        return O

    @staticmethod
    def backward(ctx, dO):
        return (*binding.marshal().fused_backward(*ctx.saved_tensors, dO, ctx.scale, ctx.causal), None, None)


def fused_attention(q, k, v, causal=False, scale=None):
    """softmax(scale * q k^T [+ causal mask]) v with gradients.  q: [B, Hq, Sq, D]; k, v:
    [B, Hkv, Sk, D] with Hkv dividing Hq; bf16 or fp16 tensors on the GPU; D a multiple of 8 up
    to 256.  scale defaults to D ** -0.5.  With causal=True query row i sees keys
    0 .. i + Sk - Sq (needs Sk >= Sq).  The backward's workspace is that of attn_bwd without one."""
    if torch._C._are_functorch_transforms_active():
        raise RuntimeError("fused_attention has no rule for function transforms (vmap, grad, jvp, ...)")
    if scale is None:
        scale = float(q.shape[-1]) ** -0.5
    out = binding.marshal().fused_attention(q, k, v, float(scale), bool(causal))
    return _RecordedAttention.apply(q, k, v, float(scale), bool(causal)) if out is None else out
