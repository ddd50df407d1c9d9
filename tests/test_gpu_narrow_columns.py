"""Head dimensions for which the products skip the kernels' last columns: the result on the same data padded
with zero columns, which takes the instances that do not skip them.  bf16 bit for bit; in fp16 the compiler
may form delta's fp32 sum with or without packed dot products, so that single dS round the other way: at most
one step of the output, or of the largest product that is summed (2^-10 of it)."""
import pytest
import torch

import paper_2601_16238_amd as attn

pytestmark = pytest.mark.gpu

# head dimensions at the edges of the narrow instances (32 of 64, 96 of 128, 192 of 256 columns); forward
# with eight, four (both forms), two and one waves, split and not; backward in one launch (four waves, one
# wave per part, grouped, eight), dK/dV with four and six pairs, split and not, dQ from kept dS and, for few
# long heads and 32 columns, recomputed, split and not
CASES = [(1, 2, 2, 300, 300, 32, 64, True), (3, 100, 100, 40, 70, 24, 64, False), (2, 2, 1, 33, 90, 32, 64, True),
         (2, 128, 128, 97, 97, 32, 64, True), (64, 8, 4, 60, 90, 32, 64, True), (1, 3, 3, 250, 256, 32, 64, False),
         (4, 64, 64, 1100, 1100, 32, 64, True), (1, 30, 15, 520, 700, 8, 64, False), (1, 2, 1, 257, 4100, 32, 64, False),
         (1, 2, 2, 128, 128, 96, 128, True), (2, 4, 2, 129, 400, 72, 128, False), (1, 16, 4, 513, 513, 96, 128, True),
         (2, 130, 130, 385, 400, 88, 128, True), (1, 1, 1, 2050, 2050, 96, 128, True), (1, 1, 1, 300, 5000, 96, 128, False),
         (1, 3, 3, 257, 290, 192, 256, True), (2, 40, 40, 200, 333, 136, 256, False), (1, 2, 1, 600, 600, 192, 256, False)]


@pytest.mark.parametrize("B,Hq,Hkv,Sq,Sk,D,full,causal", CASES)
@pytest.mark.parametrize("dtype", [torch.bfloat16, torch.float16])
def test_skipped_columns_change_nothing(B, Hq, Hkv, Sq, Sk, D, full, causal, dtype):
    print("case narrow", B, Hq, Hkv, Sq, Sk, D, causal, dtype, flush=True)
    g = torch.Generator(device="cuda")
    g.manual_seed(Sq + Sk + D)
    t = [torch.randn(s, generator=g, device="cuda").to(dtype)
         for s in ((B, Hq, Sq, D), (B, Hkv, Sk, D), (B, Hkv, Sk, D), (B, Hq, Sq, D))]
    z = [torch.nn.functional.pad(x, (0, full - D)) for x in t]

    def run(Q, K, V, dO, plain):
        O, LSE = attn.attn_fwd_rect(Q, K, V, D ** -0.5, causal)
        ws = None
        if plain:  # the backward without kept dS
            ws = torch.empty(attn.attn_bwd_rect_workspace_bytes(B, Hq, Hkv, Sq, Sk, D), dtype=torch.uint8, device="cuda")
        return O, LSE, *attn.attn_bwd_rect(Q, K, V, O, dO, LSE, D ** -0.5, causal, workspace=ws)

    for plain in (False, True):
        a, b = run(*t, plain), run(*z, plain)
        torch.cuda.synchronize()
        for name, x, y in zip(("O", "LSE", "dQ", "dK", "dV"), a, b):
            assert torch.isfinite(x).all(), name
            assert x.dim() == 3 or not y[..., D:].any(), name
            y = y[..., :D] if x.dim() == 4 else y
            if dtype == torch.bfloat16 or name in ("O", "LSE"):
                assert torch.equal(x, y), name
            else:
                x, y = x.double(), y.double()
                assert bool(((x - y).abs() <= 2.0 ** -10 * (y.abs() + y.abs().max())).all()), name


@pytest.mark.parametrize("H,Sq,Sk,D,causal", [(8, 373, 5508, 32, True), (8, 1100, 1100, 24, True), (4, 60, 4000, 32, False),
                                              (2, 257, 4100, 32, False), (16, 172, 1599, 96, False), (8, 700, 2100, 80, True)])
def test_partial_results_of_a_split_have_no_columns_that_are_skipped(H, Sq, Sk, D, causal):
    """(They would be written, and up to twice the bytes with them, only to be dropped by the merge.)"""
    print("case narrow partials", H, Sq, Sk, D, causal, flush=True)
    g = torch.Generator(device="cuda")
    g.manual_seed(Sq + Sk)
    Q = torch.randn((1, H, Sq, D), generator=g, device="cuda").bfloat16()
    K, V = (torch.randn((1, H, Sk, D), generator=g, device="cuda").bfloat16() for _ in range(2))
    wide, used = (64, 32) if D <= 64 else (128, 96)
    n = attn.attn_fwd_rect_workspace_bytes(1, H, H, Sq, Sk, D, causal)
    ws = torch.full((n,), 0xFF, dtype=torch.uint8, device="cuda")
    O, LSE = attn.attn_fwd_rect(Q, K, V, D ** -0.5, causal, workspace=ws)
    part = ws.view(torch.int32)[:H * Sq * wide].view(-1, wide)  # of the first split, which every row sees
    torch.cuda.synchronize()
    assert bool((part[:, :D] != -1).all()) and bool((part[:, used:] == -1).all())
    # ... and what lies there (here NaN) does not matter
    again = attn.attn_fwd_rect(Q, K, V, D ** -0.5, causal, workspace=ws.zero_())
    torch.cuda.synchronize()
    assert torch.equal(O, again[0]) and torch.equal(LSE, again[1])
