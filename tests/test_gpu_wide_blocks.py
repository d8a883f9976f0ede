"""The backward products of layers with Hadamard blocks of 256 columns where the GEMM applies the epilogue itself (two waves share a
block): one to several tiles per compute unit, one to five K-quads, both tile shapes, both result types, against the oracle."""
import numpy as np
import pytest
import torch

import indep
import oracle
from paper_2505_14669_amd import synth

pytestmark = pytest.mark.gpu


@pytest.fixture()
def G():
    import gpu_util
    yield gpu_util
    gpu_util.q.quartet_debug_set_gemm_plan(-1, 0)


# dW: [out x in], inner dimension tokens; dx: [tokens x in], inner dimension out.  256 x 256 tiles: 1 + 1, 15 + 6, 5 + 325 (two rounds)
@pytest.mark.parametrize("variant", [0, 1])
@pytest.mark.parametrize("t,i,o", [(256, 256, 256), (512, 768, 1280), (16640, 1280, 256)])
def test_linear_bwd_with_blocks_of_256(G, variant, t, i, o):
    block, seed = 256, 77
    x, w, dy = synth.small_matrix(1, t, i, "outliers"), synth.small_matrix(2, o, i, "normal", 0.02), synth.small_matrix(3, t, o, "normal", 1e-3)
    lin = G.LinearBlock(x, w, block)
    lin.fwd()
    ctx = lin.ctx_host()
    assert G.q.quartet_debug_set_gemm_plan(variant, 0) == 0
    dyd = G.to_dev(dy)
    lin.dx.fill_(float("nan"))
    lin.dw.fill_(float("nan"))
    lin.bwd(dyd, seed, 0)
    dx, dw = G.to_host(lin.dx, np.float32), G.to_host(lin.dw, np.float32)
    sws = oracle.sign_words(seed)
    gq = oracle.quant_bwd_sr_block(dy, block, sws, seed, 0, 0)
    wt = oracle.requant_transpose_sr_block(ctx["wq_codes"], ctx["wq_scales"], block, sws, seed, 1, 0)
    gt = oracle.quant_bwd_sr_block(dy, block, sws, seed, 2, 0, transpose=True)
    xt = oracle.requant_transpose_sr_block(ctx["xq_codes"], ctx["xq_scales"], block, sws, seed, 3, 0)
    for got, a, b, mask, k in ((dx, gq, wt, ctx["x_mask"], o), (dw, gt, xt, ctx["w_mask"], t)):
        want = oracle.grad_epilogue_block(oracle.mxfp4_gemm(*a, *b).astype(np.float32), mask, block)
        absp = indep.gemm_abs_products(*a, *b)
        assert indep.worst_excess(got, want, indep.grad_elem_bound(indep.gemm_elem_bound(absp, k), absp, oracle.FL_16_9, block)) <= 1.0
    # bf16 results are the rounded ones of the same kernel
    dx16, dw16 = torch.empty((t, i), dtype=torch.bfloat16, device="cuda"), torch.empty((o, i), dtype=torch.bfloat16, device="cuda")
    G.q.check(G.q.quartet_linear_bwd_block(dyd, t, i, o, block, lin.xq_codes, lin.xq_scales, lin.x_mask, lin.wq_codes, lin.wq_scales,
                                           lin.w_mask, seed, 0, dx16, dw16, G.q.QUARTET_DTYPE_BF16, lin.ws, lin.ws_bytes))
    for got, want in ((dx16, dx), (dw16, dw)):
        assert np.array_equal(got.view(torch.uint16).cpu().numpy().ravel(), synth.f32_to_bf16(want).ravel())


# no tokens: dW = 0; no output features: dx = 0.  The profile names the launches that there were and no other.
@pytest.mark.parametrize("t,o", [(0, 512), (512, 0)])
@pytest.mark.parametrize("dtype", [torch.float32, torch.bfloat16])
def test_empty_products_with_blocks_of_256(G, t, o, dtype):
    import ctypes
    i, u8 = 256, lambda n: torch.zeros(max(n, 256), dtype=torch.uint8, device="cuda")
    dx, dw = torch.full((t, i), float("nan"), dtype=dtype, device="cuda"), torch.full((o, i), float("nan"), dtype=dtype, device="cuda")
    ctx = [a for r in (t, o) for a in (u8(r * i // 2), u8(G.q.quartet_scale_bytes(r, i)), u8(r * i // 8))]
    out = [a if a.numel() else u8(0) for a in (dx, dw)]
    ws_bytes = G.q.quartet_linear_workspace_bytes_block(t, i, o, 256)
    G.q.check(G.q.quartet_profile_enable(16))
    try:
        G.q.check(G.q.quartet_linear_bwd_block(u8(0), t, i, o, 256, *ctx, 5, 0, *out, int(dtype == torch.bfloat16), u8(ws_bytes), ws_bytes))
        kinds, ms = (ctypes.c_int * 16)(), (ctypes.c_float * 16)()
        n = G.q.quartet_profile_read(kinds, ms, 16)
    finally:
        G.q.quartet_profile_enable(0)
    assert list(kinds)[1:n] == [3, 4, 3, 4]          # behind the operands: product, epilogue, product, epilogue
    assert not dx.any() and not dw.any()


# Blocks that take extra tiles of the second product for part of its rounds (1 of 2 and 8 of 9 with 256 x 256 tiles, 2 of 5 and 16 of 17 with
# 128 x 256), the second layer with results of more than 256 MB in both types, which go past the memory-side cache.  Against plain products on
# tiles of the same shape and the epilogue kernel: the same sums and butterflies in the same order, so the same bits.
@pytest.mark.parametrize("variant", [0, 1])
@pytest.mark.parametrize("t,i,o", [(4096, 4864, 768), (131072, 1024, 256)])
def test_wide_pair_equals_products_and_epilogues(G, variant, t, i, o):
    q, block, seed = G.q, 256, 91
    gen = torch.Generator(device="cuda").manual_seed(t + variant)
    rand = lambda *s: torch.randn(s, generator=gen, device="cuda").to(torch.bfloat16)
    quantized = lambda rows, k: (torch.empty((rows, k // 2), dtype=torch.uint8, device="cuda"), torch.empty(q.quartet_scale_bytes(rows, k), dtype=torch.uint8, device="cuda"))
    x, w, dy = rand(t, i), rand(o, i), rand(t, o)
    xq, wq = quantized(t, i), quantized(o, i)
    xm, wm = (torch.empty((r, i // 32), dtype=torch.int32, device="cuda") for r in (t, o))
    q.check(q.quartet_linear_fwd_block(x, w, t, i, o, block, torch.empty((t, o), device="cuda"), 0, *xq, xm, *wq, wm))
    n = q.quartet_linear_workspace_bytes_block(t, i, o, block)
    ws = torch.empty(n, dtype=torch.uint8, device="cuda")
    sw = q.quartet_sign_words(seed)
    g, gt, wt, xt = quantized(t, o), quantized(o, t), quantized(i, o), quantized(i, t)
    q.check(q.quartet_quant_bwd_sr_block(dy, t, o, o, 0, block, sw, seed, 0, 0, *g))
    q.check(q.quartet_requant_transpose_sr_block(*wq, i, o, block, sw, seed, 1, 0, *wt))
    q.check(q.quartet_quant_bwd_sr_block(dy, o, t, o, 1, block, sw, seed, 2, 0, *gt))
    q.check(q.quartet_requant_transpose_sr_block(*xq, i, t, block, sw, seed, 3, 0, *xt))
    assert q.quartet_debug_set_gemm_plan(variant, 0) == 0
    for dtype in (torch.float32, torch.bfloat16):
        bf16 = int(dtype == torch.bfloat16)
        dx, dw = (torch.full((r, i), float("nan"), dtype=dtype, device="cuda") for r in (t, o))
        q.check(q.quartet_linear_bwd_block(dy, t, i, o, block, *xq, xm, *wq, wm, seed, 0, dx, dw, bf16, ws, n))
        for got, a, b, mask, m, k in ((dx, g, wt, xm, t, o), (dw, gt, xt, wm, o, t)):
            acc, want = torch.empty((m, i), device="cuda"), torch.empty((m, i), dtype=dtype, device="cuda")
            q.check(q.quartet_mxfp4_gemm(*a, *b, m, i, k, 1.0, acc, 0, i))
            q.check(q.quartet_grad_epilogue_block(acc, mask, m, i, block, float(np.float32(16.0) / np.float32(9.0)), want, bf16))
            assert torch.equal(got.view(torch.int16 if bf16 else torch.int32), want.view(torch.int16 if bf16 else torch.int32))
