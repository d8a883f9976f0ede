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
