"""The transposed quantizers at the sizes where their launch changes: columns per lane of the re-quantizer blocks (2, 4, 8 by
the number of elements), the streaming and the LDS tile of the bf16 source, ragged edges of each, and the one-launch operand
conversions of wider Hadamard blocks.  Everything is compared bit for bit."""
import numpy as np
import pytest
import torch

import oracle
from paper_2505_14669_amd import synth

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def G():
    import gpu_util
    return gpu_util


def _codes(seed, rows, k):
    rng = np.random.default_rng(seed)
    return (rng.integers(0, 256, size=(rows, k // 2), dtype=np.uint8),
            rng.integers(110, 140, size=(rows, k // 32), dtype=np.uint8))


# source [k x rows]: 0.1 M, 10.7 M and 33.9 M elements = 2, 4 and 8 columns per lane; no size a multiple of a tile; rows that are not
# whole lines with 17 K-quads (columns in the grid's second dimension), whole lines, and 15 K-quads
@pytest.mark.parametrize("k,rows", [(1056, 96), (4128, 2592), (4128, 8224), (4128, 8448), (3808, 8928)])
@pytest.mark.parametrize("rounding", [0, 1])
def test_requant_every_split(G, k, rows, rounding):
    codes, scales = _codes(k + rows, k, rows)
    sw = 0x9E3779B1
    got = G.requant_transpose_sr(codes, scales, sw, 77, 3, rounding)
    want = oracle.requant_transpose_sr(codes, scales, sw, 77, 3, rounding)
    assert np.array_equal(got[0], want[0]) and np.array_equal(got[1], want[1])


@pytest.mark.parametrize("k,rows,block", [(1152, 160, 128), (4224, 2592, 64), (4352, 7840, 256)])
def test_requant_block_every_split(G, k, rows, block):
    codes, scales = _codes(k, k, rows)
    sw = oracle.sign_words(21)
    got = G.requant_transpose_sr_block(codes, scales, block, sw, 21, 1, 0)
    want = oracle.requant_transpose_sr_block(codes, scales, block, sw, 21, 1, 0)
    assert np.array_equal(got[0], want[0]) and np.array_equal(got[1], want[1])


# source [k x rows]: the line between the two tiles lies at 2048 waves of 256 rows x 32 columns for a multiple of eight K-quads, at
# 1280 otherwise
@pytest.mark.parametrize("k,rows,block", [(4064, 4040, 32), (4128, 4104, 32), (4224, 3848, 128), (4352, 4104, 256),
                                          (2528, 4064, 32), (2528, 4104, 32), (2560, 4104, 64),
                                          (5184, 8032, 64), (5248, 8040, 128)])     # two blocks share a line, K-quads rounded up
def test_quant_transposed_both_tiles(G, k, rows, block):
    x = synth.small_matrix(5, k, rows, "heavy", 1e-3)
    sw = oracle.sign_words(31)
    got = G.quant_bwd_sr_block(x, block, sw, 31, 2, 0, transpose=True)
    want = oracle.quant_bwd_sr_block(np.ascontiguousarray(x.T), block, sw, 31, 2, 0)
    assert np.array_equal(got[0], want[0]) and np.array_equal(got[1], want[1])


# the linear layer's one-launch operand conversions against the single conversions, through the gradients: both sides run
# the same products on the same tile shape, so equal operands give equal bits
@pytest.mark.parametrize("t,i,o", [(512, 768, 256), (2304, 2816, 2560), (4352, 3840, 4096)])
@pytest.mark.parametrize("block", [32, 64, 128])
def test_one_launch_operands_match_single_conversions(G, t, i, o, block):
    from paper_2505_14669_amd import binding as q
    g = torch.Generator(device=G.DEV)
    g.manual_seed(t + block)
    x, w, dy = (torch.randn(s, generator=g, device=G.DEV).to(torch.bfloat16) for s in ((t, i), (o, i), (t, o)))
    seed, words = 1234567, q.quartet_sign_words(1234567)

    def mx(rows, k):
        return (torch.empty((rows, k // 2), dtype=torch.uint8, device=G.DEV),
                torch.empty(q.quartet_scale_bytes(rows, k), dtype=torch.uint8, device=G.DEV))
    (xc, xs), (wc, ws) = mx(t, i), mx(o, i)
    xm, wm = (torch.empty((r, i // 32), dtype=torch.int32, device=G.DEV) for r in (t, o))
    y = torch.empty((t, o), device=G.DEV)
    q.check(q.quartet_linear_fwd_block(x, w, t, i, o, block, y, 0, xc, xs, xm, wc, ws, wm))
    dx, dw, dx1, dw1 = (torch.empty(s, device=G.DEV) for s in ((t, i), (o, i), (t, i), (o, i)))
    n = q.quartet_linear_workspace_bytes_block(t, i, o, block)
    q.quartet_debug_set_gemm_plan(1, 0)
    try:
        q.check(q.quartet_linear_bwd_block(dy, t, i, o, block, xc, xs, xm, wc, ws, wm, seed, 0, dx, dw, 0,
                                           torch.empty(n, dtype=torch.uint8, device=G.DEV), n))
        a, at, b, bt = mx(t, o), mx(o, t), mx(i, o), mx(i, t)
        q.check(q.quartet_quant_bwd_sr_block(dy, t, o, o, 0, block, words, seed, 0, 0, *a))
        q.check(q.quartet_requant_transpose_sr_block(wc, ws, i, o, block, words, seed, 1, 0, *b))
        q.check(q.quartet_quant_bwd_sr_block(dy, o, t, o, 1, block, words, seed, 2, 0, *at))
        q.check(q.quartet_requant_transpose_sr_block(xc, xs, i, t, block, words, seed, 3, 0, *bt))
        q.check(q.quartet_mxfp4_gemm_grad_block(*a, *b, t, i, o, block, xm, 16.0 / 9.0, dx1, 0, i))
        q.check(q.quartet_mxfp4_gemm_grad_block(*at, *bt, o, i, t, block, wm, 16.0 / 9.0, dw1, 0, i))
    finally:
        q.quartet_debug_set_gemm_plan(-1, 0)
    assert torch.equal(dx, dx1) and torch.equal(dw, dw1)
