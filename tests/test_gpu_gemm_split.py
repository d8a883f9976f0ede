"""The GEMM kernels for small problems (in-block split of the inner dimension) at the edges of their tiles, with two and four
waves, both result types and the gradient epilogue of every Hadamard block they serve, against the oracle; at sizes
around the line where the launcher goes over to the streaming kernels; and every kernel of them (waves x tile shape, plain, fused and
pairs; split_sizes.py, whose sizes test_gemm_plan.py holds to the launcher's choice) bit for bit on sums that are exact in fp32."""
import numpy as np
import pytest
import torch

import indep
import oracle
import split_sizes
from paper_2505_14669_amd import binding, synth

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def G():
    import gpu_util
    return gpu_util


def _operands(m, n, k):
    rng = np.random.default_rng(m * 7919 + n * 31 + k)
    return (rng.integers(0, 256, size=(m, k // 2), dtype=np.uint8), rng.integers(117, 137, size=(m, k // 32), dtype=np.uint8),
            rng.integers(0, 256, size=(n, k // 2), dtype=np.uint8), rng.integers(117, 137, size=(n, k // 32), dtype=np.uint8))


# fp32 accumulation of k exact products in any order: |error| <= (k/64 + 3) 2^-23 sum |a||b| per element (the streaming kernels'
# bound: one rounding per matrix-core instruction and K-step, plus the sums over the waves and the scaling)
def _check(got, want, absp, k):
    assert np.all(np.abs(got - want) <= (k / 64 + 6) * 2.0 ** -23 * absp)


@pytest.mark.parametrize("m,n,k", [(1, 1, 32), (31, 33, 256), (32, 64, 288), (33, 65, 544), (65, 129, 2784),   # two waves, ragged K-quads
                                   (7, 37, 2816), (33, 32, 3072), (64, 61, 4128), (96, 640, 3360),             # four waves
                                   (128, 2048, 4096), (1024, 1024, 1024), (264, 520, 8192), (300, 8200, 512)])
def test_split_gemm(G, m, n, k):
    a, sa, b, sb = _operands(m, n, k)
    want = oracle.mxfp4_gemm(a, sa, b, sb, alpha=0.75)
    got = G.gemm(a, sa, b, sb, alpha=0.75, ldd=n + 3)
    _check(got[:, :n], want, 0.75 * indep.gemm_abs_products(a, sa, b, sb), k)
    assert np.all(np.isnan(got[:, n:]))
    bf = G.gemm(a, sa, b, sb, alpha=0.75, bf16=True)
    assert np.array_equal(bf, synth.f32_to_bf16(G.gemm(a, sa, b, sb, alpha=0.75)))


@pytest.mark.parametrize("m,n,k,block", [(33, 96, 288, 32), (70, 192, 800, 64), (45, 384, 1056, 128), (33, 96, 2816, 32),
                                         (40, 192, 3072, 64), (65, 256, 4096, 128), (512, 512, 512, 64), (200, 768, 256, 128)])
def test_split_gemm_grad_equals_two_steps(G, m, n, k, block):
    a, sa, b, sb = _operands(m, n, k)
    mask = np.random.default_rng(k).integers(0, 2 ** 32, size=(m, n // 32), dtype=np.uint32)
    plain = G.gemm(a, sa, b, sb)
    got = G.gemm_grad_block(a, sa, b, sb, block, mask, oracle.FL_16_9)
    assert np.array_equal(got.view(np.uint32), G.grad_epilogue_block(plain, mask, block, oracle.FL_16_9).view(np.uint32))


@pytest.mark.parametrize("first,second", [((64, 96, 288), (33, 32, 544)), ((512, 256, 256), (256, 256, 512)), ((40, 64, 3072), (96, 64, 96))])
def test_split_gemm_pair(G, first, second):
    prods = []
    for i, (m, n, k) in enumerate((first, second)):
        a, sa, b, sb = _operands(m, n, k)
        mask = None if i else np.random.default_rng(m).integers(0, 2 ** 32, size=(m, n // 32), dtype=np.uint32)
        prods.append((a, sa, b, sb, mask, 1.25 + i))
    for got, (a, sa, b, sb, mask, scale) in zip(G.gemm_grad_pair(*prods), prods):
        want = oracle.grad_epilogue(oracle.mxfp4_gemm(a, sa, b, sb).astype(np.float32),
                                    np.full((a.shape[0], b.shape[0] // 32), 0xFFFFFFFF, np.uint32) if mask is None else mask, scale)
        # the transform spreads a row's errors over its 32 columns: bound by their sum
        absp = np.repeat(indep.gemm_abs_products(a, sa, b, sb).reshape(a.shape[0], -1, 32).sum(-1), 32, axis=1)
        _check(got, want, scale * absp, 2 * a.shape[1])


GRID = np.array([0, .5, 1, 1.5, 2, 3, 4, 6, 0, -.5, -1, -1.5, -2, -3, -4, -6])


def _exact_operand(rng, rows, k):
    # products are multiples of 2^-4 and at most 144 in size: with k <= 4128 every sum is exact in fp32 (below 2^24 units), in any order
    assert k * 144 * 16 < 2 ** 24
    codes = rng.integers(0, 256, size=(rows, k // 2), dtype=np.uint8)
    scales = rng.integers(126, 129, size=(rows, k // 32), dtype=np.uint8)
    values = np.empty((rows, k))
    values[:, 0::2], values[:, 1::2] = GRID[codes & 15], GRID[codes >> 4]
    return codes, scales, torch.from_numpy(values * np.repeat(2.0 ** (scales.astype(np.float64) - 127), 32, axis=1)).cuda()


def _exact_product(rng, m, n, k):
    (a, sa, va), (b, sb, vb) = _exact_operand(rng, m, k), _exact_operand(rng, n, k)
    return (a, sa, b, sb), (va @ vb.T).cpu().numpy().astype(np.float32)


@pytest.mark.parametrize("code", sorted(split_sizes.SINGLE[0]))
def test_every_split_kernel_plain(G, code):
    m, n, k = split_sizes.SINGLE[0][code]
    operands, want = _exact_product(np.random.default_rng(code), m, n, k)
    assert np.array_equal(G.gemm(*operands), want)
    assert np.array_equal(G.gemm(*operands, bf16=True), synth.f32_to_bf16(want))


@pytest.mark.parametrize("block,code", [(b, c) for b in (32, 64, 128) for c in sorted(split_sizes.SINGLE[b])])
def test_every_split_kernel_fused(G, block, code):
    m, n, k = split_sizes.SINGLE[block][code]
    rng = np.random.default_rng(code + block)
    operands, product = _exact_product(rng, m, n, k)
    mask = rng.integers(0, 2 ** 32, size=(m, n // 32), dtype=np.uint32)
    want = G.grad_epilogue_block(product, mask, block, oracle.FL_16_9)
    assert np.array_equal(G.gemm_grad_block(*operands, block, mask, oracle.FL_16_9).view(np.uint32), want.view(np.uint32))


@pytest.mark.parametrize("code", sorted(split_sizes.PAIR[32]))
def test_every_split_kernel_pair(G, code):
    t, i, o = split_sizes.PAIR[32][code]
    rng = np.random.default_rng(code)
    prods, want = [], []
    for m, n, k in ((o, i, t), (t, i, o)):
        operands, product = _exact_product(rng, m, n, k)
        mask = rng.integers(0, 2 ** 32, size=(m, n // 32), dtype=np.uint32)
        prods.append((*operands, mask, oracle.FL_16_9))
        want.append(G.grad_epilogue_block(product, mask, 32, oracle.FL_16_9))
    for got, w in zip(G.gemm_grad_pair(*prods), want):
        assert np.array_equal(got.view(np.uint32), w.view(np.uint32))


# wider Hadamard blocks reach the pair through the layer's backward pass: against the same call with the streaming kernels forced.  An fp32
# sum of k products is off by at most (k/64 + 6) 2^-23 sum |a||b|, and sum |a||b| of random signs is about sqrt(k) times the sum's size
@pytest.mark.parametrize("block,code", [(b, c) for b in (64, 128) for c in sorted(split_sizes.PAIR[b])])
def test_every_split_kernel_pair_of_wide_blocks(G, block, code):
    t, i, o = split_sizes.PAIR[block][code]
    g = torch.Generator(device=G.DEV)
    g.manual_seed(code)
    x, w, dy = (torch.randn(s, generator=g, device=G.DEV).to(torch.bfloat16) for s in ((t, i), (o, i), (t, o)))
    u8 = lambda *s: torch.empty(s, dtype=torch.uint8, device=G.DEV)
    ctx = []
    for r in (t, o):
        ctx += [u8(r, i // 2), u8(binding.quartet_scale_bytes(r, i)), torch.empty((r, i // 32), dtype=torch.int32, device=G.DEV)]
    y, n = torch.empty((t, o), device=G.DEV), binding.quartet_linear_workspace_bytes_block(t, i, o, block)
    binding.check(binding.quartet_linear_fwd_block(x, w, t, i, o, block, y, 0, *ctx))
    out = []
    try:
        for variant in (-1, 1):
            binding.check(binding.quartet_debug_set_gemm_plan(variant, 0))
            dx, dw = torch.empty((t, i), device=G.DEV), torch.empty((o, i), device=G.DEV)
            binding.check(binding.quartet_linear_bwd_block(dy, t, i, o, block, *ctx, 77, 0, dx, dw, 0, u8(n), n))
            out.append((dx, dw))
    finally:
        binding.quartet_debug_set_gemm_plan(-1, 0)
    for got, want, k in zip(*out, (o, t)):
        assert float((got - want).norm() / want.norm()) < (k / 64 + 6) * 2.0 ** -23 * k ** 0.5


# on one side of the line between two and four waves (k = 2816) a pair sums in the order its products have alone, whatever the tile
# shapes; across it the product with the smaller k may differ in the last bits.  Scales spread over 20 binades: no exact sums
@pytest.mark.parametrize("first,second,same", [((64, 96, 288), (33, 32, 2816), True), ((512, 256, 256), (256, 2048, 512), True),
                                               ((40, 64, 3072), (96, 64, 2848), True), ((40, 64, 3072), (96, 64, 2048), False)])
def test_split_pair_against_single_products(G, first, second, same):
    waves = lambda code: code // 100
    assert waves(binding.quartet_debug_gemm_plan(2, [*first, *second], 32, 256)) > 0
    prods = [(*_operands(*mnk), None, 1.0) for mnk in (first, second)]
    for i, (got, p, mnk) in enumerate(zip(G.gemm_grad_pair(*prods), prods, (first, second))):
        assert waves(binding.quartet_debug_gemm_plan(1, list(mnk), 32, 256)) > 0
        alone = G.gemm_grad_block(*p[:4], 32, None, 1.0)
        if same or i == 0:
            assert np.array_equal(got.view(np.uint32), alone.view(np.uint32))
        else:
            absp = np.repeat(indep.gemm_abs_products(*p[:4]).reshape(mnk[0], -1, 32).sum(-1), 32, axis=1)
            assert np.all(np.abs(got - alone) <= 2 * (mnk[2] / 64 + 6) * 2.0 ** -23 * absp)
