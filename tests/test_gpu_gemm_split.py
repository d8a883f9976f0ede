"""The GEMM kernels for small problems (in-block split of the inner dimension) at the edges of their tiles, with two and four
waves, both result types and the gradient epilogue of every Hadamard block they serve, against the oracle; and at the sizes
around the line where the launcher goes over to the streaming kernels."""
import numpy as np
import pytest

import indep
import oracle
from paper_2505_14669_amd import synth

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
