"""The streaming GEMM kernels where their ring of K-quads, their issue cursor and their deferred wait for result stores can go
wrong: fewer K-quads per tile than ring slots, a ragged last quad (one to seven groups), several tiles per block with full and
ragged ones in turn, two products of different inner dimensions in one launch.  Codes and scales are chosen so that every sum is
exact in fp32 (products are multiples of 2^-4 and at most 144 in size, k <= 1312: below 2^24 units), so results are
compared bit for bit with an fp64 product."""
import numpy as np
import pytest
import torch

import oracle

pytestmark = pytest.mark.gpu

GRID = np.array([0, .5, 1, 1.5, 2, 3, 4, 6, 0, -.5, -1, -1.5, -2, -3, -4, -6])


@pytest.fixture()
def G():
    import gpu_util
    from paper_2505_14669_amd import binding
    yield gpu_util
    binding.quartet_debug_set_gemm_plan(-1, 0)


def _operand(rng, rows, k):
    codes = rng.integers(0, 256, size=(rows, k // 2), dtype=np.uint8)
    scales = rng.integers(126, 129, size=(rows, k // 32), dtype=np.uint8)
    values = np.empty((rows, k))
    values[:, 0::2], values[:, 1::2] = GRID[codes & 15], GRID[codes >> 4]
    return codes, scales, torch.from_numpy(values * np.repeat(2.0 ** (scales.astype(np.float64) - 127), 32, axis=1)).cuda()


@pytest.mark.parametrize("variant,m,n", [(0, 4352 - 17, 4096 + 256), (1, 2176, 4352 - 5), (2, 2176, 2176), (2, 2176 - 9, 2176 + 64),
                                         (22, 2176, 4352), (22, 4352 - 9, 2176 + 64)])
@pytest.mark.parametrize("k", [32, 128, 160, 256, 480, 544, 768, 1312])
def test_stream_gemm_exact(G, variant, m, n, k):
    rng = np.random.default_rng(k * 8 + variant)
    (a, sa, va), (b, sb, vb) = _operand(rng, m, k), _operand(rng, n, k)
    from paper_2505_14669_amd import binding
    assert binding.quartet_debug_set_gemm_plan(variant, 0) == 0
    got = G.gemm(a, sa, b, sb)
    assert np.array_equal(got, (va @ vb.T).cpu().numpy().astype(np.float32))


@pytest.mark.parametrize("variant", [0, 1, 2, 22])
@pytest.mark.parametrize("shapes", [((2304, 4352, 288), (4096, 2304, 800)), ((2048, 2304, 1056), (2000, 2080, 96))])
def test_stream_gemm_pair_equals_single(G, variant, shapes):
    from paper_2505_14669_amd import binding
    rng = np.random.default_rng(variant)
    prods = []
    for m, n, k in shapes:
        (a, sa, _), (b, sb, _) = _operand(rng, m, k), _operand(rng, n, k)
        prods.append((a, sa, b, sb, rng.integers(0, 2 ** 32, size=(m, n // 32), dtype=np.uint32), oracle.FL_16_9))
    assert binding.quartet_debug_set_gemm_plan(variant, 0) == 0
    for got, p in zip(G.gemm_grad_pair(*prods), prods):
        want = G.grad_epilogue_block(G.gemm(*p[:4]), p[4], 32, p[5])
        assert np.array_equal(got.view(np.uint32), want.view(np.uint32))


# sizes where the launcher takes each kernel, and on both sides of lines between two: one product's plan code (quartet_debug_gemm_plan)
CHOSEN = [((4096, 4096, 256), 22), ((4097, 4096, 256), 22), ((1170, 7584, 384), 22), ((2529, 384, 1312), 222), ((46, 800, 1280), 211),
          ((3127, 1408, 1248), 22), ((4096, 2048, 512), 22), ((2048, 4097, 288), 22), ((1271, 3200, 608), 2), ((1271, 3201, 608), 22),
          ((4608, 896, 704), 2), ((4608, 897, 704), 22), ((5632, 5120, 1312), 22), ((5632, 5121, 1312), 0), ((5633, 6528, 1312), 22),
          ((5633, 6529, 1312), 1)]


@pytest.mark.parametrize("mnk,code", CHOSEN)
def test_gemm_chosen_plan_exact(G, mnk, code):
    from paper_2505_14669_amd import binding
    m, n, k = mnk
    assert binding.quartet_debug_gemm_plan(1, list(mnk), 0, torch.cuda.get_device_properties(0).multi_processor_count) == code
    rng = np.random.default_rng(m + n + k)
    (a, sa, va), (b, sb, vb) = _operand(rng, m, k), _operand(rng, n, k)
    assert np.array_equal(G.gemm(a, sa, b, sb), (va @ vb.T).cpu().numpy().astype(np.float32))


# results of 256 MB and more, which full tiles store past the memory-side cache; full and ragged tiles, every kernel, plain and with the
# gradient epilogue (against the epilogue kernel on the exact product)
@pytest.mark.parametrize("variant", [0, 1, 2, 22])
@pytest.mark.parametrize("dtype,m,n", [(torch.float32, 8192 + 100, 8192), (torch.bfloat16, 16384 + 100, 8192)])
def test_results_past_the_memory_side_cache(G, variant, dtype, m, n):
    from paper_2505_14669_amd import binding as q
    rng, k, bf16 = np.random.default_rng(variant), 288, int(dtype == torch.bfloat16)
    (a, sa, va), (b, sb, vb) = _operand(rng, m, k), _operand(rng, n, k)
    a, sa, b, sb = G.to_dev(a), G.to_dev(G.scales_to_tiled(sa)), G.to_dev(b), G.to_dev(G.scales_to_tiled(sb))
    assert q.quartet_debug_set_gemm_plan(variant, 0) == 0
    got = torch.full((m, n), float("nan"), dtype=dtype, device="cuda")
    q.check(q.quartet_mxfp4_gemm(a, sa, b, sb, m, n, k, 1.0, got, bf16, n))
    exact = (va @ vb.T).float()
    assert torch.equal(got, exact.to(dtype))
    mask = torch.from_numpy(rng.integers(-2 ** 31, 2 ** 31, size=(m, n // 32), dtype=np.int64).astype(np.int32)).cuda()
    want = torch.empty_like(got)
    q.check(q.quartet_grad_epilogue(exact, mask, m, n, float(oracle.FL_16_9), want, bf16))
    q.check(q.quartet_mxfp4_gemm_grad(a, sa, b, sb, m, n, k, mask, float(oracle.FL_16_9), got, bf16, n))
    bits = torch.int16 if bf16 else torch.int32
    assert torch.equal(got.view(bits), want.view(bits))
