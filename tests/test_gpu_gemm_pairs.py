"""Pairs of gradient products whose tiles are handed out by load (the blocks with one tile of the first product fewer take tiles of the
second in rounds of their own), and 128 x 128 tiles with two blocks per compute unit.  Codes and scales as in test_gpu_gemm_stream: every
sum is exact in fp32, so results are compared bit for bit."""
import numpy as np
import pytest
import test_gpu_gemm_stream as S

import oracle

pytestmark = pytest.mark.gpu
G = S.G


# (products (m, n, k), tile shape): on 256 compute units the first product's tiles leave 1 .. 255 blocks one tile short, and one of its
# tiles takes one to ten times as long as one of the second's.  256 x 256: 45 / 325 tiles; 128 x 256: 60 / 330, 269 (a round and 13) / 272;
# 128 x 128, with one (2) and with two blocks per compute unit (22): 90 / 330, 255 / 260, 2 / 1190
@pytest.mark.parametrize("variant,shapes", [(0, ((2304, 1280, 1312), (16640 - 9, 1280, 96))), (1, ((1500, 1280, 1056), (8448, 1280, 160))),
                                            (1, ((34432, 256, 544), (34816 - 3, 256, 32))), *((v, s) for v in (2, 22) for s in (((1152, 1280, 1312), (4224, 1280, 96)),
                                                                               ((1900, 2176, 800), (2550, 1664, 544)),
                                                                               ((128, 256, 1312), (8960 - 7, 2176, 32)))),
                                            # a first tile outlasts all tiles of the second product that the other blocks can take
                                            (0, ((256, 1280, 16640), (16640 - 9, 1280, 96))), (1, ((128, 1280, 8192), (8448, 1280, 160))),
                                            (2, ((128, 256, 14400), (8960 - 7, 2176, 32))),
                                            (22, ((128, 256, 14400), (8960 - 7, 2176, 32)))])
def test_pair_by_load_equals_single_products(G, variant, shapes):
    from paper_2505_14669_amd import binding
    rng = np.random.default_rng(variant)
    prods = []
    for m, n, k in shapes:
        (a, sa, _), (b, sb, _) = S._operand(rng, m, k), S._operand(rng, n, k)
        prods.append((a, sa, b, sb, rng.integers(0, 2 ** 32, size=(m, n // 32), dtype=np.uint32), oracle.FL_16_9))
    assert binding.quartet_debug_set_gemm_plan(variant, 0) == 0
    for got, p in zip(G.gemm_grad_pair(*prods), prods):
        want = G.grad_epilogue_block(G.gemm(*p[:4]), p[4], 32, p[5])
        assert np.array_equal(got.view(np.uint32), want.view(np.uint32))


# several rounds of tiles on every compute unit and few K-quads per tile, with one and two blocks on each: fewer quads than ring slots,
# ragged last quads, full and ragged tiles in turn
@pytest.mark.parametrize("variant", [2, 22])
@pytest.mark.parametrize("k", [32, 160, 256, 480, 544, 1312])
@pytest.mark.parametrize("m,n", [(4352, 4224), (8191, 1664 + 5)])
def test_blocks_per_compute_unit_exact(G, variant, m, n, k):
    from paper_2505_14669_amd import binding
    rng = np.random.default_rng(k)
    (a, sa, va), (b, sb, vb) = S._operand(rng, m, k), S._operand(rng, n, k)
    assert binding.quartet_debug_set_gemm_plan(variant, 0) == 0
    assert np.array_equal(G.gemm(a, sa, b, sb), (va @ vb.T).cpu().numpy().astype(np.float32))
