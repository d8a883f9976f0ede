"""Which kernel the GEMM launcher picks (host only): the choice is a function of the sizes, the Hadamard block and the chip."""
import random

import torch  # noqa: F401  (before the library, as in every program that uses both: they share one HIP runtime then)

from paper_2505_14669_amd import binding as q

CUS = 256


def plan(*mnk, block=0):
    return q.quartet_debug_gemm_plan(len(mnk) // 3, list(mnk), block, CUS)


def test_arguments_are_checked():
    E = q.QUARTET_EINVAL
    assert q.quartet_debug_gemm_plan(1, None, 0, CUS) == E and q.quartet_debug_gemm_plan(3, [32] * 9, 0, CUS) == E
    assert plan(0, 32, 32) == E and plan(32, 32, 33) == E and plan(32, 32, 32, block=48) == E and plan(32, 32, 32, block=256) == E
    assert q.quartet_debug_gemm_plan(1, [32, 32, 32], 0, 4) == E
    assert plan(2 ** 31, 32, 32) == q.QUARTET_ENOTSUP


def test_split_kernels_take_no_more_tiles_than_a_launch_can_hold():
    # one block of up to 256 threads per tile and fewer than 2^32 threads per launch: very tall narrow products stay with the
    # streaming kernels, whose grid is the chip
    assert plan(2 ** 28, 32, 32) // 100 == 2
    for mnk in ((2 ** 30, 32, 32), (2 ** 31 - 1, 1, 32), (2 ** 31 - 1, 32, 512), (2 ** 29, 40, 32)):
        assert plan(*mnk) in (0, 1, 2)
    assert plan(2 ** 29 - 32, 32, 32, 2 ** 29 - 32, 32, 32, block=32) in (0, 1, 2)


def test_four_wave_split_leaves_what_the_streaming_kernels_do_sooner():
    # measured, streaming against four waves (us): 12.8 / 13.9, 16.5 / 18.1, 12.4 / 14.0; 15.5 / 9.2, 16.4 / 9.8
    for mnk in ((377, 4096, 3936), (950, 1696, 5664), (2127, 768, 4096)):
        assert plan(*mnk) == 2
    for mnk in ((339, 2624, 5600), (104, 6592, 6240)):
        assert plan(*mnk) // 100 == 4


def test_every_forced_kernel_is_the_one_that_is_reported():
    try:
        for variant in (0, 1, 2, 22):
            assert q.quartet_debug_set_gemm_plan(variant, 0) == q.QUARTET_OK
            for mnk in ((4096, 4096, 256), (96, 96, 96), (1152, 1280, 1312, 4224, 1280, 96)):
                assert plan(*mnk) == variant and plan(*mnk, block=32) == variant
        for bad in (-2, 3, 21, 23, 222):
            assert q.quartet_debug_set_gemm_plan(bad, 0) == q.QUARTET_EINVAL
    finally:
        q.quartet_debug_set_gemm_plan(-1, 0)


def pair_plan(t, i, o, block):
    return plan(o, i, t, t, i, o, block=block)


def test_pairs_with_blocks_of_128_weigh_the_split_kernels_against_the_tiles_that_run():
    # measured, backward passes on 128 x 256 tiles against the split kernels (us): 21.6 / 13.9, 20.9 / 13.9, 30.0 / 22.8, 40.2 / 26.5, 47.5 / 38.2
    for layer, waves in (((384, 3456, 256), 2), ((512, 2176, 384), 2), ((1280, 640, 2560), 2), ((6016, 384, 640), 4), ((7808, 512, 640), 4)):
        assert pair_plan(*layer, 128) == 100 * waves + 14
    # 53.5 / 69.2, 23.4 / 30.3, 34.4 / 41.0
    for layer in ((5504, 1152, 1280), (512, 2816, 1792), (4096, 1408, 384)):
        assert pair_plan(*layer, 128) == 1


def test_one_product_runs_on_the_side_of_the_plain_one():
    rng = random.Random(4)
    for _ in range(2000):
        m, n, k = rng.randrange(1, 6000), 128 * rng.randrange(1, 40), 32 * rng.randrange(1, 200)
        assert len({plan(m, n, k, block=b) >= 100 for b in (0, 32, 64, 128)}) == 1


def test_sizes_of_the_split_tests_reach_every_kernel():
    # every shape that the launcher has, with two and four waves, wherever it can run (tiles narrower than the Hadamard block cannot)
    import split_sizes
    shapes = {0: (11, 12, 22), 32: (11, 12, 22), 64: (12, 22), 128: (14,)}
    for table in (split_sizes.SINGLE, split_sizes.PAIR):
        for block, sizes in table.items():
            assert sorted(sizes) == sorted(100 * w + s for w in (2, 4) for s in shapes[block])
    for block, sizes in split_sizes.SINGLE.items():
        for code, mnk in sizes.items():
            assert plan(*mnk, block=block) == code, (block, mnk)
    for block, sizes in split_sizes.PAIR.items():
        for code, (t, i, o) in sizes.items():
            assert plan(o, i, t, t, i, o, block=block) == code, (block, t, i, o)
