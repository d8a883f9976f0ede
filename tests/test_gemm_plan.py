"""Which kernel the GEMM launcher picks (host only): the choice is a function of the sizes, the Hadamard block and the chip."""
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
