"""Which kernel the GEMM launcher picks (host only): the choice is a function of the sizes, the Hadamard block and the chip."""
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
