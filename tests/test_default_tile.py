"""The fused adjoint's tile of a new plan where the kernels' measured times
differ most (no GPU: the choice is made when the plan is packed)."""
import numpy as np
import pytest


# times in us of the adjoint with the tile expected here, and with t2 = 32 or
# 64 on the warp-specialised kernel
@pytest.mark.parametrize("dims,q,m,rank,precision,kernel,t2", [
    ((148, 23, 49), 3, 15, 8, 0, 0, (8,)),     # 42, 60
    ((135, 27, 22), 12, 9, 8, 0, 0, (4,)),     # 49, 65
    ((90, 37, 40), 3, 30, 7, 1, 0, (4, 8)),    # 65% of the time (43 columns)
    ((152, 43, 29), 3, 13, 6, 1, 0, (4,)),     # 65%
    ((33, 33, 134), 3, 12, 6, 1, 0, (4, 8)),   # 33 and 31, 47
    ((81, 26, 61), 12, 20, 6, 0, 1, (32,)),       # FP32: the warp-specialised kernel
    ((26, 62, 144), 3, 75, 8, 1, 1, (64,)),       # 153; 276 at t2 = 8
])
def test_adjoint_tile_of_a_new_plan(dims, q, m, rank, precision, kernel, t2):
    from paper_2103_06393_amd import lib
    K = q * m
    ones = lambda n: np.full(n, 0.5 + 0.25j)  # noqa: E731
    h = lib.tv_plan_from_factors(lib.make_grid(*dims, q, m), np.full((K, 3), rank, np.int32),
                                 ones(K * rank ** 3), *(ones(K * n * rank) for n in dims),
                                 precision)
    try:
        info = lib.tv_plan_info(h)
        assert info.kernel[1] == kernel and info.tile_t2[1] in t2
    finally:
        lib.tv_plan_destroy(h)
