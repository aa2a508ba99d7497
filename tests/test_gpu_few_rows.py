"""GPU parity of the variants that calls with few rows take, at the sizes where a tile, a lane group or a wave's share
ends.  Same oracle, inputs and tolerances as the tests they reuse."""
import pytest

import test_gpu_parity as P

pytestmark = pytest.mark.gpu


# products that stream the weights: at most 8 rows per expert on average take 16-row tiles, at most 20 take 32-row tiles
@pytest.mark.parametrize("counts,d,f", [
    ([1] * 8 + [0, 0], 64, 64),                       # one block of the reduction: only the last wave has work
    ([16, 0, 17, 0, 1, 33, 0, 0, 15, 0, 0, 0, 0, 0, 0, 0, 0, 0, 0, 0], 192, 128),     # rows at and past a 16-row tile
    ([2, 0, 9] * 40 + [0] * 10, 320, 192),            # more than 64 experts; five blocks over four waves
    ([32, 33, 0, 31, 1, 64, 3, 2, 7, 0, 0, 0], 448, 320),                             # 32-row tiles
    ([20] * 130, 128, 64),                            # more than 128 experts
])
def test_streamed_products(counts, d, f):
    P.test_grouped_gemm_fwd_bwd_isolated(counts, d, f)


# Stages 1-3 in one workgroup: at most 1024 pairs
@pytest.mark.parametrize("T,E,k,eb,ec", [
    (128, 64, 8, 0, 64), (129, 64, 8, 3, 50),         # the last call of one launch, the first of two
    (65, 8, 1, 0, 8), (256, 33, 4, 1, 31), (257, 33, 3, 0, 33), (100, 130, 10, 0, 130), (14, 512, 70, 0, 512), (17, 300, 3, 299, 1)])
@pytest.mark.parametrize("renorm,gate", [(0, False), (1, True)])
def test_one_launch_routing(T, E, k, eb, ec, renorm, gate):
    P.test_route_permute_one_call(T, E, k, eb, ec, renorm, gate)
