"""Host rule for the cooperative grid of several steps per launch (no GPU): its barrier needs
every workgroup resident, and scalar registers, which the occupancy query leaves out, let at
most seven workgroups of four waves be sure of a compute unit."""
import ctypes

import pytest


@pytest.fixture(scope="module")
def grid():
    from paper_2304_11165_amd import rd

    fn = ctypes.CDLL(rd.LIB_PATH)._Z13rd_fused_gridiii
    fn.argtypes, fn.restype = [ctypes.c_int] * 3, ctypes.c_int
    return fn


@pytest.mark.parametrize("n_cu", [1, 4, 64, 255, 256, 304])
@pytest.mark.parametrize("per_cu", [0, 1, 2, 5, 6, 7, 8, 16])
def test_grid_is_resident(grid, per_cu, n_cu):
    for groups in (1, 7, 8, 9, 1791, 1792, 1793, 1979, 2048, 36933):
        n = grid(per_cu, n_cu, groups)
        assert n % 8 == 0 and 0 <= n <= min(per_cu, 7) * n_cu
        assert n <= (groups + 7) // 8 * 8
        assert n + 8 > min(min(per_cu, 7) * n_cu, (groups + 7) // 8 * 8)  # and no smaller than it need be


def test_hung_grid_is_cut(grid):
    # 160^3 packing: 1979 groups, eight workgroups per compute unit by the query
    assert grid(8, 256, 1979) == 1792
