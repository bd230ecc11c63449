"""Row blocks of an odd number of row tiles: the two halves of a workgroup differ by one tile.  First and last row count of
each, with two, three and four column tiles per wavefront, both planes and the head alone."""
import pytest

from test_gpu_gemm_ring import _check

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("N,K,split", [(1040, 1056, True), (6160, 160, True), (32008, 96, True), (528, 416, False)])
@pytest.mark.parametrize("M", [194, 222, 258, 287, 323, 351])
def test_odd_row_tiles(M, N, K, split):
    _check(M, N, K, split)
