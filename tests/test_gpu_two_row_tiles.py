"""Products of two row tiles, whose rows past the last fetch nothing: first, middle and last row counts, K ranges that end inside a
group of the packed order, both plane counts."""
import pytest

from test_gpu_gemm_ring import _check

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("N,K,split", [(48, 32, True), (1000, 160, True), (4096, 11008, True), (16384, 2048, True), (528, 416, False)])
@pytest.mark.parametrize("M", [17, 24, 31, 32])
def test_two_row_tiles(M, N, K, split):
    _check(M, N, K, split)
