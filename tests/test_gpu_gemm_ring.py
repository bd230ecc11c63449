"""The many-row projections: both row blocks of every size, ragged rows and columns, K ranges of one to many stages (fewer than
the ring has slots, odd numbers, a last range that is short or empty), and the LM head's launch at eight row tiles (one row block)
beside the shapes that the plan does not send there."""
import pytest
import torch

from paper_2411_00853_amd import workload as wl

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("N,K", [(16, 32), (100, 64), (200, 96), (1000, 160), (304, 352), (2064, 2048), (6152, 544), (4096, 11008), (22016, 224)])
@pytest.mark.parametrize("M", [193, 224, 225, 256, 257, 288, 320, 321, 352])
def test_many_rows(M, N, K):
    _check(M, N, K, True)


@pytest.mark.parametrize("M", [200, 300, 352])
def test_many_rows_head_plane_only(M):
    _check(M, 720, 736, False)


def _ring_at(M, N, K):
    """Whether the plan runs an LM head of N rows by K columns as gemm_ring_kernel"""
    from paper_2411_00853_amd import binding as sv
    look = [15] * (M // 16) + [M % 16 - 1] * (M % 16 > 0)
    return sv.spec_k_plan_step(sv.make_cfg(wl.ModelShape(1, K, 2, 2, 64, 64, N), len(look), 64, 15), look, 256).gemm_kernels >> 4 & 1


@pytest.mark.parametrize("N,K", [(16000, 64), (16008, 416), (32003, 1024)])
@pytest.mark.parametrize("M", [97, 113, 128])
def test_wide_matrices_at_eight_row_tiles(M, N, K):
    assert not _ring_at(M, N, K)
    _check(M, N, K, True)


# two K ranges and one, stages from fewer than the ring has slots on, an odd number, last column blocks of one and of all tiles
@pytest.mark.parametrize("N,K", [(32000, 2048), (32003, 4096), (31989, 2080), (50257, 1024), (50257, 96), (128256, 32)])
@pytest.mark.parametrize("M", [97, 112, 113, 128])
def test_one_row_block(M, N, K):
    assert _ring_at(M, N, K)
    _check(M, N, K, True)


@pytest.mark.parametrize("M", [100, 128])
def test_one_row_block_head_plane_only(M):
    assert _ring_at(M, 50257, 736)
    _check(M, 50257, 736, False)


def _check(M, N, K, split):
    from paper_2411_00853_amd import binding as sv
    rng = wl.Rng(M + N + K, "cpu")
    x, w = rng.normal(1, (M, K), 1.0).cuda(), rng.normal(2, (512, K), 0.02).bfloat16()
    rows = torch.arange(N) % 509          # every column of the product is one of 509, in another order per tile
    y = sv.spec_k_gemm_bf16(x, sv.spec_pack_weight(w[rows].cuda()), N, split).cpu()
    want = (x.cpu().double() @ w.double().T)[:, rows]
    scale = want.pow(2).mean().sqrt().item()
    # with the remainder 2^-18 of a result as a standard deviation, five and a half of them over two million results and as much
    # again for the order of fp32 sums; with the head alone 2^-9 of each term at most (the bounds of test_gpu_gemm_split, test_gpu_gemm)
    assert (y.double() - want).abs().max().item() < (3e-5 if split else 1.5e-2) * scale
