"""The projections where the rules of the launch shape change: three column tiles per wavefront at five and six
row tiles, two from eight row tiles on where the partial sums outweigh the weights; ragged columns and rows."""
import pytest
import torch

from paper_2411_00853_amd import workload as wl

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("N,K", [(12288, 4096), (22016, 4096), (11008, 2048), (6152, 2048), (16384, 2048), (16383, 2048)])
@pytest.mark.parametrize("M", [65, 80, 81, 96, 113, 128, 160, 177, 192])
def test_products_where_the_launch_shape_changes(M, N, K):
    from paper_2411_00853_amd import binding as sv
    rng = wl.Rng(M, "cpu")
    x, w = rng.normal(1, (M, K), 1.0).cuda(), rng.normal(2, (512, K), 0.02).bfloat16()
    rows = torch.arange(N) % 509          # every column of the product is one of 509, in another order per tile
    y = sv.spec_k_gemm_bf16(x, sv.spec_pack_weight(w[rows].cuda()), N, True).cpu()
    want = (x.cpu().double() @ w.double().T)[:, rows]
    scale = want.pow(2).mean().sqrt().item()
    # the remainder's truncation, 2^-17 of each term at most and of either sign: 2^-18 of the result as a standard
    # deviation, five and a half of them over two million results, and as much again for the order of fp32 sums
    assert (y.double() - want).abs().max().item() < 3e-5 * scale
