"""Steps of up to 16 rows, whose output and down projections finish the residual stream themselves: 4, 8 and 16 K ranges, ranges
that are short or empty, K that is no multiple of the packed order's 128 columns, widths that are no multiple of 1024 (the
row's sum of squares is added up by groups of that many columns) and, at 17 rows, the chain of launches beyond."""
import pytest
import torch

from paper_2411_00853_amd import workload as wl

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("look", [[0], [5, 0], [7, 7], [7, 8]])      # 1, 7, 16 and 17 rows
@pytest.mark.parametrize("d,heads,hd,F", [(4096, 16, 128, 2048), (2080, 32, 64, 2144), (2048, 17, 128, 6144), (1056, 8, 64, 4128),
                                          (512, 4, 64, 5664), (160, 2, 64, 96)])
def test_steps_of_few_rows(d, heads, hd, F, look):
    from test_gpu_forward import Rig
    V, B = 131, len(look)
    shape = wl.ModelShape(2, d, heads, heads, hd, F, V, dtype="bf16")
    rig = Rig(shape, B, 64, 8, seed=d + F, std=0.5 / d ** 0.5)
    rng = wl.Rng(F, "cpu")
    t0, toks = rng.randint(1, (B,), V).tolist(), rng.randint(2, (B, 8), V)
    for s in range(B):
        n = 20 + 11 * s
        rig.caches[s][:, :, :, :n] = rng.normal(20 + s, (2, 2, heads, n, hd), 0.5)
        rig.set_cache(s, n)
    got, _, _ = rig.step(list(range(B)), t0, look, toks, rng.normal(3, (B, 8, V), 1.0), rng.uniform(4, (B, 9)), 1.0)
    want = rig.oracle_logits(list(range(B)), t0, look, toks)
    assert (got - want).abs().max().item() <= 5e-3     # the bound of the other small bf16 models (test_gpu_row_scale)


# Steps of up to 16 rows against one of 17, which takes product and residual kernel: the rows they share come out alike bit for
# bit.  `inside`: which of output and down projection (bits 1 and 3) add to the residual stream themselves.
@pytest.mark.parametrize("looks", [([7, 7], [7, 8]), ([3, 3], [3, 12])])
@pytest.mark.parametrize("d,heads,hd,F,ranges,inside", [
    (4096, 16, 128, 2048, (4, 4), (0b1010, 0b1010)), (2720, 34, 64, 4128, (4, 4), (0b1010, 0b1010)), (2048, 17, 128, 4096, (4, 8), (0b0010, 0b1010)),
    (1024, 16, 64, 2048, (4, 8), (0b1010, 0b1010)), (2080, 32, 64, 2144, (8, 4), (0b1010, 0b1010)), (1056, 8, 64, 4064, (2, 16), (0b1000, 0b1000)),
    (512, 32, 64, 1568, (8, 4), (0b1010, 0b1010)), (1024, 16, 64, 5632, (4, 16), (0b0010, 0b1010))])
def test_few_rows_keep_the_bits_of_the_two_launches(d, heads, hd, F, ranges, inside, looks):
    from paper_2411_00853_amd import binding as sv
    from test_gpu_forward import Rig
    V, n = 131, sum(looks[0]) + 2
    shape = wl.ModelShape(2, d, heads, heads, hd, F, V, dtype="bf16")
    rig = Rig(shape, 2, 64, 12, seed=d + F, std=0.5 / d ** 0.5)
    few, more = (sv.spec_k_plan_step(rig.cfg, look) for look in looks)
    assert list(few.gemm_k_ranges) == list(more.gemm_k_ranges) and (few.gemm_k_ranges[1], few.gemm_k_ranges[3]) == ranges
    assert few.gemm_kernels >> 8 == inside[n == 8] and more.gemm_kernels == 0
    rng = wl.Rng(F, "cpu")
    t0, toks = rng.randint(1, (2,), V).tolist(), rng.randint(2, (2, 12), V)
    got = []
    for look in looks:
        for s in range(2):
            rig.caches[s][:, :, :, :20 + 11 * s] = wl.Rng(5, "cpu").normal(20 + s, (2, 2, heads, 20 + 11 * s, hd), 0.5)
            rig.set_cache(s, 20 + 11 * s)
        got.append(rig.step([0, 1], t0, look, toks, rng.normal(3, (2, 12, V), 1.0), rng.uniform(4, (2, 13)), 1.0)[0])
    assert torch.equal(got[0], got[1][:n])
