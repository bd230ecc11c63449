"""The per-class timing of a decoding round holds the launches that embed its rows: one a draft step and one of the verification, as
every launch of a profiled pass is in one class."""
import pytest
import torch

from paper_2411_00853_amd import workload as wl

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("dtype", ["fp32", "bf16"])
def test_a_round_counts_its_embedding(dtype):
    from paper_2411_00853_amd import binding as sv
    from test_gpu_decode import Pair
    shape = wl.ModelShape(1, 128, 2, 2, 64, 128, 211, dtype=dtype)
    K, rng = 3, wl.Rng(4, "cpu")
    pair = Pair(shape, shape, [rng.randint(b, (6 + b,), 211).tolist() for b in range(3)], 64, 4, 20)
    sv.spec_verify_profile_begin(pair.tg.h)
    sv.spec_verify_profile_begin(pair.dr.h)
    pair.round(K, rng.uniform(1, (3, 4)), rng.uniform(2, (3, 5)), 1.0)
    launches = [{c: n for c, (_, n) in sv.spec_verify_profile_end(h)[0].items()} for h in (pair.dr.h, pair.tg.h)]
    assert [l["prepare"] for l in launches] == [K, 1]
    assert [l["gemm_lm_head"] for l in launches] == [K, 1]
