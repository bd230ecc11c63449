"""Logits that leave the LM head as partial sums and are added up in the statistics pass, with rows that are not 16-byte aligned:
one chunk of 16384 columns, a column more or less, and several K ranges, every row against the oracle."""
import pytest
import torch

from paper_2411_00853_amd import workload as wl

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("d", [64, 1024])
@pytest.mark.parametrize("V", [255, 257, 4097, 16383, 16385, 18903])
def test_rows_of_any_alignment(V, d):
    from test_gpu_forward import Rig
    look = [3, 0, 2]
    shape = wl.ModelShape(1, d, 2, 2, 64, 64, V, dtype="bf16")
    rig = Rig(shape, 3, 64, 3, seed=V, std=0.5 / d ** 0.5)
    rng = wl.Rng(V, "cpu")
    t0, toks = rng.randint(1, (3,), V).tolist(), rng.randint(2, (3, 3), V)
    for s in range(3):
        n = 5 + 11 * s
        rig.caches[s][:, :, :, :n] = rng.normal(20 + s, (1, 2, 2, n, 64), 0.5)
        rig.set_cache(s, n)
    got, _, _ = rig.step([0, 1, 2], t0, look, toks, rng.normal(3, (3, 3, V), 1.0), rng.uniform(4, (3, 4)), 1.0)
    want = rig.oracle_logits([0, 1, 2], t0, look, toks)
    assert (got - want).abs().max().item() <= 5e-3     # the bound of the other small bf16 models (test_gpu_row_scale)
