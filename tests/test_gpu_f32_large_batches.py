"""The fp32 attention of large batches, whose launches have fewer positions in flight per workgroup: on both sides of the lines (four
and sixteen workgroups per compute unit, with more than 128 dims two), empty caches and caches that no trip divides: the logits and the
window's cache entries against the oracle."""
import pytest
import torch

from paper_2411_00853_amd import workload as wl

pytestmark = pytest.mark.gpu


# (row, head) workgroups of 256 compute units: 1024, 1026, 1032, 4095, 4096, 4160; 1022, 1024, 4092, 4096; 512, 513, 4104; 4160 of one lane to four dims
@pytest.mark.parametrize("heads,kv_heads,hd,B,k", [
    (4, 4, 64, 32, 7), (2, 1, 64, 57, 8), (4, 2, 24, 129, 1), (9, 3, 32, 65, 6), (8, 4, 64, 64, 7), (8, 2, 32, 65, 7), (2, 2, 128, 73, 6),
    (2, 1, 128, 64, 7), (4, 1, 128, 93, 10), (4, 2, 128, 128, 7), (2, 1, 256, 32, 7), (3, 3, 136, 171, 0), (4, 1, 136, 114, 8), (4, 2, 4, 65, 15)])
def test_large_batches(heads, kv_heads, hd, B, k):
    from test_gpu_forward import Rig
    V = 33
    shape = wl.ModelShape(1, (heads * hd + 7) // 8 * 8, heads, kv_heads, hd, 16, V, dtype="fp32")
    lens = [(0, 1, 37, 70, 141)[b % 5] for b in range(B)]
    rig = Rig(shape, B, max(lens) + k + 1, max(k, 1), seed=3, std=0.08)
    rng = wl.Rng(B + hd, "cpu")
    for b, n in enumerate(lens):
        rig.caches[b][:, :, :, :n] = rng.normal(20 + b % 5, (1, 2, kv_heads, n, hd), 1.0)
        rig.set_cache(b, n)
    t0, toks = rng.randint(1, (B,), V).tolist(), rng.randint(2, (B, max(k, 1)), V)
    dl, us = rng.normal(3, (B, max(k, 1), V), 1.0), rng.uniform(4, (B, max(k, 1) + 1))
    slots, look = list(range(B)), [k] * B
    got, _, _ = rig.step(slots, t0, look, toks, dl, us, 1.0)
    want = rig.oracle_logits(slots, t0, look, toks)
    assert (got - want).abs().max().item() <= 1e-4          # the bound of the other small fp32 models
    new = [rig.caches[b][:, :, :, n:n + k + 1] for b, n in enumerate(lens)]
    for b in range(0, B, 7):
        x = torch.zeros((1, 2, kv_heads, k + 1, hd), device="cuda")
        rig.sv.spec_kv_export(rig.h, b, lens[b], x)
        assert (x.cpu() - new[b]).abs().max().item() <= 1e-5 * max(1.0, new[b].abs().max().item())
