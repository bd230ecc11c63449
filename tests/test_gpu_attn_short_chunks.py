"""Short caches whose plan takes fewer, longer chunks, so that the attention puts queries, keys and values together itself, merged
in the workgroup where a slot is short enough: the
logits against the oracle, the window's cache entries bit for bit those of the separate rotary/append kernel (which the plan of
many short chunks, forced by the chunk knob, runs)."""
import pytest
import torch

from paper_2411_00853_amd import workload as wl

pytestmark = pytest.mark.gpu


# capacities at the ends of what the rules cover: one block, 191 and 193 positions, two chunks, four in a workgroup, more than
# eight short ones
@pytest.mark.parametrize("hd,heads,kv_heads,capacity,B,k,small", [
    (64, 4, 4, 40, 3, 5, 0), (64, 4, 4, 193, 3, 5, 0), (64, 24, 24, 900, 3, 2, 0), (64, 8, 2, 191, 2, 6, 1), (64, 8, 2, 700, 2, 6, 1),
    (128, 2, 2, 384, 3, 0, 0), (128, 2, 2, 1025, 3, 7, 0), (128, 2, 1, 2400, 2, 3, 0), (128, 8, 8, 200, 12, 3, 0),
    (64, 4, 4, 1024, 1, 6, 0), (64, 4, 4, 1060, 1, 6, 0), (128, 2, 2, 512, 3, 11, 0), (128, 4, 4, 500, 3, 11, 0)])
def test_longer_chunks_and_no_kernel_in_front(hd, heads, kv_heads, capacity, B, k, small):
    from paper_2411_00853_amd import binding as sv
    from test_gpu_forward import Rig
    V, d = 131, 256
    look = [k - b % 2 if k else 0 for b in range(B)]
    lens = [max(1, (capacity - k - 1) * (b + 1) // B) for b in range(B)]
    shape = wl.ModelShape(1, d, heads, kv_heads, hd, 64, V, dtype="bf16")
    rng = wl.Rng(capacity + hd, "cpu")
    t0, toks = rng.randint(1, (B,), V).tolist(), rng.randint(2, (B, max(k, 1)), V)
    dl, us = rng.normal(3, (B, max(k, 1), V), 1.0), rng.uniform(4, (B, max(k, 1) + 1))
    new = []
    for knob in (0, 16):
        sv.spec_k_set_attn_max_chunks(knob)
        try:
            rig = Rig(shape, B, capacity, max(k, 1), seed=9, std=0.05)
            plan = sv.spec_k_plan_step(rig.cfg, look)
            assert plan.attn_fused == (knob == 0)
            assert knob or plan.attn_small == small
            for s, n in enumerate(lens):
                rig.caches[s][:, :, :, :n] = rng.normal(20 + s, (1, 2, kv_heads, n, hd), 0.5)
                rig.set_cache(s, n)
            got, _, _ = rig.step(list(range(B)), t0, look, toks, dl, us, 1.0)
            want = rig.oracle_logits(list(range(B)), t0, look, toks)
            assert (got - want).abs().max().item() <= 5e-3     # the bound of the other small bf16 models
            rows = []
            for s, n in enumerate(lens):
                x = torch.zeros((1, 2, kv_heads, look[s] + 1, hd), dtype=torch.bfloat16, device="cuda")
                sv.spec_kv_export(rig.h, s, n, x)
                rows.append(x.cpu())
            new.append(rows)
        finally:
            sv.spec_k_set_attn_max_chunks(0)
    assert all(torch.equal(a, b) for a, b in zip(*new))
