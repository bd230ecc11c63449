"""Where the attention's plan changes between longer chunks without a kernel in front and the general one: query rows per item (12 and 13
of 128-dim heads, 8 and 9 beyond 1024 positions, 32 and 33 of 64-dim heads, 16 and 18 where items share a head) and 128-dim pairs for
four wavefronts per compute unit.  The plan on both sides, and the logits of both sides against the oracle, contiguous and on a page
pool."""
import pytest
import torch

from paper_2411_00853_amd import binding as sv
from paper_2411_00853_amd import workload as wl

# head_dim, query heads, kv heads, capacity, sequences, lookahead; inside the rule
LINES = [(128, 2, 2, 300, 3, 11, 1), (128, 2, 2, 300, 3, 12, 0), (128, 2, 2, 1500, 3, 7, 1), (128, 2, 2, 1500, 3, 8, 0),
         (64, 32, 8, 300, 5, 7, 1), (64, 33, 11, 300, 3, 10, 0), (64, 16, 2, 300, 9, 7, 1), (64, 16, 2, 300, 9, 8, 0),
         (128, 32, 32, 64, 32, 0, 1), (128, 32, 32, 64, 33, 0, 0)]
V, D = 131, 256


def model(hd, heads, kv_heads):
    return wl.ModelShape(1, D, heads, kv_heads, hd, 64, V, dtype="bf16")


@pytest.mark.parametrize("hd,heads,kv_heads,capacity,B,k,inside", LINES)
@pytest.mark.parametrize("paged", [False, True])
def test_plan(hd, heads, kv_heads, capacity, B, k, inside, paged):
    plan = sv.spec_k_plan_step(sv.make_cfg(model(hd, heads, kv_heads), B, capacity, max(k, 1)), [k] * B, 256, paged)
    assert plan.attn_fused == inside and (plan.attn_chunk_keys >= 192) == bool(inside)


@pytest.mark.gpu
@pytest.mark.parametrize("hd,heads,kv_heads,capacity,B,k,inside", LINES)
def test_logits(hd, heads, kv_heads, capacity, B, k, inside):
    from test_gpu_forward import PagedRig, Rig
    shape, K = model(hd, heads, kv_heads), max(k, 1)
    look = [k] + [k - b % 2 if k else 0 for b in range(1, B)]
    lens = [max(1, (capacity - k - 1) * (b + 1) // B) for b in range(B)]
    rng = wl.Rng(capacity + hd + k, "cpu")
    t0, toks = rng.randint(1, (B,), V).tolist(), rng.randint(2, (B, K), V)
    dl, us = rng.normal(3, (B, K, V), 1.0), rng.uniform(4, (B, K + 1))
    rig = Rig(shape, B, capacity, K, seed=9, std=0.05)
    for s, n in enumerate(lens):
        rig.caches[s][:, :, :, :n] = rng.normal(20 + s, (1, 2, kv_heads, n, hd), 0.5)
        rig.set_cache(s, n)
    paged = PagedRig(rig, B, capacity, K, sum(n // 32 + 2 for n in lens))
    for s in range(B): paged.load(rig, s)
    slots = list(range(B))
    got = [r.step(slots, t0, look, toks, dl, us, 1.0)[0] for r in (rig, paged)]
    want = rig.oracle_logits(slots, t0, look, toks)
    assert (got[0] - want).abs().max().item() <= 5e-3     # the bound of the other small bf16 models
    assert torch.equal(got[0], got[1])
