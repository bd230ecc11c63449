"""The arithmetic that every route through the bf16 decoder shares, bit for bit: a row's 1/rms from its sums of squares
(1024 columns meet in fp64, are rounded, and are added up in order) and the rotation of queries and keys.  A
draw follows the logits' last bits wherever its uniform lies next to a step of the distribution, so these may not
depend on which kernel happens to do them."""
import numpy as np
import pytest
import torch

from paper_2411_00853_amd import workload as wl

pytestmark = pytest.mark.gpu


def _inv_rms(x, eps):
    """fp32, the sums as defined above; x holds values whose squares add up exactly in fp64."""
    ss = np.zeros(x.shape[0], np.float32)
    for c in range(0, x.shape[1], 1024):
        ss += (x[:, c:c + 1024].astype(np.float64) ** 2).sum(1).astype(np.float32)
    return np.float32(1) / np.sqrt(ss / np.float32(x.shape[1]) + np.float32(eps))


@pytest.mark.parametrize("d", [64, 1024, 2048, 4096, 4608, 8192])
def test_row_scale_is_the_stated_sum(d):
    from test_gpu_forward import Rig
    V, B = 131, 24
    shape = wl.ModelShape(1, d, 2, 2, 64, 64, V, dtype="bf16")
    w = wl.make_weights(shape, 5, "cpu", std=0.02)
    for l in w["layers"]:      # the layer adds nothing: the residual stream is the embedding
        l["w_o"].zero_()
        l["w_down"].zero_()
    rng = wl.Rng(d, "cpu")
    x = (rng.randint(1, (V, d), 511) - 255) * 2 ** rng.randint(2, (V, d), 5)   # 8 significant bits: exact in bf16
    w["tok_embed"] = x.to(torch.bfloat16)
    w["final_norm"] = torch.ones(d)
    at = torch.arange(V) * 37 % d
    w["lm_head"] = torch.zeros((V, d), dtype=torch.bfloat16)
    w["lm_head"][torch.arange(V), at] = 1.0        # logit v of a row is its column at[v] times 1/rms
    rig = Rig(shape, B, 64, 0, w_cpu=w)
    t0 = rng.randint(3, (B,), V).tolist()
    got, _, _ = rig.step(list(range(B)), t0, [0] * B, torch.zeros((B, 0)), torch.zeros((B, 0, V)), torch.zeros((B, 1)), 1.0)
    rows = x[t0].numpy().astype(np.float32)
    want = rows[:, at.numpy()] * _inv_rms(rows, shape.rms_eps)[:, None]
    assert np.array_equal(got.numpy(), want)


@pytest.mark.parametrize("d,hd,heads,kv_heads", [(2048, 64, 8, 8), (1024, 128, 8, 8), (512, 64, 8, 2), (4608, 64, 2, 2), (5120, 128, 2, 2),
                                                 (8192, 64, 4, 1)])
def test_queries_finished_by_the_attention_or_before_it_are_the_same(d, hd, heads, kv_heads):
    """A cache of 160 positions takes the separate rotary kernel, one of 256 the attention that finishes queries, keys
    and values itself; one chunk of positions in both."""
    from paper_2411_00853_amd import binding as sv
    from test_gpu_forward import Rig
    V, look, lens = 131, [5, 0, 3], [100, 31, 7]
    shape = wl.ModelShape(1, d, heads, kv_heads, hd, 64, V, dtype="bf16")
    rng = wl.Rng(17, "cpu")
    t0, toks = rng.randint(1, (3,), V).tolist(), rng.randint(2, (3, 5), V)
    dl, us = rng.normal(3, (3, 5, V), 1.0), rng.uniform(4, (3, 6))
    outs = []
    sv.spec_k_set_attn_max_chunks(1)
    try:
        for capacity in (160, 256):
            rig = Rig(shape, 3, capacity, 5, seed=9, std=0.05)
            plan = sv.spec_k_plan_step(rig.cfg, look)
            assert plan.attn_fused == (capacity == 256) and plan.attn_chunks == 1
            for s, n in enumerate(lens):
                rig.caches[s][:, :, :, :n] = rng.normal(20 + s, (1, 2, kv_heads, n, hd), 0.5)
                rig.set_cache(s, n)
            got, _, _ = rig.step([0, 1, 2], t0, look, toks, dl, us, 1.0)
            want = rig.oracle_logits([0, 1, 2], t0, look, toks)
            assert (got - want).abs().max().item() <= 5e-3     # the bound of the other small bf16 models
            new = []
            for s, n in enumerate(lens):
                x = torch.zeros((1, 2, kv_heads, look[s] + 1, hd), dtype=torch.bfloat16, device="cuda")
                sv.spec_kv_export(rig.h, s, n, x)
                new.append(x.cpu())
            outs.append((got, new))
    finally:
        sv.spec_k_set_attn_max_chunks(0)
    assert torch.equal(outs[0][0], outs[1][0])
    assert all(torch.equal(a, b) for a, b in zip(outs[0][1], outs[1][1]))
