"""Draws of large batches: on both sides of the lines between a workgroup per sequence, slices whose last workgroup draws, and two
launches (the launcher's rule: slices of 2048 ids in all, and whether any sequence has proposals), every sequence's token against
the running sum of its masses in 64 bits."""
import pytest
import torch

from paper_2411_00853_amd import workload as wl
from test_gpu_draw_slices import test_shared_draws as shared_draws

pytestmark = pytest.mark.gpu

# slices of 2048 in all: 1278, 1287, 1280, 2040, 2060, 1920, 2048, 2079, 1911, 2058
@pytest.mark.parametrize("V,B", [(16385, 142), (16385, 143), (32768, 80), (40000, 102), (40000, 103), (262144, 15), (262144, 16), (65537, 63),
                                 (300001, 13), (300001, 14)])
def test_large_batches(V, B):
    shared_draws(V, B)


@pytest.mark.parametrize("V,B", [(16385, 113), (16385, 114), (32768, 64), (40001, 102), (40001, 103), (65537, 256)])
@pytest.mark.parametrize("noalloc", [False, True])
def test_no_proposals(V, B, noalloc):
    from paper_2411_00853_amd import binding as sv
    if noalloc: B = min(B, 64)
    rng = wl.Rng(V + B, "cuda")
    tl, us = rng.normal(1, (B, V), 2.0), rng.uniform(2, (B, 1))
    us[0], us[1], tl[2, 4096:12288] = 0.0, 1 - 2 ** -24, -float("inf")
    na, out = torch.full((B,), -9, dtype=torch.int32, device="cuda"), torch.full((B, 1), -9, dtype=torch.int32, device="cuda")
    if noalloc:
        sv.spec_sample_step_noalloc(V, 0, [0] * B, us, 1.0, na, out, tl)
    else:
        h = sv.spec_verify_init(sv.sampler_cfg(V, B, 0), None, None, None)
        sv.spec_verify_step(h, [0] * B, us, 1.0, na, out, target_logits_in=tl)
    torch.cuda.synchronize()
    assert not na.any()
    p = torch.softmax(tl.double(), 1)
    cdf, y = p.cumsum(1), out.long()
    at, hi, own = us[:, 0].double() * cdf[:, -1], cdf.gather(1, y)[:, 0], p.gather(1, y)[:, 0]
    # exponentials in fp32, 2 ulp each, sums in fp64: edges move by 3e-7 of the whole
    assert (own > 0).all() and (hi - own - 1e-6 <= at).all() and (at <= hi + 1e-6).all()
    if not noalloc: h.close()


@pytest.mark.parametrize("B", [31, 32])
def test_proposals_from_large_vocabularies(B):
    """The draft's draws of a decoding round beyond the plain draw's longest row, counted (2015 slices) and as two launches (2080)."""
    from test_gpu_decode import Pair
    V, K = 131073, 2
    shape = wl.ModelShape(1, 64, 1, 1, 64, 64, V, dtype="bf16")
    rng = wl.Rng(B, "cpu")
    pair = Pair(shape, shape, [rng.randint(b, (3 + b % 3,), V).tolist() for b in range(B)], 40, K, 20, std=0.1)
    du, vu = rng.uniform(100, (B, K)), rng.uniform(101, (B, K + 1))
    du[0, 0], du[1, 1] = 0.0, 1 - 2 ** -24
    g = pair.round(K, du, vu, 1.0)
    p = torch.softmax(g["draft_logits"].double(), 2)
    cdf, y = p.cumsum(2), g["draft_tokens"].long().unsqueeze(2)
    at, hi, own = du.double() * cdf[:, :, -1], cdf.gather(2, y)[:, :, 0], p.gather(2, y)[:, :, 0]
    # exponentials in fp32, 2 ulp each, sums in fp64: edges move by 3e-7 of the whole
    assert (own > 0).all() and (hi - own - 1e-6 <= at).all() and (at <= hi + 1e-6).all()
    assert (g["n_accepted"] >= 0).all()
