"""Draws from a residual without any mass: target and draft rows alike, a proposal that both exclude (0 < 0 keeps nothing).  The token is
then drawn from the target row itself; against its running sum in 64 bits, for a workgroup per sequence, slices of 2048 and of 4096
ids whose last workgroup draws, and two launches, with targets at both ends and on slices in between."""
import pytest
import torch

from paper_2411_00853_amd import workload as wl

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("V,B", [(1500, 4), (16384, 4), (16385, 4), (40001, 5), (65537, 40), (65537, 63), (32768, 80), (300001, 14)])
def test_the_target_row_is_drawn_from(V, B):
    from paper_2411_00853_amd import binding as sv
    rng = wl.Rng(V + B, "cuda")
    tl = rng.normal(1, (2 * B, V), 2.0)
    for b in range(B):                       # whole slices without mass in front, in the middle and at the end
        if b % 4 == 1: tl[2 * b, :V // 3] = -float("inf")
        if b % 4 == 2: tl[2 * b, -V // 3:] = -float("inf")
        if b % 4 == 3: tl[2 * b, V // 4:V // 2] = -float("inf")
    toks = rng.randint(3, (B, 1), V).to(torch.int32)
    tl[torch.arange(0, 2 * B, 2, device="cuda"), toks[:, 0].long()] = -float("inf")
    dl = tl[::2].clone().view(B, 1, V)
    us = rng.uniform(4, (B, 2))
    us[:4, 1] = torch.tensor([0.0, 0.0, 1 - 2 ** -24, 0.5])
    h = sv.spec_verify_init(sv.sampler_cfg(V, B, 1), None, None, None)
    na, out = torch.full((B,), -9, dtype=torch.int32, device="cuda"), torch.full((B, 2), -9, dtype=torch.int32, device="cuda")
    sv.spec_verify_step(h, [1] * B, us, 1.0, na, out, draft_tokens=toks, draft_logits=dl, target_logits_in=tl)
    torch.cuda.synchronize()
    sv.spec_verify_poll(h)
    assert not na.any() and (out[:, 1] == -1).all()
    p = torch.softmax(tl[::2].double(), 1)
    cdf, y = p.cumsum(1), out[:, :1].long()
    at, hi, own = us[:, 1].double(), cdf.gather(1, y)[:, 0], p.gather(1, y)[:, 0]
    # exponentials in fp32, 2 ulp each, sums in fp64: edges move by 3e-7 of the whole
    assert (own > 0).all() and (hi - own - 1e-6 <= at).all() and (at <= hi + 1e-6).all()
    h.close()
