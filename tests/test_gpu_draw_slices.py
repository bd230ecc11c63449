"""Draws whose row is shared out among workgroups: the token of every sequence against the running sum of its masses in 64 bits, at
vocabularies around the line to the single workgroup and around whole slices, with the slice of 2048 ids and that of 4096,
targets at the first and the last id with mass and on slices without any; two calls in a row (the count of finished slices is
back at zero) and a skipped sequence between others."""
import pytest
import torch

from paper_2411_00853_amd import workload as wl

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("V,B", [(16385, 5), (18432, 3), (20481, 64), (32768, 9), (65536, 40), (65537, 7), (128256, 20), (262144, 2), (300001, 3)])
def test_shared_draws(V, B):
    from paper_2411_00853_amd import binding as sv
    K = 3
    h = sv.spec_verify_init(sv.sampler_cfg(V, B, K), None, None, None)
    rng = wl.Rng(V + B, "cuda")
    look = [b % (K + 1) for b in range(B)]
    M = sum(look) + B
    tl, dl = rng.normal(1, (M, V), 2.0), rng.normal(2, (B, K, V), 2.0)
    row0 = [sum(look[:b]) + b for b in range(B)]
    for b in range(B):                       # whole slices without mass in front, in the middle and at the end
        rows = tl[row0[b]:row0[b] + look[b] + 1]
        if b % 4 == 1: rows[:, :9000] = -float("inf")
        if b % 4 == 2: rows[:, -9000:] = -float("inf")
        if b % 4 == 3: rows[:, 4096:12288] = -float("inf")
    toks = rng.randint(3, (B, K), V).to(torch.int32)
    skipped = B // 2
    look_ok = look[skipped] > 0
    if look_ok: toks[skipped, 0] = V
    na, out = torch.zeros(B, dtype=torch.int32, device="cuda"), torch.zeros((B, K + 1), dtype=torch.int32, device="cuda")
    for call in range(2):
        us = rng.uniform(4 + call, (B, K + 1))
        us[0, look[0]], us[1, look[1]] = 0.0, 1 - 2 ** -24
        sv.spec_verify_step(h, look, us, 1.0, na, out, draft_tokens=toks, draft_logits=dl, target_logits_in=tl)
        torch.cuda.synchronize()
        if look_ok:
            with pytest.raises(sv.SpecError): sv.spec_verify_poll(h)
        for b in range(B):
            if b == skipped and look_ok:
                assert int(na[b]) == -1 and out[b].tolist() == [-1] * (K + 1)
                continue
            a, K_b = int(na[b]), look[b]
            assert 0 <= a <= K_b
            p = torch.softmax(tl[row0[b] + a].double(), 0)
            q = torch.softmax(dl[b, a].double(), 0) if a < K_b else torch.zeros_like(p)
            for i in range(K_b):             # which proposals are kept
                x = int(toks[b, i])
                ratio = (torch.softmax(tl[row0[b] + i].double(), 0)[x] / torch.softmax(dl[b, i].double(), 0)[x]).item()
                u = float(us[b, i])
                assert i > a or abs(u - min(ratio, 1.0)) < 1e-3 or (u < ratio) == (i < a), (b, i)
            r = (p - q).clamp(min=0)
            cdf = r.cumsum(0)
            y, at = int(out[b, a]), float(us[b, K_b]) * cdf[-1].item()
            lo, hi = (cdf[y] - r[y]).item(), cdf[y].item()
            # exponentials in fp32, 2 ulp each, sums in fp64: edges move by 3e-7 of the whole
            assert r[y] > 0 and lo - 1e-6 <= at <= hi + 1e-6, (b, y, lo, at, hi)
    h.close()
