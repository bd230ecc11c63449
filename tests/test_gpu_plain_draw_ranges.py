"""Plain draws whose row is shared out among workgroups: from an LM head of several K ranges, and from whole rows (fp32 models); the token
against the running sum of the stored logits in 64 bits, a skipped sequence between others, targets at both ends."""
import pytest
import torch

from paper_2411_00853_amd import workload as wl

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("V,d,dtype,ranges", [(16385, 1024, "bf16", 4), (32771, 512, "bf16", 2), (18432, 512, "bf16", 4), (16385, 64, "fp32", 0),
                                              (32771, 64, "fp32", 0), (131072, 64, "fp32", 0)])
def test_shared_plain_draws(V, d, dtype, ranges):
    from paper_2411_00853_amd import binding as sv
    from test_gpu_forward import Rig
    B = 5
    shape = wl.ModelShape(1, d, 1, 1, 64, 64, V, dtype=dtype)
    rig = Rig(shape, B, 40, 1, w_cpu=wl.make_weights(shape, V, "cpu", std=0.1))
    if ranges: assert sv.spec_k_plan_step(rig.cfg, [0] * B, torch.cuda.get_device_properties(0).multi_processor_count).gemm_k_ranges[4] == ranges
    rng, skipped = wl.Rng(B, "cpu"), 2
    dev = lambda t: t.to(torch.int32).cuda()
    rig.kv_len.copy_(torch.tensor([40 if b == skipped else 0 for b in range(B)]))
    us = rng.uniform(4, (B, 2))
    us[0, 0], us[B - 1, 0] = 0.0, 1 - 2 ** -24
    na, out = torch.zeros(B, dtype=torch.int32, device="cuda"), torch.zeros((B, 2), dtype=torch.int32, device="cuda")
    lo = torch.zeros((B, V), device="cuda")
    last = rng.randint(7, (B,), V)
    sv.spec_verify_step(rig.h, [0] * B, us.cuda(), 1.0, na, out, seq_slot=dev(torch.arange(B)), last_token=dev(last), logits_out=lo)
    torch.cuda.synchronize()
    with pytest.raises(sv.SpecError): sv.spec_verify_poll(rig.h)
    want = rig.om.verify_rows([rig.om.new_cache() for _ in range(B)], [0] * B, [[int(t)] for t in last])
    for b in range(B):
        if b == skipped:
            assert int(na[b]) == -1 and out[b].tolist() == [-1, -1]
            continue
        l64 = lo[b].cpu().double()
        assert (l64 - want[b]).abs().max() <= (1e-4 if dtype == "fp32" else 5e-3) * max(1.0, want[b].abs().max().item())
        p = torch.softmax(l64, 0)
        cdf, y = p.cumsum(0), int(out[b, 0])
        # exponentials in fp32, 2 ulp and the rounding of their argument (2^-24 of some tens), sums in fp64
        assert int(na[b]) == 0 and int(out[b, 1]) == -1 and p[y] > 0
        assert (cdf[y] - p[y]).item() - 1e-5 <= float(us[b, 0]) * cdf[-1].item() <= cdf[y].item() + 1e-5, (b, y)
