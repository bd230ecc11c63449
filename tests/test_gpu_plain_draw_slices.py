"""Plain draws (no proposals) whose row is shared out among workgroups, from the LM head's partial sums: vocabularies around the two
lines of that route, around whole slices and with a last slice of a few ids; the token against the running sum of the stored
logits in 64 bits, two steps in a row, a skipped sequence between others, targets at the first and the last id."""
import pytest
import torch

from paper_2411_00853_amd import workload as wl

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("V,B", [(16384, 3), (16385, 5), (18432, 20), (32000, 9), (32771, 3), (131072, 2), (131073, 2)])
@pytest.mark.parametrize("temperature", [1.0, 0.05])
def test_shared_plain_draws(V, B, temperature):
    from paper_2411_00853_amd import binding as sv
    from test_gpu_forward import Rig
    shape = wl.ModelShape(1, 64, 1, 1, 64, 64, V, dtype="bf16")
    w = wl.make_weights(shape, V, "cpu", std=0.1)
    rig = Rig(shape, B, 40, 1, w_cpu=w)
    rng = wl.Rng(B, "cpu")
    dev = lambda t: t.to(torch.int32).cuda()
    skipped = B // 2
    for call in range(2):
        rig.kv_len.copy_(torch.tensor([40 if b == skipped else 0 for b in range(B)]))
        us = rng.uniform(4 + call, (B, 2))
        us[0, 0], us[B - 1, 0] = 0.0, 1 - 2 ** -24
        na, out = torch.zeros(B, dtype=torch.int32, device="cuda"), torch.zeros((B, 2), dtype=torch.int32, device="cuda")
        lo = torch.zeros((B, V), device="cuda")
        sv.spec_verify_step(rig.h, [0] * B, us.cuda(), temperature, na, out, seq_slot=dev(torch.arange(B)),
                            last_token=dev(rng.randint(7 + call, (B,), V)), logits_out=lo)
        torch.cuda.synchronize()
        with pytest.raises(sv.SpecError): sv.spec_verify_poll(rig.h)
        for b in range(B):
            if b == skipped:
                assert int(na[b]) == -1 and out[b].tolist() == [-1, -1]
                continue
            assert int(na[b]) == 0 and int(out[b, 1]) == -1
            l64 = lo[b].cpu().double()
            p = torch.exp((l64 - l64.max()) / temperature)
            p /= p.sum()
            cdf, y = p.cumsum(0), int(out[b, 0])
            at = float(us[b, 0]) * cdf[-1].item()
            # exponentials in fp32, 2 ulp and the rounding of their argument (up to 2^-24 of 40 or so at T = 0.05), sums in fp64
            assert p[y] > 0 and (cdf[y] - p[y]).item() - 1e-5 <= at <= cdf[y].item() + 1e-5, (b, y)
