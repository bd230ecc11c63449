"""Rows embedded beside the row bookkeeping: what makes the bookkeeping skip a sequence -- a token or parent out of range, a slot
that another names or that does not exist, a window that does not fit -- makes every row of it embed token 0 and attend to nothing,
so that all rows of all skipped sequences are the same bits; the others are what they are without skipped ones beside them."""
import pytest
import torch

from paper_2411_00853_amd import workload as wl

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("dtype,hd,B", [("bf16", 64, 9), ("bf16", 128, 21), ("fp32", 32, 9), ("fp32", 64, 40)])
@pytest.mark.parametrize("tree", [False, True])
def test_skipped_sequences_embed_the_first_token(dtype, hd, B, tree):
    from paper_2411_00853_amd import binding as sv
    from test_gpu_forward import Rig
    V, K, cap = 131, 5, 64
    shape = wl.ModelShape(2, 2 * hd * 3, 6, 6, hd, 96, V, dtype=dtype)
    rig = Rig(shape, B, cap, K, seed=11, std=0.05)
    rng = wl.Rng(B, "cpu")
    lens = [3 + b % 20 for b in range(B)]
    t0, toks, look = rng.randint(1, (B,), V), rng.randint(2, (B, K), V), [K - b % 3 for b in range(B)]
    parent = torch.tensor([[i - 1 if b % 2 else (i - 1) // 2 - (i < 1) for i in range(K)] for b in range(B)]).clamp(min=-1)
    slots = list(range(B))
    for b, n in enumerate(lens):
        rig.caches[b][:, :, :, :n] = rng.normal(20 + b, (2, 2, 6, n, hd), 0.5)

    def run(bad):
        for b, n in enumerate(lens): rig.set_cache(b, n)
        t, w, p, s = t0.clone(), toks.clone(), parent.clone(), torch.tensor(slots)
        if bad:
            t[1] = V
            w[2, look[2] - 1] = -1
            s[5] = s[4]                              # the second to name it is skipped
            s[6] = B
            rig.kv_len[7] = cap - look[7]            # one position too many
            if tree: p[8, 1] = 1
        dev = lambda x: x.to(torch.int32).cuda()
        na, out = torch.zeros(B, dtype=torch.int32, device="cuda"), torch.zeros((B, K + 1), dtype=torch.int32, device="cuda")
        lo = torch.zeros((sum(look) + B, V), device="cuda")
        if tree:
            sv.spec_verify_tree_step(rig.h, look, dev(p), dev(w), torch.zeros((B, K + 1, V), device="cuda"), torch.zeros((B, K + 1), device="cuda"),
                                     1.0, na, out, torch.zeros((B, K), dtype=torch.int32, device="cuda"), seq_slot=dev(s), last_token=dev(t), logits_out=lo)
        else:
            sv.spec_verify_step(rig.h, look, torch.zeros((B, K + 1), device="cuda"), 1.0, na, out, seq_slot=dev(s), last_token=dev(t),
                                draft_tokens=dev(w), draft_logits=torch.zeros((B, K, V), device="cuda"), logits_out=lo)
        torch.cuda.synchronize()
        if bad:
            with pytest.raises(sv.SpecError): sv.spec_verify_poll(rig.h)
        else: sv.spec_verify_poll(rig.h)
        return na.cpu().tolist(), lo.cpu()

    na, clean = run(False)
    assert min(na) >= 0
    na, got = run(True)
    skipped = [1, 2, 5, 6, 7] + ([8] if tree else [])
    assert [b for b in range(B) if na[b] < 0] == skipped
    rows = [sum(look[:b]) + b for b in range(B + 1)]
    first = got[rows[1]]
    for b in range(B):
        part = got[rows[b]:rows[b + 1]]
        assert torch.equal(part, first.expand_as(part) if b in skipped else clean[rows[b]:rows[b + 1]])
