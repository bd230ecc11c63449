"""The window's own keys and values in the attention: windows that begin in the middle of a 32-position
block, end in the next one, or lie across two chunks; windows of more than eight positions; each number of
wavefronts per workgroup; contiguous caches and page pools; and the separate rotary kernel, with numbers of
rows that are no multiple of its 16.  Cached values are small against the window's, so that a window position
that is lost or taken twice shows.  Vocabulary of 131: the last columns of the partial-sum reduction."""
import pytest
import torch

from paper_2411_00853_amd import workload as wl

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("lens,look", [([120, 380, 1, 31, 500], [15, 15, 9, 8, 0]), ([124, 250], [5, 3])])
@pytest.mark.parametrize("hd,heads,kv_heads,chunks,in_wg,paged", [
    (64, 16, 16, 1, True, False), (64, 16, 16, 2, True, True), (64, 16, 16, 4, True, False), (64, 16, 16, 4, False, False),
    (64, 8, 2, 0, False, False),       # four work items of a head read the same keys
    (64, 32, 8, 4, False, True),       # several row tiles
    (64, 8, 2, 8, False, True),        # short chunks: the separate rotary kernel
    (128, 8, 8, 1, True, True), (128, 8, 8, 2, True, False), (128, 8, 8, 4, True, True), (128, 8, 8, 4, False, False),
    (128, 16, 2, 0, False, True),
    (128, 8, 2, 2, False, False),      # three or four row tiles of 128 dims: the separate rotary kernel
])
def test_windows_across_blocks_and_chunks(hd, heads, kv_heads, chunks, in_wg, paged, lens, look):
    from paper_2411_00853_amd import binding as sv
    from test_gpu_forward import Rig, PagedRig, _check_step
    sv.spec_k_set_attn_max_chunks(chunks)
    if in_wg:
        sv.spec_k_set_attn_merge_min_pairs(1)
    try:
        shape = wl.ModelShape(2, 1024, heads, kv_heads, hd, 256, 131, dtype="bf16")
        B, kmax = len(lens), max(look)
        rig = Rig(shape, B, 1024, kmax, seed=3, std=0.05)
        rng = wl.Rng(17, "cpu")
        for s, n in enumerate(lens):
            rig.caches[s][:, :, :, :n] = rng.normal(20 + s, (2, 2, kv_heads, n, hd), 0.1)
            rig.set_cache(s, n)
        if paged:
            base, rig = rig, PagedRig(rig, B, 1024, kmax, n_pages=sum((n + 2 * kmax + 33) // 32 for n in lens))
            for s in range(B):
                rig.load(base, s)
        for step in range(2):      # the second one reads what the first has stored
            t0 = rng.randint(40 + step, (B,), 131).tolist()
            na = _check_step(rig, list(range(B)), t0, look, 1.0, 50 + step)[2]
            for s in range(B):
                n = rig.n[s]
                rig.n[s] = n + int(na[s]) + 1
                x = torch.zeros((2, 2, kv_heads, int(na[s]) + 1, hd), dtype=torch.bfloat16, device="cuda")
                sv.spec_kv_export(rig.h, s, n, x)
                got, want = x.cpu().float(), rig.caches[s][:, :, :, n:rig.n[s]].float()
                # both sides round to bf16, half a unit of 2^-7 of the value each, what differs before by the
                # error of the layers below (fp32 sums of some thousand terms of order 1: far below 5e-3)
                worst = ((got - want).abs() - 2 ** -7 * want.abs()).max().item()
                assert worst <= 5e-3
    finally:
        sv.spec_k_set_attn_max_chunks(0)
        sv.spec_k_set_attn_merge_min_pairs(0)


@pytest.mark.parametrize("B", [1, 64, 65, 256])
def test_sequences_dealt_out_by_length(B):
    """Ragged lengths with ties and a skipped sequence, at the edges of the prefix sums' wavefronts and with
    more rows than one decoder pass takes: every row against the oracle."""
    from test_gpu_forward import Rig
    shape = wl.ModelShape(1, 128, 2, 2, 64, 256, 131, dtype="bf16")
    rig = Rig(shape, B, 448, 2, seed=3, std=0.05)
    rng = wl.Rng(23, "cpu")
    lens = (rng.randint(1, (B,), 8) * 61 + rng.randint(2, (B,), 2)).tolist()
    look = rng.randint(3, (B,), 3).tolist()
    for s, n in enumerate(lens):
        rig.caches[s][:, :, :, :n] = rng.normal(20 + s, (1, 2, 2, n, 64), 0.3)
        rig.set_cache(s, n)
    t0 = rng.randint(4, (B,), 131).tolist()
    toks = rng.randint(5, (B, 2), 131)
    dl, us = rng.normal(6, (B, 2, 131), 1.0), rng.uniform(7, (B, 3))
    want = rig.oracle_logits(list(range(B)), t0, look, toks)
    skipped = B // 2 if B > 1 else None
    if skipped is not None:
        rig.kv_len[skipped] = 448     # its window would not fit
    rig.sv.spec_verify_step(rig.h, look, us.cuda(), 1.0, torch.zeros(B, dtype=torch.int32, device="cuda"),
                            torch.zeros((B, 3), dtype=torch.int32, device="cuda"),
                            seq_slot=torch.arange(B, dtype=torch.int32, device="cuda"),
                            last_token=torch.tensor(t0, dtype=torch.int32, device="cuda"), draft_tokens=toks.cuda(),
                            draft_logits=dl.cuda(), logits_out=(lo := torch.zeros((sum(look) + B, 131), device="cuda")))
    if skipped is not None:
        with pytest.raises(rig.sv.SpecError):
            rig.sv.spec_verify_poll(rig.h)
    keep = torch.ones(sum(look) + B, dtype=torch.bool)
    if skipped is not None:
        r0 = sum(look[:skipped]) + skipped
        keep[r0:r0 + look[skipped] + 1] = False
    assert (lo.cpu() - want)[keep].abs().max().item() <= 5e-3     # the bound of the other small bf16 models
