"""The fp32 product with what it takes over from its neighbours (norm of its input, residual addition,
SwiGLU) and the fp32 attention, through verify steps on small models whose sizes are not multiples of the
kernels' tiles, against the oracle."""
import pytest
import torch

import oracle
from paper_2411_00853_amd import workload as wl

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("M,N,K", [(1, 1, 1), (5, 17, 31), (16, 16, 32), (17, 50, 33), (33, 40, 1056), (70, 100, 129),
                                   (3, 9, 3000), (64, 5, 260)])
def test_products_at_the_edges_of_the_tiles(M, N, K):
    from paper_2411_00853_amd import binding as sv
    rng = wl.Rng(M + N + K, "cpu")
    x, w = rng.normal(1, (M, K), 1.0), rng.normal(2, (N, K), 0.05)
    y = sv.spec_k_gemm_f32(x.cuda(), w.cuda()).cpu()
    want = x.double() @ w.double().T
    # K products of fp32 rounding 2^-24 each, summed pairwise or in runs: sqrt(K) ulps of the largest partial sum
    assert (y.double() - want).abs().max().item() < 2e-7 * (K ** 0.5) * (0.05 * K ** 0.5 + want.abs().max().item())


@pytest.mark.parametrize("heads,kv_heads,head_dim,d_ffn,vocab,lens,look", [
    (4, 4, 64, 1024, 1024, [128], [4]),             # the fp32 configuration
    (3, 1, 24, 40, 77, [1, 65, 300], [3, 0, 7]),    # nothing a multiple of 16 or 32
    (2, 2, 50, 72, 130, [33], [2]),                 # head_dim not a multiple of 4
    (1, 1, 136, 24, 50, [257, 7], [5, 5]),          # more than 32 lanes per position
    (4, 2, 8, 16, 33, [20] * 9, [7] * 9),           # 72 rows: several row tiles
    (2, 2, 4, 16, 33, [70], [3]),                   # one lane per position; then four, thirty-two, and all of a wavefront
    (2, 1, 16, 16, 33, [5, 300], [3, 1]),
    (2, 2, 128, 16, 33, [33, 140], [0, 4]),
    (1, 1, 256, 16, 33, [70], [2]),
])
def test_fp32_steps_match_the_oracle(heads, kv_heads, head_dim, d_ffn, vocab, lens, look):
    from paper_2411_00853_amd import binding as sv
    d = (heads * head_dim + 7) // 8 * 8
    shape = wl.ModelShape(2, d, heads, kv_heads, head_dim, d_ffn, vocab, dtype="fp32")
    B, Kmax = len(lens), max(look)
    max_kv = max(lens) + Kmax + 1
    w = wl.make_weights(shape, 21, "cpu", std=0.08)
    for l in w["layers"]:
        l["attn_norm"] = 1 + wl.Rng(5, "cpu").normal(1, (d,), 0.2)
        l["ffn_norm"] = 1 + wl.Rng(5, "cpu").normal(2, (d,), 0.2)
    om = oracle.Model(shape, w, max_kv)
    cfg = sv.make_cfg(shape, B, max_kv, Kmax)
    dev = lambda t: t.cuda()
    weights = {k: (v.cuda() if k != "layers" else [{n: dev(t) for n, t in l.items()} for l in v]) for k, v in w.items()}
    kv = torch.zeros(sv.spec_kv_cache_bytes(cfg), dtype=torch.uint8, device="cuda")
    kv_len = torch.tensor(lens, dtype=torch.int32, device="cuda")
    h = sv.spec_verify_init(cfg, weights, kv, kv_len)
    rng = wl.Rng(31, "cpu")
    caches = []
    for b, n in enumerate(lens):
        c = om.new_cache()
        c[:, :, :, :n] = rng.normal(10 + b, (2, 2, kv_heads, n, head_dim), 1.0)
        caches.append(c)
        sv.spec_kv_import(h, b, 0, c[:, :, :, :n].contiguous().cuda())
    t0, toks = rng.randint(5, (B,), vocab), rng.randint(6, (B, max(Kmax, 1)), vocab)
    dl, us = rng.normal(7, (B, max(Kmax, 1), vocab), 1.0), rng.uniform(8, (B, Kmax + 1))
    na = torch.zeros(B, dtype=torch.int32, device="cuda")
    ot = torch.zeros((B, Kmax + 1), dtype=torch.int32, device="cuda")
    lo = torch.zeros((sum(look) + B, vocab), device="cuda")
    sv.spec_verify_step(h, look, us.cuda(), 1.0, na, ot, seq_slot=torch.arange(B, dtype=torch.int32, device="cuda"),
                        last_token=t0.cuda(), draft_tokens=toks.cuda(), draft_logits=dl.cuda(), logits_out=lo)
    torch.cuda.synchronize()
    sv.spec_verify_poll(h)
    windows = [[int(t0[b])] + toks[b, :look[b]].tolist() for b in range(B)]
    want = om.verify_rows(caches, lens, windows)
    assert (lo.cpu() - want).abs().max().item() <= 1e-4
    h.close()
