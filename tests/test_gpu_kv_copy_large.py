"""Cache copies beyond the size from which they store past the caches, against the element-wise copy: ragged positions, whole
blocks and parts of them, contiguous and paged."""
import pytest
import torch

from paper_2411_00853_amd import workload as wl

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("head_dim,paged", [(128, False), (128, True), (64, False)])
def test_streamed_copies_match_element_copies(head_dim, paged):
    from paper_2411_00853_amd import binding as sv
    layers, heads, n, pos0 = 32, 4096 // head_dim, 790, 13
    shape = wl.ModelShape(layers, 64, heads, heads, head_dim, 64, 64)
    cfg = sv.make_cfg(shape, 1, 832, 1)
    one = wl.make_weights(wl.ModelShape(1, 64, heads, heads, head_dim, 64, 64), 3, "cuda")
    layer = {k: (t if "norm" in k else sv.spec_pack_weight(t, k == "w_gate_up")) for k, t in one["layers"][0].items()}
    weights = {"tok_embed": one["tok_embed"], "final_norm": one["final_norm"], "lm_head": sv.spec_pack_weight(one["lm_head"]), "layers": [layer] * layers}
    size = sv.spec_kv_page_bytes(cfg) * 27 if paged else sv.spec_kv_cache_bytes(cfg)
    kv, kv_len = torch.zeros(size, dtype=torch.uint8, device="cuda"), torch.zeros(1, dtype=torch.int32, device="cuda")
    h = (sv.spec_verify_init_paged if paged else sv.spec_verify_init)(cfg, weights, kv, kv_len)
    dims = (layers, 2, heads, n, head_dim)
    count = torch.Size(dims).numel()
    assert 2 * count >= 384 << 20
    src = wl.Rng(4, "cuda").normal(1, (count,), 1.0, torch.bfloat16).view(dims)
    odd = torch.zeros(count + 8, dtype=torch.bfloat16, device="cuda")[1:1 + count].view(dims)   # two bytes beyond a multiple of 16
    dst = torch.zeros(dims, dtype=torch.bfloat16, device="cuda")
    sv.spec_kv_import(h, 0, pos0, src)
    sv.spec_kv_export(h, 0, pos0, odd)
    assert torch.equal(odd, src)
    sv.spec_kv_export(h, 0, pos0, dst)
    assert torch.equal(dst, src)
    head = torch.zeros((layers, 2, heads, pos0, head_dim), dtype=torch.bfloat16, device="cuda")
    sv.spec_kv_export(h, 0, 0, head)
    assert not head.any()
    h.close()
