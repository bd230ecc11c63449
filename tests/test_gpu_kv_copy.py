"""spec_kv_import / spec_kv_export: the block-wise kernels (16-byte aligned tensors) against the
element-wise ones (the same call with the tensor two bytes further on)."""
import pytest
import torch

from paper_2411_00853_amd import workload as wl

pytestmark = pytest.mark.gpu


def _handle(sv, head_dim, paged, slots=2, max_kv_len=200):
    shape = wl.ModelShape(3, 2 * head_dim, 2, 2 if head_dim == 128 else 1, head_dim, 64, 64)
    cfg = sv.make_cfg(shape, slots, max_kv_len, 1)
    w = wl.make_weights(shape, 3, "cuda")
    weights = {"tok_embed": w["tok_embed"], "final_norm": w["final_norm"], "lm_head": sv.spec_pack_weight(w["lm_head"]),
               "layers": [{n: (t if "norm" in n else sv.spec_pack_weight(t, n == "w_gate_up")) for n, t in l.items()}
                          for l in w["layers"]]}
    size = sv.spec_kv_page_bytes(cfg) * (slots * 8 + 1) if paged else sv.spec_kv_cache_bytes(cfg)
    kv = torch.zeros(size, dtype=torch.uint8, device="cuda")
    kv_len = torch.zeros(slots, dtype=torch.int32, device="cuda")
    h = (sv.spec_verify_init_paged if paged else sv.spec_verify_init)(cfg, weights, kv, kv_len)
    return h, shape


def _tensor(shape, n, odd, seed=None):
    """[layer][k|v][head][n][dim], at an address that is a multiple of 16 or two bytes beyond one."""
    size = (shape.n_layers, 2, shape.n_kv_heads, n, shape.head_dim)
    count = torch.Size(size).numel()
    flat = torch.zeros(count + 8, dtype=torch.bfloat16, device="cuda")
    t = flat[1:1 + count] if odd else flat[:count]
    assert (t.data_ptr() % 16 != 0) == odd
    if seed is not None:
        t.copy_(wl.Rng(seed, "cuda").normal(1, (count,), 1.0, torch.bfloat16))
    return t.view(size)


@pytest.mark.parametrize("head_dim", [64, 128])
@pytest.mark.parametrize("paged", [False, True])
@pytest.mark.parametrize("pos0,n", [(0, 200), (0, 1), (31, 2), (32, 32), (5, 27), (40, 100), (199, 1), (33, 63)])
def test_block_copies_match_element_copies(head_dim, paged, pos0, n):
    from paper_2411_00853_amd import binding as sv
    h, shape = _handle(sv, head_dim, paged)
    before = _tensor(shape, 200, True, 7)
    for slot in (0, 1):
        sv.spec_kv_import(h, slot, 0, before)                       # element by element
    src = _tensor(shape, n, False, 8)
    sv.spec_kv_import(h, 1, pos0, src)
    want = before.clone()
    want[:, :, :, pos0:pos0 + n] = src
    for slot, ref in ((0, before), (1, want)):
        whole = _tensor(shape, 200, True)
        sv.spec_kv_export(h, slot, 0, whole)                        # element by element
        assert torch.equal(whole, ref), slot
    part = _tensor(shape, n, False)
    sv.spec_kv_export(h, 1, pos0, part)
    assert torch.equal(part, src)
    h.close()
