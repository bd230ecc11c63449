"""The gate/up projection that finishes SwiGLU itself for more than 192 rows (single K range, sums turned around in LDS): every
number of row tiles, ragged rows and columns, to the precision of its operands: a model whose attention adds
nothing, against fp64."""
import pytest
import torch

from paper_2411_00853_amd import workload as wl

pytestmark = pytest.mark.gpu


# (two, three and four column tiles per wavefront; of four the last column block whole and partial)
@pytest.mark.parametrize("d,F,tiles", [(64, 32, 2), (96, 480, 2), (416, 11008, 3), (1056, 8192, 2), (3136, 12544, 4), (512, 12512, 4)])
@pytest.mark.parametrize("rows", [200, 225, 256, 260, 312, 320, 330, 352])
def test_swiglu_by_way_of_lds(d, F, tiles, rows):
    from paper_2411_00853_amd import binding as sv
    from test_gpu_forward import Rig
    V = 131
    B = next(b for b in range(64, 0, -1) if rows % b == 0 and rows // b <= 16)
    k = rows // B - 1
    shape = wl.ModelShape(1, d, 2, 2, 64, F, V, dtype="bf16")
    w = wl.make_weights(shape, d + rows, "cpu", std=0.1)
    w["layers"][0]["w_o"].zero_()
    w["layers"][0]["ffn_norm"] = 1 + wl.Rng(5, "cpu").normal(2, (d,), 0.2)
    rig = Rig(shape, B, 64, k, w_cpu=w)
    plan = sv.spec_k_plan_step(rig.cfg, [k] * B)
    assert plan.gate_up_swiglu_inside == 1 and plan.gemm_k_ranges[2] == 1 and plan.gemm_col_tiles[2] == tiles
    rng = wl.Rng(7, "cpu")
    t0, toks = rng.randint(3, (B,), V), rng.randint(4, (B, k), V)
    got, _, _ = rig.step(list(range(B)), t0.tolist(), [k] * B, toks, torch.zeros((B, k, V)), torch.zeros((B, k + 1)), 1.0)
    l, f64 = w["layers"][0], lambda t: t.double()
    norm = lambda x, g: x / torch.sqrt((x * x).mean(-1, keepdim=True) + shape.rms_eps) * f64(g)
    x = f64(w["tok_embed"])[torch.cat([t0[:, None], toks], 1).reshape(-1).long()]
    gu = norm(x, l["ffn_norm"]) @ f64(l["w_gate_up"]).T
    x = x + (torch.nn.functional.silu(gu[:, :F]) * gu[:, F:]) @ f64(l["w_down"]).T
    want = norm(x, w["final_norm"]) @ f64(w["lm_head"]).T
    # head and remainder carry an activation to 2^-17 of itself; three products one after the other (test_gpu_swiglu_gemm)
    assert ((got.double() - want).norm(dim=1) / want.norm(dim=1)).max().item() < 3 * 2 ** -17
