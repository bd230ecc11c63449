"""The gate/up projection that finishes SwiGLU itself, at every ending of its K loop (one, two, three and more chunks,
whole and partial), every row-tile count and number of wavefronts, to the precision of its operands: a model whose
attention adds nothing, against fp64."""
import pytest
import torch

from paper_2411_00853_amd import workload as wl

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("d", [64, 256, 384, 512, 1056])
@pytest.mark.parametrize("rows", [1, 5, 16, 17, 48, 64])
def test_swiglu_inside_the_product_keeps_the_precision_of_its_operands(d, rows):
    from paper_2411_00853_amd import binding as sv
    from test_gpu_forward import Rig
    F, V = 224, 131     # 14 pairs of column tiles: no multiple of 3 or 4 wavefronts
    shape = wl.ModelShape(1, d, 2, 2, 64, F, V, dtype="bf16")
    w = wl.make_weights(shape, d + rows, "cpu", std=0.1)
    w["layers"][0]["w_o"].zero_()
    w["layers"][0]["ffn_norm"] = 1 + wl.Rng(5, "cpu").normal(2, (d,), 0.2)
    sv.spec_k_set_swiglu_min_wgs(1)
    try:
        rig = Rig(shape, rows, 64, 0, w_cpu=w)
        assert sv.spec_k_plan_step(rig.cfg, [0] * rows).gate_up_swiglu_inside == 1
        t0 = wl.Rng(7, "cpu").randint(3, (rows,), V).tolist()
        l, f64 = w["layers"][0], lambda t: t.double()
        norm = lambda x, g: x / torch.sqrt((x * x).mean(-1, keepdim=True) + shape.rms_eps) * f64(g)
        x = f64(w["tok_embed"])[t0]
        gu = norm(x, l["ffn_norm"]) @ f64(l["w_gate_up"]).T
        x = x + (torch.nn.functional.silu(gu[:, :F]) * gu[:, F:]) @ f64(l["w_down"]).T
        want = norm(x, w["final_norm"]) @ f64(w["lm_head"]).T
        for groups in (2, 3, 4):
            sv.spec_k_set_swiglu_column_groups(groups)
            got, _, _ = rig.step(list(range(rows)), t0, [0] * rows, torch.zeros((rows, 0)), torch.zeros((rows, 0, V)),
                                 torch.zeros((rows, 1)), 1.0)
            # head and remainder carry an activation to 2^-17 of itself; three products one after the other
            off = ((got.double() - want).norm(dim=1) / want.norm(dim=1)).max().item()
            assert off < 3 * 2 ** -17, groups
    finally:
        sv.spec_k_set_swiglu_column_groups(0)
        sv.spec_k_set_swiglu_min_wgs(0)
