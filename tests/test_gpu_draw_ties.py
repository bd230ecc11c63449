"""Draws whose target falls between two halves of a row that weigh the same, with excluded ids (-inf) between them: rounding may
put the target on either side, and neither an id without mass nor one further away is ever drawn."""
import pytest
import torch

from paper_2411_00853_amd import workload as wl

pytestmark = pytest.mark.gpu


def _rows(B, V, gap):
    """B rows of a few finite logits, the same again V/2 + gap ids on; the ids that may be drawn with u = 0.5"""
    rng = wl.Rng(V + gap, "cpu")
    span = V // 2 - gap
    n = min(9, span)
    rows = torch.full((B, V), float("-inf"))
    ends = []
    for b in range(B):
        ids = torch.sort(torch.randperm(span, generator=torch.Generator().manual_seed(1000 * V + b))[:n]).values
        x = rng.normal(b, (n,), 2.0)
        rows[b, ids], rows[b, V // 2 + gap + ids] = x, x
        ends.append((int(ids[-1]), int(ids[0]) + V // 2 + gap))
    return rows, ends


@pytest.mark.parametrize("tree", [False, True])
@pytest.mark.parametrize("V,gap", [(64, 8), (256, 40), (2048, 300), (4096, 1), (8192, 700), (32768, 5000), (32770, 5000), (50257, 3), (151936, 9000)])
def test_excluded_ids_between_two_halves(V, gap, tree):
    from helpers import run_sampler_gpu
    from test_gpu_tree import run_tree_sampler
    B = 64
    rows, ends = _rows(B, V, gap)
    us, toks = torch.full((B, 2), 0.5), torch.zeros((B, 1), dtype=torch.int32)
    if tree:
        na, ot, _ = run_tree_sampler([0] * B, torch.full((B, 1), -1, dtype=torch.int32), toks, rows, torch.zeros((B, 2, V)), us, 1.0, 1)
    else:
        na, ot = run_sampler_gpu(rows, torch.zeros((B, 1, V)), toks, us, [0] * B, 1.0, 1)
    assert na.tolist() == [0] * B
    wrong = [(b, t, ends[b]) for b, t in enumerate(ot[:, 0].tolist()) if t not in ends[b]]
    assert not wrong, wrong
