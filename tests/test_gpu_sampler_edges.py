"""The sampler where its workgroups' shares end: more (row, chunk) pairs of statistics than fit in one go, numbers
of chunk masses around a multiple of eight, trees of every row count up to the largest vocabulary they take."""
import pytest

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("V,lookahead", [
    (300003, [15, 14, 2]),         # 31 rows of 19 statistics chunks
    (8 * 4096, [3, 1, 2, 0]), (8 * 4096 + 1, [3, 1, 2, 0]), (7 * 4096, [2, 3]), (16 * 4096 + 7, [3, 3]),
])
def test_sampler_at_the_edges(V, lookahead):
    from helpers import check_sampler_against_oracle, run_sampler_gpu
    from test_gpu_sampler import _random_inputs
    K = max(lookahead)
    tl, dl, toks, us = _random_inputs(V, lookahead, K, V, 0.4, 1.0)
    na, ot = run_sampler_gpu(tl, dl, toks, us, lookahead, 1.0, K)
    chk = check_sampler_against_oracle(tl, dl, toks, us, lookahead, 1.0, K, na, ot)
    assert chk.exact_accept >= len(lookahead) - 1


@pytest.mark.parametrize("V,K", [(64 * 4096, 15), (4097, 1), (4 * 4096, 4), (5 * 4096 - 3, 4)])
def test_tree_sampler_at_the_edges(V, K):
    from test_gpu_tree import check_trees, make_tree_inputs, run_tree_sampler
    B = 3
    inp = make_tree_inputs(V + K, B, K, V, 1.0, sigma=0.8)
    chk = check_trees(*inp, 1.0, K, *run_tree_sampler(*inp, 1.0, K))
    assert chk.exact_walk >= B - 1
