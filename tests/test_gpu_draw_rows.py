"""The draws of small and middle vocabularies (a workgroup per sequence holds the rows) at the ends of a wavefront's
share, of a run, of the vocabularies they take, and the target logits as they come from the LM head's partial sums."""
import pytest
import torch

from paper_2411_00853_amd import workload as wl

pytestmark = pytest.mark.gpu

VOCABS = [1, 2, 3, 4, 5, 255, 256, 257, 2047, 2048, 2049, 4095, 4096, 4097, 8192, 8193, 16384, 16385, 32767, 32768, 32769]


@pytest.mark.parametrize("V", VOCABS)
def test_accept_and_draw_at_the_ends_of_a_share(V):
    from helpers import check_sampler_against_oracle, run_sampler_gpu
    from test_gpu_sampler import _random_inputs
    lookahead = [3, 0, 1, 2, 3, 3]
    tl, dl, toks, us = _random_inputs(V, lookahead, 3, V, 0.6, 0.8)
    us[0, :] = 0.0            # the first id with mass
    us[1, :] = 0.99999994     # the last one
    us[2, 1] = 0.99999994
    na, ot = run_sampler_gpu(tl, dl, toks, us, lookahead, 0.8, 3)
    check_sampler_against_oracle(tl, dl, toks, us, lookahead, 0.8, 3, na, ot)
    assert ((ot >= -1) & (ot < V)).all()


@pytest.mark.parametrize("V", VOCABS)
def test_trees_at_the_ends_of_a_share(V):
    from test_gpu_tree import check_trees, make_tree_inputs, run_tree_sampler
    inp = make_tree_inputs(V, 6, 6, V, 0.9, sigma=0.7)
    check_trees(*inp, 0.9, 6, *run_tree_sampler(*inp, 0.9, 6))


def _model(V, dtype, B, Kmax):
    from helpers import device_weights
    from paper_2411_00853_amd import binding as sv
    shape = wl.ModelShape(1, 128, 2, 2, 64, 128, V, dtype=dtype)
    cfg = sv.make_cfg(shape, B, 64, Kmax)
    kv = torch.zeros(sv.spec_kv_cache_bytes(cfg), dtype=torch.uint8, device="cuda")
    kv_len = torch.zeros(B, dtype=torch.int32, device="cuda")
    w = wl.make_weights(shape, 3, "cpu", std=0.2)
    return sv.spec_verify_init(cfg, device_weights(shape, w), kv, kv_len), kv_len


@pytest.mark.parametrize("dtype", ["bf16", "fp32"])
@pytest.mark.parametrize("lookahead", [[0, 0, 0], [3, 0, 2]])
@pytest.mark.parametrize("V", [3, 64, 1003, 2048, 2051, 4100, 16387, 32768, 32772])
def test_step_draws_from_the_logits_it_reports(V, lookahead, dtype):
    # logits: bit for bit those of a greedy step (row sums in a kernel of their own); tokens: the oracle's on those logits
    from helpers import check_sampler_against_oracle
    from paper_2411_00853_amd import binding as sv
    B, Kmax = 3, 3
    h, kv_len = _model(V, dtype, B, Kmax)
    rng = wl.Rng(V, "cpu")
    dl = rng.normal(1, (B, Kmax, V), 1.0)
    toks = wl.pick_tokens(rng, dl, 1.0, 2)
    us = rng.uniform(3, (B, Kmax + 1))
    last = rng.randint(4, (B,), V)
    M = sum(lookahead) + B

    def step(T):
        kv_len.copy_(torch.tensor([5, 9, 2], dtype=torch.int32))
        na = torch.full((B,), -7, dtype=torch.int32, device="cuda")
        ot = torch.full((B, Kmax + 1), -7, dtype=torch.int32, device="cuda")
        lo = torch.full((M, V), 7.0, device="cuda")
        sv.spec_verify_step(h, lookahead, us.cuda(), T, na, ot, seq_slot=torch.arange(B, dtype=torch.int32, device="cuda"),
                            last_token=last.cuda(), draft_tokens=toks.cuda(), draft_logits=dl.cuda(), logits_out=lo)
        torch.cuda.synchronize()
        sv.spec_verify_poll(h)
        return na.cpu(), ot.cpu(), lo.cpu()

    greedy, (na, ot, lo) = step(0.0)[2], step(1.0)
    assert torch.equal(lo, greedy)
    check_sampler_against_oracle(lo, dl, toks, us, lookahead, 1.0, Kmax, na, ot)
    assert kv_len.cpu().tolist() == [n + int(a) + 1 for n, a in zip([5, 9, 2], na)]
    h.close()


@pytest.mark.parametrize("V", [1003, 4100, 32771])
def test_tree_step_reports_the_logits_of_a_greedy_one(V):
    from paper_2411_00853_amd import binding as sv
    B, Kmax = 2, 4
    h, kv_len = _model(V, "bf16", B, Kmax)
    rng = wl.Rng(V + 1, "cpu")
    dl, us, last = rng.normal(1, (B, Kmax + 1, V), 1.0), rng.uniform(3, (B, Kmax + 1)), rng.randint(4, (B,), V)
    toks = rng.randint(5, (B, Kmax), V)
    parent = torch.tensor([[-1, -1, 0, 1]] * B, dtype=torch.int32)

    def step(T):
        kv_len.copy_(torch.tensor([5, 9], dtype=torch.int32))
        na, ot = torch.zeros(B, dtype=torch.int32, device="cuda"), torch.zeros((B, Kmax + 1), dtype=torch.int32, device="cuda")
        path, lo = torch.zeros((B, Kmax), dtype=torch.int32, device="cuda"), torch.zeros((B * (Kmax + 1), V), device="cuda")
        sv.spec_verify_tree_step(h, [Kmax] * B, parent.cuda(), toks.cuda(), dl.cuda(), us.cuda(), T, na, ot, path,
                                 seq_slot=torch.arange(B, dtype=torch.int32, device="cuda"), last_token=last.cuda(), logits_out=lo)
        torch.cuda.synchronize()
        sv.spec_verify_poll(h)
        return lo.cpu()

    assert torch.equal(step(0.0), step(1.0))
    h.close()
