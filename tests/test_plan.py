"""Host-side planning of a step (spec_k_plan_step: decoder passes, projection launch shapes, attention
plan), checked without a GPU: invariants over a sweep of shapes, batches and lookaheads -- everything a
launch writes fits what spec_verify_init would have allocated, every variant exists, every limit of the
kernels is respected -- and the plans of the named configurations."""
import random

import pytest

from paper_2411_00853_amd import binding as sv
from paper_2411_00853_amd import workload as wl


def _plan(shape, look, max_batch=None, max_kv_len=2048, kmax=None, cu=256, paged=False):
    cfg = sv.make_cfg(shape, max_batch or len(look), max_kv_len, max(look) if kmax is None else kmax)
    return cfg, sv.spec_k_plan_step(cfg, look, cu, paged)


def _check_invariants(shape, cfg, look, p, paged, cu):
    B, rows = len(look), sum(k + 1 for k in look)
    # passes: consecutive sequences, all rows, none beyond what one launch of the projections takes
    assert p.rows == rows and 1 <= p.n_passes <= sv.PLAN_MAX_PASSES
    assert (p.n_passes == 1) == (rows <= 352)
    b0 = 0
    for g in range(p.n_passes):
        n = p.pass_seqs[g]
        assert n >= 1 and p.pass_rows[g] == sum(k + 1 for k in look[b0:b0 + n]) <= 352
        b0 += n
    assert b0 == B
    # as few passes as filling each to the brim would take, and no pass much above the mean
    fewest, acc = 1, 0
    for k in look:
        if acc + k + 1 > 352:
            fewest, acc = fewest + 1, 0
        acc += k + 1
    assert p.n_passes == fewest
    assert max(p.pass_rows[:p.n_passes]) <= -(-rows // p.n_passes) + 15
    # projections of the first pass
    dq = shape.n_q_heads * shape.head_dim
    n_in = [shape.d_model, dq, shape.d_model, shape.d_ffn, shape.d_model]
    n_out = [dq + 2 * shape.n_kv_heads * shape.head_dim, shape.d_model, 2 * shape.d_ffn, shape.d_model, shape.vocab]
    for i in range(sv.PLAN_PROJECTIONS):
        mt, nt, s, kbs = p.gemm_row_tiles[i], p.gemm_col_tiles[i], p.gemm_k_ranges[i], p.gemm_k_blocks_per_range[i]
        assert mt * 16 >= p.pass_rows[0] and mt in (1, 2, 3, 4, 5, 6, 8, 10, 12, 14, 16, 18, 20, 22)
        assert nt in (1, 2, 3, 4) and p.gemm_row_parts[i] in (1, 2) and p.gemm_col_groups[i] in (2, 3, 4)
        assert (p.gemm_row_parts[i] == 2) == (mt >= 8)
        assert s in (1, 2, 4, 8, 16) and kbs % 4 == 0 and s * kbs >= n_in[i] // 32
        with_work = -(-(n_in[i] // 32) // kbs)
        assert with_work * 8 >= s * 7, "at most one K range in eight may come out empty"
        n_pad = (n_out[i] + 15) // 16 * 16
        assert p.gemm_partial_floats[i] == s * p.pass_rows[0] * n_pad <= p.gemm_partial_capacity
        tiles_per_wg = nt * p.gemm_col_groups[i]
        # from 14 row tiles on two row blocks of eight, ten or twelve tiles; at eight row tiles one, for wide matrices
        ring = p.gemm_kernels >> i & 1
        assert ring == (mt >= 14 or (mt == 8 and nt == 4 and p.gemm_col_groups[i] == 4))
        assert p.gemm_workgroups[i] == -(-(n_pad // 16) // tiles_per_wg) * s * (2 if mt >= 14 else 1)
    # the residual inside output and down projection: few rows, a K that suits their number and the ranges, a round of workgroups
    few = p.pass_rows[0] <= 8
    for i in range(sv.PLAN_PROJECTIONS):
        s = p.gemm_k_ranges[i]
        if i == 1 and p.gate_up_swiglu_inside:
            longest = {4: 6144 if few else 3072, 8: 4096 if few else 2048, 16: 4096 if few else 2048}
        else:
            longest = {4: 6144, 8: 6144 if few else 3072, 16: 6144 if few else 4096}
        assert (p.gemm_kernels >> 8 + i & 1) == (i in (1, 3) and p.pass_rows[0] <= 16 and n_in[i] <= longest.get(s, 0)
                                                 and shape.d_model <= 16 * cu)
    # operand fragments fit their buffers; SwiGLU inside the GEMM up to four row tiles, and from 14 on with one K range
    mt = p.gemm_row_tiles[2]
    units = lambda k: (k // 32 + 4) * 2 * mt * 64
    assert p.xfrag_units == units(max(shape.d_model, dq, shape.d_ffn)) <= p.xfrag_capacity
    if mt >= 14:
        assert p.gate_up_swiglu_inside == (p.gemm_k_ranges[2] == 1)
    elif p.gate_up_swiglu_inside:
        assert mt <= 4
    # the second buffer: the normalised residual of few rows, or SwiGLU's result where the product writes it
    assert p.xfrag_act_units == (units(shape.d_model) if mt == 1 else units(shape.d_ffn) if p.gate_up_swiglu_inside else 0)
    assert p.xfrag_act_units <= p.xfrag_act_capacity
    # attention of the first pass
    group = shape.n_q_heads // shape.n_kv_heads
    window = max(look[:p.pass_seqs[0]]) + 1
    assert group % p.attn_kv_share == 0 and (group // p.attn_kv_share) * window <= 64
    assert p.attn_row_tiles == -(-(group // p.attn_kv_share) * window // 16) and 1 <= p.attn_row_tiles <= 4
    assert p.attn_chunk_keys % 32 == 0 and p.attn_chunks * p.attn_chunk_keys >= cfg.max_kv_len
    assert (p.attn_chunks - 1) * p.attn_chunk_keys < cfg.max_kv_len and 1 <= p.attn_chunks
    assert p.attn_chunks <= (16 if not paged else max(16, -(-cfg.max_kv_len // 2048)))
    assert p.attn_wavefronts in (0, 1, 2, 4, 8) and (p.attn_wavefronts == 0 or p.attn_chunks <= p.attn_wavefronts)
    if p.attn_wavefronts:                                   # chunk results of a workgroup fit 64 KiB of LDS
        assert p.attn_wavefronts * p.attn_row_tiles * 16 * (shape.head_dim + 2) * 4 <= 64 * 1024
    if p.attn_fused:
        assert not (shape.head_dim == 128 and p.attn_row_tiles >= 3) and p.attn_chunk_keys >= 192
    if paged:
        assert p.attn_chunk_keys <= 2048
    if p.attn_small:
        assert p.attn_chunks <= max(4, -(-cfg.max_kv_len // 2048) if paged else 1)
    assert p.attn_partial_floats <= p.attn_partial_capacity


@pytest.mark.parametrize("seed", range(40))
def test_plans_respect_every_limit(seed):
    r = random.Random(seed)
    for _ in range(25):
        hd = r.choice([64, 128])
        n_kv = r.choice([1, 2, 4, 8, 16, 32])
        group = r.choice([1, 2, 3, 4, 6, 8, 16])
        d = r.choice([256, 1024, 2048, 4096, 8192])
        shape = wl.ModelShape(r.choice([1, 4, 32]), d, n_kv * group, n_kv, hd, r.choice([512, 2752, 11008, 28672]),
                              r.choice([1000, 32000, 128256]))
        kmax = r.choice([0, 1, 5, 10, 15])
        max_batch = r.choice([1, 8, 32, 64, 200, 256])
        B = r.randrange(1, max_batch + 1)
        look = [r.randrange(0, kmax + 1) for _ in range(B)]
        look[r.randrange(B)] = kmax
        paged = r.random() < 0.3
        max_kv_len = r.choice([64, 1030, 2054, 4107, 16384, 32768, 131072])
        if max_kv_len < kmax + 1:
            max_kv_len = 64
        cu = r.choice([256, 256, 64, 304])
        cfg = sv.make_cfg(shape, max_batch, max_kv_len, kmax)
        p = sv.spec_k_plan_step(cfg, look, cu, paged)
        _check_invariants(shape, cfg, look, p, paged, cu)


def test_capacity_holds_for_every_batch_and_row_count():
    """What a launch writes never exceeds what init allocates, for every batch size up to the handle's
    and the full range of row counts (the check the step itself makes before launching)."""
    for shape, max_batch, kmax, max_kv in ((wl.SEVEN_B, 32, 10, 4107), (wl.ONE_B, 16, 15, 2048),
                                           (wl.ModelShape(2, 512, 64, 8, 64, 1024, 50000), 64, 15, 700)):
        cfg = sv.make_cfg(shape, max_batch, max_kv, kmax)
        for B in range(1, max_batch + 1):
            for k in (0, kmax // 2, kmax):
                p = sv.spec_k_plan_step(cfg, [k] * B, 256, False)
                assert max(p.gemm_partial_floats) <= p.gemm_partial_capacity
                assert p.attn_partial_floats <= p.attn_partial_capacity


def test_plans_of_the_named_configurations():
    w = wl.workload_7b()
    cfg, p = _plan(w.shape, list(w.lookahead), w.batch, w.max_kv_len, w.max_lookahead)
    assert p.rows == 48 and p.n_passes == 1
    assert list(p.gemm_row_tiles) == [3] * 5
    # (the launch rounds these up to whole rounds of the 8 XCDs: 250 runs as a grid of 256)
    # (the QKV projection as 256 workgroups of three wavefronts: four per workgroup would leave 64 compute units idle)
    assert list(p.gemm_workgroups) == [256, 256, 172, 256, 250] and list(p.gemm_col_groups) == [3, 2, 4, 4, 4]
    # (two column groups where a workgroup's K range stays within 2048: the output projection in 4 ranges, not the down projection)
    assert list(p.gemm_k_ranges) == [2, 4, 2, 8, 2]
    assert (p.attn_kv_share, p.attn_small, p.attn_chunks, p.attn_wavefronts, p.attn_fused) == (1, 0, 2, 2, 1)
    assert p.gate_up_swiglu_inside == 1
    w = wl.workload_1b()
    cfg, p = _plan(w.shape, list(w.lookahead), w.batch, w.max_kv_len, w.max_lookahead)
    assert p.rows == 6 and list(p.gemm_row_tiles) == [1] * 5
    assert p.gemm_kernels == 1 << 8 + 1     # the output projection adds to the residual stream; the down projection's K is 8192
    # a small launch: every query head a work item of its own, four chunks merged in the workgroup
    assert (p.attn_kv_share, p.attn_small, p.attn_chunks, p.attn_wavefronts, p.attn_fused) == (4, 1, 4, 4, 1)
    w = wl.workload_dyn()
    cfg, p = _plan(w.shape, list(w.lookahead), w.batch, w.max_kv_len, w.max_lookahead)
    assert p.rows == sum(k + 1 for k in w.lookahead) and p.n_passes == 1
    assert list(p.gemm_row_tiles) == [10] * 5 and list(p.gemm_row_parts) == [2] * 5
    assert (p.attn_kv_share, p.attn_small, p.attn_chunks, p.attn_wavefronts) == (1, 0, 1, 1)


def test_plan_of_the_many_row_step():
    # 7B shape, 352 rows: two row blocks of twelve row tiles; gate/up in one K range, with SwiGLU and the second buffer
    cfg, p = _plan(wl.SEVEN_B, [10] * 32, 32, 4107, 10)
    assert p.rows == 352 and list(p.gemm_row_tiles) == [22] * 5 and p.gemm_kernels == 0b11111
    assert list(p.gemm_workgroups) == [256, 256, 230, 256, 250] and list(p.gemm_k_ranges) == [2, 4, 1, 8, 1]
    assert p.gate_up_swiglu_inside == 1 and p.xfrag_act_units == (11008 // 32 + 4) * 2 * 22 * 64 <= p.xfrag_act_capacity
    # 128 rows: the LM head alone, as one row block
    cfg, p = _plan(wl.SEVEN_B, [15] * 8, 32, 4107, 15)
    assert p.rows == 128 and p.gemm_kernels == 0b10000 and p.gemm_workgroups[4] == 125 * p.gemm_k_ranges[4]
    assert p.gate_up_swiglu_inside == 0 and p.xfrag_act_units == 0
    # one row: the normalised residual
    cfg, p = _plan(wl.ONE_B, [0], 1, 2048, 5)
    assert p.gemm_kernels == 1 << 8 + 1 and p.xfrag_act_units == (2048 // 32 + 4) * 2 * 64


@pytest.mark.parametrize("d,dq,F,rows,want", [
    # gate/up and SwiGLU as two launches, then as one (F from 5472 on), narrow to wide
    (512, 1024, 2048, 16, 0b1010), (1024, 4096, 4096, 16, 0b1010), (1024, 4608, 4608, 9, 0), (1024, 6144, 4608, 8, 0b1010),
    (2048, 3072, 3072, 16, 0b1010), (2048, 4096, 4096, 9, 0), (2048, 5120, 4608, 8, 0b1010), (3072, 6144, 5120, 16, 0b1010),
    (1024, 2048, 5504, 16, 0b0010), (1024, 3072, 5504, 9, 0), (1024, 4096, 6144, 8, 0b1010), (1024, 4608, 6176, 8, 0),
    (2048, 2048, 5504, 8, 0b1010), (2048, 5120, 5504, 8, 0b1000), (3072, 3072, 8192, 16, 0b0010), (3072, 6144, 8192, 8, 0b0010),
    (4096, 4096, 11008, 8, 0b0010), (4096, 4096, 11008, 9, 0), (5120, 5120, 13824, 1, 0), (8192, 2048, 4096, 1, 0)])
def test_residual_inside_the_product_where_it_is_faster(d, dq, F, rows, want):
    """Each line is a measured boundary: K by rows and ranges, widths by compute units."""
    shape = wl.ModelShape(1, d, dq // 128, 4, 128, F, 1000)
    look = [rows - 1] if rows < 16 else [15]
    assert _plan(shape, look)[1].gemm_kernels >> 8 == want


@pytest.mark.parametrize("rows", [6, 48, 128, 192, 208, 352])
def test_workgroup_target_cuts_k(rows):
    """The workgroups asked for decide the K ranges at every number of rows: the fewest ranges that reach them, and with a
    target that no cut reaches as many as the shape allows."""
    look, n = [15] * (rows // 16) or [rows - 1], []
    try:
        for target in (1, 300, 700, 100000):
            sv.spec_k_set_gemm_wg_target(target)
            _, p = _plan(wl.SEVEN_B, look, 32, 4107, 15)
            n.append(list(p.gemm_k_ranges))
            for i in range(sv.PLAN_PROJECTIONS):
                s, wgs = p.gemm_k_ranges[i], p.gemm_workgroups[i]
                assert wgs >= target or target == 100000 or s == 16
                assert s == 1 or wgs // s * (s // 2) < target
    finally:
        sv.spec_k_set_gemm_wg_target(0)
    assert n[0] == [1] * 5 and n[3] == [16] * 5
    assert n[0][1] < n[1][1] <= n[2][1]     # (the output projection)


@pytest.mark.parametrize("rows", [1, 16, 32, 48, 64, 80, 128, 192, 208, 352, 1008])
def test_second_operand_buffer_holds_what_is_written_and_no_more(rows):
    """The buffer has readers up to 16 rows (d_model wide), up to 64 and above 192 (d_ffn wide): what a handle of 65 to 192 rows
    reserves is what its passes of up to 64 rows write."""
    units = lambda tiles, k: (k // 32 + 4) * 2 * tiles * 64
    for shape in (wl.SEVEN_B, wl.ONE_B, wl.ModelShape(1, 2048, 16, 16, 64, 512, 1000)):
        cfg = sv.make_cfg(shape, -(-rows // 16), 64, min(rows, 16) - 1)
        plan = lambda n: sv.spec_k_plan_step(cfg, [15] * (n // 16) + [n % 16 - 1] * (n % 16 > 0), 256)
        few, some = units(1, shape.d_model), units(min(-(-rows // 16), 4), shape.d_ffn)
        many = units(plan(min(rows, 352)).gemm_row_tiles[0], shape.d_ffn)
        want = few if rows <= 16 else max(few, some) if rows <= 192 else max(few, many)
        assert plan(1).xfrag_act_capacity == want
        try:
            sv.spec_k_set_swiglu_min_wgs(1)      # SwiGLU inside wherever it may be
            assert all(plan(n).xfrag_act_units <= want for n in range(1, rows + 1))
        finally:
            sv.spec_k_set_swiglu_min_wgs(0)


def test_steps_beyond_one_pass_and_beyond_64_rows_per_kv_head():
    shape = wl.ModelShape(2, 256, 16, 2, 64, 512, 1000)          # 8 query heads per kv head
    cfg, p = _plan(shape, [15] * 40, 40, 400, 15)
    assert p.rows == 640 and p.n_passes == 2 and list(p.pass_rows[:2]) == [320, 320]
    assert p.attn_kv_share >= 2 and (8 // p.attn_kv_share) * 16 <= 64
    cfg, p = _plan(shape, [3] * 40, 40, 400, 15)                 # 8 x 4 = 32 rows: one item per kv head would do
    assert p.n_passes == 1 and (8 // p.attn_kv_share) * 4 <= 64


def test_bad_arguments_are_refused():
    shape = wl.ModelShape(2, 256, 8, 2, 64, 512, 1000)
    cfg = sv.make_cfg(shape, 4, 100, 5)
    with pytest.raises(sv.SpecError):
        sv.spec_k_plan_step(cfg, [6, 1], 256)                    # lookahead beyond the handle's
    with pytest.raises(sv.SpecError):
        sv.spec_k_plan_step(cfg, [1] * 5, 256)                   # batch beyond the handle's
    with pytest.raises(sv.SpecError):
        sv.spec_k_plan_step(cfg, [1], 0)
    fp32 = sv.make_cfg(wl.ModelShape(2, 256, 4, 4, 64, 512, 300, dtype="fp32"), 4, 100, 5)
    with pytest.raises(sv.SpecError):
        sv.spec_k_plan_step(fp32, [1], 256)


def test_chunks_follow_the_resident_wavefronts_of_the_128_dim_fused_variant():
    """7B-shape (32 kv heads x 128): two chunks per pair as long as they fit the 1024 wavefronts the chip
    holds of that variant, one chunk where only that fits them, two again where neither does."""
    for B, chunks in ((8, 2), (16, 2), (18, 1), (20, 1), (24, 1), (27, 1), (28, 1), (32, 1), (33, 2), (48, 2)):
        cfg = sv.make_cfg(wl.SEVEN_B, B, 2054, 5)
        p = sv.spec_k_plan_step(cfg, [5] * B, 256, False)
        assert p.attn_chunks == chunks, (B, p.attn_chunks)
