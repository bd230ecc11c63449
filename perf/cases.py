"""The work that is timed: what a serving program has the verify library do, from the smallest call to the largest.

A case is a dict of sizes.  Its "kind" says which entry point it takes:

  step    spec_verify_step: the target decoder scores a window of K_b + 1 tokens per sequence over its
          KV cache, the proposals are tested, the final token is drawn, the cache length rolled back
  tree    spec_verify_tree_step: the same for a token tree per sequence
  round   spec_decode_round: the draft's K decodes, the verification and the bookkeeping
  sample  the sampling part alone on logits the caller has (a sampler-only handle, or the entry point
          that allocates nothing)
  kv      spec_kv_import and spec_kv_export: a sequence's keys and values arrive from a prefill and
          leave again (preemption, migration)

Weights, caches, logits and uniforms are random, made on the GPU from the seed alone.  Matrices have the
spread that keeps activations of unit size through a layer, the LM head gives logits with the spread
`logit_std` (2 and more: the drawn tokens carry visible probability, as a trained model's do), keys and
values are N(0, 1).  Lengths and windows of a batch follow from the case, spread over their range.
"""
import math

import torch

from paper_2411_00853_amd import binding as sv
from paper_2411_00853_amd.workload import ModelShape

EPS, THETA = 1e-5, 10000.0


# ---- cases -------------------------------------------------------------------------------------------

def _model(layers, d_model, q_heads, kv_heads, head_dim, d_ffn, vocab, dtype="bf16"):
    return {"layers": layers, "d_model": d_model, "q_heads": q_heads, "kv_heads": kv_heads, "head_dim": head_dim,
            "d_ffn": d_ffn, "vocab": vocab, "dtype": dtype}


def _step(model, batch, kv, k, kind="step", **more):
    case = dict(model, kind=kind, batch=batch, kv_min=kv[0], kv_max=kv[1], k_min=k[0], k_max=k[1], paged=False,
                temperature=1.0, logit_std=2.0)
    case.update(more)
    return case


# the shapes of workload.py: whole models and, for most cases, a few layers of them (a step is the same
# chain of kernels for every layer)
def _1b(layers):
    return _model(layers, 2048, 32, 8, 64, 8192, 32000)


def _7b(layers):
    return _model(layers, 4096, 32, 32, 128, 11008, 32000)


def listed():
    tiny = _model(2, 256, 4, 4, 64, 1024, 1024, "fp32")
    draft = {"draft_layers": 4, "draft_d_model": 2048, "draft_q_heads": 16, "draft_kv_heads": 16, "draft_d_ffn": 5504}
    return [
        # one user of the fp32 configuration: a handful of rows, launches and latency are all there is
        dict(_step(tiny, 1, (128, 128), (4, 4)), name="tiny_fp32_step"),
        # one user of the small model, a window of five proposals: the smallest bf16 call, whole model
        dict(_step(_1b(16), 1, (1024, 1024), (5, 5)), name="1b_step_batch1"),
        # the ordinary decode step (no proposals) of a draft-sized model: what a draft runs K times a round
        dict(_step(_model(4, 2048, 16, 16, 128, 5504, 32000), 8, (2048, 2048), (0, 0)), name="draft_decode_batch8"),
        # grouped heads, many users of the small model, ragged lengths
        dict(_step(_1b(4), 32, (300, 2100), (3, 3)), name="1b_block_batch32"),
        # the headline configuration, whole model: eight users, five proposals, 2048 cached tokens
        dict(_step(_7b(32), 8, (2048, 2048), (5, 5), logit_std=4.0), name="7b_step_batch8"),
        # a full server: ragged lengths, a lookahead per sequence, the paged cache
        dict(_step(_7b(4), 32, (512, 4096), (1, 7), paged=True), name="7b_block_ragged_paged"),
        # the most window rows one decoder pass takes, short prompts: the projections as a dense contraction
        dict(_step(_7b(4), 32, (64, 64), (10, 10)), name="7b_block_rows352"),
        # token trees of ten nodes
        dict(_step(_7b(4), 8, (2048, 2048), (10, 10), kind="tree", branch=3), name="7b_block_tree"),
        # a whole decoding round with the draft model of the 7B-shape configuration
        dict(_step(_7b(4), 8, (2048, 2048), (5, 5), kind="round", **draft), name="7b_block_round"),
        # a large vocabulary, many sequences, logits from elsewhere: the sampler as a stream
        {"name": "sample_batch64", "kind": "sample", "batch": 64, "vocab": 128256, "k_min": 8, "k_max": 8,
         "temperature": 0.7, "noalloc": False},
        # the sampler of a few users, called where nothing may be allocated: latency
        {"name": "sample_batch4_noalloc", "kind": "sample", "batch": 4, "vocab": 32003, "k_min": 2, "k_max": 5,
         "temperature": 1.0, "noalloc": True},
        # a prompt's keys and values arrive from the prefill; a preempted sequence leaves
        dict(_7b(32), name="7b_kv_move", kind="kv", n_pos=1333, pos0=0, slots=2, paged=False),
    ]


def _log_int(rng, lo, hi):
    return min(hi, max(lo, int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))))


def _draw_model(rng, most_layers=6):
    head_dim = rng.choice((64, 128))
    q_heads = rng.randint(512 // head_dim, 4096 // head_dim)
    groups = [g for g in (1, 1, 2, 4, 8) if q_heads % g == 0]
    d_model = q_heads * head_dim
    return _model(rng.randint(1, most_layers), d_model, q_heads, q_heads // rng.choice(groups), head_dim,
                  rng.randint(2 * d_model // 32, 4 * d_model // 32) * 32, _log_int(rng, 1000, 65536))


def _cache_bytes(c):
    return c["layers"] * 2 * c["kv_heads"] * c["head_dim"] * 2 * c["batch"] * (c["kv_max"] + c["k_max"] + 1)


def draw(rng):
    kind = rng.choices(("step", "fp32", "tree", "round", "sample", "kv"), (10, 1, 2, 1, 2, 1))[0]
    if kind == "sample":
        noalloc = rng.random() < 0.5
        k = rng.randint(0, 12)
        return {"kind": "sample", "batch": _log_int(rng, 1, 64), "vocab": _log_int(rng, 2000, 128256), "k_min": rng.randint(0, k),
                "k_max": k, "temperature": rng.choice((0.0, 0.7, 1.0, 1.3)), "noalloc": noalloc}
    if kind == "kv":
        m = _draw_model(rng, 32)
        return dict(m, kind="kv", n_pos=_log_int(rng, 1, 2048), pos0=rng.randint(0, 100), slots=rng.randint(1, 3),
                    paged=rng.random() < 0.3)
    if kind == "fp32":
        heads, head_dim = rng.randint(1, 8), rng.choice((32, 64))
        m = _model(rng.randint(1, 4), heads * head_dim, heads, heads, head_dim, rng.randint(4, 64) * 32,
                   _log_int(rng, 500, 8192), "fp32")
        n, k = _log_int(rng, 8, 1024), rng.randint(0, 7)
        return _step(m, rng.randint(1, 6), (max(1, n // 3), n), (k // 2, k))
    m = _draw_model(rng)
    batch = _log_int(rng, 1, 48)
    n = _log_int(rng, 16, 8192)
    k = rng.randint(0 if kind == "step" else 1, min(15, max(1, 400 // batch - 1)))
    if kind == "round":
        k, batch = min(k, 6), min(batch, 16)
    c = _step(m, batch, (max(4, int(n * rng.choice((0.1, 0.5, 1.0)))), n), (rng.randint(0, k) if kind == "step" else k, k),
              kind=kind, paged=rng.random() < 0.3)
    if kind == "tree":
        c["branch"] = rng.randint(1, 3)
    if kind == "round":
        heads = rng.randint(4, 16)
        c.update(draft_layers=rng.randint(1, 3), draft_d_model=heads * m["head_dim"], draft_q_heads=heads,
                 draft_kv_heads=heads, draft_d_ffn=rng.randint(heads * m["head_dim"] // 16, heads * m["head_dim"] // 8) * 32)
    if kind == "step" and rng.random() < 0.2:
        c["temperature"] = 0.0
    while _cache_bytes(c) > (6 << 30):
        c["kv_min"], c["kv_max"] = c["kv_min"] // 2 + 1, c["kv_max"] // 2 + 1
    return c


# ---- what follows from a case --------------------------------------------------------------------------

def _lens(c):
    return [c["kv_min"] + int((c["kv_max"] - c["kv_min"]) * ((b * 0.618034 + 0.35) % 1.0) + 0.5) for b in range(c["batch"])]


def _looks(c):
    return [c["k_min"] + int((c["k_max"] - c["k_min"] + 1) * ((b * 0.414214 + 0.2) % 1.0)) for b in range(c["batch"])]


def _parents(c):
    """The first `branch` nodes continue the text, every later pair continues one node."""
    return [-1 if i < c["branch"] else (i - c["branch"]) // 2 for i in range(c["k_max"])]


def _shape(c):
    return ModelShape(c["layers"], c["d_model"], c["q_heads"], c["kv_heads"], c["head_dim"], c["d_ffn"], c["vocab"],
                      dtype=c["dtype"])


def _draft_case(c):
    """The draft model of a round, as a case of its own: its cache is one token behind the target's."""
    d = dict(c, layers=c["draft_layers"], d_model=c["draft_d_model"], q_heads=c["draft_q_heads"],
             kv_heads=c["draft_kv_heads"], d_ffn=c["draft_d_ffn"])
    d["kv_min"], d["kv_max"] = c["kv_min"] - 1, c["kv_max"] - 1
    return d


# ---- inputs ------------------------------------------------------------------------------------------

def _gen(seed, stream):
    g = torch.Generator(device="cuda")
    g.manual_seed(((int(seed) * 1000003 + stream) * 7919 + 12345) % (1 << 62))
    return g


def _normal(seed, stream, shape, std=1.0, dtype=torch.float32):
    return torch.randn(shape, generator=_gen(seed, stream), device="cuda", dtype=dtype).mul_(std)


def _uniform(seed, stream, shape):
    return torch.rand(shape, generator=_gen(seed, stream), device="cuda")


def _ids(seed, stream, shape, vocab):
    return torch.randint(0, vocab, shape, generator=_gen(seed, stream), device="cuda", dtype=torch.int32)


_MATRICES = ("w_qkv", "w_o", "w_gate_up", "w_down")


def _dims(c):
    dq, dkv = c["q_heads"] * c["head_dim"], c["kv_heads"] * c["head_dim"]
    return {"w_qkv": (dq + 2 * dkv, c["d_model"]), "w_o": (c["d_model"], dq),
            "w_gate_up": (2 * c["d_ffn"], c["d_model"]), "w_down": (c["d_model"], c["d_ffn"])}


def _dtype(c):
    return torch.bfloat16 if c["dtype"] == "bf16" else torch.float32


def _matrix(c, seed, layer, name):
    """One projection matrix, rows = output features."""
    n_out, n_in = _dims(c)[name]
    return _normal(seed, 1000 + 8 * layer + _MATRICES.index(name), (n_out, n_in), 1.28 / math.sqrt(n_in), _dtype(c))


def _gain(c, seed, stream):
    return 1.0 + _normal(seed, stream, (c["d_model"],), 0.1)


def _embedding(c, seed):
    return _normal(seed, 1, (c["vocab"], c["d_model"]), 1.0, _dtype(c))


def _head(c, seed):
    return _normal(seed, 2, (c["vocab"], c["d_model"]), c["logit_std"] / math.sqrt(c["d_model"]), _dtype(c))


def _cached(c, seed, b, n):
    """Keys and values of one sequence: [layer][k|v][kv head][position][dim]."""
    return _normal(seed, 500000 + b, (c["layers"], 2, c["kv_heads"], n, c["head_dim"]), 1.0, _dtype(c))


def _pick(logits, temperature, seed, stream):
    """A token per row from softmax(logits / T)."""
    if temperature == 0:
        return logits.argmax(-1).to(torch.int32)
    u = _uniform(seed, stream, logits.shape).clamp_(1e-7, 1 - 1e-7)
    return (logits / temperature - torch.log(-torch.log(u))).argmax(-1).to(torch.int32)


def _proposals(c, seed):
    """Draft logits [batch][rows][vocab] and the tokens drawn from them (a tree has a row for the root too,
    and a node's token is drawn from its parent's row)."""
    tree = c["kind"] == "tree"
    B, K = c["batch"], c["k_max"]
    if K == 0:
        return None, None
    logits = _normal(seed, 10, (B, K + (1 if tree else 0), c["vocab"]))
    rows = logits[:, [p + 1 for p in _parents(c)]] if tree else logits
    return logits, _pick(rows, c["temperature"], seed, 11)


def _sample_inputs(c, seed):
    """Target rows that fall off as a power of the rank of a token, draft rows near them."""
    B, V, K = c["batch"], c["vocab"], c["k_max"]
    look = _looks(c)
    rank = torch.rand((sum(look) + B, V), generator=_gen(seed, 20), device="cuda").argsort(dim=1).add_(1)
    target = rank.to(torch.float32).log_().mul_(-1.1).add_(_normal(seed, 21, rank.shape, 0.5))
    draft = torch.zeros((B, max(K, 1), V), device="cuda")
    at = 0
    for b, k in enumerate(look):
        draft[b, :k] = target[at:at + k]
        at += k + 1
    draft += _normal(seed, 22, draft.shape, 0.3)
    return target, draft, _pick(draft, c["temperature"], seed, 23), _uniform(seed, 24, (B, K + 1))


# ---- prepare -------------------------------------------------------------------------------------------

def _weights(c, seed):
    pack = (lambda m, inter=False: sv.spec_pack_weight(m, inter)) if c["dtype"] == "bf16" else (lambda m, inter=False: m)
    return {"tok_embed": _embedding(c, seed), "final_norm": _gain(c, seed, 3), "lm_head": pack(_head(c, seed)),
            "layers": [dict({n: pack(_matrix(c, seed, l, n), n == "w_gate_up") for n in _MATRICES},
                            attn_norm=_gain(c, seed, 100000 + 2 * l), ffn_norm=_gain(c, seed, 100001 + 2 * l))
                       for l in range(c["layers"])]}


def _handle(c, seed, max_len, max_lookahead):
    """A handle whose cache holds the sequences' keys and values."""
    lens = _lens(c)
    cfg = sv.make_cfg(_shape(c), c["batch"], max_len, max_lookahead)
    if c["paged"]:   # a pool of the pages that the batch can touch
        size = sv.spec_kv_page_bytes(cfg) * sum((n + max_lookahead + 1 + 31) // 32 + 1 for n in lens)
    else:
        size = sv.spec_kv_cache_bytes(cfg)
    kv = torch.empty(size, dtype=torch.uint8, device="cuda")
    kv_len = torch.zeros(c["batch"], dtype=torch.int32, device="cuda")
    init = sv.spec_verify_init_paged if c["paged"] else sv.spec_verify_init
    h = init(cfg, _weights(c, seed), kv, kv_len)
    for b, n in enumerate(lens):
        sv.spec_kv_import(h, b, 0, _cached(c, seed, b, n))
    kv_len.copy_(torch.tensor(lens, dtype=torch.int32))
    return h, kv_len


def prepare(case, seed):
    c = case
    if c["kind"] == "kv":
        cfg = sv.make_cfg(_shape(dict(c, vocab=64)), c["slots"], c["pos0"] + c["n_pos"], 1)
        if c["paged"]:
            size = sv.spec_kv_page_bytes(cfg) * c["slots"] * ((c["pos0"] + c["n_pos"] + 31) // 32 + 1)
        else:
            size = sv.spec_kv_cache_bytes(cfg)
        kv = torch.empty(size, dtype=torch.uint8, device="cuda")
        kv_len = torch.zeros(c["slots"], dtype=torch.int32, device="cuda")
        init = sv.spec_verify_init_paged if c["paged"] else sv.spec_verify_init
        h = init(cfg, _stub_weights(dict(c, vocab=64)), kv, kv_len)   # weights and head play no part
        src = _cached(c, seed, 0, c["n_pos"])
        return {"case": c, "h": h, "src": src, "dst": torch.empty_like(src)}
    if c["kind"] == "sample":
        target, draft, tokens, uniforms = _sample_inputs(c, seed)
        h = None if c["noalloc"] else sv.spec_verify_init(sv.sampler_cfg(c["vocab"], c["batch"], max(c["k_max"], 1)), None, None, None)
        B, K = c["batch"], max(c["k_max"], 1)
        return {"case": c, "h": h, "target": target, "draft": draft, "tokens": tokens, "look": _looks(c), "kmax": K,
                "uniforms": uniforms if c["k_max"] else torch.cat([uniforms, uniforms], 1).contiguous(),
                "n_accepted": torch.zeros(B, dtype=torch.int32, device="cuda"),
                "out_tokens": torch.zeros((B, K + 1), dtype=torch.int32, device="cuda")}
    B, K, V = c["batch"], c["k_max"], c["vocab"]
    lens, look = _lens(c), _looks(c)
    slots = torch.arange(B, dtype=torch.int32, device="cuda")
    h, kv_len = _handle(c, seed, max(lens) + K + 1, K)
    s = {"case": c, "h": h, "kv_len": kv_len, "lens": lens, "look": look, "slots": slots, "slot_list": list(range(B)),
         "last": _ids(seed, 4, (B,), V)}
    if c["kind"] == "round":
        d = _draft_case(c)
        s["draft_lens"] = _lens(d)
        s["draft_h"], s["draft_kv_len"] = _handle(d, seed + 77, max(lens) + K + 1, K)
        s["prev"] = _ids(seed, 5, (B,), V)
        s["draft_u"], s["verify_u"] = _uniform(seed, 12, (B, K)), _uniform(seed, 13, (B, K + 1))
        s["decoder"] = sv.spec_decode_init(h, s["draft_h"], B, K + 1)
        return s
    s["draft_logits"], s["tokens"] = _proposals(c, seed)
    s["uniforms"] = _uniform(seed, 12, (B, K + 1))
    s["n_accepted"] = torch.zeros(B, dtype=torch.int32, device="cuda")
    s["out_tokens"] = torch.zeros((B, K + 1), dtype=torch.int32, device="cuda")
    s["logits"] = torch.zeros((sum(look) + B, V), device="cuda")
    if c["kind"] == "tree":
        s["parent"] = torch.tensor([_parents(c)] * B, dtype=torch.int32, device="cuda")
        s["path"] = torch.zeros((B, K), dtype=torch.int32, device="cuda")
    return s


def _stub_weights(c):
    """Weights of a handle that only holds a cache (all layers share one set)."""
    one = {n: torch.zeros(sv.spec_packed_weight_bytes(*_dims(c)[n]) // 2, dtype=torch.bfloat16, device="cuda") for n in _MATRICES}
    one["attn_norm"] = one["ffn_norm"] = torch.ones(c["d_model"], device="cuda")
    return {"tok_embed": torch.zeros((c["vocab"], c["d_model"]), dtype=torch.bfloat16, device="cuda"),
            "final_norm": one["attn_norm"], "lm_head": torch.zeros(sv.spec_packed_weight_bytes(c["vocab"], c["d_model"]) // 2,
                                                                  dtype=torch.bfloat16, device="cuda"),
            "layers": [one] * c["layers"]}


# ---- run -----------------------------------------------------------------------------------------------

def run(s):
    c = s["case"]
    kind = c["kind"]
    if kind == "kv":
        sv.spec_kv_import(s["h"], c["slots"] - 1, c["pos0"], s["src"])
        sv.spec_kv_export(s["h"], c["slots"] - 1, c["pos0"], s["dst"])
        return s["dst"]
    if kind == "sample":
        if c["noalloc"]:
            sv.spec_sample_step_noalloc(c["vocab"], s["kmax"], s["look"], s["uniforms"], c["temperature"], s["n_accepted"],
                                        s["out_tokens"], s["target"], s["tokens"], s["draft"])
        else:
            sv.spec_verify_step(s["h"], s["look"], s["uniforms"], c["temperature"], s["n_accepted"], s["out_tokens"],
                                draft_tokens=s["tokens"], draft_logits=s["draft"], target_logits_in=s["target"])
        return {"n_accepted": s["n_accepted"], "out_tokens": s["out_tokens"]}
    # every pass starts from the same text: the cache is rewound to it first
    sv.spec_kv_rollback(s["h"], s["slot_list"], s["lens"])
    if kind == "round":
        sv.spec_kv_rollback(s["draft_h"], s["slot_list"], s["draft_lens"])
        sv.spec_decode_begin(s["decoder"], s["slots"], s["prev"], s["last"])
        sv.spec_decode_round(s["decoder"], c["k_max"], s["draft_u"], s["verify_u"], c["temperature"])
        v = sv.spec_decode_get_view(s["decoder"])
        B, K, V = c["batch"], c["k_max"], c["vocab"]
        return {"target_logits": sv.device_array(v.target_logits, (B * (K + 1), V), torch.float32),
                "draft_logits": sv.device_array(v.draft_logits, (B, K, V), torch.float32),
                "draft_tokens": sv.device_array(v.draft_tokens, (B, K), torch.int32),
                "n_accepted": sv.device_array(v.n_accepted, (B,), torch.int32),
                "last_token": sv.device_array(v.last_token, (B,), torch.int32), "kv_len": s["kv_len"]}
    if kind == "tree":
        sv.spec_verify_tree_step(s["h"], s["look"], s["parent"], s["tokens"], s["draft_logits"], s["uniforms"],
                                 c["temperature"], s["n_accepted"], s["out_tokens"], s["path"], seq_slot=s["slots"],
                                 last_token=s["last"], logits_out=s["logits"])
        return {"logits": s["logits"], "n_accepted": s["n_accepted"], "out_tokens": s["out_tokens"], "path": s["path"],
                "kv_len": s["kv_len"]}
    sv.spec_verify_step(s["h"], s["look"], s["uniforms"], c["temperature"], s["n_accepted"], s["out_tokens"],
                        seq_slot=s["slots"], last_token=s["last"], draft_tokens=s["tokens"], draft_logits=s["draft_logits"],
                        logits_out=s["logits"])
    return {"logits": s["logits"], "n_accepted": s["n_accepted"], "out_tokens": s["out_tokens"], "kv_len": s["kv_len"]}


# ---- what a pass cannot do without ---------------------------------------------------------------------

def _model_work(c, lens, rows):
    """Bytes and operations of one decoder pass; rows: window tokens per sequence."""
    M, size = sum(rows), 2 if c["dtype"] == "bf16" else 4
    weights = c["layers"] * sum(a * b for a, b in _dims(c).values()) + c["vocab"] * c["d_model"]
    kv_row = 2 * c["kv_heads"] * c["head_dim"] * c["layers"] * size
    read = (weights + M * c["d_model"]) * size + sum(lens) * kv_row
    attention = sum(4 * r * (n + (r + 1) / 2) for n, r in zip(lens, rows)) * c["q_heads"] * c["head_dim"] * c["layers"]
    return read + M * kv_row + M * c["vocab"] * 4, 2 * M * weights + attention


def work(case):
    c = case
    if c["kind"] == "kv":   # read and written once each way
        return {"bytes": 4 * c["layers"] * 2 * c["kv_heads"] * c["n_pos"] * c["head_dim"] * 2, "flops": 0}
    look = _looks(c)
    drafts = 0 if c["temperature"] == 0 else (sum(look) + (c["batch"] if c["kind"] == "tree" else 0)) * c["vocab"] * 4
    if c["kind"] == "sample":
        rows = sum(look) + c["batch"]
        return {"bytes": rows * c["vocab"] * 4 + drafts, "flops": 4 * (rows + sum(look)) * c["vocab"]}
    b, f = _model_work(c, _lens(c), [k + 1 for k in look])
    if c["kind"] == "round":   # the proposals' logits are made, not read
        d = _draft_case(c)
        for i in range(c["k_max"]):
            db, df = _model_work(d, [n + (i + 1 if i else 0) for n in _lens(d)], [1 if i else 2] * c["batch"])
            b, f = b + db, f + df
        return {"bytes": b, "flops": f}
    return {"bytes": b + drafts, "flops": f}


def tolerance(case):
    if case["kind"] in ("kv", "sample"):
        return "exact"
    if case["dtype"] == "fp32":
        return {"rel": 1e-5, "max": 4e-4, "differ": 0.01}   # 0.7e-6 to 1.6e-6 off the 64-bit result
    # Long caches are 1e-5 off the 64-bit result.  With a few cached tokens it is up to 2.2e-4: sums in another
    # order move a new key or value across a rounding boundary of its bf16 storage now and then.
    return {"rel": 8e-4, "max": 0.03, "differ": 0.01}


# ---- the same in 64 bits ---------------------------------------------------------------------------------

def _rms(x, gain):
    return x / torch.sqrt((x * x).mean(-1, keepdim=True) + EPS) * gain.double()


def _rotate(x, pos):
    """x [tokens][heads][dim], dimension i paired with i + dim/2."""
    half = x.shape[-1] // 2
    freq = THETA ** (-2.0 * torch.arange(half, device=x.device, dtype=torch.float64) / x.shape[-1])
    ang = pos.double()[:, None, None] * freq
    a, b = x[..., :half], x[..., half:]
    return torch.cat([a * ang.cos() - b * ang.sin(), a * ang.sin() + b * ang.cos()], -1)


def _decode64(c, seed, lens, windows, parents=None):
    """Logits of every window token, in fp64; new keys and values are rounded to the cache's type."""
    H, G, D = c["kv_heads"], c["q_heads"] // c["kv_heads"], c["head_dim"]
    dq, dkv = c["q_heads"] * D, H * D
    depth, sees = [], []
    for w in windows:
        n = w.numel()
        if parents is None:
            depth.append(list(range(n)))
            sees.append(torch.ones(n, n, dtype=torch.bool).tril_())
        else:
            m, dep = torch.zeros(n, n, dtype=torch.bool), [0]
            m[0, 0] = True
            for i, p in enumerate(parents):
                m[i + 1] = m[p + 1]
                m[i + 1, i + 1] = True
                dep.append(dep[p + 1] + 1)
            depth.append(dep)
            sees.append(m)
    x = torch.cat([_embedding(c, seed)[w.long()] for w in windows]).double()
    pos = torch.cat([torch.tensor([n + d for d in dep], device="cuda") for n, dep in zip(lens, depth)])
    caches = [_cached(c, seed, b, n) for b, n in enumerate(lens)]
    for l in range(c["layers"]):
        qkv = _rms(x, _gain(c, seed, 100000 + 2 * l)) @ _matrix(c, seed, l, "w_qkv").double().T
        q = _rotate(qkv[:, :dq].reshape(-1, H * G, D), pos)
        k = _rotate(qkv[:, dq:dq + dkv].reshape(-1, H, D), pos).to(_dtype(c)).double()
        v = qkv[:, dq + dkv:].reshape(-1, H, D).to(_dtype(c)).double()
        out, at = [], 0
        for b, w in enumerate(windows):
            n = w.numel()
            rows = slice(at, at + n)
            at += n
            kk = torch.cat([caches[b][l, 0].double(), k[rows].transpose(0, 1)], 1).contiguous()   # [H][T][D]
            vv = torch.cat([caches[b][l, 1].double(), v[rows].transpose(0, 1)], 1).contiguous()
            qq = q[rows].reshape(n, H, G, D).permute(1, 2, 0, 3).reshape(H, G * n, D).contiguous()
            s = torch.bmm(qq, kk.transpose(1, 2).contiguous()).reshape(H, G, n, -1) / math.sqrt(D)
            s[..., lens[b]:].masked_fill_(~sees[b].to(s.device), -math.inf)
            o = torch.bmm(s.softmax(-1).reshape(H, G * n, -1), vv).reshape(H, G, n, D)
            out.append(o.permute(2, 0, 1, 3).reshape(n, dq))
        x = x + torch.cat(out) @ _matrix(c, seed, l, "w_o").double().T
        h = _rms(x, _gain(c, seed, 100001 + 2 * l)) @ _matrix(c, seed, l, "w_gate_up").double().T
        gate, up = h[:, :c["d_ffn"]], h[:, c["d_ffn"]:]
        x = x + (gate * torch.sigmoid(gate) * up) @ _matrix(c, seed, l, "w_down").double().T
    return _rms(x, _gain(c, seed, 3)) @ _head(c, seed).double().T


def exact(case, seed):
    c = case
    if c["kind"] == "kv":
        return _cached(c, seed, 0, c["n_pos"])
    if c["kind"] == "sample":   # decisions and token ids only
        return None
    lens, look, B, K, V = _lens(c), _looks(c), c["batch"], c["k_max"], c["vocab"]
    last = _ids(seed, 4, (B,), V)
    if c["kind"] != "round":
        _, tokens = _proposals(c, seed)
        windows = [torch.cat([last[b:b + 1], tokens[b, :look[b]]]) if look[b] else last[b:b + 1] for b in range(B)]
        out = {"logits": _decode64(c, seed, lens, windows, _parents(c) if c["kind"] == "tree" else None),
               "n_accepted": None, "out_tokens": None, "kv_len": None}
        return dict(out, path=None) if c["kind"] == "tree" else out
    d = _draft_case(c)
    prev, u = _ids(seed, 5, (B,), V), _uniform(seed, 12, (B, K)).double()
    windows = [torch.stack([prev[b], last[b]]) for b in range(B)]
    rows = []
    for i in range(K):   # a proposal is drawn by inverse CDF in ascending token id
        got = _decode64(d, seed + 77, _lens(d), windows).reshape(B, i + 2, V)[:, -1]
        rows.append(got)
        cdf = (got / c["temperature"]).softmax(-1).cumsum(-1)
        drawn = (cdf <= u[:, i:i + 1] * cdf[:, -1:]).sum(-1).clamp_(max=V - 1).to(torch.int32)
        windows = [torch.cat([w, drawn[b:b + 1]]) for b, w in enumerate(windows)]
    return {"target_logits": _decode64(c, seed, lens, [w[1:] for w in windows]), "draft_logits": torch.stack(rows, 1),
            "draft_tokens": None, "n_accepted": None, "last_token": None, "kv_len": None}
