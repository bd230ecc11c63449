// The decoder pass of the verify step: the order in which the kernels run for one window.
// Per layer: RMSNorm -> QKV projection -> rotary + KV append -> windowed-causal attention ->
// output projection (+residual) -> RMSNorm -> gate/up projection -> SiLU gating -> down projection
// (+residual); then the final norm and the LM head.  Every reduction of GEMM K-range partial sums
// is folded into the kernel that consumes the GEMM's result.
#include <cmath>
#include <cstring>
#include <vector>

#include "frag.h"
#include "handle.h"

namespace specv {

namespace {
struct Dims {
    int d, dq, dkv, nqkv, F, V;
};
Dims dims_of(const spec_model_cfg& c)
{
    Dims z;
    z.d = c.d_model;
    z.dq = c.n_q_heads * c.head_dim;
    z.dkv = c.n_kv_heads * c.head_dim;
    z.nqkv = z.dq + 2 * z.dkv;
    z.F = c.d_ffn;
    z.V = c.vocab;
    return z;
}
}  // namespace

int forward_init(spec_handle* h, int max_rows)
{
    const spec_model_cfg& c = h->cfg;
    const Dims z = dims_of(c);
    h->max_rows = max_rows;
    if (!h->geom.table) h->geom = make_cache_geom(c);   // a paged handle set its geometry already
    // The bf16 projections take at most GEMM_MAX_ROWS rows per launch.  A handle whose batch and
    // lookahead limits multiply to more than that is still usable: the limit then applies to the rows
    // of each step (the sum of K_b + 1), which the step checks.
    h->row_cap = c.dtype == SPEC_DTYPE_BF16 ? std::min(max_rows, GEMM_MAX_ROWS) : max_rows;
    const int all_rows = max_rows;   // the logits of a whole step, however many passes it takes
    max_rows = h->row_cap;
    int rc = SPEC_OK;
    Arena& a = h->arena;
    auto A = [&](float** p, size_t count) {
        if (rc == SPEC_OK) rc = a.alloc(reinterpret_cast<void**>(p), count * sizeof(float));
    };
    A(&h->x, (size_t)max_rows * z.d);
    if (c.dtype == SPEC_DTYPE_BF16) A(&h->q, (size_t)max_rows * z.dq);
    A(&h->logits, (size_t)all_rows * z.V);
    A(&h->cos_sin, (size_t)c.max_kv_len * c.head_dim);
    size_t part = 0;
    if (c.dtype == SPEC_DTYPE_BF16) {
        A(reinterpret_cast<float**>(&h->ssq), (size_t)max_rows * ssq_pairs(z.d) * (sizeof(double2) / sizeof(float)));
        // operand fragments: the widest GEMM input (d_model, q width or d_ffn), both planes, at the
        // row-tile count of the largest step; zeroed once so that padding blocks stay zero
        const int kmax = std::max(std::max(z.d, z.dq), z.F);
        const size_t xf_bytes = xfrag_uint4s(gemm_row_tiles(max_rows), 2, kmax) * sizeof(uint4);
        if (rc == SPEC_OK) rc = a.alloc(&h->xf, xf_bytes);
        if (rc == SPEC_OK && hipMemset(h->xf, 0, xf_bytes) != hipSuccess) rc = fail(SPEC_ERR_DEVICE, "hipMemset failed");
        // the gate/up GEMM reads h->xf while its early workgroups already write the down projection's
        // operand, which therefore has a buffer of its own (up to 16 rows the two change places)
        const size_t xa_bytes = act_frag_capacity(c, max_rows) * sizeof(uint4);
        if (rc == SPEC_OK) rc = a.alloc(&h->xf_act, xa_bytes);
        if (rc == SPEC_OK && hipMemset(h->xf_act, 0, xa_bytes) != hipSuccess) rc = fail(SPEC_ERR_DEVICE, "hipMemset failed");
        A(reinterpret_cast<float**>(&h->ssq_parts), (size_t)std::min(max_rows, 16) * (z.d / ADD_COLS) * 2);
        part = gemm_partial_capacity(c, max_rows, h->cu_count);
        const int group = c.n_q_heads / c.n_kv_heads;
        const size_t po = attn_partial_floats(c.max_kv_len, c.max_batch, c.n_kv_heads, group, c.max_lookahead + 1,
                                              c.head_dim, h->cu_count, h->geom.table != nullptr);
        A(&h->attn_part_o, po);
        A(&h->attn_part_ml, po / c.head_dim * 2);
        h->attn_part_cap = po;
    } else {
        A(&h->att, (size_t)max_rows * z.dq);
        A(&h->act, (size_t)max_rows * z.F);
        part = (size_t)max_rows * z.nqkv;   // fp32 path: the QKV result, written whole
    }
    A(&h->partial, part);
    h->partial_cap = part;
    if (rc) return rc;

    // rotary table in fp64 on the host: cos, sin of pos * theta^(-2i/hd)
    const int half = c.head_dim / 2;
    std::vector<float> tab((size_t)c.max_kv_len * c.head_dim);
    for (int pos = 0; pos < c.max_kv_len; ++pos)
        for (int i = 0; i < half; ++i) {
            const double ang = (double)pos * std::pow((double)c.rope_theta, -2.0 * i / (double)c.head_dim);
            tab[((size_t)pos * half + i) * 2 + 0] = (float)std::cos(ang);
            tab[((size_t)pos * half + i) * 2 + 1] = (float)std::sin(ang);
        }
    SPECV_HIP(hipMemcpy(h->cos_sin, tab.data(), tab.size() * sizeof(float), hipMemcpyHostToDevice));
    return SPEC_OK;
}

// partial-sum space (floats) for the largest projection at any row count up to max_rows
size_t gemm_partial_capacity(const spec_model_cfg& c, int max_rows, int cu_count)
{
    const Dims z = dims_of(c);
    const int Ns[G_COUNT] = {z.nqkv, z.d, 2 * z.F, z.d, z.V};
    const int Ks[G_COUNT] = {z.d, z.dq, z.d, z.F, z.d};
    size_t part = 0;
    for (int M = 16; M <= (max_rows + 15) / 16 * 16 && M <= GEMM_MAX_ROWS; M += 16)
        for (int i = 0; i < G_COUNT; ++i) {
            const int rows = M < max_rows ? M : max_rows;
            const size_t e = gemm_partial_elems(plan_gemm(rows, Ns[i], Ks[i], cu_count, true), rows);
            if (e > part) part = e;
        }
    return part;
}

// whether the gate/up projection of a pass of M rows finishes SwiGLU itself
bool swiglu_inside(const spec_model_cfg& c, int M, int cu_count)
{
    return gemm_swiglu_fits(M, c.d_ffn, cu_count) || gemm_ring_swiglu_fits(plan_gemm(M, 2 * c.d_ffn, c.d_model, cu_count, true));
}

size_t act_frag_units(const spec_model_cfg& c, int M, int cu_count)
{
    const int mt = gemm_row_tiles(M);
    if (mt == 1) return xfrag_uint4s(mt, 2, c.d_model);
    return swiglu_inside(c, M, cu_count) ? xfrag_uint4s(mt, 2, c.d_ffn) : 0;
}

size_t act_frag_capacity(const spec_model_cfg& c, int max_rows)
{
    // (whatever the tuning knobs say: they may change after init.  From 65 to 192 rows SwiGLU is a kernel of its own.)
    size_t n = xfrag_uint4s(1, 2, c.d_model);
    if (max_rows > 16) n = std::max(n, xfrag_uint4s(gemm_row_tiles(std::min(max_rows, 64)), 2, c.d_ffn));
    if (max_rows > 192) n = std::max(n, xfrag_uint4s(gemm_row_tiles(max_rows), 2, c.d_ffn));
    return n;
}

void projection_shapes(const spec_model_cfg& c, int* n_out, int* n_in)
{
    const Dims z = dims_of(c);
    const int Ns[G_COUNT] = {z.nqkv, z.d, 2 * z.F, z.d, z.V};
    const int Ks[G_COUNT] = {z.d, z.dq, z.d, z.F, z.d};
    for (int i = 0; i < G_COUNT; ++i) {
        n_out[i] = Ns[i];
        n_in[i] = Ks[i];
    }
}

// Decoder passes of a step of M rows when one pass takes at most cap: groups of consecutive sequences,
// as few groups as filling each to the brim would give (every pass streams all the weights), and among
// the partitions with that many groups the one whose largest group is smallest.  Returns the number of
// passes (0 if max_passes is too few).
int plan_passes(const LookaheadPack& ks, int B, int M, int cap, int* pass_seqs, int* pass_rows, int max_passes)
{
    // groups when each takes sequences while they fit under `limit`
    auto fill = [&](int limit, bool record) {
        int b0 = 0, n = 0;
        while (b0 < B) {
            int Bg = 0, Mg = 0;
            while (b0 + Bg < B && Mg + ks.k[b0 + Bg] + 1 <= limit) {
                Mg += ks.k[b0 + Bg] + 1;
                ++Bg;
            }
            if (Bg == 0) return B + 1;          // a window longer than the limit: no partition
            if (record) {
                if (n == max_passes) return 0;
                pass_seqs[n] = Bg;
                pass_rows[n] = Mg;
            }
            ++n;
            b0 += Bg;
        }
        return n;
    };
    const int fewest = fill(cap, false);
    int limit = (M + fewest - 1) / fewest;       // no partition into `fewest` groups has a smaller largest group
    while (limit < cap && fill(limit, false) > fewest) ++limit;
    return fill(limit, true);
}

// where a pass of M rows embeds them
static EmbedTo embed_to(const spec_handle* h, int M)
{
    const spec_model_cfg& c = h->cfg;
    const bool bf16 = c.dtype == SPEC_DTYPE_BF16;
    const int mt = bf16 ? gemm_row_tiles(M) : 0;
    return EmbedTo{h->tok_embed, c.dtype, c.d_model, h->x, h->ssq, bf16 ? h->layers[0].attn_norm : nullptr,
                   XOut{bf16 ? (mt == 1 ? h->xf_act : h->xf) : nullptr, mt, 2, nullptr}};
}

bool forward_embeds(const spec_handle* h, int M, EmbedTo* e)
{
    if (M < 1 || M > h->row_cap || M > EMBED_MAX_ROWS || h->cfg.d_model % 8) return false;
    *e = embed_to(h, M);
    return true;
}

int forward_run_grouped(spec_handle* h, const LookaheadPack& ks, int B, int M, float* logits_out, hipStream_t s, LogitsSrc* last,
                        bool embedded)
{
    if (last) *last = LogitsSrc{};
    if (M <= h->row_cap) return forward_run(h, h->tables, ks, B, M, logits_out, s, last, embedded);
    if (!h->group_tables.seq_row0) return fail(SPEC_ERR_SHAPE, "%d window rows exceed the %d the handle takes", M, h->row_cap);
    int pass_seqs[SPEC_PLAN_MAX_PASSES], pass_rows[SPEC_PLAN_MAX_PASSES];
    const int n_passes = plan_passes(ks, B, M, h->row_cap, pass_seqs, pass_rows, SPEC_PLAN_MAX_PASSES);
    if (n_passes == 0) return fail(SPEC_ERR_SHAPE, "a step of %d rows needs more than %d decoder passes", M, SPEC_PLAN_MAX_PASSES);
    StepTables sub = h->group_tables;
    sub.pool = h->tables.pool;
    sub.tree = h->tables.tree;
    int b0 = 0, r0 = 0;
    for (int g = 0; g < n_passes; ++g) {
        LookaheadPack kg;
        memset(&kg, 0, sizeof(kg));
        for (int i = 0; i < pass_seqs[g]; ++i) kg.k[i] = ks.k[b0 + i];
        int rc = launch_slice_tables(h->tables, sub, b0, pass_seqs[g], s);
        if (rc) return rc;
        rc = forward_run(h, sub, kg, pass_seqs[g], pass_rows[g], logits_out + (size_t)r0 * h->cfg.vocab, s);
        if (rc) return rc;
        b0 += pass_seqs[g];
        r0 += pass_rows[g];
    }
    return SPEC_OK;
}

int forward_run(spec_handle* h, const StepTables& t, const LookaheadPack& ks, int B, int M, float* logits_out, hipStream_t s,
                LogitsSrc* last, bool embedded)
{
    const spec_model_cfg& c = h->cfg;
    const Dims z = dims_of(c);
    const bool bf16 = c.dtype == SPEC_DTYPE_BF16;
    int rc;
    if (M < 1 || M > h->row_cap) return fail(SPEC_ERR_SHAPE, "%d window rows; the handle takes 1..%d per step", M, h->row_cap);
#define RUN(cls, expr)                          \
    do {                                        \
        {                                       \
            ProfScope ps_(&h->prof, cls, s);    \
            rc = (expr);                        \
        }                                       \
        if (rc) return rc;                      \
    } while (0)

    // bf16 path: every producer writes the next GEMM's operand as fragments of (value * gain); the
    // GEMM leaves K-range partial sums in h->partial, and its consumer adds them up and applies the
    // row's 1/rms where the operand was a normalised residual.  fp32 path (below): plain rows, GEMM
    // results whole, the norms, the residual additions and SwiGLU inside the GEMMs.
    struct Out {
        int n_split;
        size_t stride;
        int ld;
    };
    const int n_ssq = ssq_pairs(z.d);
    const int mt = bf16 ? gemm_row_tiles(M) : 0;
    const int planes = 2;   // activations go to the matrix cores as bf16 head + remainder
    const XOut to_xf{bf16 ? h->xf : nullptr, mt, planes, nullptr};            // operand of the next GEMM
    const NormScale scaled{h->ssq, n_ssq, z.d, c.rms_eps};
    // Up to 16 rows the output and down projections may finish the residual stream themselves (launch_gemm_add): the normalised
    // residual stays in the second fragment buffer, the attention's and SwiGLU's results in the first, and the sums of
    // squares of x come by column tile.
    const GemmPlan plan_o = plan_gemm(M, z.d, z.dq, h->cu_count, true), plan_down = plan_gemm(M, z.d, z.F, h->cu_count, true);
    const bool few = bf16 && mt == 1;
    const bool swiglu_in_gemm = bf16 && swiglu_inside(c, M, h->cu_count);
    const bool add_o = few && gemm_add_fits(plan_o, M, z.dq, h->cu_count, swiglu_in_gemm);
    const bool add_down = few && gemm_add_fits(plan_down, M, z.F, h->cu_count, false);
    void* const xn = few ? h->xf_act : h->xf;
    const XOut to_xn{bf16 ? xn : nullptr, mt, planes, nullptr};
    const SsqTiles tiles{h->ssq_parts, h->ssq, z.d / ADD_COLS};
    const SsqTiles* by_tile = nullptr;   // where the last x was written that way
    auto gemm = [&](int cls, const void* w, int N, int K, Out* o, const void* in_frags, const SsqTiles* sums) -> int {
        const GemmPlan p = plan_gemm(M, N, K, h->cu_count, true);
        // the plan follows process-wide tuning knobs; the buffer was sized with those in force at init
        if (gemm_partial_elems(p, M) > h->partial_cap)
            return fail(SPEC_ERR_SHAPE, "this step's GEMM plan (%d K ranges) needs %zu partial sums, the handle holds %zu: "
                        "set the GEMM tuning knobs before spec_verify_init", p.n_split, gemm_partial_elems(p, M),
                        h->partial_cap);
        o->n_split = p.n_split;
        o->ld = p.n_pad;
        o->stride = (size_t)M * p.n_pad;
        ProfScope ps_(&h->prof, cls, s);
        return launch_gemm_bf16(p, in_frags, w, M, N, K, h->partial, s, sums, n_ssq);
    };
    // x += in * w^T, the next product's operand and the sums of squares, in one launch or two
    auto gemm_resid = [&](int cls, const GemmPlan& p, bool add, const void* w, int K, const void* in_frags, const float* gain) -> int {
        by_tile = add ? &tiles : nullptr;
        if (add) {
            ProfScope ps_(&h->prof, cls, s);
            return launch_gemm_add(p, in_frags, w, M, z.d, K, h->x, gain, xn, h->ssq_parts, s);
        }
        Out r;
        int e = gemm(cls, w, z.d, K, &r, in_frags, nullptr);
        if (e) return e;
        ProfScope ps_(&h->prof, SPEC_PROF_GLUE, s);
        return launch_resid(h->partial, r.n_split, r.stride, r.ld, M, z.d, h->x, h->ssq, gain, to_xn, s);
    };

    if (!embedded) RUN(SPEC_PROF_GLUE, launch_embed(embed_to(h, M), t.row_tok, M, s));
    if (!bf16) {
        if (z.F % 8) return fail(SPEC_ERR_SHAPE, "d_ffn must be a multiple of 8");
        auto mul = [&](int cls, const float* in, const void* w, int N, int K, float* out, int mode, const float* gain) -> int {
            ProfScope ps_(&h->prof, cls, s);
            return launch_gemm_f32(in, (const float*)w, M, N, K, out, s, mode, gain, c.rms_eps);
        };
        for (int l = 0; l < c.n_layers; ++l) {
            const spec_layer_weights& w = h->layers[l];
            if ((rc = mul(SPEC_PROF_GEMM_QKV, h->x, w.w_qkv, z.nqkv, z.d, h->partial, F32_STORE, w.attn_norm))) return rc;
            const QkvSrc qkv{h->partial, 1, 0, z.nqkv, NormScale{nullptr, 0, 0, 0.f}, h->cos_sin};
            rc = launch_attention(c.max_kv_len, h->cu_count, t, ks, B, M, h->geom, c.n_q_heads, l, h->kv_cache, nullptr, nullptr,
                                  nullptr, 0, XOut{nullptr, 0, 0, h->att}, c.max_lookahead + 1, &h->prof, s, &qkv, h->kv_cache);
            if (rc) return rc;
            if ((rc = mul(SPEC_PROF_GEMM_O, h->att, w.w_o, z.d, z.dq, h->x, F32_ADD, nullptr))) return rc;
            if ((rc = mul(SPEC_PROF_GEMM_GATE_UP, h->x, w.w_gate_up, z.F, z.d, h->act, F32_SWIGLU, w.ffn_norm))) return rc;
            if ((rc = mul(SPEC_PROF_GEMM_DOWN, h->act, w.w_down, z.d, z.F, h->x, F32_ADD, nullptr))) return rc;
        }
        return mul(SPEC_PROF_GEMM_LM_HEAD, h->x, h->lm_head, z.V, z.d, logits_out, F32_STORE, h->final_norm);
    }
    Out o;
    const bool fuse = h->fuse_rope && attention_takes_qkv(h->geom, c.n_q_heads, ks, B, c.max_kv_len, h->cu_count);
    for (int l = 0; l < c.n_layers; ++l) {
        const spec_layer_weights& w = h->layers[l];
        rc = gemm(SPEC_PROF_GEMM_QKV, w.w_qkv, z.nqkv, z.d, &o, xn, by_tile);
        if (rc) return rc;
        if (fuse) {
            // the attention kernel adds up, scales and rotates q, k, v itself and appends k, v
            const QkvSrc qkv{h->partial, o.n_split, o.stride, o.ld, scaled, h->cos_sin};
            rc = launch_attention(c.max_kv_len, h->cu_count, t, ks, B, M, h->geom, c.n_q_heads, l, h->kv_cache,
                                  h->q, h->attn_part_o, h->attn_part_ml, h->attn_part_cap, to_xf, c.max_lookahead + 1, &h->prof, s, &qkv,
                                  h->kv_cache);
        } else {
            RUN(SPEC_PROF_GLUE, launch_rope_append(h->partial, o.n_split, o.stride, o.ld, t, M, h->geom, c.n_q_heads, l,
                                                   h->cos_sin, scaled, h->kv_cache, h->q, s));
            rc = launch_attention(c.max_kv_len, h->cu_count, t, ks, B, M, h->geom, c.n_q_heads, l, h->kv_cache,
                                  h->q, h->attn_part_o, h->attn_part_ml, h->attn_part_cap, to_xf, c.max_lookahead + 1, &h->prof, s);
        }
        if (rc) return rc;
        rc = gemm_resid(SPEC_PROF_GEMM_O, plan_o, add_o, w.w_o, z.dq, h->xf, w.ffn_norm);
        if (rc) return rc;
        void* const act = swiglu_in_gemm && !few ? h->xf_act : h->xf;
        if (swiglu_in_gemm) {
            // the gate/up GEMM applies the norm's row scale and SwiGLU itself and writes the down
            // projection's operand (into the fragment buffer that it is not reading)
            RUN(SPEC_PROF_GEMM_GATE_UP, launch_gemm_swiglu(xn, w.w_gate_up, M, z.F, z.d, h->ssq, n_ssq, z.d, c.rms_eps,
                                                   act, mt, h->cu_count, s, by_tile));
        } else {
            rc = gemm(SPEC_PROF_GEMM_GATE_UP, w.w_gate_up, 2 * z.F, z.d, &o, xn, by_tile);
            if (rc) return rc;
            RUN(SPEC_PROF_GLUE, launch_silu_mul(h->partial, o.n_split, o.stride, o.ld, M, z.F, scaled, to_xf, s));
        }
        const float* next_gain = (l + 1 < c.n_layers) ? h->layers[l + 1].attn_norm : h->final_norm;
        rc = gemm_resid(SPEC_PROF_GEMM_DOWN, plan_down, add_down, w.w_down, z.F, act, next_gain);
        if (rc) return rc;
    }
    rc = gemm(SPEC_PROF_GEMM_LM_HEAD, h->lm_head, z.V, z.d, &o, xn, by_tile);
    if (rc) return rc;
    if (last) {
        *last = LogitsSrc{h->partial, o.stride, o.n_split, o.ld, scaled, logits_out};
        return SPEC_OK;
    }
    RUN(SPEC_PROF_GLUE, launch_reduce_splits(h->partial, o.n_split, o.stride, M, z.V, o.ld, h->ssq, n_ssq, z.d, c.rms_eps,
                                             logits_out, s));
#undef RUN
    return SPEC_OK;
}

}  // namespace specv
