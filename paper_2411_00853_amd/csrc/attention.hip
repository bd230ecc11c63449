// Windowed-causal attention of the verify step: the K+1 query tokens of a sequence (times the
// query heads that share a kv head) attend over the sequence's cached positions plus the window
// tokens up to and including themselves.  All queries of a (sequence, kv head) share ONE streamed
// pass over that head's keys and values -- this is why scoring K drafts costs about as much as one
// token (the paper's observation behind speculative sampling) -- so the kernel is bound by reading
// the cache from HBM once, and is organised around that stream:
//
//  * The cache is stored in operand order (cache_layout.h): every 16-byte lane load of a key or
//    value operand is part of a contiguous 1 KiB wavefront read, and a 32-position block (keys then
//    values) is one contiguous 64*hd*2-byte run.  While one block is processed
//    the next is in flight (of 64-dim blocks that come from memory the next three, or two: see NBUF).
//  * Scores are computed transposed (S^T = K * Q^T) so that the exponentiated scores leave the
//    matrix instruction in exactly the register order the second product (O^T = V^T * P^T) wants:
//    no LDS round trip, no cross-lane movement except the 2-step maximum over a query's 4 lanes.
//  * Online softmax in fp32 (base 2), one running maximum and sum per query, per wavefront.
//  * The position range is cut into chunks across wavefronts to fill the machine; chunk results
//    (unnormalised output, maximum, sum) are merged by a second small kernel in a fixed order.
//  * Queries and probabilities enter the bf16 matrix instruction as head + remainder pairs; at a
//    handful of query rows the matrix cores are far from busy, and this keeps the only bf16
//    rounding in the path the one that the cache's storage type imposes.
#include "attention_kernel.h"

namespace specv {
namespace {

// out[m][hq][:] = sum_c w_c o_c / sum_c w_c l_c with w_c = 2^(m_c - max m), chunks in index order.
// One thread per 8 consecutive dims of a (row, query head); the result goes out as the output
// projection's operand fragments.
__global__ void __launch_bounds__(64) attn_merge_kernel(StepTables t, LookaheadPack ks, int n_kv_heads, int n_q_heads,
                                                        int hd, int max_chunks, int r_cap,
                                                        const float* __restrict__ part_o,
                                                        const float* __restrict__ part_ml, XOut xo)
{
    const int per_head = hd / 8;
    const int m = blockIdx.x;
    const int unit = blockIdx.y * 64 + threadIdx.x;       // 8-dim unit within the row
    const int hq = unit / per_head, d8 = unit % per_head;
    if (hq >= n_q_heads) return;
    const int b = t.row_seq[m];
    float v[8] = {0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f};
    if (t.seq_ok[b]) {
        const int group = n_q_heads / n_kv_heads;
        const int j = m - t.seq_row0[b];
        const int r = j * group + hq % group;
        const int total = t.seq_n[b] + ks.k[b] + 1;
        const int ck = seq_chunk_keys(total, max_chunks);
        const int n_chunks = (total + ck - 1) / ck;
        const size_t item0 = ((size_t)b * n_kv_heads + hq / group) * max_chunks;
        // Chunks are taken eight at a time, every load of a batch issued before the first use
        // (indices past the end clamped, their terms dropped), so that a batch costs one memory round
        // trip; a loop that loads, tests and then loads again per chunk pays two per chunk.  The
        // arithmetic is the plain definition: global max first, then the weighted sums in chunk order.
        constexpr int MB = 8;
        auto ml_at = [&](int c) {
            return *reinterpret_cast<const float2*>(part_ml + ((item0 + min(c, n_chunks - 1)) * r_cap + r) * 2);
        };
        float2 ml0[MB];
        float4 oa[MB], ob[MB];
#pragma unroll
        for (int i = 0; i < MB; ++i) {
            ml0[i] = ml_at(i);
            const float* po = part_o + ((item0 + min(i, n_chunks - 1)) * r_cap + r) * hd + d8 * 8;
            oa[i] = *reinterpret_cast<const float4*>(po);
            ob[i] = *reinterpret_cast<const float4*>(po + 4);
        }
        float mx = -INFINITY;
#pragma unroll
        for (int i = 0; i < MB; ++i) mx = fmaxf(mx, i < n_chunks ? ml0[i].x : -INFINITY);
        for (int c0 = MB; c0 < n_chunks; c0 += MB) {
            float2 t2[MB];
#pragma unroll
            for (int i = 0; i < MB; ++i) t2[i] = ml_at(c0 + i);
#pragma unroll
            for (int i = 0; i < MB; ++i) mx = fmaxf(mx, c0 + i < n_chunks ? t2[i].x : -INFINITY);
        }
        float den = 0.f;
        auto add = [&](bool use, float2 ml, const float4& a, const float4& bq) {
            // a chunk entirely after this query's position has max -inf and takes no part
            const bool on = use && ml.x != -INFINITY;
            const float w = on ? exp2f(ml.x - mx) : 0.f;
            den += on ? w * ml.y : 0.f;
            v[0] += on ? w * a.x : 0.f; v[1] += on ? w * a.y : 0.f; v[2] += on ? w * a.z : 0.f; v[3] += on ? w * a.w : 0.f;
            v[4] += on ? w * bq.x : 0.f; v[5] += on ? w * bq.y : 0.f; v[6] += on ? w * bq.z : 0.f; v[7] += on ? w * bq.w : 0.f;
        };
#pragma unroll
        for (int i = 0; i < MB; ++i) add(i < n_chunks, ml0[i], oa[i], ob[i]);
        for (int c0 = MB; c0 < n_chunks; c0 += MB) {
            float2 t2[MB];
#pragma unroll
            for (int i = 0; i < MB; ++i) {
                t2[i] = ml_at(c0 + i);
                const float* po = part_o + ((item0 + min(c0 + i, n_chunks - 1)) * r_cap + r) * hd + d8 * 8;
                oa[i] = *reinterpret_cast<const float4*>(po);
                ob[i] = *reinterpret_cast<const float4*>(po + 4);
            }
#pragma unroll
            for (int i = 0; i < MB; ++i) add(c0 + i < n_chunks, t2[i], oa[i], ob[i]);
        }
        const float inv = 1.0f / den;
#pragma unroll
        for (int e = 0; e < 8; ++e) v[e] *= inv;
    }
    store_x_unit(static_cast<uint4*>(xo.frags), xo.mt, xo.planes, m, unit, v);
}

// Plain fp32 attention for fp32 caches: one workgroup per (row, query head).  It takes the QKV projection as it is: the query
// is rotated here, and so are the keys of the window, which every row that sees them rotates for itself; the workgroup of a kv
// head's first query head puts its own row's key and value into the cache, which this launch reads below the window only.
// LP lanes share a position (four dims each), so keys and values are read in contiguous runs, U positions per group in flight, whose
// sums over the lanes go step by step side by side; the window and (AHEAD) the first U values are requested with the keys.  Latency:
// round trips to memory and across lanes, until a launch has more workgroups than fit (see f32_positions).  U = 8 and AHEAD against a
// rotary/append kernel in front (2.8 us), four positions in flight and the values only after the softmax: steps of two layers, four
// 64-dim heads, one sequence of 128 positions and five rows 61.9 -> 56.8 us, 1000 positions and one row 86.1 -> 76.1, six of 1024 and 48
// rows 141.7 -> 126.8.
// (That kernel, per launch of 20 (row, head) pairs at 133 and 1029 positions: 7.2 and 29.6 us; a thread per key, and one per dim
// walking all values, 9.4 and 80; the number of lanes a run-time value, each sum over the lanes a rolled loop of its own, 10.8 and 41.)
typedef float f32x4u __attribute__((ext_vector_type(4), aligned(4)));
template <int LP, int U, bool AHEAD>
__global__ void __launch_bounds__(256, U == 2 ? 8 : 1)   // (two positions are for eight workgroups on a compute unit)
attn_f32_kernel(const float* __restrict__ qkv, const float* __restrict__ cos_sin, float* cache, float* __restrict__ out, int n_q_heads,
                int layer, int ld, float scale, StepTables t, CacheGeom g)
{
    extern __shared__ float4 dyn[];
    __shared__ float red[4];
    float* osum = reinterpret_cast<float*>(dyn);   // [4][4 * LP] outputs of the wavefronts
    float* sc = osum + 16 * LP;                    // [n_keys] scores
    const int m = blockIdx.x, hq = blockIdx.y;
    const int hd = g.head_dim, half = hd >> 1;
    const int pos = t.row_pos[m], b = t.row_seq[m];
    const uint32_t wmask = t.tree ? t.row_mask[m] : 0xffffffffu;   // chains: n_keys = pos + 1 is the whole rule
    const int n_cached = t.seq_n[b], slot = t.seq_slot[b], row0 = t.seq_row0[b];
    float* dst = out + ((size_t)m * n_q_heads + hq) * hd;
    if (pos < 0) {
        for (int i = threadIdx.x; i < hd; i += 256) dst[i] = 0.f;
        return;
    }
    const int n_keys = pos + 1, window = n_keys - n_cached;   // the row's own place in the window is the last
    const int group = n_q_heads / g.n_kv_heads, hkv = hq / group;
    float* kbase = cache + cache_head_base(g, layer, slot, hkv) + plain_offset(g, 0, 0, 0);
    float* vbase = cache + cache_head_base(g, layer, slot, hkv) + plain_offset(g, 1, 0, 0);
    static_assert((LP & (LP - 1)) == 0 && LP <= 64, "a group of lanes lies within a wavefront");   // 4 * LP >= hd
    constexpr int n_grp = 256 / LP;
    const int sub = threadIdx.x & (LP - 1), grp = threadIdx.x / LP;
    const int d0 = 4 * sub;
    // four dims of a row from d0 on; a head's last lanes may have fewer
    auto load4 = [&](const float* row) -> float4 {
        if (d0 + 4 <= hd) {
            const f32x4u v = *reinterpret_cast<const f32x4u*>(row + d0);
            return make_float4(v.x, v.y, v.z, v.w);
        }
        return make_float4(d0 < hd ? row[d0] : 0.f, d0 + 1 < hd ? row[d0 + 1] : 0.f, d0 + 2 < hd ? row[d0 + 2] : 0.f, 0.f);
    };
    // the same four dims of a head turned to position p
    auto turned4 = [&](const float* row, int p) -> float4 {
        const float* cs = cos_sin + (size_t)p * hd;   // [half][2]
        float r[4], ra, rb;
        if ((hd & 7) == 0 && d0 < hd) {
            const bool lower = d0 < half;
            const int i0 = lower ? d0 : d0 - half;
            const f32x4u a = *reinterpret_cast<const f32x4u*>(row + i0), bb = *reinterpret_cast<const f32x4u*>(row + i0 + half);
            const f32x4u c0 = *reinterpret_cast<const f32x4u*>(cs + 2 * i0), c1 = *reinterpret_cast<const f32x4u*>(cs + 2 * i0 + 4);
            const float co[4] = {c0.x, c0.z, c1.x, c1.z}, si[4] = {c0.y, c0.w, c1.y, c1.w};
#pragma unroll
            for (int e = 0; e < 4; ++e) {
                rotate_pair(a[e], bb[e], co[e], si[e], ra, rb);
                r[e] = lower ? ra : rb;
            }
        } else {
#pragma unroll
            for (int e = 0; e < 4; ++e) {
                const int d = d0 + e;
                r[e] = 0.f;
                if (d < hd) {
                    const int i = d < half ? d : d - half;
                    rotate_pair(row[i], row[i + half], cs[2 * i], cs[2 * i + 1], ra, rb);
                    r[e] = d < half ? ra : rb;
                }
            }
        }
        return make_float4(r[0], r[1], r[2], r[3]);
    };
    auto turn_of = [&](int w) { return t.tree ? t.row_rope[row0 + w] : n_cached + w; };   // depth in the window, not the slot
    // U positions per group and trip, requested together (past the end: the last one again; of an empty cache the first entry, which
    // another workgroup may be writing: nothing is made of what is read)
    float4 v0[AHEAD ? U : 1];
    const int last = max(n_cached - 1, 0);
    const float4 qv = turned4(qkv + (size_t)m * ld + hq * hd, turn_of(window - 1));
    // the window's positions of this group (position k belongs to group k % n_grp), in registers from here on
    constexpr int WN = (SPEC_MAX_LOOKAHEAD + n_grp) / n_grp;
    const int w0 = (grp - n_cached) & (n_grp - 1);
    float4 kw[WN], vw[WN];
#pragma unroll
    for (int i = 0; i < WN; ++i) {
        const int w = min(w0 + i * n_grp, window - 1);
        const float* row = qkv + (size_t)(row0 + w) * ld + (n_q_heads + hkv) * hd;
        kw[i] = turned4(row, turn_of(w));
        vw[i] = load4(row + g.n_kv_heads * hd);
    }
    float mx = -INFINITY;
    auto score = [&](int k, float a, bool on) {
        if (on) {
            if (sub == 0) sc[k] = a;
            mx = fmaxf(mx, a);
        }
    };
    auto dot = [&](const float4& k) { return fmaf(qv.x, k.x, fmaf(qv.y, k.y, fmaf(qv.z, k.z, qv.w * k.w))); };
    auto scores_from = [&](int k0, bool first) {
        float4 kv[U];
#pragma unroll
        for (int i = 0; i < U; ++i) kv[i] = load4(kbase + (size_t)min(k0 + i * n_grp, last) * hd);
        if (AHEAD && first) {
#pragma unroll
            for (int i = 0; i < U; ++i) v0[i] = load4(vbase + (size_t)min(k0 + i * n_grp, last) * hd);
        }
        float a[U];
#pragma unroll
        for (int i = 0; i < U; ++i) a[i] = dot(kv[i]);
#pragma unroll
        for (int o = LP >> 1; o > 0; o >>= 1)   // the positions' sums step by step, side by side
#pragma unroll
            for (int i = 0; i < U; ++i) a[i] += __shfl_xor(a[i], o);
#pragma unroll
        for (int i = 0; i < U; ++i) score(k0 + i * n_grp, a[i] * scale, k0 + i * n_grp < n_cached);
    };
    scores_from(grp, true);   // (all groups: a barrier-free trip whose surplus positions count for nothing)
    for (int k0 = grp + U * n_grp; k0 < n_cached; k0 += U * n_grp) scores_from(k0, false);
    {
        float a[WN];
#pragma unroll
        for (int i = 0; i < WN; ++i) a[i] = dot(kw[i]);
#pragma unroll
        for (int o = LP >> 1; o > 0; o >>= 1)
#pragma unroll
            for (int i = 0; i < WN; ++i) a[i] += __shfl_xor(a[i], o);
#pragma unroll
        for (int i = 0; i < WN; ++i) {   // (a window slot that is not on this row's path: -inf)
            const int w = w0 + i * n_grp;
            score(n_cached + w, (wmask >> (w & 31)) & 1u ? a[i] * scale : -INFINITY, w < window);
        }
    }
    if (hq % group == 0) {   // this row's entry of the cache
#pragma unroll
        for (int i = 0; i < WN; ++i)
            if (w0 + i * n_grp == window - 1) {
                float* kc = kbase + (size_t)pos * hd;
                float* vc = vbase + (size_t)pos * hd;
                const float ke[4] = {kw[i].x, kw[i].y, kw[i].z, kw[i].w}, ve[4] = {vw[i].x, vw[i].y, vw[i].z, vw[i].w};
#pragma unroll
                for (int e = 0; e < 4; ++e)
                    if (d0 + e < hd) {
                        kc[d0 + e] = ke[e];
                        vc[d0 + e] = ve[e];
                    }
            }
    }
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) mx = fmaxf(mx, __shfl_xor(mx, o));
    if ((threadIdx.x & 63) == 0) red[threadIdx.x >> 6] = mx;
    __syncthreads();
    mx = fmaxf(fmaxf(red[0], red[1]), fmaxf(red[2], red[3]));
    __syncthreads();
    float z = 0.f;
    for (int k = threadIdx.x; k < n_keys; k += 256) {
        const float p = expf(sc[k] - mx);
        sc[k] = p;
        z += p;
    }
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) z += __shfl_xor(z, o);
    if ((threadIdx.x & 63) == 0) red[threadIdx.x >> 6] = z;
    __syncthreads();
    z = (red[0] + red[1]) + (red[2] + red[3]);
    float4 o4 = make_float4(0.f, 0.f, 0.f, 0.f);
    // (a position that takes no part has weight zero; its value, which may be anything, is left out)
    auto add = [&](float p, const float4& v) {
        const bool on = p != 0.f;
        o4.x = on ? fmaf(p, v.x, o4.x) : o4.x;
        o4.y = on ? fmaf(p, v.y, o4.y) : o4.y;
        o4.z = on ? fmaf(p, v.z, o4.z) : o4.z;
        o4.w = on ? fmaf(p, v.w, o4.w) : o4.w;
    };
    if constexpr (AHEAD) {
#pragma unroll
        for (int i = 0; i < U; ++i) add(grp + i * n_grp < n_cached ? sc[grp + i * n_grp] : 0.f, v0[i]);
    }
    for (int k0 = AHEAD ? grp + U * n_grp : grp; k0 < n_cached; k0 += U * n_grp) {
        float4 vv[U];
        float p[U];
#pragma unroll
        for (int i = 0; i < U; ++i) {
            const int k = k0 + i * n_grp;
            vv[i] = load4(vbase + (size_t)min(k, last) * hd);
            p[i] = k < n_cached ? sc[k] : 0.f;
        }
#pragma unroll
        for (int i = 0; i < U; ++i) add(p[i], vv[i]);
    }
#pragma unroll
    for (int i = 0; i < WN; ++i) add(w0 + i * n_grp < window ? sc[n_cached + w0 + i * n_grp] : 0.f, vw[i]);
#pragma unroll
    for (int o = LP; o < 64; o <<= 1) {
        o4.x += __shfl_xor(o4.x, o);
        o4.y += __shfl_xor(o4.y, o);
        o4.z += __shfl_xor(o4.z, o);
        o4.w += __shfl_xor(o4.w, o);
    }
    if ((threadIdx.x & 63) < LP) *reinterpret_cast<float4*>(osum + (threadIdx.x >> 6) * 4 * LP + d0) = o4;
    __syncthreads();
    if ((int)threadIdx.x < hd) {
        const int e = threadIdx.x;
        dst[e] = ((osum[e] + osum[4 * LP + e]) + (osum[8 * LP + e] + osum[12 * LP + e])) / z;
    }
}

}  // namespace

static int g_items_per_cu = 0;   // wavefront work items per compute unit to aim for; 0 = default
void set_attn_items_per_cu(int n) { g_items_per_cu = n; }
static int g_max_chunks = 16;   // most chunks per (sequence, kv head)
static bool g_max_chunks_set = false;
void set_attn_max_chunks(int n)
{
    g_max_chunks_set = n >= 1 && n <= 16;
    g_max_chunks = g_max_chunks_set ? n : 16;
}
static int g_merge_min_pairs = 0;   // fewest (sequence, kv head) pairs for merging inside the workgroup; 0 = default
void set_attn_merge_min_pairs(int n) { g_merge_min_pairs = n; }
static int g_small_positions = 2816;   // cache capacity per sequence up to which the small-launch plan applies
void set_attn_small_positions(int n) { g_small_positions = n >= 0 ? n : 2816; }

AttnPlan plan_attention(int max_kv_len, int batch, int n_kv_heads, int cu_count, bool paged)
{
    // One wavefront per (sequence, kv head, position chunk).  Measured on MI355X: a few long
    // streams beat many short ones (each wavefront keeps 16 to 24 KiB in flight and HBM likes
    // long sequential runs), so aim for two wavefronts per compute unit when every sequence is at full
    // length.  Chunks are whole 32-position cache blocks.
    AttnPlan p{};
    const long want_items = (long)(g_items_per_cu > 0 ? g_items_per_cu : 2) * cu_count;
    const long per = (long)batch * n_kv_heads;
    long chunks = want_items / per;
    if (chunks < 1) chunks = 1;
    // Never a single chunk for a long cache: the wavefront whose chunk holds the window first puts the
    // window's keys and values together (4-8 us), and with two chunks per pair the other half of the
    // wavefronts stream meanwhile (plan_launch makes the one exception, where two chunks would not all
    // be resident).
    if (chunks < 2 && max_kv_len >= 1024) chunks = 2;
    if (chunks > g_max_chunks) chunks = g_max_chunks;   // (16 unless set: the merge walks a row's chunks one after the other)
    // a paged wavefront keeps the page numbers of at most 64 blocks, whatever that makes of the chunk count
    if (paged && chunks < (max_kv_len + 2047) / 2048) chunks = (max_kv_len + 2047) / 2048;
    long keys = (max_kv_len + chunks - 1) / chunks;
    keys = (keys + 31) / 32 * 32;
    p.chunk_keys = (int)keys;
    p.max_chunks = (max_kv_len + p.chunk_keys - 1) / p.chunk_keys;
    return p;
}

// A wavefront holds at most 64 query rows (four row tiles) of one kv head: (query heads per kv head) x
// (window length).  When a step's longest window gives more, the query heads of a kv head are dealt to
// kv_share work items of group / kv_share heads each -- to the kernel they look like kv heads of their
// own that happen to read the same cache head, which is then streamed kv_share times.  The smallest
// divisor of the group that brings the rows down to 64 (a window has at most 16 rows, so one exists).
static int attn_kv_share(int group, int window)
{
    for (int s = 1; s < group; ++s)
        if (group % s == 0 && (group / s) * window <= 64) return s;
    return group;
}

size_t attn_partial_floats(int max_kv_len, int max_batch, int n_kv_heads, int group, int max_window, int hd,
                           int cu_count, bool paged)
{
    size_t worst = 0;
    for (int share = 1; share <= group; ++share) {
        if (group % share) continue;
        for (int b = 1; b <= max_batch; ++b) {
            const AttnPlan p = plan_attention(max_kv_len, b, n_kv_heads * share, cu_count, paged);
            const size_t e = (size_t)b * n_kv_heads * p.max_chunks * group * max_window * hd;
            if (e > worst) worst = e;
        }
    }
    return worst;
}


// wavefronts per workgroup for a launch with max_chunks chunks per (sequence, kv head): 1, 2, 4 or 8,
// or 0 when the chunks go to memory and attn_merge_kernel merges them
// (a workgroup sits on ONE compute unit: with few (sequence, kv head) pairs and many chunks each,
// merging inside the workgroup would leave most of the chip idle -- measured slower for the draft
// model's 64 pairs x 8 chunks -- so it needs at least half as many workgroups as compute units)
// (any_pairs: a small launch, see plan_launch, merges in the workgroup however few pairs it has)
static int merge_width(int hd, int rt, int max_chunks, int n_pairs, int cu_count, bool any_pairs)
{
    const int cw = max_chunks <= 1 ? 1 : max_chunks <= 2 ? 2 : max_chunks <= 4 ? 4 : max_chunks <= 8 ? 8 : 0;
    const int need = g_merge_min_pairs > 0 ? g_merge_min_pairs : cu_count / 2;
    return cw > 0 && merge_fits(hd, rt, cw) && (any_pairs || n_pairs >= need) ? cw : 0;
}

// What a launch does with its (sequence, kv head) pairs: how many work items share a cache head
// (attn_kv_share, at least what the row limit asks for) and how the positions are cut.
// Small launches -- at most an eighth as many pairs as compute units and short caches -- are bound by
// latency, not by the stream: there a kv
// head's query heads are spread over more work items while those still fit on half the compute units
// (duplicate reads hit L2), each item is cut into at most four chunks, and the four wavefronts merge
// inside their workgroup -- one kernel where there were three (rotary/append, chunks, merge).
// Measured at the 1B-shape (8 kv heads x 4 query heads), per step: batch 1 at 1024 positions 1.017 ->
// 0.948 ms, at 2048 1.071 -> 1.012, at 2560 1.061 -> 1.045, at 3072 1.065 -> 1.077, at 4096 1.083 ->
// 1.134 (one block in flight per wavefront: chunks of a thousand positions are latency-bound);
// batch 4 at 3072 1.214 -> 1.193, batch 8 at 2304 1.320 -> 1.279, batch 12 at 2048 1.758 -> 1.696.
// The same model as the draft of a decoding round at batch 8 (one or two rows per sequence, 2300
// positions) loses 1.8 % per round with it, so the plan stops at 32 pairs (batch 4 of this shape).
// Hence a limit on the cache capacity per sequence (counted in positions of 64-dim heads: a 128-dim
// head moves twice the bytes per position).  Only with several query heads per kv head: the work items
// of one kv head then read the same blocks and most of the traffic stays in L2; with one head per kv
// head every workgroup streams from HBM through a single compute unit, and the plan loses (7B-shape,
// 32 x 128-dim kv heads, batch 1 at 1024 positions: 3.35 -> 3.44 ms, at 2048 3.47 -> 3.73, batch 3 4.04 -> 4.07).
constexpr int BRIEF_POSITIONS = 512;    // capacity of a slot, in positions of 128-dim heads, up to which workgroups always merge
constexpr int FUSED_MIN_KEYS = 192;   // fewest positions per chunk for the attention to put queries, keys and values together itself
struct AttnLaunchPlan {
    int share;
    AttnPlan p;
    bool small;
    bool brief;   // merged inside the workgroup however few pairs there are
};
static AttnLaunchPlan plan_launch(const CacheGeom& g, bool paged, int n_q_heads, int kmax, int B, int max_kv_len,
                                  int cu_count)
{
    AttnLaunchPlan lp{};
    const int group = n_q_heads / g.n_kv_heads;
    lp.share = attn_kv_share(group, kmax + 1);
    lp.small = group >= 2 && B * g.n_kv_heads * 8 <= cu_count && (long)max_kv_len * g.head_dim <= 64L * g_small_positions
               && !g_max_chunks_set && g_merge_min_pairs == 0 && g_items_per_cu == 0;
    if (lp.small)
        for (int s = lp.share + 1; s <= group; ++s)
            if (group % s == 0 && B * g.n_kv_heads * s <= cu_count / 2) lp.share = s;
    lp.p = plan_attention(max_kv_len, B, g.n_kv_heads * lp.share, cu_count, paged);
    // The variant that puts queries, keys and values together itself needs, at 128-dim heads, more than
    // half a SIMD's registers (the prologue parks values in the accumulation registers): one wavefront
    // per SIMD, 4 per compute unit.  Where two chunks per pair overflow those slots and one chunk per pair
    // fits them, one chunk, all wavefronts resident at once, is faster (7B-shape, 2048 positions,
    // attention per layer: batch 20 161 -> 140 us, batch 24 176 -> 163, batch 28 and 32 -2 %; 32 sequences
    // of 512..4096 positions 8.74 -> 8.55 ms per step; from batch 40 on, where neither fits, two chunks win).
    // The 64-dim variants of one and two row tiles have one wavefront per SIMD as well, by a few registers; the rule was
    // measured with 128-dim heads and holds for those only.
    {
        const long pairs = (long)B * g.n_kv_heads * lp.share, slots = 4L * cu_count;
        const int rt1 = ((kmax + 1) * (group / lp.share) + 15) / 16;
        if (g.head_dim == 128 && rt1 == 1 && lp.p.max_chunks == 2 && lp.p.chunk_keys >= 192 && !lp.small && !paged
            && !g_max_chunks_set && g_items_per_cu == 0 && pairs <= slots && 2 * pairs > slots) {
            lp.p.chunk_keys = (max_kv_len + 31) / 32 * 32;
            lp.p.max_chunks = 1;
        }
    }
    // (a paged wavefront holds the page numbers of at most 64 blocks: no chunk beyond 2048 positions)
    const int few = std::max(4, paged ? (max_kv_len + 2047) / 2048 : 1);
    if (lp.small && lp.p.max_chunks > few) {
        lp.p.chunk_keys = ((max_kv_len + few - 1) / few + 31) / 32 * 32;
        lp.p.max_chunks = (max_kv_len + lp.p.chunk_keys - 1) / lp.p.chunk_keys;
    }
    const int rt = ((kmax + 1) * (group / lp.share) + 15) / 16;
    const long pairs = (long)B * g.n_kv_heads * lp.share;
    // Both rules below are for few query rows: a wavefront finishes an item's queries and the window by itself, and where several
    // items share a cache head each of them finishes the window's keys and values again.  Steps of two layers up to 330 positions,
    // without this line: 64-dim heads, 52 rows an item +0.5..+5 %, 32 rows -2..-7; 128-dim heads, 16 rows of a shared head
    // +4..+12 %, 26 and 52 rows +1..+7, 13 to 16 of a head of their own -3..+3.5, 9 to 12 rows (143 steps up to 550 positions) -8.5..+5.1,
    // -0.7 on average, up to 8 (68 steps) -21..+1, -6.6 on average.
    // And for 128-dim heads only while their wavefronts, one to a SIMD, are all resident: 1056 pairs 0..+1.4 %, 840 -3.5.
    const int rows = (kmax + 1) * (group / lp.share);
    const bool few_rows = g.head_dim == 64 ? rows <= (lp.share > 1 ? 16 : 32) : lp.share == 1 && rows <= 12 && pairs <= 4L * cu_count;
    const bool own = few_rows && !g_max_chunks_set && g_merge_min_pairs == 0 && g_items_per_cu == 0;   // (no knob set)
    auto cut = [&](int keys) {
        lp.p.chunk_keys = keys;
        lp.p.max_chunks = (max_kv_len + keys - 1) / keys;
    };
    // Short slots: a few wavefronts of one compute unit stream them in less time than chunk results through memory and the merge
    // kernel take, however few pairs there are.  Up to four chunks, merged in the workgroup; steps of four layers, 1 to 8
    // sequences, up to 127 pairs, before -> with this: 40 to 360 positions of 128-dim heads -2..-8 % (7B shape 382 -> 370 us, 8 heads of
    // a 1024 wide model 159 -> 146), of 64-dim heads -5..-8, 700 of them -2..-4.  At 700 positions of 128-dim heads -1.5..+11 %, at
    // 1100 0..+10, 1800 of 64-dim heads +1.5..+5: a compute unit's share of the stream decides, so the limit counts bytes.
    lp.brief = lp.small;
    if (own && (long)max_kv_len * g.head_dim <= 128L * BRIEF_POSITIONS) {
        lp.brief = true;
        const int keys = std::max(FUSED_MIN_KEYS, ((max_kv_len + 3) / 4 + 31) / 32 * 32);
        if (lp.p.chunk_keys < keys && merge_width(g.head_dim, rt, (max_kv_len + keys - 1) / keys, (int)pairs, cu_count, true) > 0) cut(keys);
    }
    // Chunks shorter than FUSED_MIN_KEYS would have the separate rotary/append kernel in front.  Fewer, longer chunks that do
    // without it are the faster choice (same steps, without the rule above):
    //  * 64-dim heads, a block of which is half as long to stream: 250 to 900 positions -2..-6 %, 1400 to 2500 -4..-9; short
    //    slots of the small-launch plan -3..-5
    //  * beyond 1024 positions, 128-dim heads too (9 to 16 chunks of 128 before): 1400 positions -3..-4.5 % at the 7B shape, -6..-9 with
    //    8 heads of a 1024 wide model, 2500 positions -2..-5.  Up to 8 rows: 88 steps of four layers, 1 to 16 heads of their own, 1 to
    //    23 sequences, -2.8 % on average, +2.4 at most; 9 to 12 rows, 72 of them, 0 on average, -5.6..+6.7 and most of the losses
    //    at 1300 to 2400 positions (5 sequences of 7 heads, 10 rows, 1053 to 2106 positions: a step of one layer 90.0 -> 94.7 us)
    //  * up to 384 positions with single rows, or where one or two chunks still give a quarter of the compute units a
    //    workgroup: 7B shape 8 x 300 positions -2.5 %, 32 x 48 -2; 32 prompts of 64, 352 rows -2.2 (one chunk per pair: no
    //    wavefront repeats another's queries, the kernel in front took 20 us a layer)
    // Between 384 and 1024 positions of 128-dim heads it loses (8 heads, one sequence at 550: +2.5..+6 %) and is not made.
    if (own && lp.p.chunk_keys < FUSED_MIN_KEYS && fused_fits(g.head_dim, rt)
        && (g.head_dim == 64 || lp.small || (max_kv_len > 1024 && rows <= 8) || (max_kv_len <= 2 * FUSED_MIN_KEYS && (kmax == 0 || 4 * pairs >= cu_count))))
        cut(FUSED_MIN_KEYS);
    // Two blocks: measured over 0..128 positions, 7B-shape paged step 5.04 -> 4.95 ms, decoding round 6.69 -> 6.62 ms,
    // contiguous 7B-shape, tree and long-context steps 0.2-0.7 % shorter, nothing longer (32 and 96 positions, an
    // odd number of blocks with two buffers, were slower than none).  With the window attended to from LDS: a draft model's
    // decode at batch 8 339.0 us with none, 337.9 with 32, 331.6 with 64; the other steps within 0.5 %.
    lp.p.lag_keys = 64;
    return lp;
}


AttnDescription describe_attention(const CacheGeom& g, bool paged, int n_q_heads, int kmax, int B, int max_kv_len,
                                   int max_window, int cu_count)
{
    AttnDescription d{};
    const AttnLaunchPlan lp = plan_launch(g, paged, n_q_heads, kmax, B, max_kv_len, cu_count);
    const int group = n_q_heads / (g.n_kv_heads * lp.share);
    d.share = lp.share;
    d.small = lp.small ? 1 : 0;
    d.max_chunks = lp.p.max_chunks;
    d.chunk_keys = lp.p.chunk_keys;
    d.row_tiles = ((kmax + 1) * group + 15) / 16;
    d.wavefronts = d.row_tiles >= 1 && d.row_tiles <= 4
                       ? merge_width(g.head_dim, d.row_tiles, lp.p.max_chunks, B * g.n_kv_heads * lp.share, cu_count, lp.brief)
                       : 0;
    d.fused = fused_fits(g.head_dim, d.row_tiles) && lp.p.chunk_keys >= FUSED_MIN_KEYS ? 1 : 0;
    d.partial_floats = (size_t)B * g.n_kv_heads * lp.share * lp.p.max_chunks * group * max_window * g.head_dim;
    return d;
}

bool attention_takes_qkv(const CacheGeom& g, int n_q_heads, const LookaheadPack& ks, int B, int max_kv_len, int cu_count)
{
    if (g.dtype != SPEC_DTYPE_BF16) return false;
    int kmax = 0;
    for (int b = 0; b < B; ++b) kmax = ks.k[b] > kmax ? ks.k[b] : kmax;
    const AttnLaunchPlan lp = plan_launch(g, g.table != nullptr, n_q_heads, kmax, B, max_kv_len, cu_count);
    const int rt = ((kmax + 1) * (n_q_heads / g.n_kv_heads / lp.share) + 15) / 16;
    if (!fused_fits(g.head_dim, rt)) return false;
    // Every wavefront of a (sequence, kv head) puts the queries together again: with short chunks
    // (few sequences, many chunks each) that costs more than the separate kernel it replaces
    // (measured: batch 1 at 1B-shape, 128-position chunks, 2 % slower; 256-position chunks faster).
    return lp.p.chunk_keys >= FUSED_MIN_KEYS;
}

// Lanes of attn_f32_kernel that share a position, four dims each (head_dim <= 256: spec_verify_init sees to it)
static int f32_lanes(int hd)
{
    int lp = 1;
    while (4 * lp < hd) lp *= 2;
    return lp;
}

// Positions that a group of lanes of attn_f32_kernel requests together.  Eight, with the first values ahead, while four workgroups to a
// compute unit are all there are: they take 113 registers (64-dim heads), and the scores of slots from some 8000 positions on leave room
// for no more either.  Beyond, more workgroups resident: four positions, and two from 16 workgroups to a compute unit on.
// Steps of two layers, us with a rotary/append kernel in front and four positions, with eight, four and two (1024 workgroups are four to
// a compute unit):
//   positions   4 heads of 64, 1024   8 of 64, 2 kv heads, 2048    the same, 8192 (4000: 4096)   2 of 128, 2048     2 of 256, 1024
//       8         98   96   93   91       123 127 117 115            251  286  248  244          161 173 162 159    151 162 151 155
//     100        104  101   98   99       128 128 122 123            271  294  269  271          187 192 184 183    173 193 172 181
//     400        125  123  118  121       155 162 148 148            446  455  438  421          273 270 274 264    259 295 258 264
//    1000        166  160  158  165       220 218 218 209            870  780  879  759          481 450 486 453    450 519 440 451
//    4000         -                       676 629 719  -            1666 1333 1711 1284            -                  -
// Between, two positions lose where the last few workgroups start alone: 8 heads of 64 dims, 2176 workgroups, 1000 and 2500 positions 311
// 297 308 324 and 602 558 581 653; and four against eight where these come out even (2048 workgroups of long slots, up to 16 %).
constexpr size_t LDS_BYTES = 160 * 1024;   // of a compute unit
static int f32_positions(int hd, long wgs, size_t lds, int cu_count)
{
    const bool few = hd > 128 ? wgs <= 2L * cu_count : hd > 64 ? wgs < 4L * cu_count : wgs <= 4L * cu_count;
    if (few || 5 * lds > LDS_BYTES) return 8;
    return hd <= 128 && wgs >= 16L * cu_count && 8 * lds <= LDS_BYTES ? 2 : 4;
}

int launch_attention(int max_kv_len, int cu_count, const StepTables& t, const LookaheadPack& ks, int B, int M, const CacheGeom& g,
                     int n_q_heads, int layer, const void* cache, const float* q, float* part_o, float* part_ml,
                     size_t part_cap, const XOut& xo, int max_window, Profiler* prof, hipStream_t s, const QkvSrc* qkv,
                     void* cache_w)
{
    QkvSrc src{};
    if (qkv) src = *qkv;
    const int hd = g.head_dim;
    const float scale = 1.0f / sqrtf((float)hd);
    if (g.dtype != SPEC_DTYPE_BF16) {
        if (!src.partial || src.n_split != 1 || src.ns.ssq || !cache_w) return fail(SPEC_ERR_SHAPE, "fp32 attention takes whole, normalised projections");
        // scores for one row live in LDS: positions * 4 bytes
        if ((size_t)(hd + g.t_pad) * sizeof(float) > 60 * 1024) return fail(SPEC_ERR_SHAPE, "fp32 attention supports max_kv_len up to ~15000");
        ProfScope ps(prof, SPEC_PROF_ATTENTION, s);
        const size_t lds = (size_t)(16 * f32_lanes(hd) + g.t_pad) * sizeof(float);
        const int u = f32_positions(hd, (long)M * n_q_heads, lds, cu_count);
#define SPECV_F32(LP, U)                                                                                                     \
    hipLaunchKernelGGL((attn_f32_kernel<LP, U, U == 8>), dim3(M, n_q_heads), dim3(256), lds, s, src.partial, src.cos_sin,    \
                       (float*)cache_w, xo.plain, n_q_heads, layer, src.ld, scale, t, g)
#define SPECV_ATTN_F32(LP)                 \
    case LP:                               \
        if (u == 8) SPECV_F32(LP, 8);      \
        else if (u == 4) SPECV_F32(LP, 4); \
        else SPECV_F32(LP, 2);             \
        break
        switch (f32_lanes(hd)) {
            SPECV_ATTN_F32(1);
            SPECV_ATTN_F32(2);
            SPECV_ATTN_F32(4);
            SPECV_ATTN_F32(8);
            SPECV_ATTN_F32(16);
            SPECV_ATTN_F32(32);
        default:
            if (u == 8) SPECV_F32(64, 8);
            else SPECV_F32(64, 4);
        }
#undef SPECV_F32
#undef SPECV_ATTN_F32
        SPECV_LAUNCH_CHECK("attn_f32_kernel");
        return SPEC_OK;
    }
    int kmax = 0;
    for (int b = 0; b < B; ++b) kmax = ks.k[b] > kmax ? ks.k[b] : kmax;
    const AttnLaunchPlan lp = plan_launch(g, g.table != nullptr, n_q_heads, kmax, B, max_kv_len, cu_count);
    const int share = lp.share;
    const int n_items_kv = g.n_kv_heads * share;          // (sequence, kv head) work items per sequence
    const AttnPlan p = lp.p;
    if (g.table && p.chunk_keys > 2048)
        return fail(SPEC_ERR_SHAPE, "paged attention handles chunks of up to 2048 positions, this plan has %d", p.chunk_keys);
    const int group = n_q_heads / n_items_kv;             // query heads of one work item
    const int r_cap = group * max_window;
    const size_t part_need = (size_t)B * n_items_kv * p.max_chunks * r_cap * hd;
    if (part_need > part_cap)
        return fail(SPEC_ERR_SHAPE, "this step's attention plan (%d chunks per sequence and kv head) needs %zu floats of "
                    "chunk results, the handle holds %zu: set the attention tuning knobs before spec_verify_init",
                    p.max_chunks, part_need, part_cap);
    const int rt = ((kmax + 1) * group + 15) / 16;
    const dim3 grid(p.max_chunks, n_items_kv, B), wg_grid(n_items_kv, B);
    const float sl2 = scale * 1.4426950408889634f;
    if (hd != 64 && hd != 128) return fail(SPEC_ERR_SHAPE, "bf16 attention needs head_dim 64 or 128");
    const int cw = rt >= 1 && rt <= 4 ? merge_width(hd, rt, p.max_chunks, B * n_items_kv, cu_count, lp.brief) : 0;
    int rc;
    {
        ProfScope ps(prof, SPEC_PROF_ATTENTION, s);
        // several work items per cache head: its second reader should find it in the caches
        if (share > 1)
            rc = launch_chunks_reuse(hd, rt, cw, grid, wg_grid, s, t, g, n_q_heads, share, layer, cache, q, p, r_cap, sl2,
                                     part_o, part_ml, src, cache_w, xo);
        else if (hd == 128)
            rc = launch_chunks<128, true>(rt, cw, grid, wg_grid, s, t, g, n_q_heads, share, layer, cache, q, p, r_cap, sl2,
                                          part_o, part_ml, src, cache_w, xo);
        else
            rc = launch_chunks<64, true>(rt, cw, grid, wg_grid, s, t, g, n_q_heads, share, layer, cache, q, p, r_cap, sl2,
                                         part_o, part_ml, src, cache_w, xo);
    }
    if (rc) return rc;
    if (cw > 0) return SPEC_OK;   // the workgroups merged their chunks themselves
    ProfScope ps(prof, SPEC_PROF_ATTN_MERGE, s);
    hipLaunchKernelGGL(attn_merge_kernel, dim3(M, (n_q_heads * hd / 8 + 63) / 64), dim3(64), 0, s, t, ks, n_items_kv,
                       n_q_heads, hd, p.max_chunks, r_cap, part_o, part_ml, xo);
    SPECV_LAUNCH_CHECK("attn_merge_kernel");
    return SPEC_OK;
}

}  // namespace specv
