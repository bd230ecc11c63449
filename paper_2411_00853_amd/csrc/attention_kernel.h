// The chunk kernel of the windowed-causal attention and its launch table, shared by the two
// translation units that instantiate it: attention.hip (keys and values fetched with streaming loads:
// every byte is read once per launch) and attention_reuse.hip (ordinary loads, for launches in which
// several work items stream the same cache head).  See attention.hip for the design.
#pragma once

#include "cache_layout.h"
#include "common.h"
#include "frag.h"
#include "splits.h"

namespace specv {
namespace {

__device__ __forceinline__ void split_frag(const float (&x)[8], Frag& hi, Frag& lo)
{
#pragma unroll
    for (int e = 0; e < 8; ++e) {
        const __bf16 hb = static_cast<__bf16>(x[e]);
        hi.v[e] = hb;
        lo.v[e] = static_cast<__bf16>(x[e] - static_cast<float>(hb));
    }
}

// A sequence's positions are cut into max_chunks equal runs of whole 32-position blocks (at least
// 128 positions each), from its own current length: the launch is sized for the longest sequence
// the cache can hold, but a shorter one still spreads over all of its wavefronts.
__device__ __forceinline__ int seq_chunk_keys(int total, int max_chunks)
{
    const int per = (total + max_chunks - 1) / max_chunks;
    return max((per + 31) & ~31, 128);
}

// PAGED: the blocks of a slot are looked up in the page table.  A wavefront keeps the page numbers
// of its chunk's (at most 64) blocks one per lane and broadcasts the one it needs, so the address
// of a prefetch never waits for memory.
// FUSED: the kernel takes the QKV projection's partial sums instead of finished queries: every
// wavefront adds up, scales and rotates the queries it needs, and the wavefront whose chunk holds
// window positions does the same for the window's keys and values of its kv head and stores them in
// the cache (for later steps) -- so no separate rotary/append kernel runs between the projection and the
// attention.  It attends to them from a copy in LDS that patches the blocks they belong to, so nothing waits for
// those stores, and the requests for the queries and for the window go out in one stretch, before the first of either
// is used.  (Waiting for the stores, fetching the block again and walking the two parts one after the other was
// slower: 33.8 against 31.7 us per launch for a draft model of 16 kv heads at batch 8, 237.5 against 232.8 with 32
// ragged sequences on the page pool, 52.4 against 51.4 at the 7B-shape, batch 8.)
// CW > 0: one workgroup of CW wavefronts per (sequence, kv head), wavefront c taking chunk c; the
// chunk results meet in LDS and the workgroup itself writes the merged, normalised output as the
// output projection's operand fragments (same arithmetic and order as attn_merge_kernel): no second
// kernel, no round trip of the chunk results through memory.  CW == 0: one wavefront per workgroup,
// chunk results to part_o / part_ml for attn_merge_kernel (more chunks than a workgroup can hold).
// STREAM: the keys and values are fetched with non-temporal loads.  A launch reads every byte of them
// exactly once, and marked that way they pass the caches without displacing what is reused (7B-shape:
// 58.7 -> 54.2 us per launch, Dyn 8.5 -> 7.9 ms of attention per step).  Launches in which several
// work items stream the same cache head take the other variant: there the second reader is served
// from the memory-side cache, and streaming loads cost the 1B-shape step 5 % of its attention time.
typedef unsigned int kv_u32x4 __attribute__((ext_vector_type(4)));
template <bool STREAM>
__device__ __forceinline__ kv_u32x4 kv_load(const kv_u32x4* p)
{
    if constexpr (STREAM) return __builtin_nontemporal_load(p);
    else return *p;
}

template <int HD, int RT, bool PAGED, bool FUSED, int CW, bool STREAM>
__global__ void __launch_bounds__(CW > 0 ? 64 * CW : 64)
    attn_chunk_kernel(const SeqDesc* seq_desc, const kv_u32x4* cache, int max_chunks, int lag_keys, int n_q_heads, int kv_share,
                      int layer, int r_cap, float scale_log2e, const float* __restrict__ q, StepTables t, CacheGeom g,
                      float* __restrict__ part_o, float* __restrict__ part_ml, QkvSrc src, uint16_t* cache_w, XOut xo)
{
    constexpr int STEPS = HD / 32;     // 32-dim steps of the score product
    constexpr int DT = HD / 16;        // 16-dim tiles of the output
    const int lane = threadIdx.x & 63, c16 = lane & 15, gq = lane >> 4;
    // The chunk is the same for a whole wavefront, and the compiler has to know: everything that follows from it is
    // then scalar and the loops over blocks and window positions branch instead of masking lanes.  (Taken as a
    // vector value, the compiler restored registers parked in the accumulation registers behind a masked loop, where
    // no lane was active.)
    const int wave = CW > 0 ? __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6)) : 0;
    // grid: (head items, sequences by falling length), in front of them the chunks where a workgroup takes one
    const int chunk = CW > 0 ? wave : (int)blockIdx.x;
    // kv_share > 1: the query heads of one kv head are dealt to kv_share work items ("hkv" counts those,
    // "group" is the heads of one item), which all stream the keys and values of cache head hkc
    const int n_items_kv = g.n_kv_heads * kv_share;
    const int hkv = CW > 0 ? blockIdx.x : blockIdx.y, hkc = hkv / kv_share;
    const int group = n_q_heads / n_items_kv;
    const int4* desc = reinterpret_cast<const int4*>(seq_desc + (CW > 0 ? blockIdx.y : blockIdx.z));   // scalar, like the chunk
    const int4 d0 = desc[0], d1 = desc[1];
    const int b = __builtin_amdgcn_readfirstlane(d0.x), row0 = __builtin_amdgcn_readfirstlane(d0.y);
    const int K = __builtin_amdgcn_readfirstlane(d0.z), n = __builtin_amdgcn_readfirstlane(d0.w);
    const int slot = __builtin_amdgcn_readfirstlane(d1.x), ok = __builtin_amdgcn_readfirstlane(d1.y);
    const int rows = (K + 1) * group;
    if (!ok) {
        if constexpr (CW > 0) {   // rows of a skipped sequence: zero operand rows, as the merge kernel writes them
            const float z[8] = {0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f};
            for (int u = threadIdx.x; u < rows * (HD / 8); u += 64 * CW) {
                const int r = u / (HD / 8), d8 = u % (HD / 8);
                store_x_unit(static_cast<uint4*>(xo.frags), xo.mt, xo.planes, row0 + r / group,
                             (hkv * group + r % group) * (HD / 8) + d8, z);
            }
        }
        return;
    }
    const int total = n + K + 1;
    // Equal chunks, except that the chunks before the last are lag_keys longer when the last one stays
    // long enough: its wavefront first puts the window's keys and values together (FUSED), and with a
    // shorter run to stream afterwards it ends with the others instead of after them.
    int ck = seq_chunk_keys(total, max_chunks);
    if (lag_keys > 0) {
        const int n_used = (total + ck - 1) / ck;
        if (n_used >= 2 && total - (n_used - 1) * (ck + lag_keys) >= 2 * lag_keys + 64 && (!PAGED || ck + lag_keys <= 2048))
            ck += lag_keys;
    }
    const int key0 = chunk * ck;
    const bool active = chunk < max_chunks && key0 < total;
    if constexpr (CW == 0) {
        if (!active) return;
    }
    const int dq = n_q_heads * HD;
    floatx4 acc[RT][DT];
    float m_run[RT], l_run[RT];
#pragma unroll
    for (int rt = 0; rt < RT; ++rt) {
        m_run[rt] = -INFINITY;
        l_run[rt] = 0.f;
#pragma unroll
        for (int d = 0; d < DT; ++d) acc[rt][d] = floatx4{0.f, 0.f, 0.f, 0.f};
    }
    if (active) {
    const int key1 = min(key0 + ck, total);

    const int blk0 = key0 >> 5, blk1 = (key1 + 31) >> 5;
    const kv_u32x4* head;
    int my_page = 0;
    if constexpr (PAGED) {
        head = cache + ((size_t)layer * g.n_kv_heads + hkc) * (64 * HD) / 8;   // offset inside a page
        const int p = g.table[(size_t)slot * g.blocks_per_slot + min(blk0 + lane, blk1 - 1)];
        my_page = p < 0 ? 0 : p;
    } else {
        head = cache + cache_head_base(g, layer, slot, hkc) / 8;
    }
    const size_t blk_u4 = g.blk_stride / 8;   // from one block of this head to the next (contiguous cache)

    // Blocks in registers.  128-dim heads: one processed, the next in flight (16 KiB).  64-dim blocks are half as
    // large, so of those that come from memory three are kept in flight: with one, 512 wavefronts had 4 MB under way,
    // which a memory round trip of about 1 us turns into 4.4 TB/s (28.4 -> 26.6 us at 32 sequences of 8 kv heads).
    // Out of a cache (kv_share > 1) the round trip is short and the fourth buffer only costs registers: a step at
    // the 1B shape, batch 1, takes 842 us with it and 827 without.
    // Four buffers and four ranges at a time (W0 below) take 258-268 registers at one and two row tiles: one wavefront
    // on a SIMD.  Three and two take 196-231: two.  Steps of four layers, three and two against four and four: 512 wavefronts
    // -0.3..-0.6 %, 1024 +1.0..+1.6, 2048 -0.8..-3.3, 4096 -1.4..-1.6; 1B shape, batch 32 +0.6, batch 1 +0.5, batch 8 -1.4.  The
    // variants of eight wavefronts have to fit two on a SIMD, spilled with four (36 bytes a lane), and take three:
    // 16 sequences of 15900 positions, 256 pairs, 422.6 -> 417.2 us per step.
    constexpr int NBUF = HD == 128 || !STREAM ? 2 : CW == 8 ? 3 : 4;
    kv_u32x4 kbuf[NBUF][2][STEPS], vbuf[NBUF][DT];
    // Unconditional loads: with no branch around them the compiler counts outstanding loads exactly and the
    // prefetch stays in flight.  Past the chunk's end every lane reads the same 16 bytes of its last block,
    // a few lines instead of a block nobody needs.
    auto load_block = [&](int blk, kv_u32x4(&kk)[2][STEPS], kv_u32x4(&vv)[DT]) {
        const int bb = min(blk, blk1 - 1), at = blk < blk1 ? lane : 0;
        const kv_u32x4* p;
        if constexpr (PAGED)
            p = head + (size_t)__builtin_amdgcn_readlane(my_page, bb - blk0) * (g.page_stride / 8) + at;
        else
            p = head + (size_t)bb * blk_u4 + at;
#pragma unroll
        for (int sub = 0; sub < 2; ++sub)
#pragma unroll
            for (int s = 0; s < STEPS; ++s) kk[sub][s] = kv_load<STREAM>(p + sub * (2 * HD) + s * 64);
#pragma unroll
        for (int d = 0; d < DT; ++d) vv[d] = kv_load<STREAM>(p + 4 * HD + d * 64);
    };
    load_block(blk0, kbuf[0], vbuf[0]);   // the stream starts before anything else is fetched

    // queries, pre-scaled by log2(e)/sqrt(hd), as bf16 head + remainder operand fragments
    Frag qh[RT][STEPS], ql[RT][STEPS];
    int n_vis[RT];           // cached positions below this are visible to the query (0 for padding rows)
    uint32_t wmask[RT];      // window slots (positions n + i) the query attends to
    // FUSED: a request for a row tile's queries or for eight window positions fetches the first W0 ranges of 16
    // float4 columns' worth, the row's sums of squares and its rotary factors; the rest of a longer list is
    // fetched when the request is finished.  (Two ranges where four do not fit: 128-dim heads, and eight wavefronts per workgroup.)
    constexpr int QC = 2 * STEPS, W0 = HD == 128 || CW == 8 ? 2 : 4;
    // Several lanes share a row: each fetches one pair of its sums of squares and they pass them around, so that
    // a row of up to four pairs (4096 columns) costs a lane one 16-byte load and four registers.
    auto scale_issue = [&](int m, int sub, double2& r) { r = src.ns.ssq[(size_t)m * src.ns.n_ssq + min(sub, src.ns.n_ssq - 1)]; };
    // (lane0 + i * stride: the lane that fetched pair i; the arithmetic of row_inv_rms)
    auto scale_finish = [&](int m, const double2& r, int lane0, int stride) -> float {
        const float own = (float)(r.x + r.y);
        float ss = 0.f;
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            const float v = __shfl(own, lane0 + i * stride);
            ss += i < src.ns.n_ssq ? v : 0.f;
        }
        for (int i = 4; i < src.ns.n_ssq; ++i) {
            const double2 v = src.ns.ssq[(size_t)m * src.ns.n_ssq + i];
            ss += (float)(v.x + v.y);
        }
        return 1.0f / sqrtf(ss / (float)src.ns.d + src.ns.eps);
    };
    auto range_issue = [&](const float* p, float4(&a)[W0]) {
#pragma unroll
        for (int i = 0; i < W0; ++i) a[i] = *reinterpret_cast<const float4*>(p + (size_t)min(i, src.n_split - 1) * src.stride);
    };
    auto range_finish = [&](const float4(&a)[W0]) -> float4 {   // ranges in index order
        float4 v = a[0];
#pragma unroll
        for (int i = 1; i < W0; ++i) {
            const bool on = i < src.n_split;
            v.x += on ? a[i].x : 0.f; v.y += on ? a[i].y : 0.f; v.z += on ? a[i].z : 0.f; v.w += on ? a[i].w : 0.f;
        }
        return v;
    };
    struct QRaw {
        float4 a[QC][W0], cs[STEPS / 2][4];
        double2 ss;
        const float* p;
        int m;
    };
    auto q_issue = [&](int rt, QRaw& r) {
        const int rr = rt * 16 + c16;
        const bool real = rr < rows;
        const int j = real ? rr / group : 0, hl = real ? rr % group : 0;
        r.m = row0 + j;
        r.p = src.partial + (size_t)r.m * src.ld + (hkv * group + hl) * HD + 8 * gq;   // 8 dims of every 32-dim step
        scale_issue(r.m, gq, r.ss);
#pragma unroll
        for (int c = 0; c < QC; ++c) range_issue(r.p + 32 * (c >> 1) + 4 * (c & 1), r.a[c]);
        const int rpos = t.tree ? t.row_rope[r.m] : n + j;
        const float* cs = src.cos_sin + (size_t)rpos * HD + 2 * (8 * gq);   // [HD/2][2] per position
#pragma unroll
        for (int s = 0; s < STEPS / 2; ++s)
#pragma unroll
            for (int e4 = 0; e4 < 4; ++e4) r.cs[s][e4] = *reinterpret_cast<const float4*>(cs + 2 * (32 * s) + 4 * e4);
    };
    // Add up, scale, rotate and split them: dims d and d + HD/2 (a rotary pair) sit in steps s and
    // s + STEPS/2 of the same lane.
    auto q_finish = [&](int rt, const QRaw& r, float sc) {
        const float rs = scale_finish(r.m, r.ss, c16, 16);
        float4 sums[QC];
#pragma unroll
        for (int c = 0; c < QC; ++c) sums[c] = range_finish(r.a[c]);
        if (src.n_split > W0) {
            const float* cols[QC];
#pragma unroll
            for (int c = 0; c < QC; ++c) cols[c] = r.p + 32 * (c >> 1) + 4 * (c & 1) + W0 * src.stride;
            add_splits4_many<QC, W0>(cols, src.n_split - W0, src.stride, sums);
        }
        float raw[STEPS][8];
#pragma unroll
        for (int s = 0; s < STEPS; ++s) {
            const float4 a = sums[2 * s], b = sums[2 * s + 1];
            raw[s][0] = a.x * rs; raw[s][1] = a.y * rs; raw[s][2] = a.z * rs; raw[s][3] = a.w * rs;
            raw[s][4] = b.x * rs; raw[s][5] = b.y * rs; raw[s][6] = b.z * rs; raw[s][7] = b.w * rs;
        }
#pragma unroll
        for (int s = 0; s < STEPS / 2; ++s) {
            float x0[8], x1[8];
#pragma unroll
            for (int e4 = 0; e4 < 4; ++e4) {
                const float4 c2 = r.cs[s][e4];   // cos,sin of 2 dims
                const float ca[2] = {c2.x, c2.z}, sa[2] = {c2.y, c2.w};
#pragma unroll
                for (int h2 = 0; h2 < 2; ++h2) {
                    const int e = 2 * e4 + h2;
                    rotate_pair(raw[s][e], raw[s + STEPS / 2][e], ca[h2], sa[h2], x0[e], x1[e]);
                    x0[e] *= sc;
                    x1[e] *= sc;
                }
            }
            split_frag(x0, qh[rt][s], ql[rt][s]);
            split_frag(x1, qh[rt][s + STEPS / 2], ql[rt][s + STEPS / 2]);
        }
    };
#pragma unroll
    for (int rt = 0; rt < RT; ++rt) {
        const int r = rt * 16 + c16;
        const bool real = r < rows;
        const int j = real ? r / group : 0, hl = real ? r % group : 0;
        n_vis[rt] = real ? n : 0;
        wmask[rt] = !real ? 0u : (t.tree ? t.row_mask[row0 + j] : (2u << j) - 1u);
        if constexpr (!FUSED) {
            const float sc = real ? scale_log2e : 0.f;   // rows past the window contribute zeros
            const float4* qsrc = reinterpret_cast<const float4*>(q + (size_t)(row0 + j) * dq + (hkv * group + hl) * HD + 8 * gq);
#pragma unroll
            for (int s = 0; s < STEPS; ++s) {
                const float4 a = qsrc[8 * s], b = qsrc[8 * s + 1];
                const float x[8] = {a.x * sc, a.y * sc, a.z * sc, a.w * sc, b.x * sc, b.y * sc, b.z * sc, b.w * sc};
                split_frag(x, qh[rt][s], ql[rt][s]);
            }
        }
    }
    // the window's keys [slot][dim] and values [dim][slot] (bf16), each position put there by the wavefront
    // whose chunk it falls into and read by that wavefront only
    constexpr int WK_LD = HD + 8, WV_LD = 18;
    static_assert(SPEC_MAX_LOOKAHEAD < 16, "a window has at most 16 positions");
    __shared__ __align__(16) uint16_t s_wk[FUSED ? 16 * WK_LD : 8], s_wv[FUSED ? HD * WV_LD : 8];
    if constexpr (FUSED) {
        QRaw q0;
        q_issue(0, q0);
        // The window's keys (rotated) and values of this kv head that fall into this chunk.  HD/8
        // lanes share a position (each 4 rotary pairs of the key and 8 dims of the value), so a
        // wavefront covers 8 positions per trip in rounds of 64 / (HD/8), all of a trip requested together.
        const int w0 = max(key0, n), w1 = key1;   // positions [w0, w1) are window slots of this chunk
        if (w0 < w1) {
            constexpr int HALF = HD / 2, LP = HD / 8, PPR = 64 / LP, NR = 8 / PPR;
            const int u = lane / LP, tq = lane % LP;
            const int kcol = n_q_heads * HD + hkc * HD, vcol = (n_q_heads + g.n_kv_heads) * HD + hkc * HD;
            for (int p0 = w0; p0 < w1; p0 += 8) {
                float4 raw[NR][4][W0], cs[NR][2];
                double2 ssr[NR];
                int posr[NR];
                auto col = [&](int h, int x) {
                    const float* prow = src.partial + (size_t)(row0 + (posr[h] - n)) * src.ld;
                    return x == 0 ? prow + kcol + 4 * tq : x == 1 ? prow + kcol + HALF + 4 * tq : prow + vcol + 8 * tq + 4 * (x - 2);
                };
#pragma unroll
                for (int h = 0; h < NR; ++h) {
                    posr[h] = min(p0 + PPR * h + u, w1 - 1);   // clamped: the loads are unconditional
                    const int m = row0 + (posr[h] - n);
                    scale_issue(m, tq, ssr[h]);
#pragma unroll
                    for (int x = 0; x < 4; ++x) range_issue(col(h, x), raw[h][x]);
                    const float* c2 = src.cos_sin + (size_t)(t.tree ? t.row_rope[m] : posr[h]) * HD + 2 * (4 * tq);
                    cs[h][0] = *reinterpret_cast<const float4*>(c2);
                    cs[h][1] = *reinterpret_cast<const float4*>(c2 + 4);
                }
#pragma unroll
                for (int h = 0; h < NR; ++h) {
                    const float rs = scale_finish(row0 + (posr[h] - n), ssr[h], u * LP, 1);
                    float4 kv4[4];
#pragma unroll
                    for (int x = 0; x < 4; ++x) kv4[x] = range_finish(raw[h][x]);
                    if (src.n_split > W0) {
                        const float* cols[4] = {col(h, 0) + W0 * src.stride, col(h, 1) + W0 * src.stride, col(h, 2) + W0 * src.stride,
                                                col(h, 3) + W0 * src.stride};
                        add_splits4_many<4, W0>(cols, src.n_split - W0, src.stride, kv4);
                    }
                    const float a[4] = {kv4[0].x * rs, kv4[0].y * rs, kv4[0].z * rs, kv4[0].w * rs};
                    const float bk[4] = {kv4[1].x * rs, kv4[1].y * rs, kv4[1].z * rs, kv4[1].w * rs};
                    const float v[8] = {kv4[2].x * rs, kv4[2].y * rs, kv4[2].z * rs, kv4[2].w * rs,
                                        kv4[3].x * rs, kv4[3].y * rs, kv4[3].z * rs, kv4[3].w * rs};
                    const float co[4] = {cs[h][0].x, cs[h][0].z, cs[h][1].x, cs[h][1].z};
                    const float si[4] = {cs[h][0].y, cs[h][0].w, cs[h][1].y, cs[h][1].w};
                    size_t blk;
                    if constexpr (PAGED)
                        blk = (size_t)__shfl(my_page, (posr[h] >> 5) - blk0) * g.page_stride + ((size_t)layer * g.n_kv_heads + hkc) * (64 * HD);
                    else
                        blk = cache_block_base(g, layer, slot, hkc, posr[h] >> 5);
                    if (p0 + PPR * h + u < w1) {
                        const int t32 = posr[h] & 31, w = posr[h] - n;
                        union {
                            ushort4 v;
                            uint16_t h[4];
                        } k0, k1;
#pragma unroll
                        for (int e = 0; e < 4; ++e) {
                            float ra, rb;
                            rotate_pair(a[e], bk[e], co[e], si[e], ra, rb);
                            k0.h[e] = __builtin_bit_cast(uint16_t, static_cast<__bf16>(ra));
                            k1.h[e] = __builtin_bit_cast(uint16_t, static_cast<__bf16>(rb));
                        }
                        *reinterpret_cast<ushort4*>(s_wk + w * WK_LD + 4 * tq) = k0.v;
                        *reinterpret_cast<ushort4*>(s_wk + w * WK_LD + 4 * tq + HALF) = k1.v;
                        *reinterpret_cast<ushort4*>(cache_w + blk + tiled_k_within(HD, t32, 4 * tq)) = k0.v;
                        *reinterpret_cast<ushort4*>(cache_w + blk + tiled_k_within(HD, t32, 4 * tq + HALF)) = k1.v;
#pragma unroll
                        for (int e = 0; e < 8; ++e) {
                            const uint16_t vb = __builtin_bit_cast(uint16_t, static_cast<__bf16>(v[e]));
                            s_wv[(8 * tq + e) * WV_LD + w] = vb;
                            cache_w[blk + tiled_v_within(HD, t32, 8 * tq + e)] = vb;
                        }
                    }
                }
            }
            __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");   // the copy in LDS is read by other lanes
        }
        auto q_scale = [&](int rt) { return rt * 16 + c16 < rows ? scale_log2e : 0.f; };   // rows past the window contribute zeros
        if constexpr (RT == 1) {
            q_finish(0, q0, q_scale(0));
        } else {
            QRaw q1;   // the next row tile's request goes out before a tile is finished
#pragma unroll
            for (int rt = 0; rt < RT; ++rt) {
                QRaw& cur = rt & 1 ? q1 : q0;
                if (rt + 1 < RT) q_issue(rt + 1, rt & 1 ? q0 : q1);
                q_finish(rt, cur, q_scale(rt));
            }
        }
    }

    auto process = [&](int blk, kv_u32x4(&kk)[2][STEPS], kv_u32x4(&vv)[DT]) {
        const int kbase = blk * 32;
        const bool tail = kbase + 32 > n;   // reaches the window / the end: mask per element
        if (tail) {
            if constexpr (FUSED) {   // the window's own entries from LDS
#pragma unroll
                for (int sub = 0; sub < 2; ++sub) {
                    const int w = kbase + 16 * sub + c16 - n;
                    const bool in = w >= 0 && w <= K;
#pragma unroll
                    for (int s = 0; s < STEPS; ++s) {
                        const kv_u32x4 l = *reinterpret_cast<const kv_u32x4*>(s_wk + (in ? w : 0) * WK_LD + 8 * (4 * s + gq));
                        kk[sub][s] = in ? l : kk[sub][s];
                    }
                }
#pragma unroll
                for (int d = 0; d < DT; ++d) {
#pragma unroll
                    for (int e2 = 0; e2 < 4; ++e2) {   // two positions
                        const int w = kbase + (e2 < 2 ? 4 * gq + 2 * e2 : 12 + 4 * gq + 2 * e2) - n;
                        const bool i0 = w >= 0 && w <= K, i1 = w + 1 >= 0 && w + 1 <= K;
                        const uint16_t* l = s_wv + (16 * d + c16) * WV_LD;
                        const uint32_t own = l[i0 ? w : 0] | (uint32_t)l[i1 ? w + 1 : 0] << 16;
                        const uint32_t mask = (i0 ? 0xffffu : 0u) | (i1 ? 0xffff0000u : 0u);
                        vv[d][e2] = (vv[d][e2] & ~mask) | (own & mask);
                    }
                }
            }
            // values of positions that do not exist yet may hold anything: zero them
#pragma unroll
            for (int d = 0; d < DT; ++d) {
#pragma unroll
                for (int e2 = 0; e2 < 4; ++e2) {
                    const int key = kbase + (e2 < 2 ? 4 * gq + 2 * e2 : 12 + 4 * gq + 2 * e2);
                    vv[d][e2] &= (key < total ? 0xffffu : 0u) | (key + 1 < total ? 0xffff0000u : 0u);
                }
            }
        }
#pragma unroll
        for (int rt = 0; rt < RT; ++rt) {
            floatx4 st[2];
#pragma unroll
            for (int sub = 0; sub < 2; ++sub) {
                st[sub] = floatx4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
                for (int s = 0; s < STEPS; ++s) {
                    const bf16x8 kf = __builtin_bit_cast(bf16x8, kk[sub][s]);
                    st[sub] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(kf, qh[rt][s].v, st[sub], 0, 0, 0);
                    st[sub] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(kf, ql[rt][s].v, st[sub], 0, 0, 0);
                }
            }
            float sv[8];
#pragma unroll
            for (int e = 0; e < 8; ++e) sv[e] = st[e >> 2][e & 3];
            if (tail) {
#pragma unroll
                for (int e = 0; e < 8; ++e) {
                    const int key = kbase + (e < 4 ? 4 * gq + e : 16 + 4 * gq + e - 4);
                    const int w = key - n;   // window slot, if >= 0
                    const bool vis = key < n_vis[rt] || (w >= 0 && w < 32 && ((wmask[rt] >> w) & 1u));
                    if (!vis) sv[e] = -INFINITY;
                }
            }
            float mx = sv[0];
#pragma unroll
            for (int e = 1; e < 8; ++e) mx = fmaxf(mx, sv[e]);
            mx = fmaxf(mx, __shfl_xor(mx, 16));
            mx = fmaxf(mx, __shfl_xor(mx, 32));
            // The reference exponent m_run of a row only moves when a score exceeds it by more than
            // 8 (weights stay below 2^8, far inside fp32 and the two-plane split): after the first
            // blocks that is rare, and a trip in which no row of the wavefront moves skips the
            // rescaling of the accumulators -- 32 multiplications and as many register moves each way,
            // about as many issue cycles as the block's matrix products.  Sums and outputs stay
            // relative to m_run, which is all the merge needs.
            const bool move = mx > m_run[rt] + 8.f;
            if (__builtin_amdgcn_ballot_w64(move) != 0) {
                const float m_to = move ? mx : m_run[rt];
                const float m_fin = (m_to == -INFINITY) ? 0.f : m_to;
                const float alpha = move ? __builtin_amdgcn_exp2f(m_run[rt] - m_fin) : 1.f;
                m_run[rt] = m_to;
                l_run[rt] *= alpha;
#pragma unroll
                for (int d = 0; d < DT; ++d) {
                    acc[rt][d][0] *= alpha; acc[rt][d][1] *= alpha; acc[rt][d][2] *= alpha; acc[rt][d][3] *= alpha;
                }
            }
            const float m_use = (m_run[rt] == -INFINITY) ? 0.f : m_run[rt];
            float ps = 0.f;
#pragma unroll
            for (int e = 0; e < 8; ++e) {
                sv[e] = __builtin_amdgcn_exp2f(sv[e] - m_use);   // arguments <= 8; far below -126 the result is 0
                ps += sv[e];
            }
            l_run[rt] += ps;
            Frag ph, pl;
            split_frag(sv, ph, pl);
#pragma unroll
            for (int d = 0; d < DT; ++d) {
                const bf16x8 vf = __builtin_bit_cast(bf16x8, vv[d]);
                floatx4 a = acc[rt][d];
                a = __builtin_amdgcn_mfma_f32_16x16x32_bf16(vf, ph.v, a, 0, 0, 0);
                a = __builtin_amdgcn_mfma_f32_16x16x32_bf16(vf, pl.v, a, 0, 0, 0);
                acc[rt][d] = a;
            }
        }
    };

#pragma unroll
    for (int u = 1; u < NBUF - 1; ++u) load_block(blk0 + u, kbuf[u], vbuf[u]);
    for (int blk = blk0; blk < blk1; blk += NBUF) {
#pragma unroll
        for (int u = 0; u < NBUF; ++u) {
            load_block(blk + u + NBUF - 1, kbuf[(u + NBUF - 1) % NBUF], vbuf[(u + NBUF - 1) % NBUF]);
            if (u == 0 || blk + u < blk1) process(blk + u, kbuf[u], vbuf[u]);
        }
    }
    }   // active

    if constexpr (CW == 0) {
#pragma unroll
        for (int rt = 0; rt < RT; ++rt) {
            float l = l_run[rt];
            l += __shfl_xor(l, 16);
            l += __shfl_xor(l, 32);
            const int r = rt * 16 + c16;
            if (r < rows) {
                const size_t item = ((size_t)b * n_items_kv + hkv) * max_chunks + chunk;
                float* o = part_o + (item * r_cap + r) * HD + 4 * gq;
#pragma unroll
                for (int d = 0; d < DT; ++d)
                    *reinterpret_cast<float4*>(o + 16 * d) = make_float4(acc[rt][d][0], acc[rt][d][1], acc[rt][d][2], acc[rt][d][3]);
                if (gq == 0) {
                    part_ml[(item * r_cap + r) * 2 + 0] = m_run[rt];
                    part_ml[(item * r_cap + r) * 2 + 1] = l;
                }
            }
        }
    } else {
        // chunk results of the CW wavefronts -> LDS -> merged rows as operand fragments
        __shared__ float s_o[CW][RT * 16][HD];
        __shared__ float s_m[CW][RT * 16], s_l[CW][RT * 16];
        static_assert(CW == 0 || sizeof(float) * CW * RT * 16 * (HD + 2) <= 64 * 1024, "chunk results fit in LDS");
#pragma unroll
        for (int rt = 0; rt < RT; ++rt) {
            float l = l_run[rt];
            l += __shfl_xor(l, 16);
            l += __shfl_xor(l, 32);
            const int r = rt * 16 + c16;
#pragma unroll
            for (int d = 0; d < DT; ++d)
                *reinterpret_cast<float4*>(&s_o[chunk][r][16 * d + 4 * gq]) =
                    make_float4(acc[rt][d][0], acc[rt][d][1], acc[rt][d][2], acc[rt][d][3]);
            if (gq == 0) {
                s_m[chunk][r] = m_run[rt];
                s_l[chunk][r] = l;
            }
        }
        __syncthreads();
        // out = sum_c w_c o_c / sum_c w_c l_c with w_c = 2^(m_c - max m), chunks in index order
        for (int u = threadIdx.x; u < rows * (HD / 8); u += 64 * CW) {
            const int r = u / (HD / 8), d8 = u % (HD / 8);
            float mx = -INFINITY;
#pragma unroll
            for (int c = 0; c < CW; ++c) mx = fmaxf(mx, s_m[c][r]);
            float den = 0.f;
            float v[8] = {0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f};
#pragma unroll
            for (int c = 0; c < CW; ++c) {
                const float mc = s_m[c][r];
                const bool on = mc != -INFINITY;   // a chunk entirely after this query's position (or empty)
                const float w = on ? exp2f(mc - mx) : 0.f;
                den += on ? w * s_l[c][r] : 0.f;
                const float4 a = *reinterpret_cast<const float4*>(&s_o[c][r][8 * d8]);
                const float4 bq = *reinterpret_cast<const float4*>(&s_o[c][r][8 * d8 + 4]);
                v[0] += on ? w * a.x : 0.f; v[1] += on ? w * a.y : 0.f; v[2] += on ? w * a.z : 0.f; v[3] += on ? w * a.w : 0.f;
                v[4] += on ? w * bq.x : 0.f; v[5] += on ? w * bq.y : 0.f; v[6] += on ? w * bq.z : 0.f; v[7] += on ? w * bq.w : 0.f;
            }
            const float inv = 1.0f / den;
#pragma unroll
            for (int e = 0; e < 8; ++e) v[e] *= inv;
            store_x_unit(static_cast<uint4*>(xo.frags), xo.mt, xo.planes, row0 + r / group,
                         (hkv * group + r % group) * (HD / 8) + d8, v);
        }
    }
}

// The variants with 128-dim heads and three or four row tiles have no registers left for the fused
// prologue (they would spill); those shapes keep the separate rotary/append kernel.
constexpr bool fused_fits(int hd, int rt) { return !(hd == 128 && rt >= 3); }

// Workgroups of cw wavefronts can merge their chunk results themselves when those fit in 64 KiB of
// LDS, and with 8 wavefronts only where two of them fit on a SIMD (64-dim heads, one row tile).
constexpr bool merge_fits(int hd, int rt, int cw)
{
    return cw * rt * 16 * (hd + 2) * 4 <= 64 * 1024 && (cw < 8 || (hd == 64 && rt == 1));
}

template <int HD, bool STREAM>
static int launch_chunks(int rt, int cw, dim3 grid, dim3 wg_grid, hipStream_t s, const StepTables& t,
                         const CacheGeom& g, int n_q_heads, int kv_share, int layer, const void* cache, const float* q,
                         const AttnPlan& p, int r_cap, float sl2, float* part_o, float* part_ml, const QkvSrc& src,
                         void* cache_w, const XOut& xo)
{
    const int lag_keys = src.partial ? p.lag_keys : 0;   // only the fused prologue delays a wavefront
#define SPECV_ATTN_CW(RT, PG, FU, CW_)                                                                         \
    hipLaunchKernelGGL((attn_chunk_kernel<HD, RT, PG, FU, CW_, STREAM>), CW_ > 0 ? wg_grid : grid, dim3(CW_ > 0 ? 64 * CW_ : 64), \
                       0, s, t.seq_desc, (const kv_u32x4*)cache, p.max_chunks, lag_keys, n_q_heads, kv_share, layer, r_cap, sl2, q, t, g, \
                       part_o, part_ml, src, (uint16_t*)cache_w, xo)
#define SPECV_ATTN_GO(RT, PG, FU)                                                                              \
    do {                                                                                                         \
        if (cw == 1) SPECV_ATTN_CW(RT, PG, FU, 1);                                                               \
        else if (cw == 2) { if constexpr (merge_fits(HD, RT, 2)) SPECV_ATTN_CW(RT, PG, FU, 2); }                 \
        else if (cw == 4) { if constexpr (merge_fits(HD, RT, 4)) SPECV_ATTN_CW(RT, PG, FU, 4); }                 \
        else if (cw == 8) { if constexpr (merge_fits(HD, RT, 8)) SPECV_ATTN_CW(RT, PG, FU, 8); }                 \
        else SPECV_ATTN_CW(RT, PG, FU, 0);                                                                       \
    } while (0)
#define SPECV_ATTN(RT)                                                                                           \
    do {                                                                                                         \
        if (src.partial) {                                                                                       \
            if constexpr (fused_fits(HD, RT)) {                                                                  \
                if (g.table) SPECV_ATTN_GO(RT, true, true);                                                      \
                else SPECV_ATTN_GO(RT, false, true);                                                             \
            } else {                                                                                             \
                return fail(SPEC_ERR_SHAPE, "attention variant cannot take unfinished queries");                 \
            }                                                                                                    \
        } else if (g.table) SPECV_ATTN_GO(RT, true, false);                                                      \
        else SPECV_ATTN_GO(RT, false, false);                                                                    \
    } while (0)
    switch (rt) {
    case 1: SPECV_ATTN(1); break;
    case 2: SPECV_ATTN(2); break;
    case 3: SPECV_ATTN(3); break;
    case 4: SPECV_ATTN(4); break;
    default: return fail(SPEC_ERR_SHAPE, "attention supports at most 64 query rows per kv head");
    }
#undef SPECV_ATTN
#undef SPECV_ATTN_GO
#undef SPECV_ATTN_CW
    SPECV_LAUNCH_CHECK("attn_chunk_kernel");
    return SPEC_OK;
}

}  // namespace

// launch_chunks<HD, false>, compiled in attention_reuse.hip
int launch_chunks_reuse(int hd, int rt, int cw, dim3 grid, dim3 wg_grid, hipStream_t s, const StepTables& t,
                        const CacheGeom& g, int n_q_heads, int kv_share, int layer, const void* cache,
                        const float* q, const AttnPlan& p, int r_cap, float sl2, float* part_o, float* part_ml,
                        const QkvSrc& src, void* cache_w, const XOut& xo);

}  // namespace specv
