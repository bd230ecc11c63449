// The small kernels between the GEMMs and attention.  Each one also adds up the K-range partial
// sums of the GEMM before it (fixed order), so the projections never need a separate reduction
// pass: embedding + RMSNorm, residual add + RMSNorm, SiLU gating, rotary embedding + KV append.
#include "cache_layout.h"
#include "common.h"
#include "embed.h"
#include "frag.h"
#include "splits.h"

namespace specv {
namespace {

constexpr int TPB = 256;

// x = E[token], one wavefront per (row, SSQ_CHUNK columns)
template <typename T>
__global__ void __launch_bounds__(64) embed_kernel(const T* __restrict__ E, const int32_t* __restrict__ row_tok, float* __restrict__ x,
                                                   const float* __restrict__ gain, double2* __restrict__ ssq, int d, XOut xo)
{
    const int m = blockIdx.y;
    EmbedRow<T> row;
    row.load(E, row_tok[m], blockIdx.x, d);
    embed_chunk(row, m, blockIdx.x, gridDim.x, d, x, gain, xo, ssq);
}

// One wavefront per (row, SSQ_CHUNK columns), 8 columns per lane: x += partial sums;
// ssq[m][chunk] = sum x^2 over the chunk; x * gain goes out as the next GEMM's operand.  d is a multiple of 8.
// Latency up to a hundred rows, then the partial sums and the fragment stores (16 bytes into a line each); single
// wavefronts spread best over the chip: 352 rows of 4096 with eight ranges 12.1 us as workgroups of two, 10.1
// as single ones; a wavefront per 16 rows x 32 columns, whose stores are contiguous, 10.9 (and slower at 48 rows).
__global__ void __launch_bounds__(64) resid_kernel(const float* __restrict__ partial, float* __restrict__ x, size_t split_stride,
                                                   int n_split, int ld, int d, int xmt, void* frags, const float* __restrict__ gain,
                                                   double2* __restrict__ ssq, int planes)
{
    const int m = blockIdx.y, k8 = blockIdx.x * 64 + threadIdx.x;
    double ss = 0.0;
    if (k8 * 8 < d) {
        float v[8];
        float* xp = x + (size_t)m * d + k8 * 8;
        const float4 a = *reinterpret_cast<const float4*>(xp), b = *reinterpret_cast<const float4*>(xp + 4);
        const float* pp = partial + (size_t)m * ld + k8 * 8;
        const float* cols[2] = {pp, pp + 4};
        float4 sums[2];
        sum_ranges(cols, n_split, split_stride, sums);   // up to 8 ranges in one round trip
        const float4 pa = sums[0], pb = sums[1];
        v[0] = a.x + pa.x; v[1] = a.y + pa.y; v[2] = a.z + pa.z; v[3] = a.w + pa.w;
        v[4] = b.x + pb.x; v[5] = b.y + pb.y; v[6] = b.z + pb.z; v[7] = b.w + pb.w;
        *reinterpret_cast<float4*>(xp) = make_float4(v[0], v[1], v[2], v[3]);
        *reinterpret_cast<float4*>(xp + 4) = make_float4(v[4], v[5], v[6], v[7]);
#pragma unroll
        for (int i = 0; i < 8; ++i) ss += (double)v[i] * v[i];
        emit_operand(XOut{frags, xmt, planes, nullptr}, m, k8, v, gain);
    }
    store_ssq(ssq, m, gridDim.x, blockIdx.x, ss);
}

// act[m][f] = silu(gate) * up for 8 consecutive f per thread, gate and up first scaled by the row's
// 1/rms (the FFN norm's scale, see NormScale).  The GEMM's columns come in 16-wide tiles alternating gate
// and up (see spec_pack_weight).  The result goes out as the down projection's operand.  F is a multiple of 8.
// A wavefront covers 16 rows x 32 columns, lane 16 * g + r the 8 columns from 8 * g on of row r: what it stores is
// one contiguous 1 KiB of the fragment buffer per plane, while its rows are still read in 128-byte runs.  Along a
// row every 16-byte store opened a line of its own, and those stores were most of the time (352 x 11008, one
// range: 18.6 us, 7.5 without them; this way 12.1 in the step, 20.4 before).
__global__ void __launch_bounds__(TPB) silu_mul_kernel(const float* __restrict__ partial, int n_split, size_t split_stride,
                                                       int ld, int M, int F, NormScale ns, XOut xo)
{
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const int m = blockIdx.y * 16 + (lane & 15);
    const int k8 = (blockIdx.x * (TPB / 64) + wave) * 4 + (lane >> 4), f = k8 * 8;
    if (m >= M || f >= F) return;
    const float* pg = partial + (size_t)m * ld + ((f >> 4) << 5) + (f & 15);
    const float* cols[4] = {pg, pg + 4, pg + 16, pg + 20};
    float4 sums[4];
    const float r = row_inv_rms(ns.ssq, ns.n_ssq, m, ns.d, ns.eps);
    sum_ranges(cols, n_split, split_stride, sums);   // one memory round trip for all four
    const float4 g0 = sums[0], g1 = sums[1], u0 = sums[2], u1 = sums[3];
    const float g[8] = {g0.x, g0.y, g0.z, g0.w, g1.x, g1.y, g1.z, g1.w};
    const float u[8] = {u0.x, u0.y, u0.z, u0.w, u1.x, u1.y, u1.z, u1.w};
    float v[8];
#pragma unroll
    for (int e = 0; e < 8; ++e) {
        const float ge = g[e] * r;
        v[e] = ge / (1.f + expf(-ge)) * (u[e] * r);
    }
    emit_operand(xo, m, k8, v, nullptr);
}

// Sum the partial ranges, rotate q and k heads at the row's absolute position (pairs (i, i+hd/2), angle from the
// table), write q, and put k and v -- rounded to the cache's storage type -- into the row's slot at that position.
// bf16 caches: a thread takes eight rotary pairs of a q or k head, or sixteen dims of a v head; a wavefront 16 rows x 4
// such units, so that neighbouring positions of a window, which are neighbours in the cache's tiles, are stored
// together (keys 16 bytes each in runs, values 2 bytes each).  A lane per dim along a row took 23 us for 352 rows
// of 96 128-dim heads, most of it the stores; this way 18.
__global__ void __launch_bounds__(TPB) rope_append_tiled_kernel(const float* __restrict__ partial, int n_split,
                                                                size_t split_stride, int ld, StepTables t, CacheGeom g,
                                                                int n_q_heads, int M, int layer, const float* __restrict__ cos_sin,
                                                                NormScale ns, uint16_t* cache, float* __restrict__ q_out)
{
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const int m = blockIdx.y * 16 + (lane & 15);
    const int hd = g.head_dim, half = hd >> 1, per = hd >> 4;       // units per head (a power of two)
    const int unit = (blockIdx.x * (TPB / 64) + wave) * 4 + (lane >> 4);
    const int head = unit / per, u = unit % per;
    if (m >= M || head >= n_q_heads + 2 * g.n_kv_heads) return;
    const int pos = t.row_pos[m];
    const int rope_pos = t.tree ? t.row_rope[m] : max(pos, 0);
    const int slot = t.seq_slot[t.row_seq[m]];
    const bool is_v = head >= n_q_heads + g.n_kv_heads;
    const float* row = partial + (size_t)m * ld + head * hd;
    const float* lo = is_v ? row + 16 * u : row + 8 * u;
    const float* hi = is_v ? lo + 8 : lo + half;
    const float* cols[4] = {lo, lo + 4, hi, hi + 4};
    const float rs = row_inv_rms(ns.ssq, ns.n_ssq, m, ns.d, ns.eps);   // the attention norm's row scale
    float4 sums[4];
    sum_ranges(cols, n_split, split_stride, sums);
    const float a[8] = {sums[0].x * rs, sums[0].y * rs, sums[0].z * rs, sums[0].w * rs,
                        sums[1].x * rs, sums[1].y * rs, sums[1].z * rs, sums[1].w * rs};
    const float b[8] = {sums[2].x * rs, sums[2].y * rs, sums[2].z * rs, sums[2].w * rs,
                        sums[3].x * rs, sums[3].y * rs, sums[3].z * rs, sums[3].w * rs};
    auto bits = [](float v) { return __builtin_bit_cast(uint16_t, static_cast<__bf16>(v)); };
    if (is_v) {
        if (pos < 0) return;   // row of a skipped sequence: no cache write
        uint16_t* c = cache + cache_block_base(g, layer, slot, head - n_q_heads - g.n_kv_heads, pos >> 5);
#pragma unroll
        for (int e = 0; e < 8; ++e) {
            c[tiled_v_within(hd, pos & 31, 16 * u + e)] = bits(a[e]);
            c[tiled_v_within(hd, pos & 31, 16 * u + 8 + e)] = bits(b[e]);
        }
        return;
    }
    const float* cs = cos_sin + (size_t)rope_pos * hd + 16 * u;   // [half][2]; depth in the window, not the slot
    float ra[8], rb[8];
#pragma unroll
    for (int e = 0; e < 8; e += 2) {
        const float4 c2 = *reinterpret_cast<const float4*>(cs + 2 * e);   // cos, sin of two dims
        rotate_pair(a[e], b[e], c2.x, c2.y, ra[e], rb[e]);
        rotate_pair(a[e + 1], b[e + 1], c2.z, c2.w, ra[e + 1], rb[e + 1]);
    }
    if (head < n_q_heads) {
        const bool live = pos >= 0;   // row of a skipped sequence: defined output
        float* q = q_out + (size_t)m * n_q_heads * hd + head * hd + 8 * u;
#pragma unroll
        for (int e = 0; e < 8; e += 4) {
            *reinterpret_cast<float4*>(q + e) = live ? make_float4(ra[e], ra[e + 1], ra[e + 2], ra[e + 3]) : make_float4(0.f, 0.f, 0.f, 0.f);
            *reinterpret_cast<float4*>(q + half + e) = live ? make_float4(rb[e], rb[e + 1], rb[e + 2], rb[e + 3]) : make_float4(0.f, 0.f, 0.f, 0.f);
        }
    } else if (pos >= 0) {
        uint16_t* c = cache + cache_block_base(g, layer, slot, head - n_q_heads, pos >> 5);
        Frag ka, kb;
#pragma unroll
        for (int e = 0; e < 8; ++e) {
            ka.h[e] = bits(ra[e]);
            kb.h[e] = bits(rb[e]);
        }
        *reinterpret_cast<uint4*>(c + tiled_k_within(hd, pos & 31, 8 * u)) = ka.u;
        *reinterpret_cast<uint4*>(c + tiled_k_within(hd, pos & 31, 8 * u + half)) = kb.u;
    }
}

// out[m][n] = sum of the ranges * the row's 1/rms; four columns per thread (rows of out start at any 4-byte address)
typedef float f32x4u __attribute__((ext_vector_type(4), aligned(4)));
__global__ void __launch_bounds__(TPB) reduce_splits_kernel(const float* __restrict__ partial, int n_split,
                                                            size_t split_stride, int N, int ld, NormScale ns,
                                                            float* __restrict__ out)
{
    const int m = blockIdx.y, n = (blockIdx.x * TPB + threadIdx.x) * 4;
    if (n >= N) return;
    const float* cols[1] = {partial + (size_t)m * ld + n};   // ld is a multiple of 16: the last columns are there to read
    const float r = row_inv_rms(ns.ssq, ns.n_ssq, m, ns.d, ns.eps);
    float4 v[1];
    sum_ranges(cols, n_split, split_stride, v);
    float* o = out + (size_t)m * N + n;
    if (n + 4 <= N) {
        *reinterpret_cast<f32x4u*>(o) = f32x4u{v[0].x * r, v[0].y * r, v[0].z * r, v[0].w * r};
    } else {
        const float t[4] = {v[0].x, v[0].y, v[0].z, v[0].w};
#pragma unroll
        for (int e = 0; e < 3; ++e)
            if (n + e < N) o[e] = t[e] * r;
    }
}

// plain tensor [layer][k|v][head][n_pos][hd]  <->  cache positions [pos0, pos0+n_pos) of one slot
template <bool BF16, bool TO_CACHE>
__global__ void __launch_bounds__(TPB) kv_copy_kernel(CacheGeom g, void* cache, int slot, int pos0, int n_pos, void* plain)
{
    const int hd = g.head_dim;
    const size_t total = (size_t)g.n_layers * 2 * g.n_kv_heads * n_pos * hd;
    for (size_t i = (size_t)blockIdx.x * TPB + threadIdx.x; i < total; i += (size_t)gridDim.x * TPB) {
        size_t r = i;
        const int dim = (int)(r % hd); r /= hd;
        const int p = (int)(r % n_pos); r /= n_pos;
        const int head = (int)(r % g.n_kv_heads); r /= g.n_kv_heads;
        const int kv = (int)(r % 2);
        const int layer = (int)(r / 2);
        size_t off;
        if constexpr (BF16)
            off = cache_block_base(g, layer, slot, head, (pos0 + p) >> 5)
                  + (kv ? tiled_v_within(hd, (pos0 + p) & 31, dim) : tiled_k_within(hd, (pos0 + p) & 31, dim));
        else
            off = cache_head_base(g, layer, slot, head) + plain_offset(g, kv, pos0 + p, dim);
        if constexpr (BF16) {
            uint16_t* c = static_cast<uint16_t*>(cache);
            uint16_t* q = static_cast<uint16_t*>(plain);
            if (TO_CACHE) c[off] = q[i]; else q[i] = c[off];
        } else {
            float* c = static_cast<float*>(cache);
            float* q = static_cast<float*>(plain);
            if (TO_CACHE) c[off] = q[i]; else q[i] = c[off];
        }
    }
}

// The same copy for bf16 caches whose plain tensor is 16-byte aligned, one workgroup per (layer, kv head,
// 32-position block).  Bound by memory: every byte is read and written once, in 16-byte lane accesses that
// cover whole 128-byte lines on both sides.  Keys are a permutation of 16-byte units (8 dims of a position):
// a wavefront takes 8 positions x 8 units, 128 contiguous bytes either way.  A unit of values holds 8
// positions of one dim, so values are turned around in LDS.  Element by element (the kernel above) every
// 2-byte access to the cache touched a line of its own: 699 MB read and written (7B-shape, 1333 positions) took
// 1039 us in and 935 us out; by blocks 264 us each way (5.3 TB/s; a plain copy reaches 4.8-5.2).
// STREAM: 16-byte stores non-temporal as well, for copies that the 256 MB memory-side cache cannot hold (KV_STREAM_BYTES): an import
// and an export of 699 MB each 525 -> 482 us, of 407 MB 330 -> 292, of 537 MB on the page pool 474 -> 420.  Below, what was written is
// read again out of that cache, and streaming stores cost 5 to 25 % (67 MB 45 -> 57 us, 201 MB 126 -> 142, 268 MB 170 -> 181).
typedef unsigned int kv_unit __attribute__((ext_vector_type(4)));
constexpr size_t KV_STREAM_BYTES = (size_t)384 << 20;
template <bool STREAM>
__device__ __forceinline__ void kv_store(const kv_unit& v, kv_unit* p)
{
    if constexpr (STREAM) __builtin_nontemporal_store(v, p);
    else *p = v;
}

template <int HD, bool TO_CACHE, bool STREAM>
__global__ void __launch_bounds__(TPB) kv_block_kernel(CacheGeom g, uint16_t* cache, int slot, int pos0, int n_pos,
                                                       uint16_t* plain, int blk0, int n_blk)
{
    constexpr int GROUPS = HD / 8, UNITS = 32 * GROUPS, PER = UNITS / TPB;   // 16-byte units of a part, per thread
    constexpr int LD = HD + 8;                                               // LDS row, 16-byte aligned
    __shared__ __align__(16) uint16_t rows[32 * LD];
    const int head = blockIdx.x % g.n_kv_heads;
    const int r = blockIdx.x / g.n_kv_heads;
    const int blk = blk0 + r % n_blk, layer = r / n_blk;
    const int base = blk * 32;
    const int lo = max(pos0 - base, 0), hi = min(pos0 + n_pos - base, 32);   // positions of the block that are copied
    uint16_t* kc = cache + cache_block_base(g, layer, slot, head, blk);
    uint16_t* vc = kc + 32 * HD;
    const ptrdiff_t row0 = (ptrdiff_t)base - pos0;                           // plain row of the block's position 0
    uint16_t* kp = plain + (((ptrdiff_t)layer * 2 * g.n_kv_heads + head) * n_pos + row0) * HD;
    uint16_t* vp = kp + (ptrdiff_t)g.n_kv_heads * n_pos * HD;
    auto unit = [](uint16_t* p) { return reinterpret_cast<kv_unit*>(p); };
    const int wave = threadIdx.x >> 6, lane = threadIdx.x & 63;

    kv_unit k[PER], v[PER];
    int kt[PER], kd[PER];
#pragma unroll
    for (int i = 0; i < PER; ++i) {
        const int q = i * 4 + wave;                     // 8 positions x 8 units
        kt[i] = (q / (GROUPS / 8)) * 8 + (lane & 7);
        kd[i] = (q % (GROUPS / 8)) * 8 + (lane >> 3);
    }
    auto k_cache = [&](int i) { return unit(kc + tiled_k_within(HD, kt[i], 8 * kd[i])); };
    auto k_plain = [&](int i) { return unit(kp + (ptrdiff_t)kt[i] * HD + 8 * kd[i]); };
    auto inside = [&](int t) { return t >= lo && t < hi; };
    // values: thread u takes unit (position u / GROUPS, dims 8 * (u % GROUPS)) of the plain rows and unit
    // u = 64 * dim tile + lane of the cache
    auto v_row = [&](int i) { return (i * TPB + (int)threadIdx.x) / GROUPS; };
    auto v_col = [&](int i) { return (i * TPB + (int)threadIdx.x) % GROUPS * 8; };
    auto v_cache = [&](int i) { return unit(vc + (size_t)(i * TPB + threadIdx.x) * 8); };
    auto v_dim = [&](int i) { return ((i * TPB + (int)threadIdx.x) >> 6) * 16 + (lane & 15); };
    auto v_pos = [&](int e) { return e < 4 ? 4 * (lane >> 4) + e : 12 + 4 * (lane >> 4) + e; };

    if constexpr (TO_CACHE) {
#pragma unroll
        for (int i = 0; i < PER; ++i) {
            if (inside(v_row(i))) v[i] = __builtin_nontemporal_load(unit(vp + (ptrdiff_t)v_row(i) * HD + v_col(i)));
            if (inside(kt[i])) k[i] = __builtin_nontemporal_load(k_plain(i));
        }
#pragma unroll
        for (int i = 0; i < PER; ++i)
            if (inside(v_row(i))) *unit(rows + v_row(i) * LD + v_col(i)) = v[i];
#pragma unroll
        for (int i = 0; i < PER; ++i)
            if (inside(kt[i])) kv_store<STREAM>(k[i], k_cache(i));
        __syncthreads();
#pragma unroll
        for (int i = 0; i < PER; ++i) {
            uint16_t e8[8];
#pragma unroll
            for (int e = 0; e < 8; ++e) e8[e] = rows[v_pos(e) * LD + v_dim(i)];
            if (lo == 0 && hi == 32) {
                kv_unit u;
                __builtin_memcpy(&u, e8, 16);
                kv_store<STREAM>(u, v_cache(i));
            } else {   // the block's other positions may hold entries: only these are written
#pragma unroll
                for (int e = 0; e < 8; ++e)
                    if (inside(v_pos(e))) reinterpret_cast<uint16_t*>(v_cache(i))[e] = e8[e];
            }
        }
    } else {
#pragma unroll
        for (int i = 0; i < PER; ++i) {
            v[i] = __builtin_nontemporal_load(v_cache(i));
            k[i] = __builtin_nontemporal_load(k_cache(i));
        }
#pragma unroll
        for (int i = 0; i < PER; ++i) {
            uint16_t e8[8];
            __builtin_memcpy(e8, &v[i], 16);
#pragma unroll
            for (int e = 0; e < 8; ++e) rows[v_pos(e) * LD + v_dim(i)] = e8[e];
        }
#pragma unroll
        for (int i = 0; i < PER; ++i)
            if (inside(kt[i])) kv_store<STREAM>(k[i], k_plain(i));
        __syncthreads();
#pragma unroll
        for (int i = 0; i < PER; ++i)
            if (inside(v_row(i))) kv_store<STREAM>(*unit(rows + v_row(i) * LD + v_col(i)), unit(vp + (ptrdiff_t)v_row(i) * HD + v_col(i)));
    }
}

unsigned blocks_for(size_t total)
{
    size_t b = (total + TPB - 1) / TPB;
    return (unsigned)(b > 8192 ? 8192 : (b ? b : 1));
}

}  // namespace

CacheGeom make_cache_geom(const spec_model_cfg& c)
{
    CacheGeom g{};
    g.dtype = c.dtype;
    g.n_layers = c.n_layers;
    g.n_slots = c.max_batch;
    g.n_kv_heads = c.n_kv_heads;
    g.head_dim = c.head_dim;
    if (c.dtype == SPEC_DTYPE_BF16) {
        g.t_pad = (c.max_kv_len + 31) / 32 * 32;
        g.head_stride = (size_t)64 * c.head_dim;
        g.blk_stride = (size_t)c.n_kv_heads * g.head_stride;
        g.slot_stride = (size_t)(g.t_pad / 32) * g.blk_stride;
    } else {
        g.t_pad = c.max_kv_len;
        g.head_stride = (size_t)g.t_pad * c.head_dim;
        g.slot_stride = (size_t)2 * c.n_kv_heads * g.head_stride;
    }
    g.layer_stride = (size_t)c.max_batch * g.slot_stride;
    return g;
}

int launch_embed(const EmbedTo& e, const int32_t* row_tok, int M, hipStream_t s)
{
    if (e.d % 8) return fail(SPEC_ERR_SHAPE, "d_model must be a multiple of 8");
    const dim3 grid(2 * ssq_pairs(e.d), M);
    if (e.dtype == SPEC_DTYPE_BF16)
        hipLaunchKernelGGL(embed_kernel<__bf16>, grid, dim3(64), 0, s, (const __bf16*)e.E, row_tok, e.x, e.gain, e.ssq, e.d, e.xo);
    else
        hipLaunchKernelGGL(embed_kernel<float>, grid, dim3(64), 0, s, (const float*)e.E, row_tok, e.x, e.gain, e.ssq, e.d, e.xo);
    SPECV_LAUNCH_CHECK("embed_kernel");
    return SPEC_OK;
}

int launch_resid(const float* partial, int n_split, size_t split_stride, int ld, int M, int d, float* x, double2* ssq,
                 const float* gain, const XOut& xo, hipStream_t s)
{
    if (d % 8 || ld % 4 || split_stride % 4) return fail(SPEC_ERR_SHAPE, "residual rows must be multiples of 8 wide");
    const dim3 grid(2 * ssq_pairs(d), M);
    hipLaunchKernelGGL(resid_kernel, grid, dim3(64), 0, s, partial, x, split_stride, n_split, ld, d, xo.mt, xo.frags, gain, ssq, xo.planes);
    SPECV_LAUNCH_CHECK("resid_kernel");
    return SPEC_OK;
}

int launch_silu_mul(const float* partial, int n_split, size_t split_stride, int ld, int M, int F, const NormScale& ns,
                    const XOut& xo, hipStream_t s)
{
    if (F % 8 || ld % 4 || split_stride % 4) return fail(SPEC_ERR_SHAPE, "d_ffn must be a multiple of 8");
    const int cols = 32 * (TPB / 64);   // per workgroup
    hipLaunchKernelGGL(silu_mul_kernel, dim3((F + cols - 1) / cols, (M + 15) / 16), dim3(TPB), 0, s, partial, n_split,
                       split_stride, ld, M, F, ns, xo);
    SPECV_LAUNCH_CHECK("silu_mul_kernel");
    return SPEC_OK;
}

int launch_rope_append(const float* partial, int n_split, size_t split_stride, int ld, const StepTables& t, int M,
                       const CacheGeom& g, int n_q_heads, int layer, const float* cos_sin, const NormScale& ns,
                       void* cache, float* q_out, hipStream_t s)
{
    if (g.dtype != SPEC_DTYPE_BF16) return fail(SPEC_ERR_SHAPE, "fp32 rotation is the attention's");
    if (ld % 4 || split_stride % 4) return fail(SPEC_ERR_SHAPE, "QKV rows must be multiples of 4 wide");
    const int units = (n_q_heads + 2 * g.n_kv_heads) * (g.head_dim / 16), per_wg = 4 * (TPB / 64);   // units of 16 values
    hipLaunchKernelGGL(rope_append_tiled_kernel, dim3((units + per_wg - 1) / per_wg, (M + 15) / 16), dim3(TPB), 0, s, partial, n_split,
                       split_stride, ld, t, g, n_q_heads, M, layer, cos_sin, ns, (uint16_t*)cache, q_out);
    SPECV_LAUNCH_CHECK("rope_append_tiled_kernel");
    return SPEC_OK;
}

int launch_reduce_splits(const float* partial, int n_split, size_t split_stride, int M, int N, int ld,
                         const double2* ssq, int n_ssq, int d, float eps, float* out, hipStream_t s)
{
    NormScale ns{ssq, n_ssq, d, eps};
    if (ld % 4 || split_stride % 4) return fail(SPEC_ERR_SHAPE, "partial sums must come in rows of multiples of 4");
    hipLaunchKernelGGL(reduce_splits_kernel, dim3((N + 4 * TPB - 1) / (4 * TPB), M), dim3(TPB), 0, s, partial, n_split,
                       split_stride, N, ld, ns, out);
    SPECV_LAUNCH_CHECK("reduce_splits_kernel");
    return SPEC_OK;
}

// After a tree was verified: the kept nodes' keys and values move from their window slots to the
// positions right behind the root, in path order.  Sources increase along a path and are never
// below their destination, and each thread moves the same dims in every step, so moving in place,
// one path node after the other, never overwrites an entry that is still needed.
template <bool BF16>
__global__ void __launch_bounds__(64) kv_compact_kernel(CacheGeom g, void* cache, StepTables t, int Kmax,
                                                        const int32_t* __restrict__ n_accepted,
                                                        const int32_t* __restrict__ path)
{
    const int b = blockIdx.x;
    if (!t.seq_ok[b]) return;
    const int a = n_accepted[b];
    const int n = t.seq_n[b], hd = g.head_dim;
    const int layer = blockIdx.y / g.n_kv_heads, head = blockIdx.y % g.n_kv_heads;
    const int slot = t.seq_slot[b];
    const size_t base = cache_head_base(g, layer, slot, head);   // fp32 only
    for (int k = 1; k <= a; ++k) {
        const int node = path[b * Kmax + k - 1];
        if (node < 0 || node >= Kmax) return;   // cannot happen: the walk writes a valid indices first
        const int src = n + node + 1, dst = n + k;
        if (src == dst) continue;
        for (int i = threadIdx.x; i < hd; i += 64) {
            if constexpr (BF16) {
                uint16_t* c = static_cast<uint16_t*>(cache);
                const size_t sb = cache_block_base(g, layer, slot, head, src >> 5);
                const size_t db = cache_block_base(g, layer, slot, head, dst >> 5);
                c[db + tiled_k_within(hd, dst & 31, i)] = c[sb + tiled_k_within(hd, src & 31, i)];
                c[db + tiled_v_within(hd, dst & 31, i)] = c[sb + tiled_v_within(hd, src & 31, i)];
            } else {
                float* c = static_cast<float*>(cache);
                c[base + plain_offset(g, 0, dst, i)] = c[base + plain_offset(g, 0, src, i)];
                c[base + plain_offset(g, 1, dst, i)] = c[base + plain_offset(g, 1, src, i)];
            }
        }
    }
}

int launch_kv_compact(const CacheGeom& g, void* cache, const StepTables& t, int B, int Kmax, const int32_t* n_accepted,
                      const int32_t* path, hipStream_t s)
{
    const dim3 grid(B, g.n_layers * g.n_kv_heads);
    if (g.dtype == SPEC_DTYPE_BF16)
        hipLaunchKernelGGL(kv_compact_kernel<true>, grid, dim3(64), 0, s, g, cache, t, Kmax, n_accepted, path);
    else
        hipLaunchKernelGGL(kv_compact_kernel<false>, grid, dim3(64), 0, s, g, cache, t, Kmax, n_accepted, path);
    SPECV_LAUNCH_CHECK("kv_compact_kernel");
    return SPEC_OK;
}

int launch_kv_copy(const CacheGeom& g, void* cache, int slot, int pos0, int n_pos, void* plain, bool to_cache,
                   hipStream_t s)
{
    // Whole blocks at a time wherever 16-byte accesses are possible; a tensor at an odd address and fp32 caches
    // go element by element.
    if (g.dtype == SPEC_DTYPE_BF16 && (g.head_dim == 64 || g.head_dim == 128) && (((uintptr_t)plain | (uintptr_t)cache) & 15) == 0) {
        const int blk0 = pos0 >> 5, n_blk = ((pos0 + n_pos - 1) >> 5) - blk0 + 1;
        const size_t groups = (size_t)g.n_layers * n_blk * g.n_kv_heads;
        if (groups <= 0x7fffffff) {
            const dim3 grid((unsigned)groups);
            const bool stream = (size_t)g.n_layers * 2 * g.n_kv_heads * n_pos * g.head_dim * sizeof(uint16_t) >= KV_STREAM_BYTES;
#define SPECV_KV_BLOCK(HD, IN)                                                                                                   \
    do {                                                                                                                         \
        auto* k = stream ? kv_block_kernel<HD, IN, true> : kv_block_kernel<HD, IN, false>;                                       \
        hipLaunchKernelGGL(k, grid, dim3(TPB), 0, s, g, (uint16_t*)cache, slot, pos0, n_pos, (uint16_t*)plain, blk0, n_blk);     \
    } while (0)
            if (g.head_dim == 128) {
                if (to_cache) SPECV_KV_BLOCK(128, true);
                else SPECV_KV_BLOCK(128, false);
            } else {
                if (to_cache) SPECV_KV_BLOCK(64, true);
                else SPECV_KV_BLOCK(64, false);
            }
#undef SPECV_KV_BLOCK
            SPECV_LAUNCH_CHECK("kv_block_kernel");
            return SPEC_OK;
        }
    }
    const size_t total = (size_t)g.n_layers * 2 * g.n_kv_heads * n_pos * g.head_dim;
    const dim3 grid(blocks_for(total));
    if (g.dtype == SPEC_DTYPE_BF16) {
        if (to_cache) hipLaunchKernelGGL((kv_copy_kernel<true, true>), grid, dim3(TPB), 0, s, g, cache, slot, pos0, n_pos, plain);
        else hipLaunchKernelGGL((kv_copy_kernel<true, false>), grid, dim3(TPB), 0, s, g, cache, slot, pos0, n_pos, plain);
    } else {
        if (to_cache) hipLaunchKernelGGL((kv_copy_kernel<false, true>), grid, dim3(TPB), 0, s, g, cache, slot, pos0, n_pos, plain);
        else hipLaunchKernelGGL((kv_copy_kernel<false, false>), grid, dim3(TPB), 0, s, g, cache, slot, pos0, n_pos, plain);
    }
    SPECV_LAUNCH_CHECK("kv_copy_kernel");
    return SPEC_OK;
}

}  // namespace specv
