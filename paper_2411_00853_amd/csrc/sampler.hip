// Rejection-sampling part of the verify step: softmax statistics of every target and draft row,
// the accept scan, the residual / extra-token draw and the KV length update.
//
// The procedure is the one the paper describes in its section "Speculative Sampling Results"
// (compare the two models' probabilities of each proposed token, keep a prefix, resample the
// first rejected token from a combination of the distributions, draw one more token from the
// target if nothing was rejected), with the cited works' formulas: keep x iff u*q(x) < p(x),
// resample from max(0, p - q).
//
// The vocabulary-wide work is pure streaming, so it is laid out for HBM: every logit is read once
// by the statistics pass (float4 per lane, 64 values per lane in flight); only the one or two
// rows that the final draw needs are read again.  Sums are kept in fp64 and every reduction has a
// fixed order (no floating-point atomics), so results are reproducible bit for bit.
#include "cache_layout.h"
#include "common.h"
#include "embed.h"
#include "frag.h"

#include <algorithm>
#include <cstring>
#include <mutex>

namespace specv {

namespace {

constexpr int TPB = 256;

// Exchanges inside a wavefront by DPP (a few cycles a step where a shuffle through LDS takes a hundred, and every kernel
// here is a chain of such steps).  Lanes without a source keep `old`.
enum { DPP_XOR1 = 0xb1, DPP_XOR2 = 0x4e, DPP_SHR1 = 0x111, DPP_SHR2 = 0x112, DPP_SHR4 = 0x114, DPP_SHR8 = 0x118, DPP_MIRROR = 0x140,
       DPP_HALF_MIRROR = 0x141, DPP_BCAST15 = 0x142, DPP_BCAST31 = 0x143 };
template <int CTRL, int ROWS>
__device__ __forceinline__ int dpp(int old, int v)
{
    return __builtin_amdgcn_update_dpp(old, v, CTRL, ROWS, 0xf, false);
}
template <int CTRL, int ROWS>
__device__ __forceinline__ double dpp_or_zero(double v)
{
    const uint64_t u = __builtin_bit_cast(uint64_t, v);
    const uint32_t lo = (uint32_t)dpp<CTRL, ROWS>(0, (int)(uint32_t)u), hi = (uint32_t)dpp<CTRL, ROWS>(0, (int)(uint32_t)(u >> 32));
    return __builtin_bit_cast(double, (uint64_t)hi << 32 | lo);
}
__device__ __forceinline__ double read_lane(double v, int lane)
{
    const uint64_t u = __builtin_bit_cast(uint64_t, v);
    const uint32_t lo = (uint32_t)__builtin_amdgcn_readlane((int)(uint32_t)u, lane);
    const uint32_t hi = (uint32_t)__builtin_amdgcn_readlane((int)(uint32_t)(u >> 32), lane);
    return __builtin_bit_cast(double, (uint64_t)hi << 32 | lo);
}

__device__ __forceinline__ float wave_max(float v)   // (the same for all lanes)
{
    auto step = [&](int o) { v = fmaxf(v, __builtin_bit_cast(float, o)); };
    auto bits = [&] { return __builtin_bit_cast(int, v); };
    step(dpp<DPP_XOR1, 0xf>(bits(), bits()));
    step(dpp<DPP_XOR2, 0xf>(bits(), bits()));
    step(dpp<DPP_HALF_MIRROR, 0xf>(bits(), bits()));
    step(dpp<DPP_MIRROR, 0xf>(bits(), bits()));
    step(dpp<DPP_BCAST15, 0xa>(bits(), bits()));
    step(dpp<DPP_BCAST31, 0xc>(bits(), bits()));
    return __builtin_bit_cast(float, __builtin_amdgcn_readlane(bits(), 63));
}

__device__ __forceinline__ double wave_sum(double v)   // (the same for all lanes; a fixed order)
{
    v += dpp_or_zero<DPP_XOR1, 0xf>(v);
    v += dpp_or_zero<DPP_XOR2, 0xf>(v);
    v += dpp_or_zero<DPP_HALF_MIRROR, 0xf>(v);
    v += dpp_or_zero<DPP_MIRROR, 0xf>(v);
    v += dpp_or_zero<DPP_BCAST15, 0xa>(v);
    v += dpp_or_zero<DPP_BCAST31, 0xc>(v);
    return read_lane(v, 63);
}

// inclusive running sums over the lanes (of the first 16 lanes: the first four steps)
__device__ __forceinline__ double row_scan(double v)
{
    v += dpp_or_zero<DPP_SHR1, 0xf>(v);
    v += dpp_or_zero<DPP_SHR2, 0xf>(v);
    v += dpp_or_zero<DPP_SHR4, 0xf>(v);
    v += dpp_or_zero<DPP_SHR8, 0xf>(v);
    return v;
}
__device__ __forceinline__ double wave_scan(double v)
{
    v = row_scan(v);
    v += dpp_or_zero<DPP_BCAST15, 0xa>(v);
    v += dpp_or_zero<DPP_BCAST31, 0xc>(v);
    return v;
}

// ---------------------------------------------------------------------------------------------
// Row bookkeeping.  One workgroup; thread b owns sequence b.
// ---------------------------------------------------------------------------------------------
struct PrepLds {
    int2 seq[SPEC_MAX_BATCH];   // window rows, slot
    int total[SPEC_MAX_BATCH];
};
static_assert(TPB >= SPEC_MAX_BATCH, "a thread per sequence");

// What a sequence has to know of the others: the window rows before it, all of them, and whether one before it names
// its slot.  All threads of the workgroup call.  One walk over LDS, eight entries in flight.  (With prefix sums by
// wavefront scans, a second walk for the slots and the loads behind both, the kernel took 4.8 us in a decoding round of 8
// sequences, 7.5 for trees and 9.4 for 32 ragged sequences on the page pool; this way 3.9, 7.1 and 8.9.)
struct Others {
    int row0, rows;
    bool same_slot;
};
__device__ __forceinline__ Others look_at_others(int K, int slot, int B, PrepLds& l)
{
    const int b = threadIdx.x;
    if (b < B) l.seq[b] = make_int2(K + 1, slot);
    __syncthreads();
    Others r{0, 0, false};
#pragma unroll 8
    for (int i = 0; i < B; ++i) {
        const int2 o = l.seq[i];
        r.rows += o.x;
        r.row0 += i < b ? o.x : 0;
        r.same_slot |= i < b && o.y == slot;
    }
    return r;
}

// The sequences by falling number of positions.  The attention deals its workgroups out in this order, so the
// longest ones start first and the short ones fill in behind them (32 sequences of 512..4096 positions on the page
// pool: 232 us per launch in the order of the call, 213.5..220.5 this way).  All threads of the workgroup call desc_rank.
__device__ __forceinline__ int desc_rank(int b, int B, int positions, int* total)
{
    if (b < B) total[b] = positions;
    __syncthreads();
    int rank = 0;
#pragma unroll 8
    for (int i = 0; i < B; ++i) rank += (total[i] > positions || (total[i] == positions && i < b)) ? 1 : 0;
    return rank;
}

__device__ __forceinline__ void write_desc(const StepTables& t, int rank, int b, int k, int n, int slot, int ok, int row0)
{
    int4* d = reinterpret_cast<int4*>(t.seq_desc + rank);
    d[0] = make_int4(b, row0, k, n);
    d[1] = make_int4(slot, ok, 0, 0);
}

// (a workgroup of TPB threads, all of them calling)
__device__ __forceinline__ void prepare_rows(const StepTables& t, const LookaheadPack& ks, int B, int Kmax, int V,
                                             int max_batch, int max_kv_len, int has_cache,
                                             const int32_t* __restrict__ seq_slot,
                                             const int32_t* __restrict__ last_token,
                                             const int32_t* __restrict__ draft_tokens,
                                             const int32_t* __restrict__ kv_len, int32_t* flag, PrepLds& l)
{
    const int b = threadIdx.x;
    // Two memory round trips, both under way before the first barrier: lookahead, slot and last token, then what they
    // lead to.  (Asked for behind the prefix sums, one more.)
    int K = 0, ok = 1, slot = 0, n = 0;
    int tok[SPEC_MAX_LOOKAHEAD + 1];
    if (b < B) {
        K = ks.k[b];
        slot = has_cache ? seq_slot[b] : b;
        tok[0] = last_token ? last_token[b] : 0;
#pragma unroll
        for (int i = 0; i < SPEC_MAX_LOOKAHEAD; ++i) {
            if (i >= Kmax) break;   // (the whole workgroup skips what is left of the unrolled code)
            tok[i + 1] = i < K ? draft_tokens[b * Kmax + i] : 0;
        }
        if (has_cache) n = kv_len[slot >= 0 && slot < max_batch ? slot : 0];
    }
    const Others o = look_at_others(K, slot, B, l);
    if (b < B) {
        int err = 0;
        if (has_cache) {
            if (slot < 0 || slot >= max_batch) {
                ok = 0;
                err = SPEC_ERR_INVALID_ARG;
                slot = 0;
            } else {
                // two sequences of one step must not share a slot
                if (o.same_slot) { ok = 0; err = SPEC_ERR_INVALID_ARG; }
                if (n < 0 || n + K + 1 > max_kv_len) { ok = 0; err = SPEC_ERR_KV_OVERFLOW; }
                else if (ok && !pool_cover(t.pool, slot, n, n + K + 1)) { ok = 0; err = SPEC_ERR_KV_OVERFLOW; }
            }
        }
#pragma unroll
        for (int j = 0; j <= SPEC_MAX_LOOKAHEAD; ++j) {
            if (j > Kmax) break;
            if (tok[j] < 0 || tok[j] >= V) { ok = 0; err = SPEC_ERR_TOKEN_RANGE; }
        }
        if (!ok) {
            atomicCAS(flag, 0, err);
            n = 0;
        }
    }
    const int rank = has_cache ? desc_rank(b, B, ok ? n + K + 1 : 0, l.total) : 0;
    if (b == 0) {
        t.seq_row0[B] = o.rows;
        t.seq_stat0[B] = 2 * o.rows - B;
    }
    if (b < B) {
        const int row0 = o.row0;
        if (has_cache) write_desc(t, rank, b, K, n, slot, ok, row0);
        t.seq_row0[b] = row0;
        t.seq_stat0[b] = 2 * row0 - b;
        t.arrived[b * ARRIVED_STRIDE] = 0;   // (in every call, whatever an earlier one left behind)
        t.seq_n[b] = n;
        t.seq_ok[b] = ok;
        t.seq_slot[b] = slot;
#pragma unroll
        for (int j = 0; j <= SPEC_MAX_LOOKAHEAD; ++j) {
            if (j > Kmax) break;
            if (j <= K) {
                const int r = row0 + j;
                t.row_seq[r] = b;
                t.row_pos[r] = ok ? n + j : -1;
                t.row_rope[r] = ok ? n + j : 0;
                t.row_mask[r] = (2u << j) - 1u;   // causal window: slots 0..j
                t.row_tok[r] = ok ? tok[j] : 0;
            }
        }
    }
}

__global__ void __launch_bounds__(TPB) prepare_kernel(StepTables t, LookaheadPack ks, int B, int Kmax, int V,
                                                      int max_batch, int max_kv_len, int has_cache,
                                                      const int32_t* __restrict__ seq_slot,
                                                      const int32_t* __restrict__ last_token,
                                                      const int32_t* __restrict__ draft_tokens,
                                                      const int32_t* __restrict__ kv_len, int32_t* flag)
{
    __shared__ PrepLds l;
    prepare_rows(t, ks, B, Kmax, V, max_batch, max_kv_len, has_cache, seq_slot, last_token, draft_tokens, kv_len, flag, l);
}

// A step with more window rows than one decoder pass takes is scored group by group: the row
// bookkeeping above runs once for the whole step (so that what it decides -- skipped sequences, a slot
// named twice, pages taken -- is decided once), and each pass gets the entries of its own sequences
// with rows and sequence numbers counted from the group's start.
__global__ void __launch_bounds__(TPB) slice_tables_kernel(StepTables full, StepTables sub, int b0, int Bg)
{
    const int r0 = full.seq_row0[b0], st0 = full.seq_stat0[b0];
    const int n_rows = full.seq_row0[b0 + Bg] - r0;
    __shared__ int total[SPEC_MAX_BATCH];
    const int b = threadIdx.x, at = b0 + min(b, Bg - 1);
    const int row0 = full.seq_row0[at], k = full.seq_row0[at + 1] - row0 - 1, n = full.seq_n[at], ok = full.seq_ok[at];
    const int rank = desc_rank(b, Bg, ok ? n + k + 1 : 0, total);
    if (b < Bg) write_desc(sub, rank, b, k, n, full.seq_slot[at], ok, row0 - r0);
    for (int i = threadIdx.x; i <= Bg; i += TPB) {
        sub.seq_row0[i] = full.seq_row0[b0 + i] - r0;
        sub.seq_stat0[i] = full.seq_stat0[b0 + i] - st0;
        if (i < Bg) {
            sub.seq_n[i] = full.seq_n[b0 + i];
            sub.seq_ok[i] = full.seq_ok[b0 + i];
            sub.seq_slot[i] = full.seq_slot[b0 + i];
        }
    }
    for (int r = threadIdx.x; r < n_rows; r += TPB) {
        sub.row_seq[r] = full.row_seq[r0 + r] - b0;
        sub.row_pos[r] = full.row_pos[r0 + r];
        sub.row_tok[r] = full.row_tok[r0 + r];
        sub.row_rope[r] = full.row_rope[r0 + r];
        sub.row_mask[r] = full.row_mask[r0 + r];
    }
}

// ---------------------------------------------------------------------------------------------
// Pass 1: per (row, chunk) maximum and sum of exp((l - max)/T).
// Statistics rows of sequence b: K_b+1 target rows, then K_b draft rows.
// ---------------------------------------------------------------------------------------------
// draft_rows: draft logits rows per sequence in memory (Kmax for a chain of proposals; Kmax+1 for
// a tree, whose root has a row of its own)
// Which rows the pass walks.  STAT_CHAIN / STAT_TREE: sequence b has K_b + 1 target rows and K_b
// (chain) or K_b + 1 (tree) draft rows, found from the lookaheads in the kernel arguments alone, so
// the pass does not depend on the row tables.  STAT_PLAIN: one row per sequence, its logits row taken
// from seq_row0 (a proposing model's draw, whose row is not the one the lookaheads would give).
enum { STAT_CHAIN = 0, STAT_TREE = 1, STAT_PLAIN = 2 };

// The row bookkeeping of a step that runs no decoder pass (logits supplied by the caller), done by a
// workgroup of the statistics pass (the first, which takes no chunk) instead of by a kernel of its own: the pass
// itself does not read the tables, the kernels after it do.
struct PrepIn {
    int Kmax;
    const int32_t* draft_tokens;
    int32_t* flag;
};

// The sequence b that statistics row srow belongs to, the row's number inside the sequence (local), the
// sequence's first target row (r0) and its lookahead (K), from the lookaheads in the kernel arguments.
// Every wavefront finds it for itself: lane i takes sequences i, i + 64, ... (all loads issued together,
// one memory round trip; walking the sequences one after the other costs one round trip each),
// prefix sums across the lanes place each sequence's rows, and the lane whose range holds srow answers.
__device__ __forceinline__ void find_stat_row(const LookaheadPack& ks, int B, int srow, bool tree, int* b_out,
                                              int* local_out, int* r0_out, int* K_out)
{
    constexpr int ROUNDS = SPEC_MAX_BATCH / 64;
    const int lane = threadIdx.x & 63;
    int kk[ROUNDS];
#pragma unroll
    for (int g = 0; g < ROUNDS; ++g) kk[g] = ks.k[min(g * 64 + lane, SPEC_MAX_BATCH - 1)];
    int base_st = 0, base_r = 0, b = 0, st = 0, r0 = 0, K = 0;
#pragma unroll
    for (int g = 0; g < ROUNDS; ++g) {
        if (g * 64 >= B) break;
        const int i = g * 64 + lane;
        const int k = kk[g];
        const int n = i < B ? 2 * k + 1 + (tree ? 1 : 0) : 0, r = i < B ? k + 1 : 0;
        int ps = n, pr = r;
#pragma unroll
        for (int off = 1; off < 64; off <<= 1) {
            const int a = __shfl_up(ps, off), c = __shfl_up(pr, off);
            if (lane >= off) {
                ps += a;
                pr += c;
            }
        }
        const int st_excl = base_st + ps - n;
        const bool hit = n > 0 && st_excl <= srow && srow < st_excl + n;
        const unsigned long long m = __ballot(hit);
        if (m) {
            const int src = __ffsll((long long)m) - 1;
            b = g * 64 + src;
            st = __shfl(st_excl, src);
            r0 = __shfl(base_r + pr - r, src);
            K = __shfl(k, src);
        }
        base_st += __shfl(ps, 63);
        base_r += __shfl(pr, 63);
    }
    *b_out = b;
    *local_out = srow - st;
    *r0_out = r0;
    *K_out = K;
}

// (sum of the ranges, in index order) * row scale of N float4 columns AT apart, as many loads in flight as make 32 of them
template <int S, int N>
__device__ __forceinline__ void logits_from(const float* p, size_t stride, int at, int lim, int first, float r, floatx4 (&v)[N])
{
    constexpr int W = S <= 2 ? N : N * 2 / S > 0 ? N * 2 / S : 1;   // columns at a time
#pragma unroll
    for (int i0 = 0; i0 < N; i0 += W) {
        floatx4 a[W][S];
#pragma unroll
        for (int i = 0; i < W; ++i)
#pragma unroll
            for (int q = 0; q < S; ++q)   // (columns past the end: the last ones again)
                a[i][q] = *reinterpret_cast<const floatx4*>(p + q * stride + min(first + (i0 + i) * at, lim - 4));
#pragma unroll
        for (int i = 0; i < W; ++i) {
            floatx4 t = a[i][0];
#pragma unroll
            for (int q = 1; q < S; ++q) t += a[i][q];
            v[i0 + i] = t * r;
        }
    }
}

// Rows that are not 16-byte aligned: v[i] = the logit in column i * TPB + thread of a chunk (-inf from lim on), summed over S ranges
// and written to o.  A batch's loads go out together (columns clamped, values dropped): with a branch and a run-time
// count around every load a chunk was 64 round trips one after the other (18903 logits, 41 rows: 58 us).
template <int S, int PER>
__device__ __forceinline__ void logits_by_column(const float* p, size_t stride, int lim, float r, float* o, float (&v)[PER])
{
    constexpr int N = S >= 8 ? 8 : 16;
#pragma unroll
    for (int i0 = 0; i0 < PER; i0 += N) {
        if (i0 * TPB >= lim) {   // (the same for the whole workgroup)
#pragma unroll
            for (int i = i0; i < i0 + N; ++i) v[i] = -INFINITY;
            continue;
        }
        float a[N][S];
#pragma unroll
        for (int i = 0; i < N; ++i)
#pragma unroll
            for (int q = 0; q < S; ++q) a[i][q] = p[q * stride + min((i0 + i) * TPB + (int)threadIdx.x, lim - 1)];
#pragma unroll
        for (int i = 0; i < N; ++i) {
            const int idx = (i0 + i) * TPB + threadIdx.x;
            float t = a[i][0];
#pragma unroll
            for (int q = 1; q < S; ++q) t += a[i][q];
            v[i0 + i] = idx < lim ? t * r : -INFINITY;
            if (idx < lim) o[idx] = v[i0 + i];
        }
    }
}

// SRC: target rows come as the LM head's partial sums; the workgroup adds up its chunk, writes it to src.out and goes on
// from registers (as a kernel of its own in front of this one the sum took 4.5-5.4 us a step, 9.4-15.8 at 128-352 rows).
template <bool VEC4, bool SRC>
__global__ void __launch_bounds__(TPB) stats_kernel(int prep_on, int layout, int B, int draft_rows, int V, int n_chunks,
                                                    const float* __restrict__ target,
                                                    const float* __restrict__ draft, float* __restrict__ copy_out,
                                                    float inv_T, float* __restrict__ part_max,
                                                    double* __restrict__ part_sum, size_t copy_stride,
                                                    StepTables t, LookaheadPack ks, PrepIn prep, LogitsSrc src)
{
    __shared__ float smax[TPB / 64];
    __shared__ double ssum[TPB / 64];
    __shared__ PrepLds prep_lds;
    if (prep_on && blockIdx.x == 0) {
        prepare_rows(t, ks, B, prep.Kmax, V, SPEC_MAX_BATCH, 0, 0, nullptr, nullptr, prep.draft_tokens, nullptr, prep.flag,
                     prep_lds);
        return;
    }
    const int wg = blockIdx.x - prep_on;
    const int srow = wg / n_chunks;
    const int chunk = wg % n_chunks;
    const float* row;
    int m = -1;   // target row, -1: a draft row
    if (layout == STAT_PLAIN) {
        m = t.seq_row0[srow];
        row = target + (size_t)m * V;
    } else {
        int b, local, r0, K;
        find_stat_row(ks, B, srow, layout == STAT_TREE, &b, &local, &r0, &K);
        if (local <= K) m = r0 + local;
        row = local <= K ? target + (size_t)m * V : draft + ((size_t)b * draft_rows + (local - K - 1)) * V;
    }
    const int base = chunk * STAT_CHUNK;
    const int lim = min(STAT_CHUNK, V - base);

    constexpr int PER = STAT_CHUNK / TPB;   // 64 values per lane
    float v[PER];
    // copy_out: plain-draw mode (one statistics row per sequence): keep the row for the verifier
    if (SRC && m >= 0) {
        const float rs = row_inv_rms(src.ns.ssq, src.ns.n_ssq, m, src.ns.d, src.ns.eps);
        const float* p = src.partial + (size_t)m * src.ld + base;
        float* o = src.out + (size_t)m * V + base;
        if constexpr (VEC4) {
            floatx4 x[PER / 4];
            const int first = 4 * threadIdx.x;
            switch (src.n_split) {
            case 1: logits_from<1>(p, src.stride, 4 * TPB, lim, first, rs, x); break;
            case 2: logits_from<2>(p, src.stride, 4 * TPB, lim, first, rs, x); break;
            case 4: logits_from<4>(p, src.stride, 4 * TPB, lim, first, rs, x); break;
            case 8: logits_from<8>(p, src.stride, 4 * TPB, lim, first, rs, x); break;
            default: logits_from<16>(p, src.stride, 4 * TPB, lim, first, rs, x); break;
            }
#pragma unroll
            for (int i = 0; i < PER / 4; ++i) {
                const int idx = first + i * 4 * TPB;
                const bool in = idx < lim;
                if (in) *reinterpret_cast<floatx4*>(o + idx) = x[i];
                v[4 * i + 0] = in ? x[i].x : -INFINITY; v[4 * i + 1] = in ? x[i].y : -INFINITY;
                v[4 * i + 2] = in ? x[i].z : -INFINITY; v[4 * i + 3] = in ? x[i].w : -INFINITY;
            }
        } else {
            switch (src.n_split) {
            case 1: logits_by_column<1>(p, src.stride, lim, rs, o, v); break;
            case 2: logits_by_column<2>(p, src.stride, lim, rs, o, v); break;
            case 4: logits_by_column<4>(p, src.stride, lim, rs, o, v); break;
            case 8: logits_by_column<8>(p, src.stride, lim, rs, o, v); break;
            default: logits_by_column<16>(p, src.stride, lim, rs, o, v); break;
            }
        }
    } else if constexpr (VEC4) {
        const float4* p4 = reinterpret_cast<const float4*>(row + base);
#pragma unroll
        for (int i = 0; i < PER / 4; ++i) {
            int idx = i * TPB + threadIdx.x;
            float4 x = make_float4(-INFINITY, -INFINITY, -INFINITY, -INFINITY);
            if (idx * 4 < lim) {   // lim is a multiple of 4 when VEC4
                typedef float f32x4 __attribute__((ext_vector_type(4)));
                const f32x4 y = __builtin_nontemporal_load(reinterpret_cast<const f32x4*>(p4 + idx));
                x = make_float4(y.x, y.y, y.z, y.w);
            }
            v[4 * i + 0] = x.x; v[4 * i + 1] = x.y; v[4 * i + 2] = x.z; v[4 * i + 3] = x.w;
        }
    } else {
#pragma unroll
        for (int i = 0; i < PER; ++i) {
            int idx = i * TPB + threadIdx.x;
            v[i] = idx < lim ? row[base + idx] : -INFINITY;
        }
    }
    if (VEC4 && copy_out) {   // whole 16-byte stores (the launcher checked the alignment of the copy as well)
        float4* d4 = reinterpret_cast<float4*>(copy_out + (size_t)srow * copy_stride + base);
#pragma unroll
        for (int i = 0; i < PER / 4; ++i) {
            const int idx = i * TPB + threadIdx.x;
            if (idx * 4 < lim) d4[idx] = make_float4(v[4 * i + 0], v[4 * i + 1], v[4 * i + 2], v[4 * i + 3]);
        }
    }
    if (!VEC4 && copy_out) {
        float* dst = copy_out + (size_t)srow * copy_stride + base;
#pragma unroll
        for (int i = 0; i < PER; ++i) {
            const int idx = i * TPB + (int)threadIdx.x;
            if (idx < lim) dst[idx] = v[i];
        }
    }
    float mx = -INFINITY;
#pragma unroll
    for (int i = 0; i < PER; ++i) mx = fmaxf(mx, v[i]);
    mx = wave_max(mx);
    if ((threadIdx.x & 63) == 0) smax[threadIdx.x >> 6] = mx;
    __syncthreads();
    mx = fmaxf(fmaxf(smax[0], smax[1]), fmaxf(smax[2], smax[3]));
    const float mm = (mx == -INFINITY) ? 0.f : mx;   // a chunk of -inf logits contributes nothing

    double acc = 0.0;
#pragma unroll
    for (int i = 0; i < PER; ++i) acc += (double)__expf((v[i] - mm) * inv_T);   // exp(-inf) = 0 for padding
    acc = wave_sum(acc);
    if ((threadIdx.x & 63) == 0) ssum[threadIdx.x >> 6] = acc;
    __syncthreads();
    if (threadIdx.x == 0) {
        part_max[(size_t)srow * n_chunks + chunk] = mx;
        part_sum[(size_t)srow * n_chunks + chunk] = (ssum[0] + ssum[1]) + (ssum[2] + ssum[3]);
    }
}

// Combine the chunk statistics of n_rows rows from row0 on: max of maxima, sums rescaled to it.  Every thread takes
// its share of the (row, chunk) pairs -- one exp() each instead of one thread's row of them in turn, which was the
// longest stretch of the kernels that begin with this -- and one thread per row adds them up in chunk order.
// All THREADS threads of the workgroup call; row_m and row_z are in LDS and valid after the barrier it ends with.
struct CombineLds {
    static constexpr int PAIRS = 512;
    float m[PAIRS];
    double sum[PAIRS], e[PAIRS];
};
template <int THREADS>
__device__ __forceinline__ void combine_rows(const float* part_max, const double* part_sum, int row0, int n_rows, int n_chunks,
                                             double inv_T, float* row_m, double* row_z, CombineLds& l)
{
    constexpr int PER = (CombineLds::PAIRS + THREADS - 1) / THREADS;
    const int tid = threadIdx.x;
    if (n_chunks > CombineLds::PAIRS) {   // (vocabularies of millions: a thread per row walks its chunks)
        if (tid < n_rows) {
            const float* pm = part_max + (size_t)(row0 + tid) * n_chunks;
            const double* ps = part_sum + (size_t)(row0 + tid) * n_chunks;
            float m = -INFINITY;
            for (int c = 0; c < n_chunks; ++c) m = fmaxf(m, pm[c]);
            double z = 0.0;
            for (int c = 0; c < n_chunks; ++c) z += ps[c] * exp((double)(pm[c] - m) * inv_T);
            row_m[tid] = m;
            row_z[tid] = z;
        }
        __syncthreads();
        return;
    }
    // as many rows at a time as there is room for (their pairs lie one after the other in memory)
    const int step = min(n_rows, CombineLds::PAIRS / n_chunks);
    for (int r0 = 0; r0 < n_rows; r0 += step) {
        const int rows = min(step, n_rows - r0), pairs = rows * n_chunks;
        const float* pm = part_max + (size_t)(row0 + r0) * n_chunks;
        const double* ps = part_sum + (size_t)(row0 + r0) * n_chunks;
        float mv[PER];
#pragma unroll
        for (int k = 0; k < PER; ++k) {
            const int p = tid + k * THREADS;
            mv[k] = 0.f;
            if (p < pairs) {
                mv[k] = pm[p];
                l.m[p] = mv[k];
                l.sum[p] = ps[p];
            }
        }
        __syncthreads();
        if (tid < rows) {
            float m = -INFINITY;
            for (int c = 0; c < n_chunks; ++c) m = fmaxf(m, l.m[tid * n_chunks + c]);
            row_m[r0 + tid] = m;
        }
        __syncthreads();
#pragma unroll
        for (int k = 0; k < PER; ++k) {
            const int p = tid + k * THREADS;
            if (p < pairs) l.e[p] = exp((double)(mv[k] - row_m[r0 + p / n_chunks]) * inv_T);
        }
        __syncthreads();
        if (tid < rows) {
            double z = 0.0;
            for (int c = 0; c < n_chunks; ++c) z += l.sum[tid * n_chunks + c] * l.e[tid * n_chunks + c];
            row_z[r0 + tid] = z;
        }
        __syncthreads();
    }
}

// ---------------------------------------------------------------------------------------------
// One workgroup per sequence keeps the row (or the two rows) of the draw in registers, so the accept scan, the mass and the draw -- for
// a plain draw the statistics as well -- are one launch: plain draws of up to PLAIN_MIN ids, chains of up to SLICE_MIN and, in large
// batches, DRAW_MAX (draw_route), trees of up to DRAW_MAX.  RUNS runs of 256 ids per wavefront: wavefront w holds ids [256 RUNS w, 256 RUNS (w + 1)), lane l of it
// the ids 4 l .. 4 l + 3 of every run.
// ---------------------------------------------------------------------------------------------
constexpr int DRAW_TPB = 1024, DRAW_WAVES = DRAW_TPB / 64, DRAW_MAX_RUNS = 8;
constexpr int DRAW_MAX = DRAW_WAVES * 256 * DRAW_MAX_RUNS;   // 32768
static_assert(DRAW_WAVES <= 16, "the wavefronts' sums are scanned by 16 lanes");
constexpr int SLICE_MIN = 16384;   // accept_slice_kernel beyond (draw_route): 16000 and two sequences 13.5 us in one workgroup each, 13.9 shared out, 20000 and 64 29.2 and 26.9
constexpr int PLAIN_MIN = 16384, PLAIN_MAX = 64 * 2048;   // plain_slice_kernel: beyond the one, up to the other (a lane per slice)
constexpr int STATS_MAX = 2048;                              // a row in a wavefront's registers
inline int draw_runs(int V) { return V <= 4096 ? 1 : V <= 8192 ? 2 : V <= 16384 ? 4 : 8; }
typedef float f32x4u __attribute__((ext_vector_type(4), aligned(4)));   // global memory takes 16-byte accesses at any 4-byte address

// four ids from id0 on of each of N runs of a row of V logits; past the end -inf.  WHOLE: where all of the wavefront's ids exist (id0 is
// its first id plus four times the lane) nothing is shifted, which is a seventh of a mass's arithmetic (64 sequences of 100000 25.3 ->
// 24.6 us); the tree's draw, whose registers are full, is better off without (a step of 88 rows 854 -> 868 us with it), and rows in eight
// runs have no use for it (128 registers for 95, the same time).
template <bool WHOLE = true, int N>
__device__ __forceinline__ void draw_load(const float* row, int V, int id0, floatx4 (&v)[N])
{
    if (WHOLE && __builtin_amdgcn_readfirstlane(id0) + 256 * N <= V) {   // (lane 0 has the wavefront's first ids) all of them exist
#pragma unroll
        for (int j = 0; j < N; ++j) {
            const f32x4u x = *reinterpret_cast<const f32x4u*>(row + id0 + 256 * j);
            v[j] = floatx4{x.x, x.y, x.z, x.w};
        }
    } else if (V >= 4) {   // every lane loads four ids that exist, the row's last ones shifted into place
        f32x4u x[N];
#pragma unroll
        for (int j = 0; j < N; ++j) x[j] = *reinterpret_cast<const f32x4u*>(row + min(id0 + 256 * j, V - 4));
#pragma unroll
        for (int j = 0; j < N; ++j) {
            const int id = id0 + 256 * j, sh = id - min(id, V - 4);
            v[j].x = sh == 0 ? x[j].x : sh == 1 ? x[j].y : sh == 2 ? x[j].z : sh == 3 ? x[j].w : -INFINITY;
            v[j].y = sh == 0 ? x[j].y : sh == 1 ? x[j].z : sh == 2 ? x[j].w : -INFINITY;
            v[j].z = sh == 0 ? x[j].z : sh == 1 ? x[j].w : -INFINITY;
            v[j].w = sh == 0 ? x[j].w : -INFINITY;
        }
    } else {
#pragma unroll
        for (int j = 0; j < N; ++j) {
            const int id = id0 + 256 * j;
            v[j] = floatx4{id < V ? row[id] : -INFINITY, id + 1 < V ? row[id + 1] : -INFINITY, id + 2 < V ? row[id + 2] : -INFINITY, -INFINITY};
        }
    }
}
template <int RUNS>
__device__ __forceinline__ int draw_id0() { return (threadIdx.x >> 6) * (256 * RUNS) + 4 * (threadIdx.x & 63); }

template <int N>
__device__ __forceinline__ void draw_store(float* row, int V, int id0, const floatx4 (&v)[N])
{
#pragma unroll
    for (int j = 0; j < N; ++j) {
        const int id = id0 + 256 * j;
        if (id + 4 <= V) {
            *reinterpret_cast<f32x4u*>(row + id) = f32x4u{v[j].x, v[j].y, v[j].z, v[j].w};
        } else {
            if (id < V) row[id] = v[j].x;
            if (id + 1 < V) row[id + 1] = v[j].y;
            if (id + 2 < V) row[id + 2] = v[j].z;
        }
    }
}

struct DrawLds {
    double tot[DRAW_WAVES];
    int tok;
};

// The id at which the running sum of the masses (never negative) first exceeds u times the whole (absolute: u itself), ids
// ascending; if rounding leaves no crossing, the last id with mass of the stretch looked at.  PART: the workgroup holds a part of
// the row, below is the mass of what lies before it.  run: this thread's sums of
// its four ids of every run; four(j, x): those ids' masses again.  Returns false if there is no mass (nothing drawn).  All
// threads call; the result is in l.tok for all of them.
template <int RUNS, int WAVES, bool PART = false, typename F>
__device__ __forceinline__ bool draw_locate(double (&run)[RUNS], F four, double u, bool absolute, DrawLds& l, double below = 0.0)
{
    const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
    double t = 0.0;
#pragma unroll
    for (int j = 0; j < RUNS; ++j) t += run[j];
    t = wave_sum(t);
    if (lane == 0) l.tot[wave] = t;
    __syncthreads();
    // lane w takes wavefront w's sum: the first of them whose running sum passes the target
    const double tw = lane < WAVES ? l.tot[lane] : 0.0;
    const double upto = PART ? below + row_scan(tw) : row_scan(tw), S = read_lane(upto, WAVES - 1);
    if (!absolute && !(S > 0.0)) return false;
    const double target = absolute ? u : u * S;
    // Only what has mass is picked, at each of the three levels below: lanes add the running sums up in different orders, so behind
    // the last mass before the target one may stand above it by its last bit (two halves alike and u = 0.5: an excluded id in 8 % of the draws).
    const unsigned long long over = __ballot(tw > 0.0 && upto > target), some = __ballot(tw > 0.0);   // (lanes past the wavefronts: 0)
    const int pick = over ? __ffsll((long long)over) - 1 : some ? 63 - __clzll((long long)some) : 0;
    const double before = pick > 0 ? read_lane(upto, pick - 1) : PART ? below : 0.0;
    if (wave == pick) {   // the only wavefront that looks closer: which run, which lane, which id
        int at = -1, last_run = 0;
        double c0 = before, at_before = before, last_before = before;
#pragma unroll
        for (int j = 0; j < RUNS; ++j) {
            const double r = wave_sum(run[j]);
            if (r > 0.0) { last_run = j; last_before = c0; }
            if (at < 0 && r > 0.0 && c0 + r > target) { at = j; at_before = c0; }
            c0 += r;
        }
        if (at < 0) { at = last_run; at_before = last_before; }
        double x[4];
        four(at, x);
        const double loc = (x[0] + x[1]) + (x[2] + x[3]);
        const double inc = wave_scan(loc) + at_before;
        // the first lane whose running sum passes the target; its ids one by one
        const int id0 = wave * (256 * RUNS) + 256 * at + 4 * lane;
        double cdf = inc - loc;
        int mine = -1, mine_last = -1;
#pragma unroll
        for (int e = 0; e < 4; ++e) {
            cdf += x[e];
            if (mine < 0 && x[e] > 0.0 && cdf > target) mine = id0 + e;
            if (x[e] > 0.0) mine_last = id0 + e;
        }
        if (mine < 0) mine = mine_last;   // rounding between the lane's sum and the running one
        const unsigned long long hit = __ballot(inc > target && mine >= 0), any = __ballot(mine_last >= 0);
        const int from = hit ? __ffsll((long long)hit) - 1 : any ? 63 - __clzll((long long)any) : 0;
        const int tok = __shfl(hit ? mine : mine_last, from);
        if (lane == 0) l.tok = max(tok, 0);
    }
    __syncthreads();
    return true;
}

// What a draw leaves behind; the first wavefront calls.  x: lane i holds proposal i.
__device__ __forceinline__ void draw_emit(const StepTables& t, const DrawEmit& emit, int b, int slot, int n, int K, int Kmax, int a,
                                          int y, int x, int auto_rollback, int32_t* kv_len, int32_t* n_accepted, int32_t* out_tokens)
{
    const int i = threadIdx.x;
    if (emit.tokens) {
        if (i == 0) {
            emit.tokens[b * emit.stride + emit.offset] = y;
            emit.next_token[b] = y;
            if (emit.kv_len) emit.kv_len[slot] = n + emit.kv_add;
        }
        return;
    }
    if (i <= Kmax) out_tokens[b * (Kmax + 1) + i] = i < a ? x : i == a ? y : -1;
    if (i == 0) {
        n_accepted[b] = a;
        if (kv_len) {
            const int len = n + (auto_rollback ? a : K) + 1;
            kv_len[slot] = len;
            pool_trim(t.pool, slot, len);
        }
    }
}

// a sequence that the row bookkeeping skipped; all threads call
__device__ __forceinline__ void draw_skip(const DrawEmit& emit, int b, int Kmax, int32_t* n_accepted, int32_t* out_tokens)
{
    const int i = threadIdx.x;
    if (emit.tokens) {   // an invalid id makes whoever consumes it skip the sequence too
        if (i == 0) {
            emit.tokens[b * emit.stride + emit.offset] = -1;
            emit.next_token[b] = -1;
        }
        return;
    }
    if (i == 0) n_accepted[b] = -1;
    if (i <= Kmax) out_tokens[b * (Kmax + 1) + i] = -1;
}

// After the statistics: accept scan, mass of the final draw's distribution, the draw, the results.  Rows of up to SLICE_MIN
// logits, in large batches DRAW_MAX; others are shared out (accept_slice_kernel, draw_route).  STATS: the statistics as well, a wavefront per row -- at most 31 rows of
// STATS_MAX logits, which one compute unit reads in the time that a launch takes (fp32 model of vocabulary 1024, one sequence of
// five rows: 4.3 + 5.9 us as two launches, 7.8 as one).
template <int RUNS, bool STATS>
__global__ void __launch_bounds__(DRAW_TPB) accept_draw_kernel(const int32_t* seq_stat0, const int32_t* seq_row0,
                                                               const int32_t* __restrict__ draft_tokens,
                                                               const float* __restrict__ part_max,
                                                               const double* __restrict__ part_sum, int Kmax, int V,
                                                               int n_stat_chunks, int u_stride,
                                                               const float* __restrict__ uniforms,
                                                               const float* __restrict__ target,
                                                               const float* __restrict__ draft, float inv_T_f, int auto_rollback,
                                                               int32_t* kv_len, int32_t* __restrict__ n_accepted,
                                                               int32_t* __restrict__ out_tokens, StepTables t, LookaheadPack ks)
{
    __shared__ float row_m[2 * SPEC_MAX_LOOKAHEAD + 2];
    __shared__ double row_z[2 * SPEC_MAX_LOOKAHEAD + 2];
    __shared__ int s_a;
    __shared__ double s_iz[2];
    __shared__ DrawLds l;
    const int b = blockIdx.x;
    const int st0 = seq_stat0[b], row0 = seq_row0[b], ok = t.seq_ok[b], slot = t.seq_slot[b], n = t.seq_n[b];
    const int K = ks.k[b];
    const double inv_T = (double)inv_T_f;
    const float* trow0 = target + (size_t)row0 * V;
    const float* drow0 = draft + (size_t)b * Kmax * V;
    const int i = min((int)threadIdx.x, max(K - 1, 0));   // lane i tests proposal i, all positions at once
    float lp_x = 0.f, lq_x = 0.f;
    double u = 0.0;
    int x = 0;
    if (threadIdx.x < 64 && K > 0) {
        x = draft_tokens[b * Kmax + i];
        const bool xin = x >= 0 && x < V;   // out-of-range ids were flagged by prepare; stay in bounds
        u = (double)uniforms[b * u_stride + i];
        lp_x = xin ? trow0[(size_t)i * V + x] : 0.f;
        lq_x = xin ? drow0[(size_t)i * V + x] : 0.f;
    }
    const double u_draw = (double)uniforms[b * u_stride + K];
    if (!ok) {
        draw_skip(DrawEmit{}, b, Kmax, n_accepted, out_tokens);
        return;
    }
    if constexpr (STATS) {
        for (int r = threadIdx.x >> 6; r < 2 * K + 1; r += DRAW_WAVES) {
            const float* row = r <= K ? trow0 + (size_t)r * V : drow0 + (size_t)(r - K - 1) * V;
            constexpr int N = STATS_MAX / 256;
            floatx4 v[N];
            draw_load<RUNS < 8>(row, V, 4 * (threadIdx.x & 63), v);
            float mx = -INFINITY;
#pragma unroll
            for (int j = 0; j < N; ++j) mx = fmaxf(fmaxf(mx, fmaxf(v[j].x, v[j].y)), fmaxf(v[j].z, v[j].w));
            mx = wave_max(mx);
            const float mm = mx == -INFINITY ? 0.f : mx;
            double z = 0.0;
#pragma unroll
            for (int j = 0; j < N; ++j)
#pragma unroll
                for (int e = 0; e < 4; ++e) z += (double)__expf((v[j][e] - mm) * inv_T_f);
            z = wave_sum(z);
            if ((threadIdx.x & 63) == 0) {
                row_m[r] = mx;
                row_z[r] = z;
            }
        }
        __syncthreads();
    } else {
        __shared__ CombineLds comb;
        combine_rows<DRAW_TPB>(part_max, part_sum, st0, 2 * K + 1, n_stat_chunks, inv_T, row_m, row_z, comb);
    }
    if (threadIdx.x < 64) {
        bool keep = true;
        if (K > 0) {
            const double ep = exp((double)(lp_x - row_m[i]) * inv_T);
            const double eq = exp((double)(lq_x - row_m[K + 1 + i]) * inv_T);
            keep = u * eq * row_z[i] < ep * row_z[K + 1 + i];   // u * q(x) < p(x)
        }
        const unsigned long long failed = __ballot(!keep && (int)threadIdx.x < K);
        const int first = failed ? __builtin_ctzll(failed) : K;
        if (threadIdx.x < 2) s_iz[threadIdx.x] = 1.0 / row_z[threadIdx.x == 0 ? first : first < K ? K + 1 + first : 0];
        if (threadIdx.x == 0) s_a = first;
    }
    __syncthreads();
    const int a = s_a;
    const bool residual = a < K;
    const float mp = row_m[a], mq = residual ? row_m[K + 1 + a] : 0.f;
    const double izp = s_iz[0], izq = s_iz[1];
    const float* prow = trow0 + (size_t)a * V;            // a == K: the extra-token row
    const float* qrow = drow0 + (size_t)(residual ? a : 0) * V;
    auto mass = [&](float lp, float lq) {
        const double pv = (double)__expf((lp - mp) * inv_T_f) * izp, qv = residual ? (double)__expf((lq - mq) * inv_T_f) * izq : 0.0;
        return pv > qv ? pv - qv : 0.0;
    };
    double run[RUNS];
    {
        floatx4 p[RUNS], q[RUNS];
        draw_load<RUNS < 8>(prow, V, draw_id0<RUNS>(), p);
        if (residual) draw_load<RUNS < 8>(qrow, V, draw_id0<RUNS>(), q);
#pragma unroll
        for (int j = 0; j < RUNS; ++j)
            run[j] = (mass(p[j].x, q[j].x) + mass(p[j].y, q[j].y)) + (mass(p[j].z, q[j].z) + mass(p[j].w, q[j].w));
    }
    auto four = [&](int j, double (&x)[4]) {   // (read again rather than kept: both rows are 64 registers)
        floatx4 p[1], q[1];
        draw_load<RUNS < 8>(prow, V, draw_id0<RUNS>() + 256 * j, p);
        if (residual) draw_load<RUNS < 8>(qrow, V, draw_id0<RUNS>() + 256 * j, q);
#pragma unroll
        for (int e = 0; e < 4; ++e) x[e] = mass(p[0][e], q[0][e]);
    };
    if (!draw_locate<RUNS, DRAW_WAVES>(run, four, u_draw, false, l)) {   // no mass left (impossible in exact arithmetic): draw from p_a, which sums to 1
        __syncthreads();
        auto plain = [&](float lp) { return (double)__expf((lp - mp) * inv_T_f) * izp; };
        floatx4 p[RUNS];
        draw_load<RUNS < 8>(prow, V, draw_id0<RUNS>(), p);
#pragma unroll
        for (int j = 0; j < RUNS; ++j) run[j] = (plain(p[j].x) + plain(p[j].y)) + (plain(p[j].z) + plain(p[j].w));
        draw_locate<RUNS, DRAW_WAVES>(run, [&](int j, double (&x)[4]) {
            floatx4 p1[1];
            draw_load<RUNS < 8>(prow, V, draw_id0<RUNS>() + 256 * j, p1);
#pragma unroll
            for (int e = 0; e < 4; ++e) x[e] = plain(p1[0][e]);
        }, u_draw, true, l);
    }
    if (threadIdx.x < 64) draw_emit(t, DrawEmit{}, b, slot, n, K, Kmax, a, l.tok, x, auto_rollback, kv_len, n_accepted, out_tokens);
}

// The same for longer rows: a workgroup per sequence and slice of 1024 RUNS ids.  Every workgroup repeats the accept scan (a handful
// of scalars) and sums the mass of its slice; whichever of a sequence's workgroups comes last finds the slice that the
// target falls on, reads it again and draws.  The mass of an id is two exponentials and a few fp64 operations, 84 issue
// cycles for a wavefront's 64: a row of 32000 in one workgroup of 1024 threads spent 4 to 5 us on them alone, and two
// launches (masses, then draw) a launch and another chain of round trips.  The sampling part alone, us before and now: 4
// sequences of 32003 16.4 -> 14.1, 8 of 32000 17.7 -> 14.2, 32 of 32000 19.7 -> 17.0, one of 128256 18.5 -> 13.9, 16 of 128256 29.0
// -> 24.7.
//
// No workgroup waits for another: each stores its mass with an atomic store at device scope, waits until that has arrived, and then
// counts itself; the one that counts last sees all masses.  The row bookkeeping in front has set the count to zero.  The accesses are
// relaxed (a release would write back the XCD's whole L2); what orders them is gfx950's own: vmcnt counts stores, which leave it
// when they have arrived where they are visible, and accesses at device scope pass the XCD's L2 in both directions.
//
// COUNTED = false: the masses only, slice_draw_kernel draws.  Where a launch has many workgroups per compute unit, the round trip of
// the count is time that none of them can use (see draw_route).

// The rows a draw takes its masses from, in slices of 1024 RUNS ids: p at temperature, less q where a proposal was rejected.
template <int RUNS>
struct SliceRows {
    static constexpr int SLICE = TPB * 4 * RUNS;
    const float *prow, *qrow;
    double izp, izq;
    float mp, mq, inv_T;
    int V;

    __device__ __forceinline__ double mass(float lp, float lq, bool with_q) const
    {
        const double pv = (double)__expf((lp - mp) * inv_T) * izp, qv = with_q ? (double)__expf((lq - mq) * inv_T) * izq : 0.0;
        return pv > qv ? pv - qv : 0.0;
    }
    // a thread's sums of its four ids of every run of a slice
    __device__ __forceinline__ void sums_of(int c, bool with_q, double (&run)[RUNS]) const
    {
        floatx4 p[RUNS], q[RUNS];
        const int id0 = c * SLICE + draw_id0<RUNS>();
        draw_load(prow, V, id0, p);
        if (with_q) draw_load(qrow, V, id0, q);
#pragma unroll
        for (int j = 0; j < RUNS; ++j)
            run[j] = (mass(p[j].x, q[j].x, with_q) + mass(p[j].y, q[j].y, with_q)) + (mass(p[j].z, q[j].z, with_q) + mass(p[j].w, q[j].w, with_q));
    }
    __device__ __forceinline__ double total(const double (&run)[RUNS], DrawLds& l) const   // of the workgroup, the same for all threads
    {
        double sum = 0.0;
#pragma unroll
        for (int j = 0; j < RUNS; ++j) sum += run[j];
        sum = wave_sum(sum);
        if ((threadIdx.x & 63) == 0) l.tot[threadIdx.x >> 6] = sum;
        __syncthreads();
        static_assert(TPB == 256, "four sums");
        return (l.tot[0] + l.tot[1]) + (l.tot[2] + l.tot[3]);
    }

    // The id that u times the whole falls on, once the masses of all slices are there.  All threads of the workgroup call.
    __device__ __forceinline__ int draw(const double* masses, int n_slices, bool residual, double u, DrawLds& l) const
    {
        const int lane = threadIdx.x & 63;
        double run[RUNS];
        // The slice that the running sum passes u times the whole in, as draw_locate looks among wavefronts: every wavefront for
        // itself, 64 slices at a time
        auto mass_of = [&](int c) { return c < n_slices ? __hip_atomic_load(masses + c, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) : 0.0; };
        const double first64 = mass_of(lane);
        double S = 0.0;
        for (int c0 = 0; c0 < n_slices; c0 += 64) S += wave_sum(c0 == 0 ? first64 : mass_of(c0 + lane));
        int pick = -1;
        bool with_q = residual;
        double below = 0.0, goal = u * S;
        if (S > 0.0) {
            double before = 0.0;
            for (int c0 = 0; c0 < n_slices; c0 += 64) {
                const double m = c0 == 0 ? first64 : mass_of(c0 + lane), upto = before + wave_scan(m);
                const unsigned long long over = __ballot(m > 0.0 && upto > goal), some = __ballot(m > 0.0);
                if (over || some) {
                    const int at = over ? __ffsll((long long)over) - 1 : 63 - __clzll((long long)some);
                    pick = c0 + at;
                    below = at > 0 ? read_lane(upto, at - 1) : before;
                }
                if (over) break;
                before = read_lane(upto, 63);
            }
        } else {   // no mass left (impossible in exact arithmetic): draw from p_a, which sums to 1, slice by slice
            with_q = false;
            goal = u;
            double before = 0.0;
            for (int c = 0; c < n_slices; ++c) {
                sums_of(c, false, run);
                const double sum = total(run, l);
                __syncthreads();
                if (sum > 0.0 || pick < 0) {
                    pick = c;
                    below = before;
                }
                before += sum;
                if (before > goal) break;
            }
        }
        sums_of(pick, with_q, run);
        __syncthreads();
        // (ids of the slice; a row's end lies inside the last one)
        draw_locate<RUNS, TPB / 64, true>(run, [&](int j, double (&m4)[4]) {
            floatx4 p[1], q[1];
            const int id0 = pick * SLICE + draw_id0<RUNS>() + 256 * j;
            draw_load(prow, V, id0, p);
            if (with_q) draw_load(qrow, V, id0, q);
#pragma unroll
            for (int e = 0; e < 4; ++e) m4[e] = mass(p[0][e], q[0][e], with_q);
        }, goal, true, l, below);
        return min(pick * SLICE + l.tok, V - 1);
    }
};

template <int RUNS, bool COUNTED>
__global__ void __launch_bounds__(TPB) accept_slice_kernel(const int32_t* seq_stat0, const int32_t* seq_row0,
                                                           const int32_t* __restrict__ draft_tokens,
                                                           const float* __restrict__ part_max,
                                                           const double* __restrict__ part_sum, int Kmax, int V,
                                                           int n_stat_chunks, int u_stride,
                                                           const float* __restrict__ uniforms,
                                                           const float* __restrict__ target,
                                                           const float* __restrict__ draft, float inv_T_f, int auto_rollback,
                                                           int32_t* kv_len, int32_t* __restrict__ n_accepted,
                                                           int32_t* __restrict__ out_tokens, double* slice_mass, DrawnRow* drawn,
                                                           StepTables t, DrawEmit emit, LookaheadPack ks)
{
    __shared__ float row_m[2 * SPEC_MAX_LOOKAHEAD + 2];
    __shared__ double row_z[2 * SPEC_MAX_LOOKAHEAD + 2];
    __shared__ int s_a, s_last;
    __shared__ double s_iz[2];
    __shared__ DrawLds l;
    __shared__ CombineLds comb;
    const int b = blockIdx.y, slice = blockIdx.x, n_slices = gridDim.x;
    const int st0 = seq_stat0[b], row0 = seq_row0[b], ok = t.seq_ok[b], slot = t.seq_slot[b], n = t.seq_n[b];
    const int K = ks.k[b];
    const double inv_T = (double)inv_T_f;
    const float* trow0 = target + (size_t)row0 * V;
    const float* drow0 = draft + (size_t)b * Kmax * V;
    // lane i tests proposal i (all positions at once: only the first failure matters); padding lanes repeat the last
    // proposal and are masked out.  Its logits are requested before the statistics are put together.
    const int i = min((int)threadIdx.x, max(K - 1, 0));
    float lp_x = 0.f, lq_x = 0.f;
    double u = 0.0;
    int x = 0;
    if (threadIdx.x < 64 && K > 0) {
        x = draft_tokens[b * Kmax + i];
        const bool xin = x >= 0 && x < V;   // out-of-range ids were flagged by prepare; stay in bounds
        u = (double)uniforms[b * u_stride + i];
        lp_x = xin ? trow0[(size_t)i * V + x] : 0.f;
        lq_x = xin ? drow0[(size_t)i * V + x] : 0.f;
    }
    const double u_draw = COUNTED ? (double)uniforms[b * u_stride + K] : 0.0;
    if (!ok) {
        if (COUNTED && slice == 0) draw_skip(emit, b, Kmax, n_accepted, out_tokens);
        return;
    }
    combine_rows<TPB>(part_max, part_sum, st0, 2 * K + 1, n_stat_chunks, inv_T, row_m, row_z, comb);
    if (threadIdx.x < 64) {
        bool keep = true;
        if (K > 0) {
            const double ep = exp((double)(lp_x - row_m[i]) * inv_T);
            const double eq = exp((double)(lq_x - row_m[K + 1 + i]) * inv_T);
            keep = u * eq * row_z[i] < ep * row_z[K + 1 + i];   // u * q(x) < p(x)
        }
        const unsigned long long failed = __ballot(!keep && (int)threadIdx.x < K);
        const int first = failed ? __builtin_ctzll(failed) : K;
        if (threadIdx.x < 2) s_iz[threadIdx.x] = 1.0 / row_z[threadIdx.x == 0 ? first : first < K ? K + 1 + first : 0];
        if (threadIdx.x == 0) s_a = first;
    }
    __syncthreads();
    const int a = s_a;
    const bool residual = a < K;
    const SliceRows<RUNS> rows{trow0 + (size_t)a * V,            // a == K: the extra-token row
                               drow0 + (size_t)(residual ? a : 0) * V, s_iz[0], s_iz[1], row_m[a], residual ? row_m[K + 1 + a] : 0.f, inv_T_f, V};
    double* masses = slice_mass + (size_t)b * n_slices;
    double run[RUNS];
    rows.sums_of(slice, residual, run);
    const double sum = rows.total(run, l);
    if constexpr (COUNTED) {
        if (threadIdx.x == 0) {
            __hip_atomic_store(masses + slice, sum, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            asm volatile("s_waitcnt vmcnt(0)" ::: "memory");   // (the mass has arrived before it is counted: see above)
            s_last = __hip_atomic_fetch_add(t.arrived + b * ARRIVED_STRIDE, 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) == n_slices - 1;
        }
        __syncthreads();
        if (!s_last) return;
        const int y = rows.draw(masses, n_slices, residual, u_draw, l);
        if (threadIdx.x < 64) draw_emit(t, emit, b, slot, n, K, Kmax, a, y, x, auto_rollback, kv_len, n_accepted, out_tokens);
    } else if (threadIdx.x == 0) {
        masses[slice] = sum;
        if (slice == 0) drawn[b] = DrawnRow{rows.izp, rows.izq, rows.mp, rows.mq, a, 0};
    }
}

// The draw behind accept_slice_kernel<RUNS, false>: one workgroup per sequence, the bits of the other route.
template <int RUNS>
__global__ void __launch_bounds__(TPB) slice_draw_kernel(const int32_t* seq_row0, const double* slice_mass, const DrawnRow* drawn,
                                                         const float* __restrict__ uniforms, int u_stride, int n_slices, int Kmax, int V,
                                                         const float* __restrict__ target, const float* __restrict__ draft, float inv_T_f,
                                                         int auto_rollback, int32_t* kv_len, const int32_t* __restrict__ draft_tokens,
                                                         int32_t* __restrict__ n_accepted, int32_t* __restrict__ out_tokens, StepTables t,
                                                         DrawEmit emit, LookaheadPack ks)
{
    __shared__ DrawLds l;
    const int b = blockIdx.x, K = ks.k[b];
    const int row0 = seq_row0[b], ok = t.seq_ok[b], slot = t.seq_slot[b], n = t.seq_n[b];
    const int x = K > 0 ? draft_tokens[b * Kmax + min((int)threadIdx.x, K - 1)] : 0;
    const double u = (double)uniforms[b * u_stride + K];
    if (!ok) {
        draw_skip(emit, b, Kmax, n_accepted, out_tokens);
        return;
    }
    const DrawnRow d = drawn[b];
    const SliceRows<RUNS> rows{target + (size_t)(row0 + d.a) * V, draft + ((size_t)b * Kmax + (d.a < K ? d.a : 0)) * V, d.izp, d.izq, d.mp, d.mq, inv_T_f, V};
    const int y = rows.draw(slice_mass + (size_t)b * n_slices, n_slices, d.a < K, u, l);
    if (threadIdx.x < 64) draw_emit(t, emit, b, slot, n, K, Kmax, d.a, y, x, auto_rollback, kv_len, n_accepted, out_tokens);
}

// A plain draw (no proposals): maximum, weights and draw of one row per sequence, which comes whole or as the LM head's
// partial sums (SRC; written to src.out on the way).  The draft model's draw was four launches (row sum, statistics, mass, draw).
template <bool SRC, int RUNS>
__global__ void __launch_bounds__(DRAW_TPB) plain_draw_kernel(const int32_t* seq_row0, const float* __restrict__ target,
                                                              const float* __restrict__ uniforms, int u_stride, int V, int Kmax,
                                                              float inv_T_f, int auto_rollback, int32_t* kv_len,
                                                              int32_t* __restrict__ n_accepted, int32_t* __restrict__ out_tokens,
                                                              StepTables t, DrawEmit emit, LogitsSrc src)
{
    __shared__ float s_max[DRAW_WAVES];
    __shared__ DrawLds l;
    const int b = blockIdx.x, lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const int m = seq_row0[b], ok = t.seq_ok[b], slot = t.seq_slot[b], n = t.seq_n[b];
    const double u = (double)uniforms[b * u_stride];
    const int first = draw_id0<RUNS>();
    floatx4 v[RUNS];
    if constexpr (SRC) {
        const float rs = row_inv_rms(src.ns.ssq, src.ns.n_ssq, m, src.ns.d, src.ns.eps);
        const float* p = src.partial + (size_t)m * src.ld;   // (a row has ld >= V columns, a multiple of 16, to read)
        switch (src.n_split) {
        case 1: logits_from<1>(p, src.stride, 256, src.ld, first, rs, v); break;
        case 2: logits_from<2>(p, src.stride, 256, src.ld, first, rs, v); break;
        case 4: logits_from<4>(p, src.stride, 256, src.ld, first, rs, v); break;
        case 8: logits_from<8>(p, src.stride, 256, src.ld, first, rs, v); break;
        default: logits_from<16>(p, src.stride, 256, src.ld, first, rs, v); break;
        }
#pragma unroll
        for (int j = 0; j < RUNS; ++j) {
            const int id = first + 256 * j;
            if (id >= V) v[j].x = -INFINITY;
            if (id + 1 >= V) v[j].y = -INFINITY;
            if (id + 2 >= V) v[j].z = -INFINITY;
            if (id + 3 >= V) v[j].w = -INFINITY;
        }
        draw_store(src.out + (size_t)m * V, V, first, v);
    } else {
        draw_load(target + (size_t)m * V, V, draw_id0<RUNS>(), v);
    }
    if (emit.logits_copy) draw_store(emit.logits_copy + (size_t)b * emit.copy_stride, V, first, v);
    if (!ok) {
        draw_skip(emit, b, Kmax, n_accepted, out_tokens);
        return;
    }
    // the weights relative to the row's maximum are all a draw needs: their sum takes the place of the normaliser
    float mw = -INFINITY;
#pragma unroll
    for (int j = 0; j < RUNS; ++j) mw = fmaxf(fmaxf(mw, fmaxf(v[j].x, v[j].y)), fmaxf(v[j].z, v[j].w));
    mw = wave_max(mw);
    if (lane == 0) s_max[wave] = mw;
    __syncthreads();
    const float mp = wave_max(s_max[lane % DRAW_WAVES]);
    double run[RUNS];
#pragma unroll
    for (int j = 0; j < RUNS; ++j) {
#pragma unroll
        for (int e = 0; e < 4; ++e) v[j][e] = __expf((v[j][e] - mp) * inv_T_f);
        run[j] = ((double)v[j].x + (double)v[j].y) + ((double)v[j].z + (double)v[j].w);
    }
    // (no mass at all takes a row without a finite logit; the draw is then what rounding makes of it)
    if (!draw_locate<RUNS, DRAW_WAVES>(run, [&](int j, double (&x)[4]) {
            floatx4 e4 = v[0];
#pragma unroll
            for (int i = 1; i < RUNS; ++i)
#pragma unroll
                for (int e = 0; e < 4; ++e) e4[e] = j == i ? v[i][e] : e4[e];
#pragma unroll
            for (int e = 0; e < 4; ++e) x[e] = (double)e4[e];
        }, u, false, l)) {
        if (threadIdx.x == 0) l.tok = 0;
        __syncthreads();
    }
    if (threadIdx.x < 64) draw_emit(t, emit, b, slot, n, 0, Kmax, 0, l.tok, 0, auto_rollback, kv_len, n_accepted, out_tokens);
}

// The same for rows of more than PLAIN_MIN ids, shared out as accept_slice_kernel shares them: a workgroup per sequence and 2048 ids
// finishes and stores its part of the row and leaves that part's maximum and sum of weights; the last one brings the parts
// to one maximum, finds the part that the target falls on, makes its logits again and draws.  In one workgroup the row's
// partial sums, its stores (the logits and the draft's copy of them) and its exponentials were a compute unit's share of all three.
// Steps of two layers, one row a sequence, 1, 8 and 48 sequences: vocabulary 20000 95.6 -> 91.2, 96.7 -> 92.3 and 139.8 -> 137.4 us,
// 50257 (before: statistics, then accept_slice_kernel) 109.9 -> 100.5, 112.7 -> 101.7 and 159.4 -> 146.8, 128256 132.5 -> 125.9, 136.0 ->
// 127.6 and 194.9 -> 175.6; 12000 0 to +0.6 %.  Draft decode of 8 rows 288.0 -> 284.5, decoding round 2165 -> 2146.
template <bool SRC>
__global__ void __launch_bounds__(TPB) plain_slice_kernel(const int32_t* seq_row0, const float* __restrict__ target,
                                                          const float* __restrict__ uniforms, int u_stride, int V, int Kmax,
                                                          float inv_T_f, int auto_rollback, int32_t* kv_len,
                                                          int32_t* __restrict__ n_accepted, int32_t* __restrict__ out_tokens,
                                                          double* slice_mass, StepTables t, DrawEmit emit, LogitsSrc src)
{
    constexpr int RUNS = 2, WAVES = TPB / 64, SLICE = TPB * 4 * RUNS;
    __shared__ float s_max[WAVES];
    __shared__ int s_last;
    __shared__ DrawLds l;
    const int b = blockIdx.y, slice = blockIdx.x, n_slices = gridDim.x, lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const int m = seq_row0[b], ok = t.seq_ok[b], slot = t.seq_slot[b], n = t.seq_n[b];
    const double u = (double)uniforms[b * u_stride];
    float rs = 1.f;
    if constexpr (SRC) rs = row_inv_rms(src.ns.ssq, src.ns.n_ssq, m, src.ns.d, src.ns.eps);
    auto logits = [&](int first, floatx4 (&v)[RUNS]) {   // a thread's ids of a slice; past the end -inf
        if constexpr (SRC) {
            const float* p = src.partial + (size_t)m * src.ld;   // (a row has ld >= V columns, a multiple of 16, to read)
            switch (src.n_split) {
            case 1: logits_from<1>(p, src.stride, 256, src.ld, first, rs, v); break;
            case 2: logits_from<2>(p, src.stride, 256, src.ld, first, rs, v); break;
            case 4: logits_from<4>(p, src.stride, 256, src.ld, first, rs, v); break;
            case 8: logits_from<8>(p, src.stride, 256, src.ld, first, rs, v); break;
            default: logits_from<16>(p, src.stride, 256, src.ld, first, rs, v); break;
            }
#pragma unroll
            for (int j = 0; j < RUNS; ++j)
#pragma unroll
                for (int e = 0; e < 4; ++e)
                    if (first + 256 * j + e >= V) v[j][e] = -INFINITY;
        } else {
            draw_load(target + (size_t)m * V, V, first, v);
        }
    };
    floatx4 v[RUNS];
    const int first = slice * SLICE + draw_id0<RUNS>();
    logits(first, v);
    if constexpr (SRC) draw_store(src.out + (size_t)m * V, V, first, v);
    if (emit.logits_copy) draw_store(emit.logits_copy + (size_t)b * emit.copy_stride, V, first, v);
    if (!ok) {
        if (slice == 0) draw_skip(emit, b, Kmax, n_accepted, out_tokens);
        return;
    }
    float mw = -INFINITY;
#pragma unroll
    for (int j = 0; j < RUNS; ++j) mw = fmaxf(fmaxf(mw, fmaxf(v[j].x, v[j].y)), fmaxf(v[j].z, v[j].w));
    mw = wave_max(mw);
    if (lane == 0) s_max[wave] = mw;
    __syncthreads();
    // weights relative to the slice's own maximum (a slice without a finite logit: all of them zero)
    auto weights = [&](float mp, double (&run)[RUNS], floatx4 (&x)[RUNS]) {
#pragma unroll
        for (int j = 0; j < RUNS; ++j) {
#pragma unroll
            for (int e = 0; e < 4; ++e) x[j][e] = mp == -INFINITY ? 0.f : __expf((x[j][e] - mp) * inv_T_f);
            run[j] = ((double)x[j].x + (double)x[j].y) + ((double)x[j].z + (double)x[j].w);
        }
    };
    double run[RUNS];
    const float mp = fmaxf(fmaxf(s_max[0], s_max[1]), fmaxf(s_max[2], s_max[3]));
    weights(mp, run, v);
    const double part = wave_sum(run[0] + run[1]);
    static_assert(RUNS == 2 && WAVES == 4, "two runs, four wavefronts");
    if (lane == 0) l.tot[wave] = part;
    __syncthreads();
    double* parts = slice_mass + (size_t)b * n_slices * 2;   // maximum and sum of every slice
    if (threadIdx.x == 0) {
        __hip_atomic_store(parts + 2 * slice, (double)mp, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        __hip_atomic_store(parts + 2 * slice + 1, (l.tot[0] + l.tot[1]) + (l.tot[2] + l.tot[3]), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        asm volatile("s_waitcnt vmcnt(0)" ::: "memory");   // (they have arrived before they are counted: see accept_slice_kernel)
        s_last = __hip_atomic_fetch_add(t.arrived + b * ARRIVED_STRIDE, 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) == n_slices - 1;
    }
    __syncthreads();
    if (!s_last) return;
    // (at most 64 slices: PLAIN_MAX)
    const bool in = lane < n_slices;
    const float mc = in ? (float)__hip_atomic_load(parts + 2 * lane, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) : -INFINITY;
    const double sc = in ? __hip_atomic_load(parts + 2 * lane + 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) : 0.0;
    const float mx = wave_max(mc);
    const double f = sc > 0.0 ? exp((double)(mc - mx) * (double)inv_T_f) : 0.0, mass = sc * f;   // to the row's maximum
    const double upto = wave_scan(mass), goal = u * read_lane(upto, 63);
    const unsigned long long over = __ballot(mass > 0.0 && upto > goal), some = __ballot(mass > 0.0);
    int tok = 0;   // (no mass at all takes a row without a finite logit)
    if (some) {
        const int pick = over ? __ffsll((long long)over) - 1 : 63 - __clzll((long long)some);
        const double below = pick > 0 ? read_lane(upto, pick - 1) : 0.0, scale = read_lane(f, pick);
        const float mpick = __shfl(mc, pick);
        floatx4 x[RUNS];
        logits(pick * SLICE + draw_id0<RUNS>(), x);
        weights(mpick, run, x);
#pragma unroll
        for (int j = 0; j < RUNS; ++j) run[j] *= scale;
        __syncthreads();
        draw_locate<RUNS, WAVES, true>(run, [&](int j, double (&m4)[4]) {
#pragma unroll
            for (int e = 0; e < 4; ++e) m4[e] = (double)(j == 0 ? x[0][e] : x[1][e]) * scale;
        }, goal, true, l, below);
        tok = min(pick * SLICE + l.tok, V - 1);
    }
    if (threadIdx.x < 64) draw_emit(t, emit, b, slot, n, 0, Kmax, 0, tok, 0, auto_rollback, kv_len, n_accepted, out_tokens);
}

// ---------------------------------------------------------------------------------------------
// Temperature 0.  Pass 1: per (target row, chunk) the maximum and the lowest id that holds it.
// Pass 2 (one wavefront per sequence): combine the chunks of each window row in ascending order,
// compare with the proposals, emit.
// ---------------------------------------------------------------------------------------------
__global__ void __launch_bounds__(TPB) argmax_kernel(int V, int n_chunks, const float* __restrict__ target,
                                                     float* __restrict__ part_max, int32_t* __restrict__ part_idx)
{
    __shared__ float sv[TPB / 64];
    __shared__ int si[TPB / 64];
    const int row = blockIdx.x / n_chunks, chunk = blockIdx.x % n_chunks;
    const float* p = target + (size_t)row * V;
    const int base = chunk * STAT_CHUNK;
    const int lim = min(STAT_CHUNK, V - base);
    float best = -INFINITY;
    int bi = 0x7fffffff;
    for (int i = threadIdx.x; i < lim; i += TPB) {   // ascending ids per thread: '>' keeps the first maximum
        const float x = p[base + i];
        if (x > best || bi == 0x7fffffff) {
            best = x;
            bi = base + i;
        }
    }
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) {
        const float ob = __shfl_xor(best, o);
        const int oi = __shfl_xor(bi, o);
        if (ob > best || (ob == best && oi < bi)) {
            best = ob;
            bi = oi;
        }
    }
    if ((threadIdx.x & 63) == 0) {
        sv[threadIdx.x >> 6] = best;
        si[threadIdx.x >> 6] = bi;
    }
    __syncthreads();
    if (threadIdx.x == 0) {
        for (int w = 1; w < TPB / 64; ++w)
            if (sv[w] > best || (sv[w] == best && si[w] < bi)) {
                best = sv[w];
                bi = si[w];
            }
        part_max[(size_t)row * n_chunks + chunk] = best;
        part_idx[(size_t)row * n_chunks + chunk] = bi;
    }
}

__global__ void __launch_bounds__(64) greedy_emit_kernel(StepTables t, LookaheadPack ks, int Kmax, int n_chunks,
                                                         const float* __restrict__ part_max,
                                                         const int32_t* __restrict__ part_idx,
                                                         const int32_t* __restrict__ draft_tokens, int auto_rollback,
                                                         int32_t* kv_len, int32_t* __restrict__ n_accepted,
                                                         int32_t* __restrict__ out_tokens, DrawEmit emit)
{
    const int b = blockIdx.x;
    if (threadIdx.x != 0) return;
    if (emit.tokens) {   // a proposing model's step (every K_b = 0): the most likely token of the sequence's row
        int y = -1;
        if (t.seq_ok[b]) {
            const size_t r = (size_t)t.seq_row0[b] * n_chunks;
            float best = part_max[r];
            y = part_idx[r];
            for (int c = 1; c < n_chunks; ++c)
                if (part_max[r + c] > best) {
                    best = part_max[r + c];
                    y = part_idx[r + c];
                }
            if (emit.kv_len) emit.kv_len[t.seq_slot[b]] = t.seq_n[b] + emit.kv_add;
        }
        emit.tokens[b * emit.stride + emit.offset] = y;
        emit.next_token[b] = y;
        return;
    }
    int32_t* o = out_tokens + b * (Kmax + 1);
    if (!t.seq_ok[b]) {
        n_accepted[b] = -1;
        for (int i = 0; i <= Kmax; ++i) o[i] = -1;
        return;
    }
    const int K = ks.k[b];
    int a = 0;
    for (int j = 0; j <= K; ++j) {
        const size_t r = (size_t)(t.seq_row0[b] + j) * n_chunks;
        float best = part_max[r];
        int bi = part_idx[r];
        for (int c = 1; c < n_chunks; ++c)
            if (part_max[r + c] > best) {   // chunks ascend in id: a later equal maximum does not win
                best = part_max[r + c];
                bi = part_idx[r + c];
            }
        if (j < K && draft_tokens[b * Kmax + j] == bi) {
            o[a++] = bi;
            continue;
        }
        o[a] = bi;
        break;
    }
    for (int i = a + 1; i <= Kmax; ++i) o[i] = -1;
    n_accepted[b] = a;
    if (kv_len) {
        kv_len[t.seq_slot[b]] = t.seq_n[b] + (auto_rollback ? a : K) + 1;
        pool_trim(t.pool, t.seq_slot[b], t.seq_n[b] + (auto_rollback ? a : K) + 1);
    }
}

// Temperature 0 on a tree: from the root, move to the first child (index order) whose token is the
// most likely token of the current node's row; otherwise that token ends the step.
__global__ void __launch_bounds__(64) tree_greedy_kernel(StepTables t, LookaheadPack ks, int Kmax, int n_chunks,
                                                         const float* __restrict__ part_max,
                                                         const int32_t* __restrict__ part_idx,
                                                         const int32_t* __restrict__ parent,
                                                         const int32_t* __restrict__ tokens, int auto_rollback,
                                                         int32_t* kv_len, int32_t* __restrict__ n_accepted,
                                                         int32_t* __restrict__ out_tokens, int32_t* __restrict__ path)
{
    const int b = blockIdx.x;
    if (threadIdx.x != 0) return;
    int32_t* o = out_tokens + b * (Kmax + 1);
    int32_t* pth = path + b * Kmax;
    if (!t.seq_ok[b]) {
        n_accepted[b] = -1;
        for (int i = 0; i <= Kmax; ++i) o[i] = -1;
        for (int i = 0; i < Kmax; ++i) pth[i] = -1;
        return;
    }
    const int N = ks.k[b];
    int cur = -1, a = 0;
    for (;;) {
        const size_t r = (size_t)(t.seq_row0[b] + cur + 1) * n_chunks;
        float best = part_max[r];
        int bi = part_idx[r];
        for (int c = 1; c < n_chunks; ++c)
            if (part_max[r + c] > best) {
                best = part_max[r + c];
                bi = part_idx[r + c];
            }
        int next = -1;
        for (int c = cur + 1; c < N; ++c)
            if (parent[b * Kmax + c] == cur && tokens[b * Kmax + c] == bi) { next = c; break; }
        o[a] = bi;
        if (next < 0) break;
        pth[a++] = next;
        cur = next;
    }
    for (int i = a + 1; i <= Kmax; ++i) o[i] = -1;
    for (int i = a; i < Kmax; ++i) pth[i] = -1;
    n_accepted[b] = a;
    if (kv_len) {
        // with auto_rollback the kept path is still to be moved: its pages go back after that
        // (tree_trim_kernel), never here
        kv_len[t.seq_slot[b]] = t.seq_n[b] + (auto_rollback ? a : N) + 1;
        if (!auto_rollback) pool_trim(t.pool, t.seq_slot[b], t.seq_n[b] + N + 1);
    }
}

// ---------------------------------------------------------------------------------------------
// Token trees.  Window slot 0 is the sequence's last token (the root), slot i+1 is node i; the
// nodes come in topological order with parent[i] = -1 (child of the root) or an index < i.
// ---------------------------------------------------------------------------------------------
typedef uint16_t TreeMasks[SPEC_MAX_LOOKAHEAD + 1][TPB];
// (a workgroup of TPB threads, all of them calling)
__device__ __forceinline__ void prepare_tree_rows(const StepTables& t, const LookaheadPack& ks, int B, int Kmax, int V, int max_batch,
                                                  int max_kv_len, int has_cache, const int32_t* __restrict__ seq_slot,
                                                  const int32_t* __restrict__ last_token, const int32_t* __restrict__ parent,
                                                  const int32_t* __restrict__ tokens, const int32_t* __restrict__ kv_len, int32_t* flag,
                                                  PrepLds& l, TreeMasks& s_mask)
{
    const int b = threadIdx.x;
    const int N = b < B ? ks.k[b] : 0;
    int ok = 1, slot = 0, n = 0;
    int tok[SPEC_MAX_LOOKAHEAD + 1], par[SPEC_MAX_LOOKAHEAD];
    if (b < B) {
        // all of a sequence's nodes requested together
        tok[0] = last_token ? last_token[b] : 0;
#pragma unroll
        for (int i = 0; i < SPEC_MAX_LOOKAHEAD; ++i) {
            tok[i + 1] = i < N ? tokens[b * Kmax + i] : 0;
            par[i] = i < N ? parent[b * Kmax + i] : -1;
        }
        slot = has_cache ? seq_slot[b] : b;
        if (has_cache) n = kv_len[slot >= 0 && slot < max_batch ? slot : 0];
    }
    const Others o = look_at_others(N, slot, B, l);   // (the loads above are under way meanwhile)
    if (b < B) {
        int err = 0;
        if (has_cache) {
            if (slot < 0 || slot >= max_batch) {
                ok = 0;
                err = SPEC_ERR_INVALID_ARG;
                slot = 0;
            } else {
                if (o.same_slot) { ok = 0; err = SPEC_ERR_INVALID_ARG; }
                if (n < 0 || n + N + 1 > max_kv_len) { ok = 0; err = SPEC_ERR_KV_OVERFLOW; }
                else if (ok && !pool_cover(t.pool, slot, n, n + N + 1)) { ok = 0; err = SPEC_ERR_KV_OVERFLOW; }
            }
        }
        if (tok[0] < 0 || tok[0] >= V) { ok = 0; err = SPEC_ERR_TOKEN_RANGE; }
#pragma unroll
        for (int i = 0; i < SPEC_MAX_LOOKAHEAD; ++i) {
            if (tok[i + 1] < 0 || tok[i + 1] >= V) { ok = 0; err = SPEC_ERR_TOKEN_RANGE; }
            if (par[i] < -1 || par[i] >= i) { ok = 0; err = SPEC_ERR_INVALID_ARG; }
        }
        if (!ok) {
            atomicCAS(flag, 0, err);
            n = 0;
        }
    }
    const int rank = has_cache ? desc_rank(b, B, ok ? n + N + 1 : 0, l.total) : 0;
    if (b == 0) {   // statistics rows: target and draft row of the root and of every node
        t.seq_row0[B] = o.rows;
        t.seq_stat0[B] = 2 * o.rows;
    }
    if (b < B) {
        const int row0 = o.row0;
        if (has_cache) write_desc(t, rank, b, N, n, slot, ok, row0);
        t.seq_row0[b] = row0;
        t.seq_stat0[b] = 2 * row0;
        t.seq_n[b] = n;
        t.seq_ok[b] = ok;
        t.seq_slot[b] = slot;
        // slot j's set of slots on its path (itself included); its depth is their number
#pragma unroll
        for (int j = 0; j <= SPEC_MAX_LOOKAHEAD; ++j) {
            if (j <= N) {
                uint32_t mask = 1u;
                if (j > 0) mask = s_mask[ok ? par[j - 1] + 1 : 0][b] | (1u << j);   // its parent's slot
                s_mask[j][b] = (uint16_t)mask;
                const int r = row0 + j;
                t.row_seq[r] = b;
                t.row_pos[r] = ok ? n + j : -1;
                t.row_rope[r] = ok ? n + __popc(mask) - 1 : 0;
                t.row_mask[r] = mask;
                t.row_tok[r] = ok ? tok[j] : 0;
            }
        }
    }
}

__global__ void __launch_bounds__(TPB) prepare_tree_kernel(StepTables t, LookaheadPack ks, int B, int Kmax, int V,
                                                           int max_batch, int max_kv_len, int has_cache,
                                                           const int32_t* __restrict__ seq_slot,
                                                           const int32_t* __restrict__ last_token,
                                                           const int32_t* __restrict__ parent,
                                                           const int32_t* __restrict__ tokens,
                                                           const int32_t* __restrict__ kv_len, int32_t* flag)
{
    __shared__ TreeMasks s_mask;
    __shared__ PrepLds l;
    prepare_tree_rows(t, ks, B, Kmax, V, max_batch, max_kv_len, has_cache, seq_slot, last_token, parent, tokens, kv_len, flag, l, s_mask);
}

// ---------------------------------------------------------------------------------------------
// The row bookkeeping and the embedding in one launch: the first workgroup does the one, a wavefront per (row, SSQ_CHUNK
// columns) of the others the other, which has no need of the tables.  The embedding of a few rows and the bookkeeping take a
// launch and two or three round trips each, one behind the other before: a step of the fp32 configuration 65.9 -> 63.8 us, draft
// decode of 8 rows 289.3 -> 288.1; the same 2 us or so of longer steps are less than their runs differ.
// A row of a sequence that the bookkeeping skips embeds token 0, as from the tables, so every wavefront looks at its
// sequence for itself: slot, cached length, tokens, parents.  (A page pool that runs dry is only seen by the
// bookkeeping: those rows embed their tokens.  The caller may see what becomes of them in logits_out, where a skipped
// sequence's rows are unspecified; nothing else reads it.)
// ---------------------------------------------------------------------------------------------
struct RowPack {
    uint16_t r[EMBED_MAX_ROWS];   // 16 * sequence + place in its window
};
static_assert(SPEC_MAX_LOOKAHEAD < 16 && SPEC_MAX_BATCH <= 4096, "a row's sequence and place in 16 bits");

template <typename T, bool TREE>
__global__ void __launch_bounds__(TPB) prepare_embed_kernel(const T* __restrict__ E, const int32_t* __restrict__ seq_slot,
                                                            const int32_t* __restrict__ last_token, const int32_t* __restrict__ parent,
                                                            const int32_t* __restrict__ tokens, const int32_t* __restrict__ kv_len,
                                                            int32_t* flag, int B, int Kmax, int V, int max_batch, int max_kv_len, int M,
                                                            int chunks, EmbedTo e, StepTables t, LookaheadPack ks, RowPack rows)
{
    __shared__ TreeMasks s_mask;
    __shared__ PrepLds l;
    if (blockIdx.x == 0) {
        if constexpr (TREE) prepare_tree_rows(t, ks, B, Kmax, V, max_batch, max_kv_len, 1, seq_slot, last_token, parent, tokens, kv_len, flag, l, s_mask);
        else prepare_rows(t, ks, B, Kmax, V, max_batch, max_kv_len, 1, seq_slot, last_token, tokens, kv_len, flag, l);
        return;
    }
    const int item = (blockIdx.x - 1) * (TPB / 64) + __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
    const int m = item / chunks;
    if (m >= M) return;
    const int at = rows.r[m], b = at >> 4, j = at & 15, K = ks.k[b], lane = threadIdx.x & 63;
    const int slot = seq_slot[b], first = last_token[b];
    int tok = 0, par = -1;
    if (lane < K) {
        tok = tokens[b * Kmax + lane];
        if (TREE) par = parent[b * Kmax + lane];
    }
    const int own = j == 0 ? first : __builtin_amdgcn_readlane(tok, j - 1);
    EmbedRow<T> row;   // (asked for before the cached length has arrived)
    row.load(E, own >= 0 && own < V ? own : 0, item % chunks, e.d);
    bool bad = first < 0 || first >= V || tok < 0 || tok >= V || par < -1 || (par >= lane && lane < K);
    for (int i = lane; i < b; i += 64) bad |= seq_slot[i] == slot;   // two sequences of a step must not share a slot
    const int n = kv_len[slot >= 0 && slot < max_batch ? slot : 0];
    bad |= slot < 0 || slot >= max_batch || n < 0 || n + K + 1 > max_kv_len;
    if (__ballot(bad)) row.load(E, 0, item % chunks, e.d);
    embed_chunk(row, m, item % chunks, chunks, e.d, e.x, e.gain, e.xo, e.ssq);
}

template <bool TREE>
int launch_prepare_embed(const EmbedTo& e, const StepTables& t, const LookaheadPack& ks, int B, int Kmax, int V, int max_batch, int max_kv_len,
                         const int32_t* seq_slot, const int32_t* last_token, const int32_t* parent, const int32_t* tokens,
                         const int32_t* kv_len, int32_t* flag, hipStream_t s)
{
    RowPack rows;
    int M = 0;
    for (int b = 0; b < B; ++b)
        for (int j = 0; j <= ks.k[b]; ++j) {
            if (M == EMBED_MAX_ROWS) return fail(SPEC_ERR_SHAPE, "more than %d rows embedded beside their bookkeeping", EMBED_MAX_ROWS);
            rows.r[M++] = (uint16_t)(16 * b + j);
        }
    const int chunks = 2 * ssq_pairs(e.d);
    const dim3 grid(1 + (M * chunks + TPB / 64 - 1) / (TPB / 64));
    if (e.dtype == SPEC_DTYPE_BF16)
        hipLaunchKernelGGL((prepare_embed_kernel<__bf16, TREE>), grid, dim3(TPB), 0, s, (const __bf16*)e.E, seq_slot, last_token, parent,
                           tokens, kv_len, flag, B, Kmax, V, max_batch, max_kv_len, M, chunks, e, t, ks, rows);
    else
        hipLaunchKernelGGL((prepare_embed_kernel<float, TREE>), grid, dim3(TPB), 0, s, (const float*)e.E, seq_slot, last_token, parent,
                           tokens, kv_len, flag, B, Kmax, V, max_batch, max_kv_len, M, chunks, e, t, ks, rows);
    SPECV_LAUNCH_CHECK("prepare_embed_kernel");
    return SPEC_OK;
}

constexpr int TREE_TPB = 1024;   // the walk is one workgroup per sequence: make it a big one
constexpr int TREE_CHUNKS = 64;  // its final draw keeps the masses of as many chunks of RES_CHUNK ids

struct TreeOut {
    int32_t* n_accepted;   // [B]
    int32_t* out_tokens;   // [B][Kmax+1]
    int32_t* path;         // [B][Kmax] kept node indices root-down, then -1
};

// Of the lanes of a wavefront whose running sum inc (own share loc, of PER ids with the masses x) passes the target, the first one
// that has mass: which of its ids the target falls on, the first whose running sum passes it (rounding between that sum and inc: the
// last id with mass).  -1 for the other lanes.  The lanes add up in different orders, so neighbours' ranges [inc - loc, inc) may
// leave a gap or overlap by rounding: a lane is not asked whether the target lies in its range.
template <int PER>
__device__ __forceinline__ int lowest_crossing(const double* x, double loc, double inc, double target)
{
    const unsigned long long over = __ballot(loc > 0.0 && inc > target);
    if (!over || (int)(threadIdx.x & 63) != __ffsll((long long)over) - 1) return -1;
    double cdf = inc - loc;
    int first = -1, last = -1;
#pragma unroll
    for (int i = 0; i < PER; ++i) {
        cdf += x[i];
        if (first < 0 && x[i] > 0.0 && cdf > target) first = i;
        if (x[i] > 0.0) last = i;
    }
    return first >= 0 ? first : last;
}

// The walk of one sequence's tree (one workgroup).  At the current node r starts as the target
// distribution p; a child with token x is kept iff u * q(x) < r(x); every rejection replaces r by
// max(0, r - q) renormalised.  r is never materialised: r_k(v) is recomputed from p(v), q(v) and the
// masses S_1..S_k of the earlier levels, so a rejection costs one pass over the two logits rows.
// One compute unit does a sequence: the passes are bound by its fp64 rate (divisions by the masses most of all) and by
// memory round trips.  8 sequences, 10 nodes, vocabulary 32000: 77 us with full divisions, 8 elements in flight and a
// barrier per chunk of the final draw; 59 as it is.
__global__ void __launch_bounds__(TREE_TPB) tree_walk_kernel(StepTables t, LookaheadPack ks, int Kmax, int V,
                                                        int n_stat_chunks, const float* __restrict__ target,
                                                        const float* __restrict__ draft,
                                                        const int32_t* __restrict__ parent,
                                                        const int32_t* __restrict__ tokens,
                                                        const float* __restrict__ uniforms, float inv_T_f,
                                                        const float* __restrict__ part_max,
                                                        const double* __restrict__ part_sum, int auto_rollback,
                                                        int32_t* kv_len, TreeOut out)
{
    constexpr int MAXN = SPEC_MAX_LOOKAHEAD;
    __shared__ float row_m[2 * MAXN + 2];
    __shared__ double row_z[2 * MAXN + 2];
    __shared__ double level_S[MAXN + 1];     // level_S[k]: mass of the unnormalised r_k, k >= 1
    __shared__ double level_I[MAXN + 1];     // 1 / level_S[k]
    __shared__ double wsum[TREE_TPB / 64];
    __shared__ double r[RES_CHUNK + TREE_TPB];   // 4 consecutive ids per lane, a word of padding between lanes
    __shared__ int s_tok, s_chunk;
    __shared__ double s_val, s_before, s_target;
    const int b = blockIdx.x;
    const int N = ks.k[b];
    if (!t.seq_ok[b]) {
        if (threadIdx.x == 0) out.n_accepted[b] = -1;
        for (int i = threadIdx.x; i <= Kmax; i += TREE_TPB) out.out_tokens[b * (Kmax + 1) + i] = -1;
        for (int i = threadIdx.x; i < Kmax; i += TREE_TPB) out.path[b * Kmax + i] = -1;
        return;
    }
    const double inv_T = (double)inv_T_f;
    const int st0 = t.seq_stat0[b];
    __shared__ CombineLds comb;
    combine_rows<TREE_TPB>(part_max, part_sum, st0, 2 * N + 2, n_stat_chunks, inv_T, row_m, row_z, comb);
    const float* trow0 = target + (size_t)t.seq_row0[b] * V;
    const float* drow0 = draft + (size_t)b * (Kmax + 1) * V;
    const int32_t* par = parent + b * Kmax;
    const int32_t* tok = tokens + b * Kmax;

    int cur = -1, level = 0, a = 0;
    const float* prow = trow0;
    const float* qrow = drow0;
    float mp = row_m[0], mq = row_m[N + 1];
    double izp = 1.0 / row_z[0], izq = 1.0 / row_z[N + 1];
    // x / level_S[k], rounded as a division is: y is the rounded reciprocal, the remainder of the rounded product is
    // exact, and one step with it gives the rounded quotient (Markstein 1990; masses and values stay far from the ends
    // of the exponent range).  3 fp64 instructions instead of 11, for each element and level.
    auto div_S = [&](double x, int k) -> double {
        const double y = level_I[k], q = x * y;
        return fma(fma(-q, level_S[k], x), y, q);
    };
    // r_level(v) from the two rows (level and the masses are uniform over the workgroup)
    auto resid = [&](float lp, float lq, int lev) -> double {
        double pv = (double)__expf((lp - mp) * inv_T_f) * izp;
        if (lev > 0) {
            const double qv = (double)__expf((lq - mq) * inv_T_f) * izq;
            pv = pv > qv ? pv - qv : 0.0;
            for (int k = 1; k < lev; ++k) {
                pv = div_S(pv, k);
                pv = pv > qv ? pv - qv : 0.0;
            }
        }
        return pv;
    };
    auto block_sum = [&](double v) -> double {
        v = wave_sum(v);
        __syncthreads();
        if ((threadIdx.x & 63) == 0) wsum[threadIdx.x >> 6] = v;
        __syncthreads();
        double tot = 0.0;
#pragma unroll
        for (int w = 0; w < TREE_TPB / 64; ++w) tot += wsum[w];   // fixed order
        return tot;
    };

    // What the test of node c needs from memory does not depend on the walk (a node is always tested
    // against its parent's rows): lane c fetches it for all nodes at once, and every thread then
    // takes the same decisions from LDS -- no load and no barrier per tested node.
    __shared__ int s_par[MAXN], s_ntok[MAXN];
    __shared__ double s_ep[MAXN], s_eq[MAXN], s_u[MAXN];
    if ((int)threadIdx.x < N) {
        const int c = threadIdx.x;
        const int pr = par[c] + 1;                 // row of the parent (0: the root)
        const int x = tok[c];
        s_par[c] = par[c];
        s_ntok[c] = x;
        s_u[c] = (double)uniforms[b * (Kmax + 1) + c];
        s_ep[c] = exp((double)(trow0[(size_t)pr * V + x] - row_m[pr]) * inv_T);
        s_eq[c] = exp((double)(drow0[(size_t)pr * V + x] - row_m[N + 1 + pr]) * inv_T);
    }
    __syncthreads();

    for (int c = 0; c < N; ++c) {
        if (s_par[c] != cur) continue;
        bool keep;
        {
            const double u = s_u[c], ep = s_ep[c], eq = s_eq[c];
            if (level == 0) {
                keep = u * eq * row_z[cur + 1] < ep * row_z[N + 1 + cur + 1];   // u q(x) < p(x), division-free
            } else {
                const double qx = eq * izq;
                double rx = ep * izp;
                rx = rx > qx ? rx - qx : 0.0;
                for (int k = 1; k < level; ++k) {
                    rx = rx / level_S[k];
                    rx = rx > qx ? rx - qx : 0.0;
                }
                keep = u * qx * level_S[level] < rx;   // u q(x) < r(x) / S
            }
        }
        if (keep) {
            if (threadIdx.x == 0) {
                out.path[b * Kmax + a] = c;
                out.out_tokens[b * (Kmax + 1) + a] = s_ntok[c];
            }
            ++a;
            cur = c;
            level = 0;
            prow = trow0 + (size_t)(c + 1) * V;
            qrow = drow0 + (size_t)(c + 1) * V;
            mp = row_m[c + 1];
            mq = row_m[N + 1 + c + 1];
            izp = 1.0 / row_z[c + 1];
            izq = 1.0 / row_z[N + 1 + c + 1];
            continue;
        }
        // rejected: mass of max(0, r/S - q)
        double acc = 0.0;
        constexpr int UN = 16;
        for (int v0 = threadIdx.x; v0 < V; v0 += UN * TREE_TPB) {
            // sixteen elements per trip, loads first (indices past the end clamped, their terms dropped)
            float lpv[UN], lqv[UN];
#pragma unroll
            for (int k = 0; k < UN; ++k) {
                const int v = min(v0 + k * TREE_TPB, V - 1);
                lpv[k] = prow[v];
                lqv[k] = qrow[v];
            }
#pragma unroll
            for (int k = 0; k < UN; ++k) {
                double pv = resid(lpv[k], lqv[k], level);
                if (level > 0) pv = div_S(pv, level);
                const double qv = (double)__expf((lqv[k] - mq) * inv_T_f) * izq;
                if (v0 + k * TREE_TPB < V) acc += pv > qv ? pv - qv : 0.0;
            }
        }
        const double S_new = block_sum(acc);
        if (S_new > 0.0) {   // <= 0 cannot happen in exact arithmetic; then r stays as it is
            if (threadIdx.x == 0) {
                level_S[level + 1] = S_new;
                level_I[level + 1] = 1.0 / S_new;
            }
            ++level;
        }
        __syncthreads();
    }

    // final draw from r_level of the current node: chunk masses, then a scan inside one chunk.  The loads of four
    // chunks are in flight at a time, and the chunks' sums over the wavefronts meet behind one barrier.
    const int n_res_chunks = (V + RES_CHUNK - 1) / RES_CHUNK;   // at most TREE_CHUNKS: the launch wrapper sees to it
    constexpr int PER = RES_CHUNK / TREE_TPB, GR = 4, WAVES = TREE_TPB / 64;
    __shared__ double mass[TREE_CHUNKS], mass_w[TREE_CHUNKS * WAVES];
    for (int c0 = 0; c0 < n_res_chunks; c0 += GR) {
        float lpv[GR][PER], lqv[GR][PER];
#pragma unroll
        for (int g = 0; g < GR; ++g)
#pragma unroll
            for (int k = 0; k < PER; ++k) {
                const int v = min((c0 + g) * RES_CHUNK + (int)threadIdx.x + k * TREE_TPB, V - 1);
                lpv[g][k] = prow[v];
                lqv[g][k] = qrow[v];
            }
#pragma unroll
        for (int g = 0; g < GR; ++g) {
            double acc = 0.0;
#pragma unroll
            for (int k = 0; k < PER; ++k)
                if ((c0 + g) * RES_CHUNK + (int)threadIdx.x + k * TREE_TPB < V) acc += resid(lpv[g][k], lqv[g][k], level);
            acc = wave_sum(acc);
            if ((threadIdx.x & 63) == 0 && c0 + g < n_res_chunks) mass_w[(c0 + g) * WAVES + (threadIdx.x >> 6)] = acc;
        }
    }
    __syncthreads();
    if ((int)threadIdx.x < n_res_chunks) {
        double m = 0.0;
#pragma unroll
        for (int w = 0; w < WAVES; ++w) m += mass_w[threadIdx.x * WAVES + w];   // fixed order
        mass[threadIdx.x] = m;
    }
    __syncthreads();
    double total = 0.0;   // meaningful in thread 0
    if (threadIdx.x == 0)
        for (int cc = 0; cc < n_res_chunks; ++cc) total += mass[cc];
    if (threadIdx.x == 0) {
        const double target_mass = (double)uniforms[b * (Kmax + 1) + N] * total;
        double c0 = 0.0, last_before = 0.0;
        int pick = -1, last_pos = -1;
        for (int cc = 0; cc < n_res_chunks; ++cc) {
            if (mass[cc] > 0.0) { last_pos = cc; last_before = c0; }
            if (c0 + mass[cc] > target_mass) { pick = cc; break; }
            c0 += mass[cc];
        }
        if (pick < 0) { pick = last_pos; c0 = last_before; }
        if (pick < 0) { pick = 0; c0 = 0.0; }
        s_chunk = pick;
        s_before = c0;
        s_target = target_mass;
        s_tok = V;   // none yet
    }
    __syncthreads();
    {
        const int base = s_chunk * RES_CHUNK;
        const int lim = min(RES_CHUNK, V - base);
        const double before = s_before, target_mass = s_target;
        {
            float lpv[PER], lqv[PER];
#pragma unroll
            for (int k = 0; k < PER; ++k) {
                const int i = min((int)threadIdx.x + k * TREE_TPB, lim - 1);
                lpv[k] = prow[base + i];
                lqv[k] = qrow[base + i];
            }
#pragma unroll
            for (int k = 0; k < PER; ++k) {
                const int i = threadIdx.x + k * TREE_TPB;
                r[i + i / PER] = i < lim ? resid(lpv[k], lqv[k], level) : 0.0;
            }
        }
        __syncthreads();
        double loc = 0.0;
        int my_last = -1;
#pragma unroll
        for (int i = 0; i < PER; ++i) {
            const double x = r[threadIdx.x * (PER + 1) + i];
            loc += x;
            if (x > 0.0) my_last = base + threadIdx.x * PER + i;
        }
        double inc = wave_scan(loc);
        if ((threadIdx.x & 63) == 63) wsum[threadIdx.x >> 6] = inc;
        __syncthreads();
        double off = before;
        for (int wv = 0; wv < (int)(threadIdx.x >> 6); ++wv) off += wsum[wv];
        inc += off;
        const int at = lowest_crossing<PER>(r + threadIdx.x * (PER + 1), loc, inc, target_mass);
        if (at >= 0) atomicMin(&s_tok, base + threadIdx.x * PER + at);
        int wl = my_last;
#pragma unroll
        for (int o = 32; o > 0; o >>= 1) wl = max(wl, __shfl_xor(wl, o));
        __syncthreads();
        int* scratch = reinterpret_cast<int*>(wsum);
        if ((threadIdx.x & 63) == 0) scratch[threadIdx.x >> 6] = wl;
        __syncthreads();
        if (threadIdx.x == 0) {
            int y = s_tok;
            if (y >= V) {
                y = -1;
                for (int w = 0; w < TREE_TPB / 64; ++w) y = max(y, scratch[w]);
            }
            if (y < 0) y = 0;
            out.n_accepted[b] = a;
            int32_t* o = out.out_tokens + b * (Kmax + 1);
            o[a] = y;
            for (int i = a + 1; i <= Kmax; ++i) o[i] = -1;
            for (int i = a; i < Kmax; ++i) out.path[b * Kmax + i] = -1;
            if (kv_len) {
                // with auto_rollback the kept path is still to be moved: its pages go back after
                // that (tree_trim_kernel), never here
                kv_len[t.seq_slot[b]] = t.seq_n[b] + (auto_rollback ? a : N) + 1;
                if (!auto_rollback) pool_trim(t.pool, t.seq_slot[b], t.seq_n[b] + N + 1);
            }
        }
    }
}

// The same walk with the current node's r in registers, for vocabularies of up to DRAW_MAX: a node's rows are read and
// their exponentials taken once, a rejection is 10 fp64 instructions an id (r / S - q in place; the same values as above),
// and the final draw looks up what is there.  q's weights sit in LDS, each thread's own.
// 8 sequences, 10 nodes, vocabulary 32000: 62.0 us as the kernel above, 26.4 as this one.
template <int RUNS>
__global__ void __launch_bounds__(DRAW_TPB) tree_draw_kernel(const int32_t* seq_stat0, const int32_t* seq_row0,
                                                             const float* __restrict__ part_max, const double* __restrict__ part_sum,
                                                             const int32_t* __restrict__ parent, const int32_t* __restrict__ tokens,
                                                             int Kmax, int V, int n_stat_chunks, float inv_T_f,
                                                             const float* __restrict__ uniforms, const float* __restrict__ target,
                                                             const float* __restrict__ draft, int auto_rollback, int32_t* kv_len,
                                                             TreeOut out, StepTables t, LookaheadPack ks)
{
    constexpr int MAXN = SPEC_MAX_LOOKAHEAD;
    __shared__ float row_m[2 * MAXN + 2];
    __shared__ double row_z[2 * MAXN + 2];
    __shared__ double level_S[MAXN + 1];     // level_S[k]: mass of the unnormalised r_k, k >= 1
    __shared__ double level_I[MAXN + 1];     // 1 / level_S[k]
    __shared__ double tot[2][DRAW_WAVES];
    __shared__ floatx4 qw[RUNS][DRAW_TPB];
    __shared__ DrawLds l;
    __shared__ CombineLds comb;
    __shared__ int s_par[MAXN], s_ntok[MAXN];
    __shared__ double s_ep[MAXN], s_eq[MAXN], s_u[MAXN];
    const int b = blockIdx.x, lane = threadIdx.x & 63;
    const int st0 = seq_stat0[b], row0 = seq_row0[b], ok = t.seq_ok[b], slot = t.seq_slot[b], n_cached = t.seq_n[b];
    const int N = ks.k[b];
    if (!ok) {
        const int i = threadIdx.x;
        if (i == 0) out.n_accepted[b] = -1;
        if (i <= Kmax) out.out_tokens[b * (Kmax + 1) + i] = -1;
        if (i < Kmax) out.path[b * Kmax + i] = -1;
        return;
    }
    const double inv_T = (double)inv_T_f;
    const float* trow0 = target + (size_t)row0 * V;
    const float* drow0 = draft + (size_t)b * (Kmax + 1) * V;
    // what the tests need from memory does not depend on the walk: lane c fetches it for node c
    float lp_x = 0.f, lq_x = 0.f;
    int pr = 0;
    if ((int)threadIdx.x < N) {
        const int c = threadIdx.x, x = tokens[b * Kmax + c];
        pr = parent[b * Kmax + c] + 1;             // row of the parent (0: the root)
        s_par[c] = pr - 1;
        s_ntok[c] = x;
        s_u[c] = (double)uniforms[b * (Kmax + 1) + c];
        lp_x = trow0[(size_t)pr * V + x];
        lq_x = drow0[(size_t)pr * V + x];
    }
    const double u_draw = (double)uniforms[b * (Kmax + 1) + N];
    combine_rows<DRAW_TPB>(part_max, part_sum, st0, 2 * N + 2, n_stat_chunks, inv_T, row_m, row_z, comb);
    if ((int)threadIdx.x < N) {
        s_ep[threadIdx.x] = exp((double)(lp_x - row_m[pr]) * inv_T);
        s_eq[threadIdx.x] = exp((double)(lq_x - row_m[N + 1 + pr]) * inv_T);
    }
    __syncthreads();

    int cur = -1, level = 0, a = 0;
    double izp = 1.0 / row_z[0], izq = 1.0 / row_z[N + 1];
    double r[RUNS][4];
    int applied = -1;                              // levels of the current node that r has been through (-1: not read yet)
    // x / level_S[k], rounded as a division is (see tree_walk_kernel)
    auto div_S = [&](double x, double S, double y) -> double {
        const double q = x * y;
        return fma(fma(-q, S, x), y, q);
    };
    auto fetch = [&] {                             // r = p, qw = q's weights
        const float* prow = trow0 + (size_t)(cur + 1) * V;
        const float* qrow = drow0 + (size_t)(cur + 1) * V;
        const float mp = row_m[cur + 1], mq = row_m[N + 1 + cur + 1];
        // both rows under way together; q's weights leave the registers before p's values, twice as wide, fill them
        floatx4 p[RUNS], q[RUNS];
        draw_load<false>(qrow, V, draw_id0<RUNS>(), q);
        draw_load<false>(prow, V, draw_id0<RUNS>(), p);
        __builtin_amdgcn_sched_barrier(0);
#pragma unroll
        for (int j = 0; j < RUNS; ++j) {
#pragma unroll
            for (int e = 0; e < 4; ++e) q[j][e] = __expf((q[j][e] - mq) * inv_T_f);
            qw[j][threadIdx.x] = q[j];
        }
        __builtin_amdgcn_sched_barrier(0);
#pragma unroll
        for (int j = 0; j < RUNS; ++j) {
#pragma unroll
            for (int e = 0; e < 4; ++e) r[j][e] = (double)__expf((p[j][e] - mp) * inv_T_f) * izp;
            __builtin_amdgcn_sched_barrier(0);
        }
    };
    // r through the levels up to `upto`: r = max(0, r / S - q) each; the thread's share of the last one's mass
    auto bring = [&](int upto) -> double {
        double acc = 0.0;
        if (applied < 0) {
            fetch();
            applied = 0;
        }
        for (; applied < upto; ++applied) {
            const double S = applied > 0 ? level_S[applied] : 1.0, I = applied > 0 ? level_I[applied] : 1.0;
            acc = 0.0;
#pragma unroll
            for (int j = 0; j < RUNS; ++j) {
                const floatx4 q = qw[j][threadIdx.x];
#pragma unroll
                for (int e = 0; e < 4; ++e) {
                    const double qv = (double)q[e] * izq;
                    const double pv = div_S(r[j][e], S, I);   // (level 0: by 1, which changes nothing)
                    r[j][e] = pv > qv ? pv - qv : 0.0;
                    acc += r[j][e];
                }
                __builtin_amdgcn_sched_barrier(0);
            }
        }
        return acc;
    };
    int flip = 0;
    for (int c = 0; c < N; ++c) {
        if (s_par[c] != cur) continue;
        bool keep;
        {
            const double u = s_u[c], ep = s_ep[c], eq = s_eq[c];
            if (level == 0) {
                keep = u * eq * row_z[cur + 1] < ep * row_z[N + 1 + cur + 1];   // u q(x) < p(x), division-free
            } else {
                const double qx = eq * izq;
                double rx = ep * izp;
                rx = rx > qx ? rx - qx : 0.0;
                for (int k = 1; k < level; ++k) {
                    rx = rx / level_S[k];
                    rx = rx > qx ? rx - qx : 0.0;
                }
                keep = u * qx * level_S[level] < rx;   // u q(x) < r(x) / S
            }
        }
        if (keep) {
            if (threadIdx.x == 0) {
                out.path[b * Kmax + a] = c;
                out.out_tokens[b * (Kmax + 1) + a] = s_ntok[c];
            }
            ++a;
            cur = c;
            level = 0;
            applied = -1;
            izp = 1.0 / row_z[c + 1];
            izq = 1.0 / row_z[N + 1 + c + 1];
            continue;
        }
        const double acc = wave_sum(bring(level + 1));
        if (lane == 0) tot[flip][threadIdx.x >> 6] = acc;
        __syncthreads();
        const double S_new = wave_sum(lane < DRAW_WAVES ? tot[flip][lane] : 0.0);
        flip ^= 1;
        if (S_new > 0.0) {
            ++level;
            if (threadIdx.x == 0) {
                level_S[level] = S_new;
                level_I[level] = 1.0 / S_new;
            }
        } else {
            applied = -1;   // cannot happen in exact arithmetic; then r stays as it was, to be put together again
        }
        __syncthreads();
    }
    bring(level);
    double run[RUNS];
#pragma unroll
    for (int j = 0; j < RUNS; ++j) run[j] = (r[j][0] + r[j][1]) + (r[j][2] + r[j][3]);
    if (!draw_locate<RUNS, DRAW_WAVES>(run, [&](int j, double (&x)[4]) {
#pragma unroll
            for (int e = 0; e < 4; ++e) x[e] = r[0][e];
#pragma unroll
            for (int i = 1; i < RUNS; ++i)
#pragma unroll
                for (int e = 0; e < 4; ++e) x[e] = j == i ? r[i][e] : x[e];
        }, u_draw, false, l)) {
        if (threadIdx.x == 0) l.tok = 0;   // a row without mass
        __syncthreads();
    }
    const int i = threadIdx.x;
    if (i >= a && i <= Kmax) out.out_tokens[b * (Kmax + 1) + i] = i == a ? l.tok : -1;
    if (i >= a && i < Kmax) out.path[b * Kmax + i] = -1;
    if (i == 0) {
        out.n_accepted[b] = a;
        if (kv_len) {
            // with auto_rollback the kept path is still to be moved: its pages go back after
            // that (tree_trim_kernel), never here
            kv_len[slot] = n_cached + (auto_rollback ? a : N) + 1;
            if (!auto_rollback) pool_trim(t.pool, slot, n_cached + N + 1);
        }
    }
}

// kv_len[slot] = len where 0 <= len <= kv_len[slot]; anything else leaves the slot alone and flags.
__global__ void __launch_bounds__(TPB) rollback_kernel(RollbackPack p, int n, int max_batch, int32_t* kv_len,
                                                       int32_t* flag, PagePool pool)
{
    const int i = threadIdx.x;
    if (i >= n) return;
    const int slot = p.slot[i], len = p.len[i];
    if (slot < 0 || slot >= max_batch) { atomicCAS(flag, 0, (int)SPEC_ERR_INVALID_ARG); return; }
    if (len < 0 || len > kv_len[slot]) { atomicCAS(flag, 0, (int)SPEC_ERR_ROLLBACK); return; }
    kv_len[slot] = len;
    pool_trim(pool, slot, len);
}

// Paged cache, after a tree step's compaction: hand back the pages beyond the new length.  The walk
// cannot do it: a kept node's keys and values may still sit in a block above n + a + 1 until
// kv_compact_kernel has moved them (n = 28, kept node in window slot 4: position 32 is in the
// second block, the new length 30 needs the first only).
__global__ void __launch_bounds__(TPB) tree_trim_kernel(StepTables t, int B, const int32_t* __restrict__ n_accepted)
{
    const int b = threadIdx.x;
    if (b >= B || !t.seq_ok[b]) return;
    const int a = n_accepted[b];
    if (a >= 0) pool_trim(t.pool, t.seq_slot[b], t.seq_n[b] + a + 1);
}

__global__ void pool_cover_kernel(PagePool pool, int slot, int pos0, int pos1, int32_t* flag)
{
    if (threadIdx.x == 0 && blockIdx.x == 0 && !pool_cover(pool, slot, pos0, pos1)) atomicCAS(flag, 0, (int)SPEC_ERR_KV_OVERFLOW);
}

}  // namespace

int launch_prepare(const StepTables& t, const LookaheadPack& ks, int B, int Kmax, int V, int max_batch,
                   int max_kv_len, bool has_cache, const int32_t* seq_slot, const int32_t* last_token,
                   const int32_t* draft_tokens, const int32_t* kv_len, int32_t* flag, hipStream_t s, const EmbedTo* embed)
{
    if (embed)
        return launch_prepare_embed<false>(*embed, t, ks, B, Kmax, V, max_batch, max_kv_len, seq_slot, last_token, nullptr, draft_tokens,
                                           kv_len, flag, s);
    hipLaunchKernelGGL(prepare_kernel, dim3(1), dim3(TPB), 0, s, t, ks, B, Kmax, V, max_batch, max_kv_len,
                       has_cache ? 1 : 0, seq_slot, last_token, draft_tokens, kv_len, flag);
    SPECV_LAUNCH_CHECK("prepare_kernel");
    return SPEC_OK;
}

int launch_greedy(const StepTables& t, const SamplerWorkspace& w, const LookaheadPack& ks, int B, int Kmax, int V,
                  int M, const float* target_logits, const int32_t* draft_tokens, int auto_rollback, int32_t* kv_len,
                  int32_t* n_accepted, int32_t* out_tokens, const DrawEmit* emit, Profiler* prof, hipStream_t s)
{
    DrawEmit em{};
    if (emit) em = *emit;
    const int n_chunks = (V + STAT_CHUNK - 1) / STAT_CHUNK;
    {
        ProfScope ps(prof, SPEC_PROF_SAMPLER_STATS, s);
        hipLaunchKernelGGL(argmax_kernel, dim3((unsigned)M * n_chunks), dim3(TPB), 0, s, V, n_chunks, target_logits,
                           w.part_max, w.part_idx);
        SPECV_LAUNCH_CHECK("argmax_kernel");
    }
    ProfScope ps(prof, SPEC_PROF_SAMPLER_DRAW, s);
    hipLaunchKernelGGL(greedy_emit_kernel, dim3(B), dim3(64), 0, s, t, ks, Kmax, n_chunks, w.part_max, w.part_idx,
                       draft_tokens, auto_rollback, kv_len, n_accepted, out_tokens, em);
    SPECV_LAUNCH_CHECK("greedy_emit_kernel");
    return SPEC_OK;
}

int launch_tree_greedy(const StepTables& t, const SamplerWorkspace& w, const LookaheadPack& ks, int B, int Kmax, int V,
                       int M, const float* target_logits, const int32_t* parent, const int32_t* tokens,
                       int auto_rollback, int32_t* kv_len, int32_t* n_accepted, int32_t* out_tokens, int32_t* path,
                       Profiler* prof, hipStream_t s)
{
    const int n_chunks = (V + STAT_CHUNK - 1) / STAT_CHUNK;
    {
        ProfScope ps(prof, SPEC_PROF_SAMPLER_STATS, s);
        hipLaunchKernelGGL(argmax_kernel, dim3((unsigned)M * n_chunks), dim3(TPB), 0, s, V, n_chunks, target_logits,
                           w.part_max, w.part_idx);
        SPECV_LAUNCH_CHECK("argmax_kernel");
    }
    ProfScope ps(prof, SPEC_PROF_SAMPLER_DRAW, s);
    hipLaunchKernelGGL(tree_greedy_kernel, dim3(B), dim3(64), 0, s, t, ks, Kmax, n_chunks, w.part_max, w.part_idx,
                       parent, tokens, auto_rollback, kv_len, n_accepted, out_tokens, path);
    SPECV_LAUNCH_CHECK("tree_greedy_kernel");
    return SPEC_OK;
}

int launch_prepare_tree(const StepTables& t, const LookaheadPack& ks, int B, int Kmax, int V, int max_batch,
                        int max_kv_len, bool has_cache, const int32_t* seq_slot, const int32_t* last_token,
                        const int32_t* parent, const int32_t* tokens, const int32_t* kv_len, int32_t* flag,
                        hipStream_t s, const EmbedTo* embed)
{
    if (embed)
        return launch_prepare_embed<true>(*embed, t, ks, B, Kmax, V, max_batch, max_kv_len, seq_slot, last_token, parent, tokens, kv_len,
                                          flag, s);
    hipLaunchKernelGGL(prepare_tree_kernel, dim3(1), dim3(TPB), 0, s, t, ks, B, Kmax, V, max_batch, max_kv_len,
                       has_cache ? 1 : 0, seq_slot, last_token, parent, tokens, kv_len, flag);
    SPECV_LAUNCH_CHECK("prepare_tree_kernel");
    return SPEC_OK;
}

int launch_tree_sampler(const StepTables& t, const SamplerWorkspace& w, const LookaheadPack& ks, int B, int Kmax,
                        int V, int n_stat_rows, const float* target_logits, const float* draft_logits,
                        const int32_t* parent, const int32_t* tokens, const float* uniforms, float temperature,
                        int auto_rollback, int32_t* kv_len, int32_t* n_accepted, int32_t* out_tokens,
                        int32_t* path, Profiler* prof, hipStream_t s, const LogitsSrc* src)
{
    const int n_stat_chunks = (V + STAT_CHUNK - 1) / STAT_CHUNK;
    if ((V + RES_CHUNK - 1) / RES_CHUNK > TREE_CHUNKS)
        return fail(SPEC_ERR_SHAPE, "tree verification supports vocabularies up to %d", TREE_CHUNKS * RES_CHUNK);
    const float inv_T = 1.0f / temperature;
    const bool vec4 = (V % 4 == 0) && ((reinterpret_cast<uintptr_t>(target_logits) & 15) == 0)
                      && ((reinterpret_cast<uintptr_t>(draft_logits) & 15) == 0);
    dim3 g1((unsigned)n_stat_rows * n_stat_chunks);
    {
        ProfScope ps(prof, SPEC_PROF_SAMPLER_STATS, s);
        const LogitsSrc from = src ? *src : LogitsSrc{};
        auto* k = from.partial ? (vec4 ? stats_kernel<true, true> : stats_kernel<false, true>)
                               : (vec4 ? stats_kernel<true, false> : stats_kernel<false, false>);
        hipLaunchKernelGGL(k, g1, dim3(TPB), 0, s, 0, (int)STAT_TREE, B, Kmax + 1, V, n_stat_chunks, target_logits, draft_logits,
                           (float*)nullptr, inv_T, w.part_max, w.part_sum, (size_t)0, t, ks, PrepIn{}, from);
        SPECV_LAUNCH_CHECK("stats_kernel");
    }
    ProfScope ps(prof, SPEC_PROF_SAMPLER_DRAW, s);
    TreeOut o{n_accepted, out_tokens, path};
    if (V <= DRAW_MAX) {
        const int runs = draw_runs(V);
        auto* k = runs == 1 ? tree_draw_kernel<1> : runs == 2 ? tree_draw_kernel<2> : runs == 4 ? tree_draw_kernel<4> : tree_draw_kernel<8>;
        hipLaunchKernelGGL(k, dim3(B), dim3(DRAW_TPB), 0, s, t.seq_stat0, t.seq_row0, w.part_max, w.part_sum, parent, tokens, Kmax, V,
                           n_stat_chunks, inv_T, uniforms, target_logits, draft_logits, auto_rollback, kv_len, o, t, ks);
        SPECV_LAUNCH_CHECK("tree_draw_kernel");
        return SPEC_OK;
    }
    hipLaunchKernelGGL(tree_walk_kernel, dim3(B), dim3(TREE_TPB), 0, s, t, ks, Kmax, V, n_stat_chunks, target_logits,
                       draft_logits, parent, tokens, uniforms, inv_T, w.part_max, w.part_sum, auto_rollback, kv_len, o);
    SPECV_LAUNCH_CHECK("tree_walk_kernel");
    return SPEC_OK;
}

int launch_rollback(const RollbackPack& p, int n, int max_batch, int32_t* kv_len, int32_t* flag, const PagePool& pool,
                    hipStream_t s)
{
    hipLaunchKernelGGL(rollback_kernel, dim3(1), dim3(TPB), 0, s, p, n, max_batch, kv_len, flag, pool);
    SPECV_LAUNCH_CHECK("rollback_kernel");
    return SPEC_OK;
}

int launch_slice_tables(const StepTables& full, const StepTables& sub, int b0, int Bg, hipStream_t s)
{
    hipLaunchKernelGGL(slice_tables_kernel, dim3(1), dim3(TPB), 0, s, full, sub, b0, Bg);
    SPECV_LAUNCH_CHECK("slice_tables_kernel");
    return SPEC_OK;
}

int launch_tree_trim(const StepTables& t, int B, const int32_t* n_accepted, hipStream_t s)
{
    if (!t.pool.table) return SPEC_OK;
    hipLaunchKernelGGL(tree_trim_kernel, dim3(1), dim3(TPB), 0, s, t, B, n_accepted);
    SPECV_LAUNCH_CHECK("tree_trim_kernel");
    return SPEC_OK;
}

int launch_pool_cover(const PagePool& pool, int slot, int pos0, int pos1, int32_t* flag, hipStream_t s)
{
    if (!pool.table) return SPEC_OK;
    hipLaunchKernelGGL(pool_cover_kernel, dim3(1), dim3(64), 0, s, pool, slot, pos0, pos1, flag);
    SPECV_LAUNCH_CHECK("pool_cover_kernel");
    return SPEC_OK;
}

// How a draw behind the statistics is launched.  Beyond SLICE_MIN ids by the workgroups that slices of 2048 ids would give, up to
// four, five or eight per compute unit: from there on, a round trip for the count that every workgroup makes before it can leave costs more
// than a launch.  The sampling part, us, as one workgroup per sequence, counted (slices of 2048, more than 1024 of them 4096) and
// as two launches:
//                                          no proposals           three proposals
//    64 sequences of 32768 (1024 of 2048)  16.1  16.0  19.1       24.5  23.1  22.8
//    80              32768 (1280)          16.5  16.8  20.1       27.2  28.0  26.5
//   100              32768 (1600)          17.1  18.6  21.1       30.5  32.6  30.6
//   256              32768 (4096)          25.4  32.1  29.2       55.7  63.2  59.8
//    64              50257 (1600)           -    17.7  17.8        -    36.5  36.8
//   100              40000 (2000)           -    20.1  21.2        -    36.3  36.4
//   100              50257 (2500)           -    22.8  20.7        -    50.2  48.3
//    24             128256 (1512)           -    16.6  16.0        -    29.5  29.0
//    64             128256 (4032)           -    27.6  24.3        -    58.0  56.4
//   256             128256 (16128)          -    89.0  63.0        -   203.5 182.4
// (Two launches that combined the statistics in the first and walked the masses one by one in the second took 26.9 and 60.4 for 64
// of 128256, 67.2 and 190.5 for 256.)
enum DrawRoute { DRAW_ONE_WG, DRAW_COUNTED, DRAW_TWO_LAUNCHES };
static DrawRoute draw_route(int B, int V, bool any_proposals)
{
    const long wgs = (long)B * ((V + 2047) / 2048);
    if (V <= SLICE_MIN) return DRAW_ONE_WG;
    if (V <= DRAW_MAX) return wgs < (any_proposals ? 1280 : 1024) ? DRAW_COUNTED : DRAW_ONE_WG;
    return wgs < 2048 ? DRAW_COUNTED : DRAW_TWO_LAUNCHES;
}

int launch_sampler(const StepTables& t, const SamplerWorkspace& w, const LookaheadPack& ks, int B, int Kmax,
                   int V, int n_stat_rows, const float* target_logits, const float* draft_logits,
                   const int32_t* draft_tokens, const float* uniforms, int u_stride, float temperature,
                   int auto_rollback, int32_t* kv_len, int32_t* n_accepted, int32_t* out_tokens,
                   const DrawEmit* emit, Profiler* prof, hipStream_t s, int32_t* prepare_flag, const LogitsSrc* src)
{
    const int n_stat_chunks = (V + STAT_CHUNK - 1) / STAT_CHUNK;
    const float inv_T = 1.0f / temperature;
    PrepIn prep{};
    const int prep_on = prepare_flag ? 1 : 0;
    if (prepare_flag) {   // no decoder pass ran: the statistics pass fills the row tables itself
        prep.Kmax = Kmax;
        prep.draft_tokens = draft_tokens;
        prep.flag = prepare_flag;
    }
    const int layout = emit ? (int)STAT_PLAIN : (int)STAT_CHAIN;
    DrawEmit em{};
    if (emit) {
        if (n_stat_rows != B) return fail(SPEC_ERR_INVALID_ARG, "a plain draw needs every lookahead to be 0");
        em = *emit;
    }
    const bool vec4 = (V % 4 == 0) && ((reinterpret_cast<uintptr_t>(target_logits) & 15) == 0)
                      && ((reinterpret_cast<uintptr_t>(draft_logits) & 15) == 0)
                      && ((reinterpret_cast<uintptr_t>(em.logits_copy) & 15) == 0) && (em.copy_stride % 4 == 0);
    const LogitsSrc from = src ? *src : LogitsSrc{};
    if (n_stat_rows == B && V <= PLAIN_MAX && !prepare_flag) {   // nothing to test: one launch
        ProfScope ps(prof, SPEC_PROF_SAMPLER_DRAW, s);
        if (V > PLAIN_MIN) {
            hipLaunchKernelGGL(from.partial ? plain_slice_kernel<true> : plain_slice_kernel<false>, dim3((V + 2047) / 2048, B), dim3(TPB), 0, s,
                               t.seq_row0, target_logits, uniforms, u_stride, V, Kmax, inv_T, auto_rollback, kv_len, n_accepted,
                               out_tokens, w.slice_mass, t, em, from);
            SPECV_LAUNCH_CHECK("plain_slice_kernel");
            return SPEC_OK;
        }
        const int runs = draw_runs(V);
        auto* k = from.partial ? (runs == 1 ? plain_draw_kernel<true, 1> : runs == 2 ? plain_draw_kernel<true, 2> : plain_draw_kernel<true, 4>)
                               : (runs == 1 ? plain_draw_kernel<false, 1> : runs == 2 ? plain_draw_kernel<false, 2> : plain_draw_kernel<false, 4>);
        hipLaunchKernelGGL(k, dim3(B), dim3(DRAW_TPB), 0, s, t.seq_row0, target_logits, uniforms, u_stride, V, Kmax, inv_T,
                           auto_rollback, kv_len, n_accepted, out_tokens, t, em, from);
        SPECV_LAUNCH_CHECK("plain_draw_kernel");
        return SPEC_OK;
    }
    const bool stats_inside = V <= STATS_MAX && !emit && !prepare_flag && !from.partial;
    dim3 g1((unsigned)n_stat_rows * n_stat_chunks + prep_on);
    if (!stats_inside) {
    ProfScope ps(prof, SPEC_PROF_SAMPLER_STATS, s);
    auto* k = from.partial ? (vec4 ? stats_kernel<true, true> : stats_kernel<false, true>)
                           : (vec4 ? stats_kernel<true, false> : stats_kernel<false, false>);
    hipLaunchKernelGGL(k, g1, dim3(TPB), 0, s, prep_on, layout, B, Kmax, V, n_stat_chunks, target_logits, draft_logits,
                       em.logits_copy, inv_T, w.part_max, w.part_sum, em.copy_stride, t, ks, prep, from);
    SPECV_LAUNCH_CHECK("stats_kernel");
    }
    ProfScope ps(prof, SPEC_PROF_SAMPLER_DRAW, s);
    const int route = draw_route(B, V, n_stat_rows > B);
    if (route == DRAW_ONE_WG && !emit) {
        const int runs = draw_runs(V);
        auto* k = stats_inside ? accept_draw_kernel<1, true> : runs == 1 ? accept_draw_kernel<1, false> : runs == 2 ? accept_draw_kernel<2, false>
                  : runs == 4 ? accept_draw_kernel<4, false> : accept_draw_kernel<8, false>;
        hipLaunchKernelGGL(k, dim3(B), dim3(DRAW_TPB), 0, s, t.seq_stat0, t.seq_row0, draft_tokens, w.part_max,
                           w.part_sum, Kmax, V, n_stat_chunks, u_stride, uniforms, target_logits, draft_logits, inv_T, auto_rollback,
                           kv_len, n_accepted, out_tokens, t, ks);
        SPECV_LAUNCH_CHECK("accept_draw_kernel");
        return SPEC_OK;
    }
    const bool counted = route == DRAW_COUNTED;
    const int runs = counted && (long)B * ((V + 2047) / 2048) <= 1024 ? 2 : 4;   // (slice_masses has the room)
    const int slices = (V + 1024 * runs - 1) / (1024 * runs);
    auto* k = !counted ? accept_slice_kernel<4, false> : runs == 2 ? accept_slice_kernel<2, true> : accept_slice_kernel<4, true>;
    hipLaunchKernelGGL(k, dim3(slices, B), dim3(TPB), 0, s, t.seq_stat0, t.seq_row0, draft_tokens, w.part_max, w.part_sum, Kmax, V,
                       n_stat_chunks, u_stride, uniforms, target_logits, draft_logits, inv_T, auto_rollback, kv_len, n_accepted,
                       out_tokens, w.slice_mass, w.drawn, t, em, ks);
    SPECV_LAUNCH_CHECK("accept_slice_kernel");
    if (counted) return SPEC_OK;
    hipLaunchKernelGGL(slice_draw_kernel<4>, dim3(B), dim3(TPB), 0, s, t.seq_row0, w.slice_mass, w.drawn, uniforms, u_stride, slices, Kmax, V,
                       target_logits, draft_logits, inv_T, auto_rollback, kv_len, draft_tokens, n_accepted, out_tokens, t, em, ks);
    SPECV_LAUNCH_CHECK("slice_draw_kernel");
    return SPEC_OK;
}

}  // namespace specv

// ---------------------------------------------------------------------------------------------
// The sampling part of the verify step for callers that cannot allocate: no handle, no hipMalloc.
// The row tables and the sampler's workspace (chunk statistics, slice masses, the error flag) live in one device array of fixed size instead of a handle's arena.
// ---------------------------------------------------------------------------------------------
namespace specv {
namespace {

constexpr int NA_MAX_BATCH = SPEC_NOALLOC_MAX_BATCH;
constexpr int NA_MAX_VOCAB = SPEC_NOALLOC_MAX_VOCAB;
constexpr int NA_MAX_ROWS = NA_MAX_BATCH * (SPEC_MAX_LOOKAHEAD + 1);
constexpr int NA_MAX_STAT = NA_MAX_BATCH * (2 * SPEC_MAX_LOOKAHEAD + 1);
constexpr int NA_STAT_CHUNKS = (NA_MAX_VOCAB + STAT_CHUNK - 1) / STAT_CHUNK;
constexpr int NA_RES_CHUNKS = (NA_MAX_VOCAB + RES_CHUNK - 1) / RES_CHUNK;

struct NoAllocScratch {
    double part_sum[(size_t)NA_MAX_STAT * NA_STAT_CHUNKS];
    double slice_mass[(size_t)NA_MAX_BATCH * NA_RES_CHUNKS];
    DrawnRow drawn[NA_MAX_BATCH];
    float part_max[(size_t)NA_MAX_STAT * NA_STAT_CHUNKS];
    int32_t part_idx[(size_t)NA_MAX_STAT * NA_STAT_CHUNKS];
    int32_t arrived[NA_MAX_BATCH * ARRIVED_STRIDE];
    int32_t seq_row0[NA_MAX_BATCH + 1], seq_stat0[NA_MAX_BATCH + 1];
    int32_t seq_n[NA_MAX_BATCH], seq_ok[NA_MAX_BATCH], seq_slot[NA_MAX_BATCH];
    int32_t row_seq[NA_MAX_ROWS], row_pos[NA_MAX_ROWS], row_tok[NA_MAX_ROWS], row_rope[NA_MAX_ROWS];
    uint32_t row_mask[NA_MAX_ROWS];
    int32_t flag[4];
};
static_assert(sizeof(NoAllocScratch) <= (size_t)640 * 1024, "the fixed workspace is meant to stay modest");

// Every GPU the library runs on holds its own copy of this array until the process ends.  In host
// code the name is only a handle for hipGetSymbolAddress: kernels get the address looked up below.
static __device__ __align__(256) unsigned char scratch[sizeof(NoAllocScratch)];

constexpr int NA_MAX_DEVICES = 64;
NoAllocScratch* g_scratch_ptr[NA_MAX_DEVICES];   // per device; written once, under g_scratch_lock
std::mutex g_scratch_lock;

// Address of the current device's copy of the array (looked up on the first call on that device).
int scratch_of_current_device(NoAllocScratch** out)
{
    int dev = -1;
    SPECV_HIP(hipGetDevice(&dev));
    if (dev < 0 || dev >= NA_MAX_DEVICES) return fail(SPEC_ERR_DEVICE, "device index %d is not supported", dev);
    std::lock_guard<std::mutex> guard(g_scratch_lock);
    if (!g_scratch_ptr[dev]) {
        void* p = nullptr;
        SPECV_HIP(hipGetSymbolAddress(&p, HIP_SYMBOL(scratch)));
        if (!p) return fail(SPEC_ERR_DEVICE, "hipGetSymbolAddress returned no address for the fixed workspace");
        g_scratch_ptr[dev] = static_cast<NoAllocScratch*>(p);
    }
    *out = g_scratch_ptr[dev];
    return SPEC_OK;
}

}  // namespace
}  // namespace specv

using namespace specv;

extern "C" int spec_sample_step_noalloc(int32_t vocab, int32_t max_lookahead, const spec_step_args* args,
                                        const spec_step_out* out, void* stream)
{
    if (!args || !out) return fail(SPEC_ERR_INVALID_ARG, "NULL args or out");
    if (vocab < 1 || vocab > NA_MAX_VOCAB)
        return fail(SPEC_ERR_SHAPE, "vocab %d outside 1..%d (the fixed workspace is sized for that)", vocab, NA_MAX_VOCAB);
    if (max_lookahead < 0 || max_lookahead > SPEC_MAX_LOOKAHEAD)
        return fail(SPEC_ERR_SHAPE, "max_lookahead %d outside 0..%d", max_lookahead, SPEC_MAX_LOOKAHEAD);
    const int B = args->batch, Kmax = max_lookahead;
    if (B < 1 || B > NA_MAX_BATCH)
        return fail(SPEC_ERR_SHAPE, "batch %d outside 1..%d (the fixed workspace is sized for that)", B, NA_MAX_BATCH);
    if (!args->target_logits_in) return fail(SPEC_ERR_INVALID_ARG, "target_logits_in is NULL: this entry point runs no decoder pass");
    if (!args->lookahead) return fail(SPEC_ERR_INVALID_ARG, "lookahead is NULL");
    if (!(args->temperature >= 0.f)) return fail(SPEC_ERR_INVALID_ARG, "temperature must be >= 0");
    const bool greedy = args->temperature == 0.f;
    if (!greedy && !args->uniforms) return fail(SPEC_ERR_INVALID_ARG, "uniforms is NULL");
    if (!out->n_accepted || !out->out_tokens) return fail(SPEC_ERR_INVALID_ARG, "n_accepted or out_tokens is NULL");
    LookaheadPack ks;
    memset(&ks, 0, sizeof(ks));
    int M = 0, n_stat = 0, any_draft = 0;
    for (int b = 0; b < B; ++b) {
        const int k = args->lookahead[b];
        if (k < 0 || k > Kmax) return fail(SPEC_ERR_INVALID_ARG, "lookahead[%d] = %d outside 0..%d", b, k, Kmax);
        ks.k[b] = (uint8_t)k;
        M += k + 1;
        n_stat += 2 * k + 1;
        any_draft |= k;
    }
    if (any_draft && (!args->draft_tokens || (!greedy && !args->draft_logits)))
        return fail(SPEC_ERR_INVALID_ARG, "draft_tokens or draft_logits is NULL");
    NoAllocScratch* w = nullptr;
    int rc = scratch_of_current_device(&w);
    if (rc) return rc;
    hipStream_t s = (hipStream_t)stream;
    // the array keeps the last call's contents: every entry that is read was written earlier in this call (the flag is
    // where the row bookkeeping reports; a call without a handle has no poll that would read it)
    StepTables t{};
    t.seq_row0 = w->seq_row0;
    t.seq_stat0 = w->seq_stat0;
    t.seq_n = w->seq_n;
    t.seq_ok = w->seq_ok;
    t.seq_slot = w->seq_slot;
    t.row_seq = w->row_seq;
    t.row_pos = w->row_pos;
    t.row_tok = w->row_tok;
    t.row_rope = w->row_rope;
    t.row_mask = w->row_mask;
    t.arrived = w->arrived;
    t.tree = 0;
    SamplerWorkspace sw{};
    sw.part_max = w->part_max;
    sw.part_sum = w->part_sum;
    sw.slice_mass = w->slice_mass;
    sw.drawn = w->drawn;
    sw.part_idx = w->part_idx;
    if (greedy) {   // the greedy rule's kernels read the tables from the start
        rc = launch_prepare(t, ks, B, Kmax, vocab, NA_MAX_BATCH, 0, false, nullptr, nullptr, args->draft_tokens, nullptr,
                            w->flag, s);
        if (rc) return rc;
    }
    if (out->logits_out) {
        // a copy node, not an allocation; callers under capture simply pass logits_out = NULL
        SPECV_HIP(hipMemcpyAsync(out->logits_out, args->target_logits_in, (size_t)M * vocab * sizeof(float),
                                 hipMemcpyDeviceToDevice, s));
    }
    if (greedy)
        return launch_greedy(t, sw, ks, B, Kmax, vocab, M, args->target_logits_in, args->draft_tokens, 0, nullptr,
                             out->n_accepted, out->out_tokens, nullptr, nullptr, s);
    return launch_sampler(t, sw, ks, B, Kmax, vocab, n_stat, args->target_logits_in, args->draft_logits,
                          args->draft_tokens, args->uniforms, Kmax + 1, args->temperature, 0, nullptr, out->n_accepted,
                          out->out_tokens, nullptr, nullptr, s, w->flag);
}
