// The decoder's projections: Y[M][N] = X[M][K] * W[N][K]^T with a handful of rows (M = number of
// window tokens in flight) against large bf16 weight matrices.  This is a real dense contraction,
// so it runs on the matrix cores (v_mfma_f32_16x16x32_bf16), but at these M it is bound by
// streaming W from HBM exactly once, and the kernel is organised around that stream:
//
//  * W is stored in tile order (spec_pack_weight): the 16x32 operand tile a wavefront needs is one
//    contiguous 1 KiB block, and the tiles a wavefront walks along K follow each other in memory,
//    so every lane issues plain 16-byte loads that coalesce perfectly and each wave streams a
//    contiguous region.  The loads for the next K chunk are in flight while the current one is
//    multiplied (two register buffers), and nothing but W goes through that pipe.
//  * X (a few hundred KiB, L2 resident) arrives already as bf16 operand fragments (frag.h), written
//    that way by the kernel that produced it, and is staged through LDS once per workgroup and K
//    chunk with plain 16-byte copies, shared by the four wavefronts, double buffered.  With two
//    planes each activation is a bf16 head plus a bf16 remainder (two matrix instructions): the
//    matrix cores have ample slack at these shapes, and activation rounding drops to ~2^-17.
//  * RMSNorm costs nothing here: the producer multiplies by the gain, and the row's 1/rms factors
//    out of the dot product, so the consumer of the GEMM's result applies it as a row scale.
//  * K is cut into ranges across workgroups so that the grid fills all 256 compute units even when
//    N is small; range sums are left in a partial buffer in a fixed order and added up by the
//    consumer kernel (no floating-point atomics: bit-reproducible).
#include <type_traits>

#include "common.h"
#include "frag.h"

namespace specv {
namespace {

// Workgroup index -> (K range, column block).  Workgroups are dealt round-robin to the 8 XCDs, each
// with its own L2; ranges are assigned so that all workgroups of one K range run on one XCD and the
// slice of X they share stays in that L2.  n_split is a power of two.
__device__ __forceinline__ void map_block(int i, int n_split, int* s, int* nb)
{
    const int x = i & 7, j = i >> 3;
    if (n_split >= 8) {
        const int hi = n_split >> 3;
        *s = x + 8 * (j % hi);
        *nb = j / hi;
    } else {
        const int per = 8 / n_split;
        *s = x % n_split;
        *nb = j * per + x / n_split;
    }
}

typedef unsigned int u32x4 __attribute__((ext_vector_type(4)));
constexpr int WPACK_KG = 4;   // K blocks per group of the packed weight order

// All global loads below are unconditional (addresses clamped into range, W zeroed by selects past
// the K range): with no branch around a load the compiler can count outstanding loads exactly, so
// a wait for X never turns into a wait for the whole W stream.
// RS = 2 (many row tiles): eight wavefronts per workgroup, two row halves x four column groups.
// A wavefront then holds the accumulators of MTW = ceil(MT/2) row tiles only, which fits two
// wavefronts per SIMD: the matrix instruction issues faster with a second wavefront to alternate
// with (measured: one 16x16x32 product per 19-20 cycles and SIMD instead of 22-26), and the
// other wavefront's products cover this one's waits.
// EPI = 1 (gate/up projection with a single K range, NT == 2, columns packed so that a gate tile and
// its up tile are neighbours): instead of leaving sums for another kernel, the workgroup applies the
// row scale of the preceding norm, computes silu(gate) * up and writes the result as operand
// fragments of the down projection.  One kernel and one round of partial sums less per layer.
// CG: wavefronts (column groups of NT tiles) per workgroup, 4 unless the launch picks fewer.  With a
// single K range every workgroup streams all of X through its compute unit next to its share of W;
// three wavefronts per workgroup put the 7B-shape gate/up projection on 230 compute units instead of
// 172, and the same stream ran in 32.5 instead of 37.8 us (stand-alone, epilogue removed; without
// any X traffic both take 30 us): what a compute unit can pull from L2 per unit of time, X included,
// is the limit there, not HBM.
struct SwigluOut {
    const double2* ssq; // NormScale of the rows (sums of squares in n_ssq pairs of chunks)
    int n_ssq, d;
    float eps;
    uint4* frags;       // fragment buffer of the down projection's operand
    int mt, planes;
    SsqTiles tiles;     // one row tile: the sums of squares as gemm_add_kernel leaves them (tiles.parts == NULL: ssq)
};

// The sums of squares of N groups of 1024 columns of a row, from group q on, from the sums over ADD_COLS columns each, by
// eight neighbouring lanes (sub 0..7; every lane gets the sums; 0 past the end): one memory round trip.  d is a multiple
// of 32, so the sums come in pairs.
template <int N>
__device__ __forceinline__ void ssq_group_sums(const double* row, int n_parts, int q, int sub, double (&sums)[N])
{
    constexpr int PER = 2 * SSQ_CHUNK / ADD_COLS / 8;   // sums per lane
    const int i0 = q * 8 * PER + sub * PER;
    double2 v[N][PER / 2];
#pragma unroll
    for (int j = 0; j < N; ++j)
#pragma unroll
        for (int i = 0; i < PER / 2; ++i) v[j][i] = *reinterpret_cast<const double2*>(row + min(i0 + j * 8 * PER + 2 * i, n_parts - 2));
#pragma unroll
    for (int j = 0; j < N; ++j) {
        sums[j] = 0.0;
#pragma unroll
        for (int i = 0; i < PER / 2; ++i) sums[j] += i0 + j * 8 * PER + 2 * i < n_parts ? v[j][i].x + v[j][i].y : 0.0;
#pragma unroll
        for (int o = 1; o < 8; o *= 2) sums[j] += __shfl_xor(sums[j], o);
    }
}

template <int MT, int NT, int KC, int PLANES, int RS = 1, int EPI = 0, int CG = 4>
__global__ void __launch_bounds__(64 * CG * RS) gemm_skinny_kernel(const u32x4* __restrict__ Xf, const u32x4* __restrict__ Wp,
                                                          float* __restrict__ partial, int M, int n_tiles,
                                                          int kb_total, int kb_per_split, int n_split, int n_blocks,
                                                          SwigluOut so)
{
    if constexpr (MT == 1 && EPI == 0) {
        // Eight more workgroups where gemm_add_kernel wrote the operand (the XCDs' turns stay as they are): the first
        // makes the row sums that the consumer of this product scales with, beside the product.
        if (so.tiles.parts && blockIdx.x + 8 >= gridDim.x) {
            if (blockIdx.x + 8 > gridDim.x || threadIdx.x >= 128) return;
            const int m = min((int)threadIdx.x >> 3, M - 1);
            for (int q = 0; q < so.n_ssq; q += 2) {
                double ss[2];
                ssq_group_sums(so.tiles.parts + (size_t)m * so.tiles.n_parts, so.tiles.n_parts, q, threadIdx.x & 7, ss);
                if ((threadIdx.x & 7) == 0 && (int)threadIdx.x >> 3 == m) {
                    so.tiles.ssq_out[(size_t)m * so.n_ssq + q] = make_double2(ss[0], 0.0);
                    if (q + 1 < so.n_ssq) so.tiles.ssq_out[(size_t)m * so.n_ssq + q + 1] = make_double2(ss[1], 0.0);
                }
            }
            return;
        }
    }
    constexpr int CHUNK_U4 = KC * PLANES * MT * 64;     // 16-byte units per X chunk (contiguous in Xf)
    constexpr int TPBK = 64 * CG * RS;                    // threads per workgroup: CG column groups x RS row halves
    constexpr int UPT = (CHUNK_U4 + TPBK - 1) / TPBK;     // per thread
    __shared__ u32x4 xs[2][CHUNK_U4];                   // two chunk buffers
    __shared__ float rsv[EPI == 1 ? MT * 16 : 1];       // SwiGLU: row scales

    int split, nblk;
    map_block(blockIdx.x, n_split, &split, &nblk);
    if (nblk >= n_blocks) return;
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    constexpr int MTW = (MT + RS - 1) / RS;               // row tiles of one wavefront
    const int a0 = (wave % RS) * MTW;                       // its first row tile
    const int tile0 = (nblk * CG + wave / RS) * NT;
    const int kb0 = split * kb_per_split;
    const int kb1 = min(kb0 + kb_per_split, kb_total);

    floatx4 acc[MTW][NT];
#pragma unroll
    for (int a = 0; a < MTW; ++a)
#pragma unroll
        for (int i = 0; i < NT; ++i) acc[a][i] = floatx4{0.f, 0.f, 0.f, 0.f};

    u32x4 wa[KC][NT], wb[KC][NT];
    u32x4 xr[UPT];
    int xoff[UPT];
#pragma unroll
    for (int u = 0; u < UPT; ++u) xoff[u] = min(u * TPBK + (int)threadIdx.x, CHUNK_U4 - 1);   // surplus threads repeat
    // Two row tiles: X through a buffer descriptor, whose bound makes rows past the last fetch nothing (their zeros are never
    // stored).  Steps of four layers, 17 to 24 rows: 7B shape -2.0..-2.2 %, 3072 wide -2.3..-2.5, 1B shape -1.5..-1.8, 1536 and 1024 wide
    // -0.9 and -0.1..-0.4; 32 rows -1.1, -0.9 and 0.  One row tile within 0.5 % either way, three +4 % at 48 rows, four mixed.
    constexpr bool X_BUFFER = MT == 2;
    const __amdgpu_buffer_rsrc_t xbuf = __builtin_amdgcn_make_buffer_rsrc(const_cast<u32x4*>(Xf), 0, (kb_total + XFRAG_PAD_KB) * PLANES * MT * 1024, 0x00027000);
    uint32_t xbyte[UPT];
    if constexpr (X_BUFFER) {
#pragma unroll
        for (int u = 0; u < UPT; ++u) xbyte[u] = ((xoff[u] >> 6) % MT) * 16 + (xoff[u] & 15) < M ? xoff[u] * 16u : 0x40000000u;
    }

    // W tile order: [K group of 4 blocks][column tile][block in group][lane] -- the chunk a workgroup
    // reads in one step (its 4*NT tiles, KC blocks) is one contiguous run, and workgroups of
    // neighbouring column blocks read neighbouring runs
    const u32x4* wbase[NT];
#pragma unroll
    for (int i = 0; i < NT; ++i) wbase[i] = Wp + (size_t)min(tile0 + i, n_tiles - 1) * (WPACK_KG * 64) + lane;
    const size_t group_stride = (size_t)n_tiles * (WPACK_KG * 64);

    // Up to four row tiles the weights are fetched with streaming (non-temporal) loads: each is read once
    // per launch by one wavefront, and marked that way the stream leaves the caches to what is reused (the
    // X fragments, the partial sums, a small model's keys and values).  Measured, same box: 7B-shape step
    // 4.934 -> 4.877 ms, 1B-shape 0.947 -> 0.890 ms (its 34 MB of keys and values stay in the memory-side
    // cache from step to step).  From five row tiles on it is a wash (72 rows +0.4 %, 88-96 rows -0.5 %),
    // and where two wavefronts of a workgroup fetch the same tile (RS = 2) the second would miss: 157 rows
    // +6..10 % GEMM time.  Those keep ordinary loads.
    constexpr bool W_STREAM = RS == 1 && MT <= 4;
    // Loads past the end of the range are redirected to its last block (a cache hit, no new HBM
    // traffic); the products of such blocks are suppressed by mask_w.
    auto load_w = [&](int kbase, u32x4(&dst)[KC][NT]) {
#pragma unroll
        for (int c = 0; c < KC; ++c) {
            const int kb = min(kbase + c, kb1 - 1);
            const size_t off = (size_t)(kb / WPACK_KG) * group_stride + (kb % WPACK_KG) * 64;
#pragma unroll
            for (int i = 0; i < NT; ++i) {
                if constexpr (W_STREAM) dst[c][i] = __builtin_nontemporal_load(&wbase[i][off]);
                else dst[c][i] = wbase[i][off];
            }
        }
    };
    auto mask_w = [&](int kbase, u32x4(&w)[KC][NT]) {   // K blocks past the range contribute nothing
#pragma unroll
        for (int c = 0; c < KC; ++c) {
            const bool ok = kbase + c < kb1;
#pragma unroll
            for (int i = 0; i < NT; ++i) w[c][i] = ok ? w[c][i] : u32x4{0u, 0u, 0u, 0u};
        }
    };
    auto load_x = [&](int kbase) {
        // fragment buffers carry XFRAG_PAD_KB zeroed blocks past kb_total, so the last chunk of the
        // last range may overhang
        const int kb = min(kbase, kb1 - 1);
        if constexpr (X_BUFFER) {
#pragma unroll
            for (int u = 0; u < UPT; ++u) xr[u] = __builtin_amdgcn_raw_buffer_load_b128(xbuf, xbyte[u], kb * (PLANES * MT * 1024), 0);
        } else {
            const u32x4* src = Xf + (size_t)kb * (PLANES * MT * 64);
#pragma unroll
            for (int u = 0; u < UPT; ++u) xr[u] = src[xoff[u]];
        }
    };
    auto store_x = [&](int buf) {
#pragma unroll
        for (int u = 0; u < UPT; ++u) xs[buf][xoff[u]] = xr[u];
    };
    // fragment of the wavefront's a-th row tile (RS = 2 and odd MT: the second half's last tile does
    // not exist; it re-reads the tile before it and its results are dropped)
    auto x_frag = [&](int buf, int c, int plane, int a) {
        const int row_tile = RS == 1 ? a : min(a0 + a, MT - 1);
        return __builtin_bit_cast(bf16x8, xs[buf][((c * PLANES + plane) * MT + row_tile) * 64 + lane]);
    };
    auto compute = [&](const u32x4(&w)[KC][NT], int buf) {
        if constexpr (MT >= 3) {
            // One wavefront per SIMD: nothing else fills the matrix pipeline while this wave waits
            // for an LDS read, so the fragments of row tile t+1 are requested before the products of
            // tile t are issued, and the instruction order is pinned (2 LDS reads, then the 2*NT
            // products of the previous reads); left to itself the scheduler reads, waits, multiplies.
            bf16x8 xh = x_frag(buf, 0, 0, 0), xl = xh;
            if constexpr (PLANES == 2) xl = x_frag(buf, 0, 1, 0);
            __builtin_amdgcn_sched_group_barrier(0x100, PLANES, 0);            // LDS reads of tile 0
#pragma unroll
            for (int t = 0; t < KC * MTW; ++t) {
                const int c = t / MTW, a = t % MTW;
                bf16x8 nh = xh, nl = xl;
                if (t + 1 < KC * MTW) {
                    nh = x_frag(buf, (t + 1) / MTW, 0, (t + 1) % MTW);
                    nl = nh;
                    if constexpr (PLANES == 2) nl = x_frag(buf, (t + 1) / MTW, 1, (t + 1) % MTW);
                }
#pragma unroll
                for (int i = 0; i < NT; ++i)
                    acc[a][i] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(xh, __builtin_bit_cast(bf16x8, w[c][i]), acc[a][i], 0, 0, 0);
                if constexpr (PLANES == 2) {
#pragma unroll
                    for (int i = 0; i < NT; ++i)
                        acc[a][i] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(xl, __builtin_bit_cast(bf16x8, w[c][i]), acc[a][i], 0, 0, 0);
                }
                __builtin_amdgcn_sched_group_barrier(0x100, PLANES, 0);        // LDS reads of tile t+1
                __builtin_amdgcn_sched_group_barrier(0x008, PLANES * NT, 0);   // products of tile t
                xh = nh;
                xl = nl;
            }
            return;
        }
#pragma unroll
        for (int c = 0; c < KC; ++c)
#pragma unroll
            for (int a = 0; a < MT; ++a) {
                const bf16x8 xh = x_frag(buf, c, 0, a);
                bf16x8 xl = xh;
                if constexpr (PLANES == 2) xl = x_frag(buf, c, 1, a);
#pragma unroll
                for (int i = 0; i < NT; ++i) {
                    const bf16x8 wf = __builtin_bit_cast(bf16x8, w[c][i]);
                    acc[a][i] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(xh, wf, acc[a][i], 0, 0, 0);
                    if constexpr (PLANES == 2)
                        acc[a][i] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(xl, wf, acc[a][i], 0, 0, 0);
                }
            }
    };

    if constexpr (MT >= 8) {
        // Many row tiles: a chunk's products take about as long as a memory round trip, and with two W
        // buffers the loads of chunk j+2 can only be issued after the products of chunk j (they reuse
        // its registers), so products and waiting alternate instead of overlapping.  A third W buffer
        // lets the loads of chunk j+2 go out BEFORE the products of chunk j, and three X register
        // sets keep the fragments of chunks j+2..j+4 in flight (X is the larger of the two streams
        // here and misses L2 as often as not).  One K block per chunk (KC == 1): no chunk is partial,
        // nothing needs masking; loads past the range are redirected to its last block and their
        // chunks never multiplied.
        static_assert(MT < 8 || KC == 1, "the three-buffer pipeline takes one K block per chunk");
        u32x4 wc[KC][NT];
        u32x4 x0[UPT], x1[UPT], x2[UPT];
        auto load_xs = [&](int kbase, u32x4(&dst)[UPT]) {
            const u32x4* src = Xf + (size_t)min(kbase, kb1 - 1) * (PLANES * MT * 64);
#pragma unroll
            for (int u = 0; u < UPT; ++u) dst[u] = src[xoff[u]];
        };
        auto store_xs = [&](int buf, const u32x4(&from)[UPT]) {
#pragma unroll
            for (int u = 0; u < UPT; ++u) xs[buf][xoff[u]] = from[u];
        };
        const int n_chunks = kb1 - kb0;
        // step j: W of chunk j+2 requested, chunk j multiplied, chunk j+1's X (set xn, fetched three
        // steps ago) put into the other LDS buffer, chunk j+4's X requested into the same set
        auto step = [&](int j, const u32x4(&cur)[KC][NT], u32x4(&ahead)[KC][NT], u32x4(&xn)[UPT]) {
            load_w(kb0 + j + 2, ahead);
            compute(cur, j & 1);
            store_xs((j + 1) & 1, xn);
            load_xs(kb0 + j + 4, xn);
            __syncthreads();
        };
        load_w(kb0, wa);
        __builtin_amdgcn_sched_barrier(0);
        load_xs(kb0, x0);
        load_xs(kb0 + 1, x1);
        load_xs(kb0 + 2, x2);
        load_w(kb0 + 1, wb);
        store_xs(0, x0);
        load_xs(kb0 + 3, x0);
        __syncthreads();
        int j = 0;
        for (; j + 3 <= n_chunks; j += 3) {
            step(j, wa, wc, x1);
            step(j + 1, wb, wa, x2);
            step(j + 2, wc, wb, x0);
        }
        if (j < n_chunks) {
            step(j, wa, wc, x1);
            if (j + 1 < n_chunks) step(j + 1, wb, wa, x2);
        }
    } else {
    // The W stream starts first; afterwards X loads are always issued before the W loads of the same
    // step, so that waiting for X (older) leaves the W loads (younger) in flight.
    load_w(kb0, wa);
    __builtin_amdgcn_sched_barrier(0);   // keep the first W loads ahead of everything else
    load_x(kb0);
    store_x(0);
    load_x(kb0 + KC);
    load_w(kb0 + KC, wb);
    if constexpr (MT == 1 && EPI == 1) {
        if (so.tiles.parts) {   // here, where the stream's first round trips cover it (eight lanes a row)
            if (threadIdx.x < 128) {
                const int m = min((int)threadIdx.x >> 3, M - 1);
                float ss = 0.f;
                for (int q = 0; q < so.n_ssq; q += 2) {   // (past the end a group is 0)
                    double two[2];
                    ssq_group_sums(so.tiles.parts + (size_t)m * so.tiles.n_parts, so.tiles.n_parts, q, threadIdx.x & 7, two);
                    ss += (float)two[0];
                    ss += (float)two[1];
                }
                if ((threadIdx.x & 7) == 0) rsv[threadIdx.x >> 3] = 1.0f / sqrtf(ss / (float)so.d + so.eps);
            }
        }
    }
    __syncthreads();
    // Chunk j is multiplied from LDS buffer j%2 while chunk j+1's X (already in registers) is copied
    // into the other buffer and the loads of chunk j+2 are issued.  The main loop runs while both of
    // its prefetches are inside the range; the last one to three chunks are finished below without
    // loading anything past the range.  Only the last chunk can be partial (mask_w).
    const int n_chunks = (kb1 - kb0 + KC - 1) / KC;
    int j = 0;
    for (; j + 3 < n_chunks; j += 2) {
        const int kbase = kb0 + j * KC;
        compute(wa, 0);
        store_x(1);
        load_x(kbase + 2 * KC);
        load_w(kbase + 2 * KC, wa);
        __syncthreads();
        compute(wb, 1);
        store_x(0);
        load_x(kbase + 3 * KC);
        load_w(kbase + 3 * KC, wb);
        __syncthreads();
    }
    {
        const int kbase = kb0 + j * KC;
        const int left = n_chunks - j;   // 1, 2 or 3 (0 only for an empty range)
        if (left == 3) {
            compute(wa, 0);
            store_x(1);
            load_x(kbase + 2 * KC);
            load_w(kbase + 2 * KC, wa);
            __syncthreads();
            compute(wb, 1);
            store_x(0);
            __syncthreads();
            mask_w(kbase + 2 * KC, wa);
            compute(wa, 0);
        } else if (left == 2) {
            compute(wa, 0);
            store_x(1);
            __syncthreads();
            mask_w(kbase + KC, wb);
            compute(wb, 1);
        } else if (left == 1) {
            mask_w(kbase, wa);
            compute(wa, 0);
        }
    }
    }   // MT < 8

    const int g = lane >> 4, c = lane & 15;
    if constexpr (EPI == 1) {
        static_assert(EPI == 0 || (NT == 2 && RS == 1), "the SwiGLU epilogue pairs the two column tiles of a wavefront");
        static_assert(EPI == 0 || sizeof(xs) >= CG * MT * 256 * sizeof(float), "tile staging fits the X chunk buffers");
        // The accumulators are read next, by vector instructions, which have to wait seven states for the last products.
        // The compiler's own wait is lost where the branches above meet (one row tile: two states; the last
        // product's remainder was missing from rows 0, 4, 8 and 12, 1.6e-4 of their values), so it is written out here,
        // and the accumulators pass through it.
#pragma unroll
        for (int a = 0; a < MT; ++a) asm volatile("s_nop 15" : "+a"(acc[a][0]), "+a"(acc[a][1]));
        __syncthreads();                                      // everyone is done with the X chunk buffers
        float* tw = reinterpret_cast<float*>(&xs[0][0]) + wave * (MT * 256);   // [MT*16 rows][16 units]
        for (int m = threadIdx.x; m < MT * 16 && !(MT == 1 && so.tiles.parts); m += TPBK)
            rsv[m] = m < M ? row_inv_rms(so.ssq, so.n_ssq, m, so.d, so.eps) : 0.f;
        __syncthreads();
#pragma unroll
        for (int a = 0; a < MT; ++a)
#pragma unroll
            for (int r = 0; r < 4; ++r) {
                const int ml = a * 16 + 4 * g + r;
                const float rs = rsv[ml];
                const float ge = acc[a][0][r] * rs, ue = acc[a][1][r] * rs;
                tw[ml * 16 + c] = ge / (1.f + expf(-ge)) * ue;
            }
        __syncthreads();
        if (tile0 + 1 < n_tiles) {
            const int f0 = (tile0 >> 1) * 16;                 // first FFN unit of this tile pair
            for (int u = lane; u < MT * 32; u += 64) {
                const int row = u >> 1, oct = u & 1;
                if (row < M) {
                    const float4 lo4 = *reinterpret_cast<const float4*>(tw + row * 16 + oct * 8);
                    const float4 hi4 = *reinterpret_cast<const float4*>(tw + row * 16 + oct * 8 + 4);
                    const float v[8] = {lo4.x, lo4.y, lo4.z, lo4.w, hi4.x, hi4.y, hi4.z, hi4.w};
                    store_x_unit(so.frags, so.mt, so.planes, row, (f0 >> 3) + oct, v);
                }
            }
        }
        return;
    }
    const int n_pad = n_tiles * 16;
    float* out = partial + (size_t)split * M * n_pad;
#pragma unroll
    for (int a = 0; a < MTW; ++a)
#pragma unroll
        for (int i = 0; i < NT; ++i) {
            const int tile = tile0 + i;
            if (tile < n_tiles && a0 + a < MT) {
#pragma unroll
                for (int r = 0; r < 4; ++r) {
                    const int m = (a0 + a) * 16 + 4 * g + r;
                    if (m < M) out[(size_t)m * n_pad + tile * 16 + c] = acc[a][i][r];
                }
            }
        }
}

// ---- few rows, the projections that end in the residual stream ---------------------------------------------
// x += X * W^T for up to 16 rows, with what follows it in the chain: the new x times the next norm's gain as operand
// fragments and the sums of squares of the new x.  A step of a few rows is a chain of launches that are mostly latency, and
// cut into K ranges across workgroups these two projections needed a launch of their own to add the ranges up.  Here a
// workgroup takes ADD_COLS columns and wavefront r the r-th K range, with the sums of the ranges met in LDS: the
// products and additions are those of the cut across workgroups, in the same order (bit for bit the same x).  Nothing
// else is shared, so both operands go straight into registers, DEPTH groups of four K blocks ahead.
// Each workgroup reads all of X: the loads of X are two thirds of all, which is what limits this to one row tile and to K up
// to 6144.  2048 columns, us by trace, product and residual kernel before, this now (128 workgroups): K = 2048 4.3 + 3.1 -> 4.2,
// K = 5504 6.6 + 3.8 -> 8.6, K = 8192 7.5 + 3.1 -> 11.4 (eight columns per workgroup, twice the workgroups: no faster).
// 1B shape, batch 1, 787 -> 773 us a step (790 with its down projection, K = 8192, this way), draft decode of 8 rows
// 302 -> 291, decoding round 2217 -> 2184.
// The row's whole sum of squares spans all workgroups: it leaves as one fp64 sum per row and workgroup, and the next
// product adds those up (ssq_group_sums).
template <int RANGES>
__global__ void __launch_bounds__(64 * RANGES) gemm_add_kernel(const u32x4* __restrict__ Xf, const u32x4* __restrict__ Wp, float* __restrict__ x,
                                                               const float* __restrict__ gain, int M, int n_tiles, int kb_total,
                                                               int kb_per_range, uint16_t* __restrict__ frags, double* __restrict__ parts)
{
    constexpr int PLANES = 2;
    constexpr int DEPTH = RANGES > 8 ? 1 : 3;   // register buffers (128 registers a wavefront with sixteen of them, 256 with eight)
    static_assert(RANGES >= 4, "a thread for every element");
    __shared__ float red[RANGES][16 * ADD_COLS];
    const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6)), g = lane >> 4, c = lane & 15;
    const int n0 = blockIdx.x * ADD_COLS;
    const int group0 = wave * (kb_per_range / WPACK_KG);
    const int n = (min(kb_per_range, kb_total - wave * kb_per_range) + WPACK_KG - 1) / WPACK_KG;   // groups (none or less: an empty range)
    // lanes past the last row ask past the end of the buffer: they get zeros and fetch nothing
    const __amdgpu_buffer_rsrc_t xb = __builtin_amdgcn_make_buffer_rsrc(const_cast<u32x4*>(Xf), 0, kb_total * PLANES * 1024, 0x00027000);
    const uint32_t x_lane = c < M ? lane * 16u : 0x40000000u;
    const u32x4* wp = Wp + (size_t)blockIdx.x * (WPACK_KG * 64);
    const size_t group_stride = (size_t)n_tiles * (WPACK_KG * 64);
    struct Group {
        u32x4 w[WPACK_KG], x[WPACK_KG][PLANES];
    };
    Group buf[DEPTH];
    auto load = [&](int i, Group& d) {
        const int group = group0 + i;
#pragma unroll
        for (int j = 0; j < WPACK_KG; ++j) d.w[j] = __builtin_nontemporal_load(wp + group * group_stride + j * 64 + (uint32_t)lane);
#pragma unroll
        for (int j = 0; j < WPACK_KG; ++j) {   // (past the last block the packed weights are zeros)
            const int kb = min(group * WPACK_KG + j, kb_total - 1);
#pragma unroll
            for (int p = 0; p < PLANES; ++p) d.x[j][p] = __builtin_amdgcn_raw_buffer_load_b128(xb, x_lane, (kb * PLANES + p) * 1024, 0);
        }
    };
    floatx4 acc = {0.f, 0.f, 0.f, 0.f};
    auto multiply = [&](const Group& d) {
#pragma unroll
        for (int j = 0; j < WPACK_KG; ++j)
#pragma unroll
            for (int p = 0; p < PLANES; ++p)
                acc = __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8, d.x[j][p]), __builtin_bit_cast(bf16x8, d.w[j]), acc, 0, 0, 0);
    };
    // the last groups, with no branch between a load and its use (the compiler then knows which loads a wait is for):
    // HAVE of them in flight, MORE to come (fewer than DEPTH, in the buffers of the first ones)
    auto finish = [&](int i, auto have, auto more) {
#pragma unroll
        for (int j = 0; j < decltype(more)::value; ++j) {
            multiply(buf[j]);
            load(i + decltype(have)::value + j, buf[j]);
        }
#pragma unroll
        for (int j = decltype(more)::value; j < decltype(have)::value; ++j) multiply(buf[j]);
#pragma unroll
        for (int j = 0; j < decltype(more)::value; ++j) multiply(buf[j]);
    };
    auto start = [&](auto have) {
#pragma unroll
        for (int j = 0; j < decltype(have)::value; ++j) load(j, buf[j]);
    };
    float x_old = 0.f, gn = 0.f;   // (requested with the first operands)
    if ((int)threadIdx.x < M * ADD_COLS) {
        x_old = x[(size_t)(threadIdx.x / ADD_COLS) * (n_tiles * 16) + n0 + threadIdx.x % ADD_COLS];
        gn = gain[n0 + threadIdx.x % ADD_COLS];
    }
    using I0 = std::integral_constant<int, 0>;
    using I1 = std::integral_constant<int, 1>;
    using I2 = std::integral_constant<int, 2>;
    using ID = std::integral_constant<int, DEPTH>;
    if (n >= DEPTH) {
        start(ID{});
        int i = 0;
        for (; i + 2 * DEPTH <= n; i += DEPTH)
#pragma unroll
            for (int j = 0; j < DEPTH; ++j) {
                multiply(buf[j]);
                load(i + DEPTH + j, buf[j]);
            }
        switch (n - i - DEPTH) {
        case 0: finish(i, ID{}, I0{}); break;
        case 1: if constexpr (DEPTH > 1) finish(i, ID{}, I1{}); break;
        default: if constexpr (DEPTH > 2) finish(i, ID{}, I2{}); break;
        }
    } else if (n == 1) {
        start(I1{});
        finish(0, I1{}, I0{});
    } else if (DEPTH > 2 && n == 2) {
        start(I2{});
        finish(0, I2{}, I0{});
    }
#pragma unroll
    for (int r = 0; r < 4; ++r) red[wave][(4 * g + r) * ADD_COLS + c] = acc[r];
    __syncthreads();
    const int row = threadIdx.x / ADD_COLS, col = n0 + threadIdx.x % ADD_COLS;
    if (row >= M) return;   // (all lanes of a row alike)
    float sum = red[0][threadIdx.x];
#pragma unroll
    for (int w = 1; w < RANGES; ++w) sum += red[w][threadIdx.x];
    const float v = x_old + sum;
    x[(size_t)row * (n_tiles * 16) + col] = v;
    uint16_t* f = frags + ((size_t)(col >> 5) * PLANES * 64 + ((col >> 3) & 3) * 16 + row) * 8 + (col & 7);
    {
#pragma clang fp contract(off)   // the product is rounded before it is split, as by resid_kernel
        const float o = v * gn;
        const __bf16 head = static_cast<__bf16>(o);
        *f = __builtin_bit_cast(uint16_t, head);
        f[64 * 8] = __builtin_bit_cast(uint16_t, static_cast<__bf16>(o - static_cast<float>(head)));
    }
    double ss = (double)v * v;
#pragma unroll
    for (int s = 1; s < ADD_COLS; s *= 2) ss += __shfl_xor(ss, s);
    if (col == n0) parts[(size_t)row * n_tiles + blockIdx.x] = ss;
}

// ---- many rows ---------------------------------------------------------------------------------------------
// The product for more than 192 rows (and, at 97..128 rows, of matrices wide enough for four column tiles per wavefront, e.g. the
// LM head): a tile of 112..176 rows x 128..256 columns per workgroup, both operands fetched straight into LDS
// (global_load_lds: no registers on the way, so the accumulators of that many tiles fit eight wavefronts, two on every
// SIMD) through a ring of stages of one K block.
//
// What bounds it is the matrix instruction's rate together with the LDS reads that feed it: an X fragment read feeds NT
// products, and the two overlap only as far as the other wavefront of the SIMD has something to do.  The kernel above
// takes all rows in one workgroup, which leaves registers for two column tiles per wavefront (one LDS read per two
// products, and X, the larger operand by far, fetched anew for every 96 or 128 columns); two row blocks of half the rows
// take three or four, with W fetched twice.  7B shape, us per launch (QKV, gate/up, output, down, LM head), before and now:
//   256 rows  59.9 109.5 23.1 46.9 122.6    50.3  90.7 22.4 43.6 109.4
//   320       73.5 136.3 27.9 57.3 151.2    60.6 109.1 27.9 55.4 142.2
//   352       84.8 157.6 31.2 65.8 173.7    67.9 121.9 30.0 58.6 151.9   (1.04 PFLOP/s of issued products at QKV)
// (launches repeated, row blocks of 8, 10 and 12 tiles; means of a trace of nine single steps of 352 rows, QKV and gate/up: 91.4
// 170.3 before, 74.2 137.6 now)
// Row blocks of an odd number of tiles (7, 9, 11: the halves of a workgroup differ by one, and every SIMD gets one of each) are
// no longer multiplied as the next even one.  Steps of four layers, 208, 272, 288 and 352 rows: 7B shape 1124 -> 1102 us, 1307 ->
// 1276, 1348 -> 1294, 1519 -> 1490, 1B shape 632 -> 596, 721 -> 678, 742 -> 688, 804 -> 748.  Less than the products saved:
// at 352 rows a stage takes 1600-1700 cycles of which its products are 1060, the rest waiting for the slowest wavefront at the
// barrier, and a launch spends 14 us before the first stage and after the last (counters in a copy of the kernel).
// Tried: four wavefronts with 32x32x16 products (one per SIMD: fetching, LDS reads and products add up instead of overlapping,
// 85 and 158 us at 352 rows); fetching on two wavefronts of their own; from 65 to 192 rows, where W from memory is half of the
// time, this kernel and the one above are within 5 % of each other either way, except for the LM head at eight row tiles
// (71.6 -> 63.3).
//
// A stage: 2 MT X tiles of 1 KiB (head plane, remainder plane) and 4 NT W tiles, requested by all wavefronts alike, S - 1 stages
// ahead.  Stage i's products run while its last fragments and then stage i + 1's first ones are read: the barrier stands L tiles
// before a stage's end, where all of stage i is in registers (its slot is free) and stage i + 1 has landed.  The
// requests are not known to the compiler, which sees no load at all in this kernel; every wait is written here.
// (m0 is none of the registers that the compiler hands out, about which it warns; it may set m0 for an instruction of its own.)
#pragma clang diagnostic push
#pragma clang diagnostic ignored "-Winline-asm"
template <bool STREAM>
__device__ __forceinline__ void fetch_to_lds(const char* base, uint32_t offset, uint32_t lds)   // 16 bytes per lane, to lds + 16 * lane
{
    if constexpr (STREAM) asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %1, %2 nt" ::"s"(lds), "v"(offset), "s"(base) : "memory", "m0");
    else asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %1, %2" ::"s"(lds), "v"(offset), "s"(base) : "memory", "m0");
}
#pragma clang diagnostic pop
template <int N>
__device__ __forceinline__ void wait_fetches()   // at most N requests of this wavefront still under way
{
    static_assert(N < 64, "the counter has six bits");
    asm volatile("s_waitcnt vmcnt(%0)" ::"n"(N) : "memory");
}
__device__ __forceinline__ void wait_lds_reads() { asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory"); }
__device__ __forceinline__ void workgroup_barrier()
{
    __builtin_amdgcn_s_barrier();
    asm volatile("" ::: "memory");
}

constexpr int RING_GROUPS = 4;   // column groups of a workgroup; times two row halves: eight wavefronts
constexpr int ring_stages(int mt, int nt, int planes) { return 160 / (planes * mt + RING_GROUPS * nt) < 6 ? 160 / (planes * mt + RING_GROUPS * nt) : 6; }

// SwiGLU of sums that lie in LDS ([16 n_tiles rows][cols], rows ld floats apart), gate and up tiles of 16 columns in turn: a
// wavefront takes 16 rows x 32 results, whose fragments are contiguous (as silu_mul_kernel).  Row tile t of the sums is row
// tile row_tile(t) of the workgroup (negative: none), counted from row m0 on.
template <typename RowTile>
__device__ __forceinline__ void swiglu_from_lds(const float* sums, int ld, const float* row_scale, int n_tiles, int cols, int f0, int F, int m0, int M,
                                                int wave, int waves, int lane, const SwigluOut& so, RowTile row_tile)
{
    const int blocks = cols / 64, r16 = lane & 15, g = lane >> 4;
    for (int u = wave; u < n_tiles * blocks; u += waves) {
        const int t = u / blocks, fl = (u % blocks) * 32 + 8 * g, rt = row_tile(t);
        const int m = m0 + rt * 16 + r16;
        const float* p = sums + (t * 16 + r16) * ld + ((fl >> 4) << 5) + (fl & 15);
        float v[8];
        const float r = row_scale[max(rt, 0) * 16 + r16];
#pragma unroll
        for (int e = 0; e < 8; e += 4) {
            const float4 ga = *reinterpret_cast<const float4*>(p + e), up = *reinterpret_cast<const float4*>(p + 16 + e);
            const float gs[4] = {ga.x, ga.y, ga.z, ga.w}, us[4] = {up.x, up.y, up.z, up.w};
#pragma unroll
            for (int i = 0; i < 4; ++i) {
                const float ge = gs[i] * r;
                v[e + i] = ge / (1.f + expf(-ge)) * (us[i] * r);
            }
        }
        if (rt >= 0 && m < M && f0 + fl < F) store_x_unit(so.frags, so.mt, so.planes, m, (f0 + fl) >> 3, v);
    }
}

// STREAM: W by streaming loads (one row block: read once)
// SWIGLU (gate/up projection, single K range): the workgroup finishes SwiGLU and writes the down projection's operand; its sums go
// through LDS, where the ring was, because a wavefront's column tiles are no whole pairs and a fragment takes 32 columns.  7B
// shape, 352 rows: gate/up 122 -> 124 us, and the silu_mul_kernel of 12 us behind it gone (a step of four layers -3 %).
template <int MT, int NT, int PLANES, bool STREAM, bool SWIGLU>
__global__ void __launch_bounds__(512, 1) gemm_ring_kernel(const char* __restrict__ Xf, const char* __restrict__ Wp, float* __restrict__ partial,
                                                           int M, int mt, int n_tiles, int kb_total, int kb_per_split, int n_split,
                                                           int row_blocks, int n_blocks, SwigluOut so)
{
    constexpr int XT = PLANES * MT, ST = XT + RING_GROUPS * NT, U = (ST + 7) / 8;   // KiB tiles per stage; requests per wavefront
    constexpr int S = ring_stages(MT, NT, PLANES), L = 2;                            // read ahead, row tiles
    constexpr int G0 = (MT + 1) / 2, G1 = MT / 2;                                    // row tiles of the two halves
    static_assert(G1 > L && S >= 3, "tile shape");
    constexpr int GP = (G0 + 1) / 2, COLS = RING_GROUPS * NT * 16, LD = COLS + 4;   // SwiGLU: row tiles of a pass; its sums in LDS
    static_assert((2 * GP * 16 * LD + MT * 16) * 4 <= S * ST * 1024 && MT * 16 <= 512, "the sums of a pass fit the ring");
    __shared__ u32x4 lds[S * ST * 64];
    const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
    // Wavefronts i and i + 4 share a SIMD: they take different halves, so that an odd number of row tiles loads all SIMDs alike.
    // The halves of an odd number run two instantiations of `run` and meet in barriers of both: the hardware counts wavefronts, not
    // places in the code, and either half comes to as many -- one before the first stage, one a stage, and with SWIGLU two for
    // each of the ceil(G0 / GP) passes, also where the shorter half has no tile left.
    const int half = (MT % 2 ? wave ^ (wave >> 2) : wave) & 1, a0 = half * G0, group = wave >> 1;
    // row blocks of the same columns follow each other on one XCD (map_block's order otherwise): the second reads W from its L2
    const int x = blockIdx.x & 7, j = blockIdx.x >> 3;
    int split, nblk;
    map_block(x + 8 * (j / row_blocks), n_split, &split, &nblk);
    if (nblk >= n_blocks) return;
    const int t0 = (j % row_blocks) * MT, c0 = nblk * RING_GROUPS * NT;   // first row and column tile
    const int kb0 = split * kb_per_split, n = min(kb_per_split, kb_total - kb0);   // stages (none or less: an empty range)

    const uint32_t lds0 = (uint32_t)(uintptr_t)(__attribute__((address_space(3))) void*)lds + wave * 1024;
    const char* xbase = Xf + (size_t)kb0 * PLANES * mt * 1024;
    const char* wbase = Wp + (size_t)(kb0 / WPACK_KG) * n_tiles * (WPACK_KG * 1024) + (kb0 % WPACK_KG) * 1024;
    // tile 8 u + wave of a stage, rows and columns past the end the last ones again (never stored)
    uint32_t offset[U];
#pragma unroll
    for (int u = 0; u < U; ++u) {
        const int tile = min(u * 8 + wave, ST - 1);
        offset[u] = (tile < XT ? (uint32_t)((tile / MT) * mt + min(t0 + tile % MT, mt - 1)) * 1024u
                               : (uint32_t)min(c0 + tile - XT, n_tiles - 1) * (WPACK_KG * 1024u)) + lane * 16;
    }
    int requested = 0, slot_to = 0;
    auto request = [&](int u) {
        const uint32_t to = lds0 + (uint32_t)(slot_to * ST + u * 8) * 1024u;
        const int tile = u * 8 + wave;
        if (u * 8 + 8 <= XT || (u * 8 < XT && tile < XT)) fetch_to_lds<false>(xbase, offset[u], to);
        else if (u * 8 + 8 <= ST || tile < ST) fetch_to_lds<STREAM>(wbase, offset[u], to);
        else fetch_to_lds<false>(wave < XT ? xbase : wbase, offset[0], to - u * 8192u);   // (its first tile again: every wavefront counts U a stage)
    };
    auto advance = [&]() {
        xbase += (size_t)PLANES * mt * 1024;
        wbase += (kb0 + requested) % WPACK_KG == WPACK_KG - 1 ? (size_t)n_tiles * (WPACK_KG * 1024) - (WPACK_KG - 1) * 1024 : (size_t)1024;
        slot_to = slot_to + 1 == S ? 0 : slot_to + 1;
        ++requested;
    };
    auto landed = [&](int stage) {   // the stages up to this one
        if (requested - 1 - stage >= S - 2) wait_fetches<(S - 2) * U>();
        else wait_fetches<0>();
    };
    auto run = [&](auto tiles_of_half) {
        constexpr int G = decltype(tiles_of_half)::value;
        floatx4 acc[G][NT];
#pragma unroll
        for (int a = 0; a < G; ++a)
#pragma unroll
            for (int i = 0; i < NT; ++i) acc[a][i] = floatx4{0.f, 0.f, 0.f, 0.f};

        const u32x4* xl = lds + a0 * 64 + lane;
        const u32x4* wl = lds + (XT + group * NT) * 64 + lane;
        constexpr int R = 4;   // ring of X fragments in registers: tile g of a stage at g % R
        bf16x8 xh[R], xr[R], wf[2][NT];
        auto read_x = [&](int slot, int g, int at) {
            xh[at] = __builtin_bit_cast(bf16x8, xl[(slot * ST + g) * 64]);
            if constexpr (PLANES == 2) xr[at] = __builtin_bit_cast(bf16x8, xl[(slot * ST + MT + g) * 64]);
        };
        auto read_w = [&](int slot, int i) { return __builtin_bit_cast(bf16x8, wl[(slot * ST + i) * 64]); };
        float scale = 0.f;   // SwiGLU: of row threadIdx.x
        if (n > 0) {
            for (int i = min(n, S - 1); i > 0; --i) {
#pragma unroll
                for (int u = 0; u < U; ++u) request(u);
                advance();
            }
            // (behind the first requests, so that the wait for it costs nothing)
            if constexpr (SWIGLU) scale = row_inv_rms(so.ssq, so.n_ssq, min(t0 * 16 + (int)threadIdx.x, M - 1), so.d, so.eps);
            landed(0);
            workgroup_barrier();
            int stage = 0, slot = 0;
#pragma unroll
            for (int i = 0; i < NT; ++i) wf[0][i] = wf[1][i] = read_w(0, i);
#pragma unroll
            for (int g = 0; g < L; ++g) read_x(0, g, g);
            auto step = [&](auto set) {   // which of the two sets of W fragments the stage is in
                constexpr int cur = decltype(set)::value;
                const bool more = requested < n;
                const int next = slot + 1 == S ? 0 : slot + 1;
#pragma unroll
                for (int g = 0; g < G; ++g) {
                    if (g == G - L) {
                        if (more) advance();
                        wait_lds_reads();
                        landed(min(stage + 1, n - 1));
                        workgroup_barrier();
#pragma unroll
                        for (int i = 0; i < NT; ++i) wf[cur ^ 1][i] = read_w(next, i);   // (after the last stage: never used)
                    }
                    if (g + L < G) read_x(slot, g + L, (g + L) % R);
                    else read_x(next, g + L - G, (g + L) % R);
                    if (g < G - L && more) {
#pragma unroll
                        for (int u = g; u < U; u += G - L) request(u);
                    }
#pragma unroll
                    for (int i = 0; i < NT; ++i) acc[g][i] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(xh[g % R], wf[cur][i], acc[g][i], 0, 0, 0);
                    if constexpr (PLANES == 2) {
#pragma unroll
                        for (int i = 0; i < NT; ++i) acc[g][i] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(xr[g % R], wf[cur][i], acc[g][i], 0, 0, 0);
                    }
                    __builtin_amdgcn_sched_barrier(0);
                }
                if constexpr (G % R != 0) {   // the next stage's first fragments to where it looks for them
                    bf16x8 h[L], r[L];
#pragma unroll
                    for (int g = 0; g < L; ++g) { h[g] = xh[(G + g) % R]; r[g] = xr[(G + g) % R]; }
#pragma unroll
                    for (int g = 0; g < L; ++g) { xh[g] = h[g]; xr[g] = r[g]; }
                }
                slot = next;
                ++stage;
            };
            if (n & 1) step(std::integral_constant<int, 1>{});   // (both sets hold stage 0)
            while (stage < n) {
                step(std::integral_constant<int, 0>{});
                step(std::integral_constant<int, 1>{});
            }
            wait_lds_reads();
            wait_fetches<0>();
        }
        if constexpr (SWIGLU) {
            float* sums = reinterpret_cast<float*>(lds);
            float* scales = sums + 2 * GP * 16 * LD;
            const int g = lane >> 4, c = lane & 15;
#pragma unroll
            for (int p0 = 0; p0 < G0; p0 += GP) {   // (as many for either half)
                __syncthreads();   // everyone is done with the ring, and with the pass before
                if (p0 == 0 && (int)threadIdx.x < MT * 16) scales[threadIdx.x] = scale;
#pragma unroll
                for (int a = 0; a < GP; ++a)
                    if (p0 + a < G) {
#pragma unroll
                        for (int i = 0; i < NT; ++i)
#pragma unroll
                            for (int r = 0; r < 4; ++r)
                                sums[((half * GP + a) * 16 + 4 * g + r) * LD + (group * NT + i) * 16 + c] = acc[p0 + a][i][r];
                    }
                __syncthreads();
                swiglu_from_lds(sums, LD, scales, 2 * GP, COLS, nblk * (COLS / 2), n_tiles * 8, t0 * 16, M, wave, 8, lane, so, [&](int t) {
                    const int a = p0 + t % GP;
                    return a < (t < GP ? G0 : G1) ? (t / GP) * G0 + a : -1;
                });
            }
            return;
        }
        const int n_pad = n_tiles * 16, g4 = lane >> 4, c16 = lane & 15;
        float* out = partial + (size_t)split * M * n_pad;
#pragma unroll
        for (int a = 0; a < G; ++a)
#pragma unroll
            for (int i = 0; i < NT; ++i) {
                const int tile = c0 + group * NT + i;
                if (tile < n_tiles) {
#pragma unroll
                    for (int r = 0; r < 4; ++r) {
                        const int m = (t0 + a0 + a) * 16 + 4 * g4 + r;
                        if (m < M) out[(size_t)m * n_pad + tile * 16 + c16] = acc[a][i][r];
                    }
                }
            }
    };
    if (G0 == G1 || half == 0) run(std::integral_constant<int, G0>{});
    else run(std::integral_constant<int, G1>{});
}

// zero a fragment buffer (a kernel rather than a memset node, so that the call can be captured in a graph)
__global__ void __launch_bounds__(256) zero_kernel(uint4* __restrict__ p, size_t n)
{
    for (size_t i = (size_t)blockIdx.x * 256 + threadIdx.x; i < n; i += (size_t)gridDim.x * 256) p[i] = make_uint4(0, 0, 0, 0);
}

// fp32 row-major X[M][K] (optionally times gain[K]) -> fragment buffer
__global__ void __launch_bounds__(256) pack_x_kernel(const float* __restrict__ X, const float* __restrict__ gain, int M,
                                                     int K, int mt_count, int planes, uint4* __restrict__ xf)
{
    const int units = K / 8;
    for (int i = blockIdx.x * 256 + threadIdx.x; i < M * units; i += gridDim.x * 256) {
        const int m = i / units, k8 = i % units;
        const float4 a = *reinterpret_cast<const float4*>(X + (size_t)m * K + k8 * 8);
        const float4 b = *reinterpret_cast<const float4*>(X + (size_t)m * K + k8 * 8 + 4);
        float v[8] = {a.x, a.y, a.z, a.w, b.x, b.y, b.z, b.w};
        if (gain)
#pragma unroll
            for (int e = 0; e < 8; ++e) v[e] *= gain[k8 * 8 + e];
        store_x_unit(xf, mt_count, planes, m, k8, v);
    }
}

// The product for the small fp32 configurations, on the fp32 matrix instruction (v_mfma_f32_16x16x4_f32).  These
// calls are a handful of rows against matrices of a megabyte: what bounds them is the number of dependent memory
// round trips, so one workgroup takes a 16-column block of W over ALL of K -- eight wavefronts with interleaved
// 32-column slabs, every load of four slabs requested before the first product, sums met in LDS -- and does
// what its neighbours in the chain would need a launch for: the norm of its input (x * gain is multiplied, the row's
// 1/rms, formed from the very columns that pass by, scales the result), the residual addition, SwiGLU.
// At d = 256 with 5 rows a product took 8.9-32 us (15.8 on average) with K in 8-32 dependent slabs of 32 through LDS, 4.1
// this way; with the launches that it takes over (a step of that model had 29, now 18) the step went from 256 to 83 us.
typedef float f32x4u __attribute__((ext_vector_type(4), aligned(4)));   // global memory takes 16-byte accesses at any 4-byte address
constexpr int F32_WAVES = 8;

// MT row tiles of 16, NT column tiles: 2 for F32_SWIGLU (a gate tile and its up tile, N rows of W further on)
template <int MT, int NT, bool NORM>
__global__ void __launch_bounds__(64 * F32_WAVES) gemm_f32_kernel(const float* __restrict__ X, const float* __restrict__ W,
                                                                  const float* __restrict__ gain, float eps, int mode,
                                                                  float* __restrict__ Y, int M, int N, int K)
{
    constexpr int SLAB = 32, AHEAD = MT * NT <= 2 ? 4 : 2;   // slabs whose loads are requested together
    __shared__ float red[F32_WAVES][MT * NT][256];
    __shared__ double ss_part[F32_WAVES][MT * 16];
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const int r16 = lane & 15, g = lane >> 4;
    const int n0 = blockIdx.x * 16, m0 = blockIdx.y * (MT * 16);
    const float* xrow[MT];
    const float* wrow[NT];
#pragma unroll
    for (int a = 0; a < MT; ++a) xrow[a] = X + (size_t)min(m0 + a * 16 + r16, M - 1) * K + 4 * g;
#pragma unroll
    for (int t = 0; t < NT; ++t) wrow[t] = W + (size_t)(min(n0 + r16, N - 1) + t * N) * K + 4 * g;
    floatx4 acc[MT][NT];
    double ss[MT];
#pragma unroll
    for (int a = 0; a < MT; ++a) {
        ss[a] = 0.0;
#pragma unroll
        for (int t = 0; t < NT; ++t) acc[a][t] = floatx4{0.f, 0.f, 0.f, 0.f};
    }
    // four consecutive columns from p + k on; beyond K zeros (both operands, so nothing is added there)
    auto load4 = [&](const float* p, int k) -> floatx4 {
        if (k + 4 * g + 4 <= K) {
            const f32x4u v = *reinterpret_cast<const f32x4u*>(p + k);
            return floatx4{v.x, v.y, v.z, v.w};
        }
        floatx4 v = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
        for (int e = 0; e < 4; ++e)
            if (k + 4 * g + e < K) v[e] = p[k + e];
        return v;
    };
    auto full4 = [](const float* p) -> floatx4 {
        const f32x4u v = *reinterpret_cast<const f32x4u*>(p);
        return floatx4{v.x, v.y, v.z, v.w};
    };
    auto multiply = [&](const floatx4 (&x)[MT], const floatx4 (&w)[NT], const floatx4& gn) {
#pragma unroll
        for (int a = 0; a < MT; ++a) {
            if constexpr (NORM) {
#pragma unroll
                for (int e = 0; e < 4; ++e) ss[a] += (double)x[a][e] * x[a][e];
            }
#pragma unroll
            for (int e = 0; e < 4; ++e)
#pragma unroll
                for (int t = 0; t < NT; ++t)
                    acc[a][t] = __builtin_amdgcn_mfma_f32_16x16x4f32(NORM ? x[a][e] * gn[e] : x[a][e], w[t][e], acc[a][t], 0, 0, 0);
        }
    };
    const int stride = F32_WAVES * SLAB;
    int k = wave * SLAB;
    const floatx4 one = {1.f, 1.f, 1.f, 1.f};
    for (; k + (AHEAD - 1) * stride + SLAB <= K; k += AHEAD * stride) {
        floatx4 x[AHEAD][2][MT], w[AHEAD][2][NT], gn[AHEAD][2];
#pragma unroll
        for (int i = 0; i < AHEAD; ++i)
#pragma unroll
            for (int h = 0; h < 2; ++h) {
                const int kk = k + i * stride + 16 * h;
#pragma unroll
                for (int t = 0; t < NT; ++t) w[i][h][t] = full4(wrow[t] + kk);
#pragma unroll
                for (int a = 0; a < MT; ++a) x[i][h][a] = full4(xrow[a] + kk);
                gn[i][h] = NORM ? full4(gain + 4 * g + kk) : one;
            }
#pragma unroll
        for (int i = 0; i < AHEAD; ++i)
#pragma unroll
            for (int h = 0; h < 2; ++h) multiply(x[i][h], w[i][h], gn[i][h]);
    }
    for (; k < K; k += stride) {
        floatx4 x[2][MT], w[2][NT], gn[2];
#pragma unroll
        for (int h = 0; h < 2; ++h) {
            const int kk = k + 16 * h;
#pragma unroll
            for (int t = 0; t < NT; ++t) w[h][t] = load4(wrow[t], kk);
#pragma unroll
            for (int a = 0; a < MT; ++a) x[h][a] = load4(xrow[a], kk);
            gn[h] = NORM ? load4(gain + 4 * g, kk) : one;
        }
#pragma unroll
        for (int h = 0; h < 2; ++h) multiply(x[h], w[h], gn[h]);
    }
#pragma unroll
    for (int a = 0; a < MT; ++a) {
#pragma unroll
        for (int t = 0; t < NT; ++t)
#pragma unroll
            for (int r = 0; r < 4; ++r) red[wave][a * NT + t][(4 * g + r) * 16 + r16] = acc[a][t][r];
        if constexpr (NORM) {
            ss[a] += __shfl_xor(ss[a], 16);
            ss[a] += __shfl_xor(ss[a], 32);
            if (g == 0) ss_part[wave][a * 16 + r16] = ss[a];
        }
    }
    __syncthreads();
    for (int i = threadIdx.x; i < MT * 256; i += 64 * F32_WAVES) {
        const int a = i >> 8, row = (i >> 4) & 15, col = i & 15;
        const int m = m0 + a * 16 + row, n = n0 + col;
        float v[NT];
#pragma unroll
        for (int t = 0; t < NT; ++t) {
            v[t] = 0.f;
#pragma unroll
            for (int w = 0; w < F32_WAVES; ++w) v[t] += red[w][a * NT + t][i & 255];
        }
        if constexpr (NORM) {
            double sum = 0.0;
#pragma unroll
            for (int w = 0; w < F32_WAVES; ++w) sum += ss_part[w][a * 16 + row];
            const float inv = 1.0f / sqrtf((float)sum / (float)K + eps);
#pragma unroll
            for (int t = 0; t < NT; ++t) v[t] *= inv;
        }
        if (m < M && n < N) {
            float* y = Y + (size_t)m * N + n;
            if constexpr (NT == 2) *y = v[0] / (1.f + expf(-v[0])) * v[1];
            else *y = mode == F32_ADD ? *y + v[0] : v[0];
        }
    }
}

__global__ void __launch_bounds__(256) pack_weight_kernel(const uint16_t* __restrict__ src, uint4* __restrict__ dst,
                                                          int n_out, int n_in, int n_tiles, int interleave)
{
    const int kb_total = n_in / 32;
    const int kb_pad = (kb_total + WPACK_KG - 1) / WPACK_KG * WPACK_KG;
    const size_t total = (size_t)n_tiles * kb_pad * 64;
    for (size_t i = (size_t)blockIdx.x * 256 + threadIdx.x; i < total; i += (size_t)gridDim.x * 256) {
        // i = ((group * n_tiles + tile) * WPACK_KG + block in group) * 64 + lane
        const int lane = (int)(i & 63);
        size_t r = i >> 6;
        const int kbi = (int)(r % WPACK_KG); r /= WPACK_KG;
        const int j = (int)(r % n_tiles);
        const int kb = (int)(r / n_tiles) * WPACK_KG + kbi;
        int row = j * 16 + (lane & 15);
        if (interleave) row = ((j & 1) ? n_out / 2 : 0) + (j >> 1) * 16 + (lane & 15);
        uint4 v = make_uint4(0, 0, 0, 0);
        if (row < n_out && kb < kb_total)
            v = *reinterpret_cast<const uint4*>(src + (size_t)row * n_in + kb * 32 + (lane >> 4) * 8);
        dst[i] = v;
    }
}

template <int MT, int NT, int KC, int RS, int CG>
int launch_groups(const GemmPlan& p, const void* xf, const void* w, int M, int K, int n_tiles, float* partial,
                  hipStream_t s, const SsqTiles* job, int n_ssq)
{
    const int n_blocks = (n_tiles + CG * NT - 1) / (CG * NT);
    int grid = n_blocks * p.n_split;
    if (p.n_split < 8) grid = (n_blocks + (8 / p.n_split) - 1) / (8 / p.n_split) * 8;
    SwigluOut so{};
    if (job) {   // (one row tile)
        so.tiles = *job;
        so.n_ssq = n_ssq;
        grid += 8;
    }
    if (p.planes == 2)
        hipLaunchKernelGGL((gemm_skinny_kernel<MT, NT, KC, 2, RS, 0, CG>), dim3(grid), dim3(64 * CG * RS), 0, s, (const u32x4*)xf,
                           (const u32x4*)w, partial, M, n_tiles, K / 32, p.kb_per_split, p.n_split, n_blocks, so);
    else
        hipLaunchKernelGGL((gemm_skinny_kernel<MT, NT, KC, 1, RS, 0, CG>), dim3(grid), dim3(64 * CG * RS), 0, s, (const u32x4*)xf,
                           (const u32x4*)w, partial, M, n_tiles, K / 32, p.kb_per_split, p.n_split, n_blocks, so);
    SPECV_LAUNCH_CHECK("gemm_skinny_kernel");
    return SPEC_OK;
}

template <int MT, int NT, int KC, int RS = 1>
int launch_variant(const GemmPlan& p, const void* xf, const void* w, int M, int K, int n_tiles, float* partial,
                   hipStream_t s, const SsqTiles* job, int n_ssq)
{
    if constexpr (RS == 2 || (MT <= 4 && NT == 2)) {
        if (p.cg == 3) return launch_groups<MT, NT, KC, RS, 3>(p, xf, w, M, K, n_tiles, partial, s, job, n_ssq);
    }
    if constexpr (MT <= 4 && NT == 2) {
        if (p.cg == 2) return launch_groups<MT, NT, KC, RS, 2>(p, xf, w, M, K, n_tiles, partial, s, job, n_ssq);
    }
    if constexpr (MT == 8 && NT == 4) return fail(SPEC_ERR_SHAPE, "eight row tiles by four column tiles in four groups: gemm_ring_kernel's");
    else return launch_groups<MT, NT, KC, RS, 4>(p, xf, w, M, K, n_tiles, partial, s, job, n_ssq);
}

template <int MT, int NT, bool STREAM>
int launch_ring(const GemmPlan& p, const void* xf, const void* w, int M, int K, int n_tiles, float* partial, hipStream_t s, const SwigluOut* swiglu)
{
    const int row_blocks = gemm_row_blocks(p), n_blocks = (n_tiles + RING_GROUPS * NT - 1) / (RING_GROUPS * NT);
    int grid = n_blocks * p.n_split;
    if (p.n_split < 8) grid = (n_blocks + (8 / p.n_split) - 1) / (8 / p.n_split) * 8;   // (a multiple of eight either way)
    auto* k = swiglu ? gemm_ring_kernel<MT, NT, 2, false, true>
                     : p.planes == 2 ? gemm_ring_kernel<MT, NT, 2, STREAM, false> : gemm_ring_kernel<MT, NT, 1, STREAM, false>;
    hipLaunchKernelGGL(k, dim3(grid * row_blocks), dim3(512), 0, s, (const char*)xf, (const char*)w, partial, M, p.mt, n_tiles, K / 32,
                       p.kb_per_split, p.n_split, row_blocks, n_blocks, swiglu ? *swiglu : SwigluOut{});
    SPECV_LAUNCH_CHECK("gemm_ring_kernel");
    return SPEC_OK;
}

struct Variant {
    int mt, nt, kc;   // row tiles, column tiles per wave, K blocks per LDS chunk
};
// row tiles -> (column tiles per wave, K blocks per LDS chunk); LDS = 2 buffers * planes * mt * kc KiB.
// Up to 4 row tiles there is a second, wider variant (4 column tiles per wave, 2 K blocks per
// chunk) for matrices with many columns.
// From 6 row tiles on the matrix cores and the LDS reads of X start to matter: several column tiles
// per wave (each X fragment read from LDS feeds that many products) keep LDS traffic per W byte down.
// From 8 row tiles on the workgroup has eight wavefronts (two row halves) and the three-buffer
// pipeline of one K block per chunk (see the kernel): both measured slower at 6 row tiles (88
// rows), faster from 8 on (120 rows -6 %, 160 -7 %, 250 and 320 -20 %).  Those variants come in
// even row-tile counts only: the two row halves of a workgroup take ceil(mt/2) tiles each, so an
// odd count costs what the next even one does.
// (14 row tiles and more: gemm_ring_kernel, see plan_ring; even counts here too, for its two row blocks.)
constexpr Variant kVariants[] = {{1, 2, 4}, {2, 2, 4}, {3, 2, 4}, {4, 2, 2}, {5, 4, 2}, {6, 4, 2},
                                 {8, 4, 1}, {10, 4, 1}, {12, 4, 1}, {14, 3, 1}, {16, 3, 1}, {18, 3, 1},
                                 {20, 3, 1}, {22, 3, 1}};
constexpr int kWideMaxMt = 4;
// column tiles from which the wide variant is taken (up to 4 row tiles) and below which 5-12 row tiles
// take two tiles per wavefront.  The wide variant fills the chip from 340 tiles on, but between that
// and 1000 tiles (the 7B-shape QKV projection: 768) the narrow one does with half the K ranges -- half
// the partial sums for the attention kernel to add up: step 5.088 -> 5.057 ms, decoding round with the
// configuration's draft (QKV of 384 tiles) 7.15 -> 7.07 ms.
constexpr int kWideMinTiles = 340;
constexpr int kWideMinTilesFewRows = 1000;

const Variant* pick_variant(int M)
{
    const int mt = (M + 15) / 16;
    for (const Variant& v : kVariants)
        if (v.mt >= mt) return &v;
    return nullptr;
}

int g_wg_target = 0;   // workgroups per launch to aim for; 0 = two thirds of the compute units
int g_balance_groups = 1;   // many-row launches: four column groups of three tiles instead of three of four

}  // namespace

void set_gemm_wg_target(int t) { g_wg_target = t; }

int gemm_row_tiles(int M)
{
    const Variant* v = pick_variant(M);
    return v ? v->mt : 0;
}

// K ranges are whole K groups of the packed order, so cutting a short K too finely leaves ranges with nothing in them --
// workgroups that only write zeros for the consumer to add; no cut that leaves more than one range in eight empty.
static int blocks_per_range(int kb_total, int n) { return ((kb_total + n - 1) / n + WPACK_KG - 1) / WPACK_KG * WPACK_KG; }
static bool ranges_have_work(int kb_total, int n)
{
    const int per = blocks_per_range(kb_total, n);
    return (kb_total + per - 1) / per * 8 >= n * 7;
}

// Launch shape of gemm_ring_kernel: two row blocks of half the row tiles each; column tiles per wavefront and K ranges by the
// cheapest of what fits, counted in cycles: rounds of workgroups over the chip x stages x a stage's time -- its matrix
// instructions (32 cycles per pair of tiles and SIMD) plus 0.6 of its LDS reads -- plus, per range, writing the partial sums and
// reading them back.  (By row tiles, not rows: the space for the partial sums is reserved by row tiles.)  Calibrated on the 7B, 1B and 2048-wide shapes at 256, 320 and 352 rows, where it picks the best of
// the shapes measured or one within 3 % of it: QKV of the 7B shape three tiles and two ranges (256 workgroups), gate/up three
// and one (230), output two and four, down (K = 11008) four and eight, LM head four and one (250).
static void plan_ring(GemmPlan& p, int n_tiles, int kb_total, int cu_count)
{
    p.ring = p.mt / 2;
    p.cg = RING_GROUPS;
    auto may_cut = [&](int s) { return blocks_per_range(kb_total, s) >= 2 * WPACK_KG && ranges_have_work(kb_total, s); };
    double best = 0.0;
    for (int nt = 2; nt <= 4; ++nt)
        for (int s = 1; s <= 16; s *= 2) {
            if (s > 1 && !may_cut(s)) break;
            const int wgs = (n_tiles + RING_GROUPS * nt - 1) / (RING_GROUPS * nt) * 2 * s;
            // a workgroup target that the caller set: the fewest ranges that reach it, or as many as the shape allows
            if (g_wg_target > 0 && wgs < g_wg_target && s < 16 && may_cut(2 * s)) continue;
            const int rounds = (wgs + cu_count - 1) / cu_count;
            const double stage = 32.0 * p.ring * nt + 0.6 * 64.0 * (p.ring + nt);
            const double cost = rounds * blocks_per_range(kb_total, s) * stage + 0.0025 * s * p.mt * 16 * p.n_pad;
            if (best == 0.0 || cost < best) {
                best = cost;
                p.nt = nt;
                p.n_split = s;
            }
            if (g_wg_target > 0) break;
        }
    p.kb_per_split = blocks_per_range(kb_total, p.n_split);
}

GemmPlan plan_gemm(int M, int N, int K, int cu_count, bool split_x)
{
    GemmPlan p{};
    const Variant* v = pick_variant(M);
    p.mt = v ? v->mt : 0;
    p.nt = v ? v->nt : 1;
    p.planes = split_x ? 2 : 1;
    int kc = v ? v->kc : 4;
    p.n_pad = (N + 15) / 16 * 16;
    const int n_tiles = p.n_pad / 16;
    if (p.mt <= kWideMaxMt && n_tiles >= kWideMinTilesFewRows) {
        p.nt = 4;
        kc = 2;
    }
    // 5 to 12 row tiles and few columns (the 4096-column output and down projections): two column tiles
    // per wavefront instead of four -- twice the column blocks, so half the K ranges fill the chip and
    // half the partial sums are written and read back (16 ranges x 157 rows x 4096 columns were 41 MB
    // against 33.5 MB of weights).  Costs LDS reads per product, gains more: step -3 % at 88 rows,
    // projections and their consumers -0.3 ms of 6.6 at 157 rows.
    if (p.mt >= 5 && p.mt <= 12 && n_tiles < kWideMinTiles) p.nt = 2;
    p.cg = 4;
    p.rs = p.mt >= 8 ? 2 : 1;
    const int kb_total = K / 32;
    if (p.mt >= 14) {
        plan_ring(p, n_tiles, kb_total, cu_count);
        return p;
    }
    // K ranges: a power of two, just enough of them that the launch has about `target` workgroups.
    // Measured on MI355X: every launch pays a few microseconds of ramp-up and tail whatever its
    // size, and long-lived workgroups stream best, so fewer, longer ranges win as long as roughly
    // two thirds of the compute units have a workgroup; more ranges only add partial-sum traffic
    // (M*N*4 bytes each way per range).  At most 16 ranges, each at least two LDS chunks long.
    const int target = g_wg_target > 0 ? g_wg_target : (2 * cu_count) / 3;
    auto ranges_for = [&](int blocks_x) {
        int n = 1;
        while (n < 16 && blocks_x * n < target && (kb_total + 2 * n - 1) / (2 * n) >= 2 * kc
               && ranges_have_work(kb_total, 2 * n))
            n *= 2;
        return n;
    };
    // Few rows and few columns (up to four row tiles, under 340 column tiles: the 4096-column projections, a small
    // model's QKV): two column groups per workgroup.  Twice the column blocks fill the chip with half the K ranges,
    // i.e. half the partial sums for the launch to write and for its consumer to add up, and two wavefronts per
    // compute unit stream as fast as four (stand-alone read of 33 and 90 MB: 4.7 and 5.8 TB/s either way).  1B-shape
    // step 0.884 -> 0.850 ms (its attention adds up four QKV ranges instead of eight), batch 8 1.242 -> 1.205,
    // decoding round -0.3 %.  Only while a workgroup's K range stays within 2048: a workgroup stages all rows of
    // X over its range, and at 2752 (the 7B-shape down projection in four ranges) the launch was 1.7 us slower,
    // as much as its consumers gained; at 2048 (K = 8192) and below it costs the launch nothing.
    if (p.mt <= 4 && p.nt == 2 && n_tiles < kWideMinTiles) {
        const int n2 = ranges_for((n_tiles + 2 * p.nt - 1) / (2 * p.nt));
        if ((kb_total + n2 - 1) / n2 * 32 <= 2048) p.cg = 2;
    }
    // The same for wider matrices from 8 row tiles on, where the partial sums, written and read back (8 bytes per column
    // for each range and row), move at least as much as the weights (2 K bytes).  Measured in steps of three layers with
    // two tiles per wavefront against four, 113, 128, 176 and 192 rows: models 1024 wide -0.4..-5.9 %, 1536 -1.4..-3.1,
    // 2048 (FFN 5504 and 8192) -2.6..-7.6, 2560 -3.4..-6.4, 3072 -1.8..-4.5.  At K = 4096 (0.5 to 0.75 times the weights: the
    // 7B-shape QKV) it costs 0.3 to 1.0 % and is not made.
    if (p.mt >= 8 && p.nt == 4) {
        const int s4 = ranges_for((n_tiles + 15) / 16);
        if (8 * s4 * 16 * p.mt >= 2 * K && ranges_for((n_tiles + 7) / 8) < s4) p.nt = 2;
    }
    const int wg_x = (n_tiles + p.cg * p.nt - 1) / (p.cg * p.nt);
    const int s = ranges_for(wg_x);
    p.n_split = s;
    // Few rows, two column tiles per wavefront: three column groups per workgroup where four leave more than a
    // fifth of the compute units without a workgroup and three fill them (7B-shape QKV: 192 workgroups of four
    // wavefronts -> 256 of three).  A read stream of that size (100 MB) runs 10 % faster from 256 workgroups than
    // from 192, and since the weights are fetched with streaming loads the GEMM follows: QKV 25.5 -> 22.5 us per
    // launch, 7B-shape step 4.915 -> 4.853 ms, 1B-shape 0.897 -> 0.884, decoding round 6.67 -> 6.58 ms (before the
    // streaming loads the same change gained nothing).  With four tiles per wavefront or five to seven row tiles
    // it is mixed (72 rows -1 %, 88-96 rows +1.3..1.6 % per step) and is not made.
    if (p.mt <= 4 && p.nt == 2) {
        const int wg3 = (n_tiles + 3 * p.nt - 1) / (3 * p.nt) * s;
        if (p.cg == 4 && wg_x * s * 5 < cu_count * 4 && wg3 <= cu_count) p.cg = 3;
    }
    // Many rows (the eight-wavefront variants): the matrix instructions set the pace, so compute units
    // without a workgroup are lost time; three column groups per workgroup instead of four when that
    // brings the launch from under four fifths of the compute units to at most all of them
    // (157 rows: QKV 192 -> 256 workgroups, gate/up 172 -> 230; GEMM time of that step -6 %).
    if (p.mt >= 8 && p.rs == 2) {
        const int wg3 = (n_tiles + 3 * p.nt - 1) / (3 * p.nt) * s;
        if (wg_x * s * 5 < cu_count * 4 && wg3 <= cu_count) {
            // Twelve column tiles per workgroup either way; as four column groups of three tiles the
            // workgroup keeps eight wavefronts, two on every SIMD, where three groups of four tiles
            // put two wavefronts on two SIMDs and one on the others (the loaded ones set the pace).
            if (p.nt == 4 && g_balance_groups) p.nt = 3;
            else p.cg = 3;
        }
    }
    // Five and six row tiles: the same, as four column groups of three tiles (7B-shape, 88 rows: QKV 192 -> 256
    // workgroups, gate/up 172 -> 230).  Steps of three layers with and without, 72, 88 and 96 rows: 7B shape -1.2..-1.4 %,
    // 2048 wide with an FFN of 5504 -1.7..-2.4, 1536 wide -1.9..-2.6; 1024, 2560 and 3072 wide and an FFN of 8192, where it is
    // not made or changes little, within 0.5 %.
    if (p.mt >= 5 && p.mt <= 6 && p.nt == 4) {
        const int wg3 = (n_tiles + 4 * 3 - 1) / (4 * 3) * s;
        if (wg_x * s * 5 < cu_count * 4 && wg3 <= cu_count) p.nt = 3;
    }
    // ranges start on a K group of the packed order so that every chunk is one contiguous run
    p.kb_per_split = blocks_per_range(kb_total, s);
    // eight row tiles with four column tiles per wavefront (the LM head): one row block of the ring (32000 x 4096 at 128 rows
    // 71.6 -> 63.3 us, 112 rows 72.5 -> 62.4; with three tiles per wavefront or ten and twelve row tiles no difference)
    if (p.mt == 8 && p.nt == 4 && p.cg == 4) p.ring = 8;
    return p;
}

size_t gemm_partial_elems(const GemmPlan& p, int M) { return (size_t)p.n_split * M * p.n_pad; }

static int launch_ring_plan(const GemmPlan& p, const void* x_frags, const void* w_packed, int M, int N, int K, float* partial, hipStream_t s,
                            const SwigluOut* swiglu)
{
    const int n_tiles = (N + 15) / 16;
#define SPECV_RING(MT_, NT_, STREAM_)                                                                              \
    if (p.ring == MT_ && p.nt == NT_ && (p.mt <= MT_) == STREAM_) return launch_ring<MT_, NT_, STREAM_>(p, x_frags, w_packed, M, K, n_tiles, partial, s, swiglu)
    SPECV_RING(8, 4, true);
    SPECV_RING(7, 2, false);
    SPECV_RING(7, 3, false);
    SPECV_RING(7, 4, false);
    SPECV_RING(8, 2, false);
    SPECV_RING(8, 3, false);
    SPECV_RING(8, 4, false);
    SPECV_RING(9, 2, false);
    SPECV_RING(9, 3, false);
    SPECV_RING(9, 4, false);
    SPECV_RING(10, 2, false);
    SPECV_RING(10, 3, false);
    SPECV_RING(10, 4, false);
    SPECV_RING(11, 2, false);
    SPECV_RING(11, 3, false);
    SPECV_RING(11, 4, false);
#undef SPECV_RING
    return fail(SPEC_ERR_SHAPE, "no GEMM variant for %d rows (%d row tiles, %d column tiles per wave)", M, p.mt, p.nt);
}

int launch_gemm_bf16(const GemmPlan& p, const void* x_frags, const void* w_packed, int M, int N, int K, float* partial,
                     hipStream_t s, const SsqTiles* job, int n_ssq)
{
    if (job && p.mt != 1) return fail(SPEC_ERR_SHAPE, "row sums by column tiles are for one row tile, got %d", p.mt);
    if (M < 1 || M > GEMM_MAX_ROWS) return fail(SPEC_ERR_SHAPE, "GEMM supports 1..%d rows, got %d", GEMM_MAX_ROWS, M);
    if (K % 32) return fail(SPEC_ERR_SHAPE, "GEMM needs K %% 32 == 0, got %d", K);
    const int n_tiles = (N + 15) / 16;
    if (p.ring) return launch_ring_plan(p, x_frags, w_packed, M, N, K, partial, s, nullptr);
#define SPECV_GEMM(MT_, NT_, KC_, ...)                                                                  \
    if (p.mt == MT_ && p.nt == NT_ && p.rs == (1, ##__VA_ARGS__))                                         \
        return launch_variant<MT_, NT_, KC_, ##__VA_ARGS__>(p, x_frags, w_packed, M, K, n_tiles, partial, s, job, n_ssq)
    SPECV_GEMM(1, 4, 2);
    SPECV_GEMM(2, 4, 2);
    SPECV_GEMM(3, 4, 2);
    SPECV_GEMM(4, 4, 2);
    SPECV_GEMM(1, 2, 4);
    SPECV_GEMM(2, 2, 4);
    SPECV_GEMM(3, 2, 4);
    SPECV_GEMM(4, 2, 2);
    SPECV_GEMM(5, 2, 2);
    SPECV_GEMM(6, 2, 2);
    SPECV_GEMM(5, 3, 2);
    SPECV_GEMM(6, 3, 2);
    SPECV_GEMM(5, 4, 2);
    SPECV_GEMM(6, 4, 2);
    SPECV_GEMM(8, 2, 1, 2);
    SPECV_GEMM(10, 2, 1, 2);
    SPECV_GEMM(12, 2, 1, 2);
    SPECV_GEMM(8, 3, 1, 2);
    SPECV_GEMM(10, 3, 1, 2);
    SPECV_GEMM(12, 3, 1, 2);
    SPECV_GEMM(8, 4, 1, 2);
    SPECV_GEMM(10, 4, 1, 2);
    SPECV_GEMM(12, 4, 1, 2);
#undef SPECV_GEMM
    return fail(SPEC_ERR_SHAPE, "no GEMM variant for %d rows (%d row tiles, %d column tiles per wave)", M, p.mt, p.nt);
}

// Where the residual product is the faster route, from steps of six and eight layers with and without it: widths 512 to 8192, K
// 1024 to 6144, 1 to 16 rows.  What tells against it:
//  * The reads of X, which every workgroup makes, grow with K.  Up to eight rows they take one 128-byte line per 8 columns of K and
//    plane, from nine on two.
//  * More than four ranges means a narrow matrix: few workgroups (a column tile each), each with a long stream to read.
//  * In front of the product that finishes SwiGLU (sums_again) the row sums are added up by every workgroup of it.
//  * More workgroups than compute units: steps of 5120 wide models 0.6 to 3.1 % slower, of 6144 by 6144 2.5 to 9 %.
// Gain of the step at the longest K taken, and at the next one measured (in brackets):
//                 up to 8 rows                                          9 to 16 rows
//   4 ranges      6144 +4..+5.5 % (not measured beyond)                 6144 0..+0.6
//   8             6144 +0.2..+0.9                                       3072 +1.2..+2.2 (4096 -0.3..-1.1, 5504 -1.8)
//   16            6144 -0.3..+0.5                                       4096 -0.1..+1.6 (6144 -5)
//   sums_again, 4 6144 +1..+2.2                                         3072 +0.3..+0.9 (4096 -0.4..-0.8)
//   8 and 16      4096 +0.6..+1.8 (5120 -0.9..-1.3, 6144 -0.8..-2.7)    2048 +0.6..+1.5 (3072 -0.7..+0.5)
bool gemm_add_fits(const GemmPlan& p, int M, int K, int cu_count, bool sums_again)
{
    if (p.mt != 1 || p.planes != 2 || p.n_pad % 32 || p.n_pad / ADD_COLS > cu_count) return false;
    if (p.n_split != 4 && p.n_split != 8 && p.n_split != 16) return false;
    if (sums_again) return K <= (p.n_split == 4 ? 6144 : 4096) / (M <= 8 ? 1 : 2);
    return K <= (M <= 8 || p.n_split == 4 ? 6144 : p.n_split == 8 ? 3072 : 4096);
}

int launch_gemm_add(const GemmPlan& p, const void* x_frags, const void* w_packed, int M, int d, int K, float* x, const float* gain,
                    void* out_frags, double* parts, hipStream_t s)
{
    if (!gemm_add_fits(p, M, K, d / ADD_COLS, false) || M < 1 || M > 16 || d != p.n_pad || K % 32 || K < 32)
        return fail(SPEC_ERR_SHAPE, "no residual GEMM for %d rows of %d x %d", M, d, K);
#define SPECV_ADD(R_)                                                                                                          \
    if (p.n_split == R_) {                                                                                                     \
        hipLaunchKernelGGL(gemm_add_kernel<R_>, dim3(d / ADD_COLS), dim3(64 * R_), 0, s, (const u32x4*)x_frags, (const u32x4*)w_packed, \
                           x, gain, M, d / 16, K / 32, p.kb_per_split, (uint16_t*)out_frags, parts);                           \
    }
    SPECV_ADD(4)
    SPECV_ADD(8)
    SPECV_ADD(16)
#undef SPECV_ADD
    SPECV_LAUNCH_CHECK("gemm_add_kernel");
    return SPEC_OK;
}

namespace {
int g_swiglu_min_wgs = 0;   // 0: a third of the compute units
int g_swiglu_cg = 0;        // 0: chosen by swiglu_column_groups; 2, 3, 4: forced (tests)
}
void set_swiglu_min_wgs(int n) { g_swiglu_min_wgs = n; }
void set_swiglu_column_groups(int n) { g_swiglu_cg = n >= 2 && n <= 4 ? n : 0; }

// The gate/up projection can finish SwiGLU itself when it runs as ONE K range of 128-column
// workgroups (narrow variants, up to 4 row tiles) and that still gives enough workgroups.
bool gemm_swiglu_fits(int M, int F, int cu_count)
{
    const int mt = gemm_row_tiles(M);
    if (mt < 1 || mt > 4 || F % 16) return false;   // (6 row tiles measured, with four and with three wavefronts per workgroup: the narrow GEMM loses more than the kernel saved)
    const int wgs = (2 * F / 16 + 7) / 8;
    // measured: 172 workgroups (F = 11008) step -1.9 %, 128 workgroups (F = 8192) -3.5 %
    return wgs >= (g_swiglu_min_wgs > 0 ? g_swiglu_min_wgs : cu_count / 3);
}

// So does the many-row kernel wherever its launch has a single K range.
bool gemm_ring_swiglu_fits(const GemmPlan& p) { return p.ring && p.mt >= 14 && p.n_split == 1; }

template <int MT, int KC, int CG>
static int launch_swiglu_cg(const void* xf, const void* w, int M, int K, int n_tiles, const SwigluOut& so,
                            hipStream_t s)
{
    const int n_blocks = (n_tiles + 2 * CG - 1) / (2 * CG);
    const int grid = (n_blocks + 7) / 8 * 8;       // map_block deals workgroups to the 8 XCDs
    const int kb = K / 32;
    hipLaunchKernelGGL((gemm_skinny_kernel<MT, 2, KC, 2, 1, 1, CG>), dim3(grid), dim3(64 * CG), 0, s, (const u32x4*)xf,
                       (const u32x4*)w, nullptr, M, n_tiles, kb, (kb + WPACK_KG - 1) / WPACK_KG * WPACK_KG, 1, n_blocks, so);
    SPECV_LAUNCH_CHECK("gemm_skinny_kernel (SwiGLU)");
    return SPEC_OK;
}

// wavefronts per workgroup of the SwiGLU GEMM: as few as still give no more workgroups than compute
// units (the number of wavefronts in the launch is the same either way, one per pair of column tiles;
// fewer per workgroup spread them, and the X traffic, over more compute units)
static int swiglu_column_groups(int n_tiles, int cu_count)
{
    for (int cg = 2; cg < 4; ++cg)
        if ((n_tiles + 2 * cg - 1) / (2 * cg) <= cu_count) return cg;
    return 4;
}

template <int MT, int KC>
static int launch_swiglu_variant(const void* xf, const void* w, int M, int K, int n_tiles, const SwigluOut& so,
                                 int cu_count, hipStream_t s)
{
    switch (g_swiglu_cg > 0 ? g_swiglu_cg : swiglu_column_groups(n_tiles, cu_count)) {
    case 2: return launch_swiglu_cg<MT, KC, 2>(xf, w, M, K, n_tiles, so, s);
    case 3: return launch_swiglu_cg<MT, KC, 3>(xf, w, M, K, n_tiles, so, s);
    default: return launch_swiglu_cg<MT, KC, 4>(xf, w, M, K, n_tiles, so, s);
    }
}

int launch_gemm_swiglu(const void* x_frags, const void* w_gate_up, int M, int F, int K, const double2* ssq, int n_ssq, int d,
                       float eps, void* act_frags, int act_mt, int cu_count, hipStream_t s,
                       const SsqTiles* tiles)
{
    if (tiles && gemm_row_tiles(M) != 1) return fail(SPEC_ERR_SHAPE, "row sums by column tiles are for one row tile, got %d rows", M);
    if (K % 32 || F % 16) return fail(SPEC_ERR_SHAPE, "SwiGLU GEMM needs K %% 32 == 0 and F %% 16 == 0");
    const SwigluOut so{ssq, n_ssq, d, eps, static_cast<uint4*>(act_frags), act_mt, 2, tiles ? *tiles : SsqTiles{}};
    const int n_tiles = 2 * F / 16;
    switch (gemm_row_tiles(M)) {
    case 1: return launch_swiglu_variant<1, 4>(x_frags, w_gate_up, M, K, n_tiles, so, cu_count, s);
    case 2: return launch_swiglu_variant<2, 4>(x_frags, w_gate_up, M, K, n_tiles, so, cu_count, s);
    case 3: return launch_swiglu_variant<3, 4>(x_frags, w_gate_up, M, K, n_tiles, so, cu_count, s);
    case 4: return launch_swiglu_variant<4, 2>(x_frags, w_gate_up, M, K, n_tiles, so, cu_count, s);
    default: break;
    }
    const GemmPlan p = plan_gemm(M, 2 * F, K, cu_count, true);
    if (!gemm_ring_swiglu_fits(p)) return fail(SPEC_ERR_SHAPE, "no SwiGLU GEMM variant for %d rows", M);
    return launch_ring_plan(p, x_frags, w_gate_up, M, 2 * F, K, nullptr, s, &so);
}

int launch_pack_x(const float* x, const float* gain, int M, int K, int mt_count, int planes, void* x_frags, hipStream_t s)
{
    const int total = M * (K / 8);
    int blocks = (total + 255) / 256;
    if (blocks > 4096) blocks = 4096;
    hipLaunchKernelGGL(pack_x_kernel, dim3(blocks), dim3(256), 0, s, x, gain, M, K, mt_count, planes, (uint4*)x_frags);
    SPECV_LAUNCH_CHECK("pack_x_kernel");
    return SPEC_OK;
}

int launch_gemm_f32(const float* x, const float* w, int M, int N, int K, float* y, hipStream_t s, int mode,
                    const float* gain, float eps)
{
    // row tiles per workgroup: up to four share a workgroup's reads of W
    const int mt = M <= 16 ? 1 : M <= 32 ? 2 : 4;
    const dim3 grid((N + 15) / 16, (M + 16 * mt - 1) / (16 * mt));
#define SPECV_F32(NT, NORM)                                                                                             \
    do {                                                                                                                \
        auto* k = mt == 1 ? gemm_f32_kernel<1, NT, NORM> : mt == 2 ? gemm_f32_kernel<2, NT, NORM> : gemm_f32_kernel<4, NT, NORM>; \
        hipLaunchKernelGGL(k, grid, dim3(64 * F32_WAVES), 0, s, x, w, gain, eps, mode, y, M, N, K);                     \
    } while (0)
    if (mode == F32_SWIGLU) {
        if (!gain) return fail(SPEC_ERR_SHAPE, "the fp32 SwiGLU product normalises its input");
        SPECV_F32(2, true);
    } else if (gain) {
        SPECV_F32(1, true);
    } else {
        SPECV_F32(1, false);
    }
#undef SPECV_F32
    SPECV_LAUNCH_CHECK("gemm_f32_kernel");
    return SPEC_OK;
}

}  // namespace specv

using namespace specv;

extern "C" size_t spec_packed_weight_bytes(int32_t n_out, int32_t n_in)
{
    if (n_out <= 0 || n_in <= 0 || n_in % 32) return 0;
    const size_t kb_pad = (size_t)(n_in / 32 + WPACK_KG - 1) / WPACK_KG * WPACK_KG;
    return (size_t)((n_out + 15) / 16) * kb_pad * 1024;
}

extern "C" int spec_pack_weight(const void* src, void* dst, int32_t n_out, int32_t n_in, int32_t interleave_halves,
                                void* stream)
{
    if (!src || !dst || n_out <= 0 || n_in <= 0) return fail(SPEC_ERR_INVALID_ARG, "spec_pack_weight: bad pointer or size");
    if (n_in % 32) return fail(SPEC_ERR_SHAPE, "spec_pack_weight: n_in must be a multiple of 32");
    if (interleave_halves && (n_out % 32)) return fail(SPEC_ERR_SHAPE, "spec_pack_weight: interleaving needs n_out/2 %% 16 == 0");
    if (((uintptr_t)src & 15) || ((uintptr_t)dst & 15)) return fail(SPEC_ERR_INVALID_ARG, "spec_pack_weight: 16-byte alignment");
    const int n_tiles = (n_out + 15) / 16;
    const size_t total = spec_packed_weight_bytes(n_out, n_in) / 16;
    size_t blocks = (total + 255) / 256;
    if (blocks > 65536) blocks = 65536;
    hipLaunchKernelGGL(pack_weight_kernel, dim3((unsigned)blocks), dim3(256), 0, (hipStream_t)stream,
                       (const uint16_t*)src, (uint4*)dst, n_out, n_in, n_tiles, interleave_halves ? 1 : 0);
    SPECV_LAUNCH_CHECK("pack_weight_kernel");
    return SPEC_OK;
}

extern "C" void spec_k_set_gemm_wg_target(int32_t workgroups) { set_gemm_wg_target(workgroups); }
extern "C" void spec_k_set_gemm_balance_groups(int32_t on) { g_balance_groups = on != 0; }
extern "C" void spec_k_set_swiglu_min_wgs(int32_t workgroups) { set_swiglu_min_wgs(workgroups); }
extern "C" void spec_k_set_swiglu_column_groups(int32_t groups) { set_swiglu_column_groups(groups); }
extern "C" void spec_k_set_attn_items_per_cu(int32_t items) { set_attn_items_per_cu(items); }
extern "C" void spec_k_set_attn_merge_min_pairs(int32_t pairs) { set_attn_merge_min_pairs(pairs); }
extern "C" void spec_k_set_attn_max_chunks(int32_t chunks) { set_attn_max_chunks(chunks); }
extern "C" void spec_k_set_attn_small_positions(int32_t positions) { set_attn_small_positions(positions); }

extern "C" size_t spec_k_gemm_workspace_bytes(int32_t M, int32_t N, int32_t K)
{
    if (M < 1 || M > GEMM_MAX_ROWS || N < 1 || K < 32 || K % 32) return 0;
    GemmPlan p = plan_gemm(M, N, K, 256, true);
    // partial sums of the widest plan (16 ranges) + the X fragment buffer (both planes)
    const size_t part = (size_t)16 * M * p.n_pad * sizeof(float);
    return part + xfrag_uint4s(p.mt, 2, K) * sizeof(uint4) + 256;
}

extern "C" int spec_k_gemm_bf16(const float* x, const void* w_packed, float* y, int32_t M, int32_t N, int32_t K,
                                int32_t split_x, void* workspace, void* stream)
{
    if (!x || !w_packed || !y || !workspace) return fail(SPEC_ERR_INVALID_ARG, "spec_k_gemm_bf16: null pointer");
    if (M < 1 || M > GEMM_MAX_ROWS || N < 1 || K < 32 || K % 32) return fail(SPEC_ERR_SHAPE, "spec_k_gemm_bf16: unsupported shape");
    GemmPlan p = plan_gemm(M, N, K, 256, split_x != 0);
    float* partial = (float*)workspace;
    char* xf = (char*)workspace + (((size_t)16 * M * p.n_pad * sizeof(float) + 255) & ~(size_t)255);
    const size_t n_xf = xfrag_uint4s(p.mt, p.planes, K);
    hipLaunchKernelGGL(zero_kernel, dim3((unsigned)((n_xf + 255) / 256 < 2048 ? (n_xf + 255) / 256 : 2048)), dim3(256), 0,
                       (hipStream_t)stream, (uint4*)xf, n_xf);
    SPECV_LAUNCH_CHECK("zero_kernel");
    int rc = launch_pack_x(x, nullptr, M, K, p.mt, p.planes, xf, (hipStream_t)stream);
    if (rc) return rc;
    rc = launch_gemm_bf16(p, xf, w_packed, M, N, K, partial, (hipStream_t)stream);
    if (rc) return rc;
    return launch_reduce_splits(partial, p.n_split, (size_t)M * p.n_pad, M, N, p.n_pad, nullptr, 0, 0, 0.f, y,
                                (hipStream_t)stream);
}

extern "C" int spec_k_gemm_f32(const float* x, const float* w, float* y, int32_t M, int32_t N, int32_t K, void* stream)
{
    if (!x || !w || !y || M < 1 || N < 1 || K < 1) return fail(SPEC_ERR_INVALID_ARG, "spec_k_gemm_f32: bad argument");
    return launch_gemm_f32(x, w, M, N, K, y, (hipStream_t)stream);
}
