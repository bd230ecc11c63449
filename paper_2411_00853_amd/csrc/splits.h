// Adding up the K-range partial sums a GEMM leaves behind (fixed order: range 0, 1, 2, ...).
#pragma once

#include <hip/hip_runtime.h>
#include <stddef.h>

namespace specv {

// out += N float4 columns of one row, all loads of a batch of (up to) W ranges issued before the first addition
// (indices past the end clamped, values dropped), so that the memory latency is paid once per batch: summing
// the columns one after the other makes N dependent round trips (the compiler keeps each sum's loads next
// to its additions).  Ranges are added in index order.
template <int N, int W>
__device__ __forceinline__ void add_splits4_many(const float* const (&p)[N], int n_split, size_t stride, float4 (&out)[N])
{
    for (int s0 = 0; s0 < n_split; s0 += W) {
        float4 a[N][W];
#pragma unroll
        for (int x = 0; x < N; ++x)
#pragma unroll
            for (int i = 0; i < W; ++i)
                a[x][i] = *reinterpret_cast<const float4*>(p[x] + (size_t)min(s0 + i, n_split - 1) * stride);
#pragma unroll
        for (int x = 0; x < N; ++x)
#pragma unroll
            for (int i = 0; i < W; ++i) {
                const bool ok = s0 + i < n_split;
                out[x].x += ok ? a[x][i].x : 0.f; out[x].y += ok ? a[x][i].y : 0.f;
                out[x].z += ok ? a[x][i].z : 0.f; out[x].w += ok ? a[x][i].w : 0.f;
            }
    }
}

// The same with as many loads as there are ranges (1, 2, 4 or 8; more come in batches of 8): the clamped
// loads above cost the kernels that run over many rows more than the bytes they need.
template <int S, int N>
__device__ __forceinline__ void sum_exact(const float* const (&p)[N], size_t stride, float4 (&out)[N])
{
    float4 a[N][S];
#pragma unroll
    for (int i = 0; i < S; ++i)
#pragma unroll
        for (int x = 0; x < N; ++x) a[x][i] = *reinterpret_cast<const float4*>(p[x] + i * stride);
#pragma unroll
    for (int x = 0; x < N; ++x) {
        out[x] = a[x][0];
#pragma unroll
        for (int i = 1; i < S; ++i) {
            out[x].x += a[x][i].x; out[x].y += a[x][i].y; out[x].z += a[x][i].z; out[x].w += a[x][i].w;
        }
    }
}

template <int N>
__device__ __forceinline__ void sum_ranges(const float* const (&p)[N], int n_split, size_t stride, float4 (&out)[N])
{
    switch (n_split) {
    case 1: sum_exact<1>(p, stride, out); break;
    case 2: sum_exact<2>(p, stride, out); break;
    case 4: sum_exact<4>(p, stride, out); break;
    case 8: sum_exact<8>(p, stride, out); break;
    default:
#pragma unroll
        for (int x = 0; x < N; ++x) out[x] = make_float4(0.f, 0.f, 0.f, 0.f);
        add_splits4_many<N, 8>(p, n_split, stride, out);
        break;
    }
}

}  // namespace specv
