// The embedding of a window row, shared by the two kernels that do it: beside the row bookkeeping (sampler.hip) and on its own,
// for steps of several decoder passes (elementwise.hip).
#pragma once

#include "common.h"
#include "frag.h"

namespace specv {

// Emit 8 consecutive values of a row as the next GEMM's operand: x * gain, as fragments (the fp32 path has none:
// its GEMM takes the plain rows).
__device__ __forceinline__ void emit_operand(const XOut& xo, int m, int k8, const float (&v)[8], const float* __restrict__ gain)
{
    if (!xo.frags) return;
    float g[8];
#pragma unroll
    for (int e = 0; e < 8; ++e) g[e] = v[e] * (gain ? gain[k8 * 8 + e] : 1.f);
    store_x_unit(static_cast<uint4*>(xo.frags), xo.mt, xo.planes, m, k8, g);
}

// the sum of squares of one of a row's chunks of SSQ_CHUNK columns, from its 64 lanes' sums
__device__ __forceinline__ void store_ssq(double2* ssq, int m, int chunks, int chunk, double ss)
{
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) ss += __shfl_xor(ss, o);
    if ((threadIdx.x & 63) == 0) reinterpret_cast<double*>(ssq)[(size_t)m * chunks + chunk] = ss;
}

// One wavefront: x = E[token] for SSQ_CHUNK columns of row m, 8 per lane (the two calls around whatever the load of the row covers),
// with the sum of squares and the next operand.  d is a multiple of 8.  (ssq == NULL, the fp32 path: its GEMM sums the squares itself)
template <typename T>
struct EmbedRow {
    typedef T t8 __attribute__((ext_vector_type(8), aligned(sizeof(T))));
    t8 v;
    __device__ __forceinline__ void load(const T* __restrict__ E, int token, int chunk, int d)
    {
        const int k8 = chunk * 64 + (threadIdx.x & 63);
        v = *reinterpret_cast<const t8*>(E + (size_t)token * d + min(k8 * 8, d - 8));
    }
};
template <typename T>
__device__ __forceinline__ void embed_chunk(const EmbedRow<T>& row, int m, int chunk, int chunks, int d, float* __restrict__ x,
                                            const float* __restrict__ gain, const XOut& xo, double2* __restrict__ ssq)
{
    const int k8 = chunk * 64 + (threadIdx.x & 63);
    double ss = 0.0;
    if (k8 * 8 < d) {
        float v[8];
#pragma unroll
        for (int i = 0; i < 8; ++i) v[i] = static_cast<float>(row.v[i]);
        float* xp = x + (size_t)m * d + k8 * 8;
        *reinterpret_cast<float4*>(xp) = make_float4(v[0], v[1], v[2], v[3]);
        *reinterpret_cast<float4*>(xp + 4) = make_float4(v[4], v[5], v[6], v[7]);
#pragma unroll
        for (int i = 0; i < 8; ++i) ss += (double)v[i] * v[i];
        emit_operand(xo, m, k8, v, gain);
    }
    if (ssq) store_ssq(ssq, m, chunks, chunk, ss);
}

}  // namespace specv
