// The sum of a weight gradient's parts: device code shared by the launches of mfma_wgrad.hip and sums.hip.
#pragma once

#include "nm_common.h"

namespace nm {

// One sum as the definition has it (see DefinedDw), in the plain kernel's blocks.
template <typename TS>
__device__ __forceinline__ float defined_dw(const Geom &g, const TS *x, const TS *dy, const TS *y, int co, int ci, int k)
{
    const int off = k * g.dil - g.pad;
    float z = 0.f;
#pragma clang loop unroll(disable)
    for (int b = 0; b < g.B && z == z; ++b) {
        const int len = valid_len(g, b);
        const size_t at = ((size_t)b * g.Cout + co) * g.To;
        const TS *xr = x + ((size_t)b * g.Cin + ci) * g.T;
#pragma clang loop unroll(disable)
        for (int t0 = 0; t0 < g.To && z == z; t0 += 64) {
            float part = 0.f;
#pragma clang loop unroll(disable)
            for (int t = t0; t < min(t0 + 64, g.To); ++t) {
                const int tau = t * g.stride + off;
                if (tau < 0 || tau >= len) continue;
                const float gv = y && !(load_as_f32(y, at + t) > 0.f) ? 0.f : load_as_f32(dy, at + t);
                part = fmaf(gv, load_as_f32(xr, (size_t)tau), part);
            }
            z += part;
        }
    }
    return z;
}
__device__ __forceinline__ float defined_dw(const Geom &g, const DefinedDw &q, int co, int ci, int k)
{
    return q.f32 ? defined_dw(g, (const float *)q.x, (const float *)q.dy, (const float *)q.y, co, ci, k)
                 : defined_dw(g, (const bf16_t *)q.x, (const bf16_t *)q.dy, (const bf16_t *)q.y, co, ci, k);
}

// dw[co][ci][k] = (accumulate ? dw : 0) + scale[co] * sum_s part[s][k][co][ci] for Cin % 4 == 0 and 16-byte aligned dw: a block of 256
// threads per (co, 256 ci), 16-byte loads along ci (a wavefront reads 1 KiB contiguous per partial row) and 16-byte stores of the
// transposed tile ([256][K+1] floats of LDS).  MEND, MANY: as for wgrad_reduce_kernel.
constexpr int kReduce4Ci = 256;
template <bool MEND, bool MANY>
__device__ __forceinline__ void reduce4_block(float *tile, int cb, int co, const float *__restrict__ part, float *__restrict__ dw,
                                              const float *__restrict__ scale, int S, int K, int Cout, int Cin, int accumulate,
                                              const Geom &own, const DefinedDw &defined)
{
    typedef float f32x4 __attribute__((ext_vector_type(4)));
    const int ci0 = cb * kReduce4Ci;
    const int l = threadIdx.x & 63, kq = threadIdx.x >> 6;
    const int ci = ci0 + 4 * l;
    const size_t plane = (size_t)Cout * Cin;
    const float factor = scale ? scale[co] : 1.f;
    for (int k = kq; k < K; k += 4) {
        f32x4 sum = {0.f, 0.f, 0.f, 0.f};
        if (ci < Cin) {
            const float *src = part + ((size_t)k * Cout + co) * Cin + ci;
#pragma unroll MANY ? 8 : 1
            for (int sp = 0; sp < S; ++sp) sum += *reinterpret_cast<const f32x4 *>(src + (size_t)sp * K * plane);
            if constexpr (MEND) {
                const float all = (sum[0] + sum[1]) + (sum[2] + sum[3]);  // a NaN (or an infinity) if one of them is
                if (__builtin_expect(made_again(all, defined.infinities), 0)) {
#pragma clang loop unroll(disable)
                    for (int e = 0; e < 4; ++e) {
                        const float one = e == 0 ? sum[0] : e == 1 ? sum[1] : e == 2 ? sum[2] : sum[3];
                        if (!made_again(one, defined.infinities)) continue;
                        const float z = defined_dw(own, defined, co, ci + e, k);
                        if (e == 0) sum[0] = z; else if (e == 1) sum[1] = z; else if (e == 2) sum[2] = z; else sum[3] = z;
                    }
                }
            }
        }
#pragma unroll
        for (int e = 0; e < 4; ++e) tile[(4 * l + e) * (K + 1) + k] = sum[e] * factor;
    }
    __syncthreads();
    const int nci = min(kReduce4Ci, Cin - ci0);
    const int n = nci * K;  // a multiple of 4
    float *dst = dw + ((size_t)co * Cin + ci0) * K;
    for (int e0 = threadIdx.x * 4; e0 < n; e0 += 1024) {
        f32x4 v;
#pragma unroll
        for (int e = 0; e < 4; ++e) {
            const int c = (e0 + e) / K, k = (e0 + e) - c * K;
            v[e] = tile[c * (K + 1) + k];
        }
        f32x4 *o = reinterpret_cast<f32x4 *>(dst + e0);
        *o = accumulate ? *o + v : v;
    }
}

struct SplitSum;
hipError_t launch_split_sum(const SplitSum &sum, hipStream_t s);  // that one alone
// both sums in one launch (sums.hip): first, and reduce4_block's (mend: own and defined are given)
hipError_t launch_both_sums(const SplitSum &first, const float *part, float *dw, const float *scale, int S, int K, int Cout, int Cin,
                            bool accumulate, bool mend, const Geom &own, const DefinedDw &defined, hipStream_t s);

}  // namespace nm
