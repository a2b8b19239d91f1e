// Float32 storage on the matrix cores: what the two engines (f32_conv.hip, f32_terms.hip) share.
#pragma once

#include "nm_common.h"

namespace nm {

typedef float f32x16 __attribute__((ext_vector_type(16)));
typedef float f32x4 __attribute__((ext_vector_type(4)));

// All staging loads are buffer loads without branches (a branch around a load makes the next one wait for it): what a
// lane does not want lies beyond the tensor and reads zeros.  The host keeps weights, dz and batch items below 2 GiB.
constexpr uint32_t kFar = 0x80000000u;
__device__ __forceinline__ __amdgpu_buffer_rsrc_t rsrc(const float *p, size_t n)
{
    return __builtin_amdgcn_make_buffer_rsrc((void *)p, 0, (int)(n * sizeof(float)), 0x00020000);
}
__device__ __forceinline__ float load1(__amdgpu_buffer_rsrc_t r, uint32_t off)
{
    return __uint_as_float(__builtin_amdgcn_raw_buffer_load_b32(r, off, 0, 0));
}
__device__ __forceinline__ f32x4 load4(__amdgpu_buffer_rsrc_t r, uint32_t off)
{
    return __builtin_bit_cast(f32x4, __builtin_amdgcn_raw_buffer_load_b128(r, off, 0, 0));
}

struct F32ConvParams {
    int B, M, R, Tin, Tout, K, stride, dil, padL;
    int nmt, ntt;
    int w_stride;   // LDS: floats per output channel (forward), per reduction channel (input gradient)
    int x_stride;   // LDS: floats per reduction channel of the window
    int W;          // window length
    int flush;      // chunks between two additions to the second accumulators
    int relu;
    const float *in;               // [B][R][Tin]
    const float *w;                // forward [M][R][K]; input gradient [R][M][K], taps flipped here
    const float *rscale;           // input gradient: optional factors of the reduction channels, folded into one operand
    const float *scale, *shift;    // optional [M]
    const float *res;              // optional, layout of out
    float *out;                    // [B][M][Tout]
    const int *len_in, *len_out;   // optional [B]
    bool infinities;               // infinite sums are made again too
    int nsplit;                    // workgroups that share a tile's reduction channels
    float *part;                   // their sums [nsplit][B][M][Tout] (nsplit > 1)
};

// One output as the definition has it, the sums as the plain kernels take them.  The kernels of both engines also multiply zeros
// for the padding: with a non-finite weight that makes a NaN of a sum that has no such product, so a NaN is made again here.
template <bool FLIP>
__device__ __forceinline__ float defined_sum(const F32ConvParams &p, const float *in, int len, int m, int t)
{
    float z = 0.f;
#pragma clang loop unroll(disable)
    for (int r0 = 0; r0 < p.R && z == z; r0 += 8) {
        float part = 0.f;
#pragma clang loop unroll(disable)
        for (int r = r0; r < min(r0 + 8, p.R); ++r) {
            const float *w = p.w + ((size_t)(FLIP ? r : m) * (FLIP ? p.M : p.R) + (FLIP ? m : r)) * p.K;
            const float f = p.rscale ? p.rscale[r] : 1.f;
#pragma clang loop unroll(disable)
            for (int k = 0; k < p.K; ++k) {
                const int j = FLIP ? p.K - 1 - k : k, tau = t * p.stride - p.padL + j * p.dil;
                if (tau >= 0 && tau < len) part = fmaf(w[k], in[(size_t)r * p.Tin + tau] * f, part);
            }
        }
        z += part;
    }
    return z;
}

// there: not behind the outputs' valid length, where they are zero
__device__ __forceinline__ void finish_output(const F32ConvParams &p, float v, bool there, int m, size_t o)
{
    if (p.scale) v *= p.scale[m];
    if (p.shift) v += p.shift[m];
    if (!there) v = 0.f;
    if (p.res) v += p.res[o];
    if (p.relu) v = v > 0.f ? v : 0.f;
    p.out[o] = v;
}

// f32_terms.hip: the sums p.part (p.nsplit > 1) or the outputs, on tiles of 32 channels x 32*nt steps
bool f32_terms_conv_supported(int R, int K, int stride, int dil);
void f32_terms_plan(int B, int M, int R, int Tout, int K, int most_parts, int *nt, int *nsplit);
hipError_t launch_f32_terms_conv(const F32ConvParams &p, bool flip, int nt, hipStream_t s);
bool f32_terms_wgrad_supported(const Geom &g);
int f32_terms_wgrad_parts(const Geom &g, int most, double *cost);  // at most `most`; cost: estimated us
hipError_t launch_f32_terms_wgrad(const Geom &g, int S, const float *x, const float *dz, float *part, hipStream_t s);

}  // namespace nm
