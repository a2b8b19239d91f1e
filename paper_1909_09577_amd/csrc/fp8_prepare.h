// 8-bit operands: the code conversion, and the passes that write a call's operands (fp8_prepare.hip).
#pragma once

#include "nm_common.h"

namespace nm {

constexpr float kE4M3Max = 448.0f;

// ---------------------------------------------------------------------------------------------
// E4M3 conversion: round to nearest, ties to even, saturating at +-448.  The hardware conversion
// (v_cvt_pk_fp8_f32, two values per instruction) rounds to nearest even; the saturation is made explicit by
// clamping first.  Inputs are finite by contract (a NaN gives a NaN code).
__device__ __forceinline__ float clamp_e4m3(float v) { return __builtin_fminf(__builtin_fmaxf(v, -448.0f), 448.0f); }
// codes of a, b, c, d in bytes 0..3
__device__ __forceinline__ uint32_t e4m3_pack4(float a, float b, float c, float d)
{
    int r = __builtin_amdgcn_cvt_pk_fp8_f32(clamp_e4m3(a), clamp_e4m3(b), 0, false);
    r = __builtin_amdgcn_cvt_pk_fp8_f32(clamp_e4m3(c), clamp_e4m3(d), r, true);
    return (uint32_t)r;
}
__device__ __forceinline__ uint32_t f32_to_e4m3(float f) { return e4m3_pack4(f, 0.f, 0.f, 0.f) & 0xffu; }


// src [B][C][T] (or src*[y>0]) -> codes [B][C/64][Tp][64], row r standing for time r - pad, zero rows elsewhere; copy (optional): the
// masked values in the layout of src.  src NULL: nothing.
struct Fp8Quant {
    const void *src, *y;
    const float *scale;  // [1]
    unsigned char *codes;
    void *copy;
    int B, C, T, Tp, pad;
};
// w [Cout][Cin][K] -> A-fragment order.  Forward: [Cout/64][Cin/64][K][2][64 lanes][32] codes of w, lane l holding row l%32 and 32
// channels 32*(l/32) .. of the chunk, row_scales[Cout].  Flipped: [Cin/64][Cout/64][K][2][64][32] codes of
// w[co][ci][K-1-k]*scale[co] (scale NULL: 1), row_scales[Cin].  w NULL: nothing.
struct Fp8Pack {
    const void *w;
    const float *scale, *row_scales;
    unsigned char *out;
    int Cin, Cout, K;
    bool flip;
};
// all of them in one launch
hipError_t fp8_prepare(const Fp8Pack &pack, const Fp8Quant &first, const Fp8Quant &second, hipStream_t s);

}  // namespace nm
