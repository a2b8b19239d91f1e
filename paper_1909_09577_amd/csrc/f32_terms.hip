// Float32 mode on the bfloat16 matrix instructions: every float32 operand is the sum of three bfloat16 terms, exactly
// (x = h + m + l, h the rounded value, m the rounded remainder, l what is left: 24 bits in three times 8, signs included), and a
// product is h*h' + (h*m' + m*h') + (h*l' + l*h' + m*m'), the terms left out being below 2^-26 of it.  Products of two
// bfloat16 values are exact in float32.  Six v_mfma_f32_32x32x16_bf16 of 32 cycles do what eight v_mfma_f32_32x32x2_f32 of 64 do.
// h*h' and the five corrections are summed in accumulators of their own, so that the rounding of the small terms costs
// nothing, and a chain of additions has one link per 16 products where the float32 instruction has eight.
// Operands are multiplied by 2^16 first and the sums by 2^-32 last: every float32 number, the denormal ones included, is then a multiple
// of 2^-133, which is what bfloat16 terms resolve (unscaled, operands below 2^-109 lost digits, those of 2^-126 all but nine).
// An operand that is infinite, or rounds to infinity, makes a NaN here, and leading products of rounded values can add up to an infinity
// where the sum is finite (unscaled, x = w = 2^64*(1 - 2^-10): 2^128 less the corrections).  Sums that are not finite are made again from
// the definition's products; so are, then, those of operands from 2^112 on and those that reach 2^96.
//
// Measured (4 x 256 -> 256 channels, K = 11, T = 400; the float32 instructions of f32_conv.hip before): forward 50.0 -> 24.5 us,
// input gradient 49.9 -> 22.9, weight gradient 34.2 -> 24.7 and its sum of four parts instead of seven 9.2 -> 6.7.  What bounds a
// convolution: its products alone take 11 us of that (at the 1.65 GHz these phases run at), splitting and LDS accesses alone as
// long; two wavefronts per SIMD overlap them to 16, the rest is the first loads and the sum of the wavefronts.
#include "f32_conv.h"

namespace nm {
namespace {

typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));

constexpr int kTermWaves = 8;  // two per SIMD: one splits and reads while the other multiplies
constexpr int kRows = 32;      // output channels of a tile
constexpr float kLift = 65536.f, kDrop = 1.f / (kLift * kLift);  // of an operand, of a sum

// two floats -> three packed pairs of terms
__device__ __forceinline__ void split2(float a, float b, uint32_t &h, uint32_t &m, uint32_t &l)
{
    h = pack_bf16x2(a, b);
    a -= __uint_as_float(h << 16);
    b -= __uint_as_float(h & 0xffff0000u);
    m = pack_bf16x2(a, b);
    a -= __uint_as_float(m << 16);
    b -= __uint_as_float(m & 0xffff0000u);
    l = pack_bf16x2(a, b);
}
__device__ __forceinline__ void split8(const float (&v)[8], bf16x8 (&t)[3])
{
    u32x4 h, m, l;
#pragma unroll
    for (int j = 0; j < 4; ++j) {
        uint32_t a, b, c;
        split2(v[2 * j], v[2 * j + 1], a, b, c);
        h[j] = a; m[j] = b; l[j] = c;
    }
    t[0] = __builtin_bit_cast(bf16x8, h);
    t[1] = __builtin_bit_cast(bf16x8, m);
    t[2] = __builtin_bit_cast(bf16x8, l);
}
// main[n] += a*b[n], rest[n] += the corrections; the tiles take turns so that no instruction waits for the one before it
template <int N>
__device__ __forceinline__ void multiply_terms(const bf16x8 (&a)[3], const bf16x8 (&b)[N][3], f32x16 (&main)[N], f32x16 (&rest)[N])
{
    constexpr int ia[5] = {2, 0, 1, 1, 0}, ib[5] = {0, 2, 1, 0, 1};  // small ones first
#pragma unroll
    for (int n = 0; n < N; ++n) main[n] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(a[0], b[n][0], main[n], 0, 0, 0);
#pragma unroll
    for (int i = 0; i < 5; ++i)
#pragma unroll
        for (int n = 0; n < N; ++n) rest[n] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(a[ia[i]], b[n][ib[i]], rest[n], 0, 0, 0);
}

// ---- forward pass and input gradient (stride 1, dilation 1) -------------------------------------------------------------
// A workgroup owns 32 output channels x 32*NT time steps of one batch item; its eight wavefronts take eight reduction
// channels in turn and add their sums through LDS at the end.  A wavefront works on its own: no barrier before that.
// An instruction multiplies eight channels of two taps (lane half h: tap 2i + h; the absent tap of an odd K has zero
// weights), so that a wavefront stages only eight channels' weights at a time, which is what lets eight of them fit the LDS.
// Weights lie in LDS as in memory (float32; rows of 8*K floats and four more, input gradient: 32*K), are gathered eight
// channels at a time (at most two lanes a bank) and split in registers; samples are split once, while they are staged, to rows
// of one time step: three terms of eight channels, 48 bytes, an odd multiple of 16, so that 16-byte reads of
// consecutive rows hit all banks.  The next chunk is held in registers meanwhile.
template <int NT, bool FLIP, int KT>
struct TermsConv {
    static constexpr int TN = 32 * NT, PAIRS = (KT + 1) / 2;
    static constexpr int XROWS = TN + 2 * PAIRS - 1, XBYTES = XROWS * 48;
    static constexpr int WSTRIDE = FLIP ? kRows * KT : 8 * KT + 4;  // floats
    static constexpr int WBYTES = (FLIP ? 8 : kRows) * WSTRIDE * 4;
    static constexpr int WAVE = XBYTES + WBYTES;                    // (multiples of 16)
    static constexpr int RED = kTermWaves * kRows * TN * 4;
    static constexpr int LDS = kTermWaves * WAVE > RED ? kTermWaves * WAVE : RED;
    // weights: eight lanes read 128 bytes of a row, eight rows at a time; a rest of two columns is one load for all rows
    static constexpr bool WREST = !FLIP && 2 * KT % 8 == 2;
    static constexpr int WCOLS = FLIP ? KT : (2 * KT + 7) / 8 - WREST, WGROUPS = FLIP ? 1 : 4;
    static constexpr int XFULL = XROWS / 64, XTAIL = XROWS % 64;    // rows that whole wavefronts hold, and the rest
};

template <int NT, bool FLIP, int KT, bool SPLIT>
__global__ __launch_bounds__(64 * kTermWaves) __attribute__((amdgpu_waves_per_eu(2, 2))) void f32_conv_kernel(const F32ConvParams p)
{
    using Q = TermsConv<NT, FLIP, KT>;
    extern __shared__ __align__(16) unsigned char smem[];
    constexpr int TN = Q::TN;
    const int lane = threadIdx.x & 63;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int mt = (int)blockIdx.x % p.nmt, col = (int)blockIdx.x / p.nmt;
    const int b = col / p.ntt, t0 = (col - b * p.ntt) * TN, m0 = mt * kRows;
    const int chunks = (p.R + 7) / 8;
    int first = wave, end = chunks;
    if constexpr (SPLIT) {
        first = (int)blockIdx.y * chunks / p.nsplit + wave;
        end = ((int)blockIdx.y + 1) * chunks / p.nsplit;
    }
    const int len = [&] {
        const int l = p.len_in ? p.len_in[b] : p.Tin;
        return l < 0 ? 0 : (l < p.Tin ? l : p.Tin);
    }();
    const float *xb = p.in + (size_t)b * p.R * p.Tin;
    unsigned char *xs = smem + wave * Q::WAVE;
    float *ws = reinterpret_cast<float *>(xs + Q::XBYTES);
    const int tau0 = t0 - p.padL;

    // weights: row lane/8 (of its group), 16-byte column lane%8 (+8 per load); a row is 2*KT (input gradient 8*KT) columns
    const int wrow = lane >> 3, wcol = lane & 7;
    f32x4 wv[Q::WGROUPS][Q::WCOLS];
    uint32_t woff[Q::WGROUPS];
#pragma unroll
    for (int g = 0; g < Q::WGROUPS; ++g)
        woff[g] = FLIP ? (uint32_t)((wrow * p.M + m0) * KT + 4 * wcol) * 4u : (uint32_t)((m0 + 8 * g + wrow) * p.R * KT + 4 * wcol) * 4u;
    const bool wlast = FLIP || 8 * (Q::WCOLS - 1) + wcol < 2 * KT;  // the lane's last column lies in the row
    const int rrow = lane >> 1, rcol = 8 * Q::WCOLS + (lane & 1);
    f32x4 wr = {};
    // samples: whole wavefronts hold eight channels of 64 steps; the rest of the window two channels of 16 steps at most
    constexpr bool kTailPairs = Q::XTAIL > 0 && Q::XTAIL <= 16;
    constexpr int kFullGroups = Q::XFULL + (Q::XTAIL > 16 ? 1 : 0);
    float xv[kFullGroups][8], xt[2];
    uint32_t xoff[kFullGroups], xtoff = 0;
#pragma unroll
    for (int f = 0; f < kFullGroups; ++f) {
        const int c = 64 * f + lane, tau = tau0 + c;
        xoff[f] = c < Q::XROWS && tau >= 0 && tau < len ? (uint32_t)tau * 4u : kFar;
    }
    if constexpr (kTailPairs) {
        const int c = 64 * Q::XFULL + (lane & 15), tau = tau0 + c;
        xtoff = c < Q::XROWS && tau >= 0 && tau < len ? (uint32_t)(2 * (lane >> 4) * p.Tin + tau) * 4u : kFar;
    }
    auto load_chunk = [&](int c) {
        if (c >= end) return;
        const size_t at = FLIP ? (size_t)c * 8 * p.M * KT : (size_t)c * 8 * KT;
        const __amdgpu_buffer_rsrc_t rs_w = rsrc(p.w + at, (size_t)p.M * p.R * KT - at);
#pragma unroll
        for (int g = 0; g < Q::WGROUPS; ++g)
#pragma unroll
            for (int i = 0; i < Q::WCOLS; ++i)
                wv[g][i] = load4(rs_w, (i + 1 < Q::WCOLS || wlast ? woff[g] : kFar) + 128u * i);
        if constexpr (Q::WREST) wr = load4(rs_w, (uint32_t)((m0 + rrow) * p.R * KT + 4 * rcol) * 4u);
        const __amdgpu_buffer_rsrc_t rs_x = rsrc(xb + (size_t)c * 8 * p.Tin, (size_t)(p.R - c * 8) * p.Tin);
#pragma unroll
        for (int f = 0; f < kFullGroups; ++f)
#pragma unroll
            for (int j = 0; j < 8; ++j) xv[f][j] = load1(rs_x, xoff[f] + (uint32_t)(j * p.Tin) * 4u);
        if constexpr (kTailPairs) {
            xt[0] = load1(rs_x, xtoff);
            xt[1] = load1(rs_x, xtoff + (uint32_t)p.Tin * 4u);
        }
    };
    auto store_chunk = [&](int c) {
#pragma unroll
        for (int g = 0; g < Q::WGROUPS; ++g)
#pragma unroll
            for (int i = 0; i < Q::WCOLS; ++i)
                if (i + 1 < Q::WCOLS || wlast)
                    *reinterpret_cast<f32x4 *>(ws + (8 * g + wrow) * Q::WSTRIDE + 4 * (wcol + 8 * i)) = wv[g][i] * kLift;
        if constexpr (Q::WREST) *reinterpret_cast<f32x4 *>(ws + rrow * Q::WSTRIDE + 4 * rcol) = wr * kLift;
        auto factor = [&](int r) { return FLIP && p.rscale ? p.rscale[min(r, p.R - 1)] * kLift : kLift; };
#pragma unroll
        for (int j = 0; j < 8; ++j) {
            const float f = factor(c * 8 + j);
#pragma unroll
            for (int q = 0; q < kFullGroups; ++q) xv[q][j] *= f;
        }
        if constexpr (kTailPairs) {
#pragma unroll
            for (int i = 0; i < 2; ++i) xt[i] *= factor(c * 8 + 2 * (lane >> 4) + i);
        }
#pragma unroll
        for (int f = 0; f < kFullGroups; ++f)
            if (64 * (f + 1) <= Q::XROWS || 64 * f + lane < Q::XROWS) {
                bf16x8 t[3];
                split8(xv[f], t);
#pragma unroll
                for (int q = 0; q < 3; ++q) *reinterpret_cast<bf16x8 *>(xs + (64 * f + lane) * 48 + 16 * q) = t[q];
            }
        if constexpr (kTailPairs) {
            if ((lane & 15) < Q::XTAIL) {
                uint32_t t[3];
                split2(xt[0], xt[1], t[0], t[1], t[2]);
#pragma unroll
                for (int q = 0; q < 3; ++q)
                    *reinterpret_cast<uint32_t *>(xs + (64 * Q::XFULL + (lane & 15)) * 48 + 16 * q + 4 * (lane >> 4)) = t[q];
            }
        }
    };

    f32x16 main[NT], rest[NT];
#pragma unroll
    for (int n = 0; n < NT; ++n)
#pragma unroll
        for (int r = 0; r < 16; ++r) main[n][r] = rest[n][r] = 0.f;
    const int l32 = lane & 31, h = lane >> 5;
    const float *a0 = FLIP ? ws + l32 * KT + KT - 1 - h : ws + l32 * Q::WSTRIDE + h;
    const unsigned char *x0 = xs + (l32 + h) * 48;
    auto gather = [&](int i, float(&v)[8]) {
#pragma unroll
        for (int j = 0; j < 8; ++j) v[j] = FLIP ? a0[j * Q::WSTRIDE - 2 * i] : a0[j * KT + 2 * i];
        if (2 * i + 1 >= KT && h) {  // the absent tap
#pragma unroll
            for (int j = 0; j < 8; ++j) v[j] = 0.f;
        }
    };
    load_chunk(first);
    for (int c = first; c < end; c += kTermWaves) {
        store_chunk(c);
        // (a wavefront's LDS operations execute in order: this only keeps the compiler from moving them)
        __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
        __builtin_amdgcn_wave_barrier();
        __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
        load_chunk(c + kTermWaves);
        // while a pair of taps multiplies, the next pair's samples are read, its weights split and those of the one behind it gathered
        constexpr int kAhead = NT < 3 ? 2 : 1;  // sets of samples (three tiles leave no registers for two)
        float v[2][8];
        bf16x8 fa[2][3], fb[kAhead][NT][3];
        auto read = [&](int i) {
#pragma unroll
            for (int n = 0; n < NT; ++n)
#pragma unroll
                for (int q = 0; q < 3; ++q) fb[i % kAhead][n][q] = *reinterpret_cast<const bf16x8 *>(x0 + (32 * n + 2 * i) * 48 + 16 * q);
        };
        gather(0, v[0]);
        if (kAhead == 2) read(0);
        gather(1, v[1]);
        split8(v[0], fa[0]);
#pragma unroll
        for (int i = 0; i < Q::PAIRS; ++i) {
            __builtin_amdgcn_sched_barrier(0);
            if (kAhead == 1) read(i);
            if (kAhead == 2 && i + 1 < Q::PAIRS) read(i + 1);
            if (i + 1 < Q::PAIRS) split8(v[(i + 1) & 1], fa[(i + 1) & 1]);
            if (i + 2 < Q::PAIRS) gather(i + 2, v[i & 1]);
            multiply_terms<NT>(fa[i & 1], fb[i % kAhead], main, rest);
            if (kAhead == 2) {
#pragma unroll
                for (int n = 0; n < 6 * NT; ++n) {  // a read and a few splitting instructions behind every product
                    __builtin_amdgcn_sched_group_barrier(0x008, 1, 0);
                    __builtin_amdgcn_sched_group_barrier(0x100, 2 / NT, 0);
                    __builtin_amdgcn_sched_group_barrier(0x002, 8 / NT, 0);
                }
            }
        }
        __builtin_amdgcn_sched_barrier(0);
        __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
        __builtin_amdgcn_wave_barrier();
        __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
    }

    // the wavefronts' sums, added in order; one thread then finishes each output
    __syncthreads();
    float *lds = reinterpret_cast<float *>(smem), *red = lds + wave * kRows * TN;
#pragma unroll
    for (int n = 0; n < NT; ++n)
#pragma unroll
        for (int r = 0; r < 16; ++r) red[(8 * (r >> 2) + 4 * h + (r & 3)) * TN + n * 32 + l32] = main[n][r] + rest[n][r];
    __syncthreads();
    int lim = p.Tout;
    if (p.len_out) {
        const int l = p.len_out[b];
        lim = l < 0 ? 0 : (l < lim ? l : lim);
    }
#pragma unroll
    for (int e0 = 0; e0 < kRows * TN; e0 += 64 * kTermWaves) {
        const int e = e0 + (int)threadIdx.x, m = m0 + e / TN, t = t0 + e % TN;
        if (m >= p.M || t >= p.Tout) continue;
        float v = 0.f;
#pragma unroll
        for (int q = 0; q < kTermWaves; ++q) v += lds[q * kRows * TN + e];
        v *= kDrop;
        if constexpr (SPLIT) {
            p.part[(size_t)blockIdx.y * p.B * p.M * p.Tout + ((size_t)b * p.M + m) * p.Tout + t] = v;
        } else {
            if (made_again(v, true) && t < lim) v = defined_sum<FLIP>(p, xb, len, m, t);
            finish_output(p, v, t < lim, m, ((size_t)b * p.M + m) * p.Tout + t);
        }
    }
}

template <int NT, bool FLIP, int KT, bool SPLIT>
hipError_t launch_conv_t(F32ConvParams p, hipStream_t s)
{
    using Q = TermsConv<NT, FLIP, KT>;
    static_assert(Q::LDS <= 160 * 1024 && Q::WAVE % 16 == 0, "LDS of a workgroup");
    p.nmt = (p.M + kRows - 1) / kRows;
    p.ntt = (p.Tout + Q::TN - 1) / Q::TN;
    void (*kern)(const F32ConvParams) = f32_conv_kernel<NT, FLIP, KT, SPLIT>;
    static LdsOptIn opt_in;
    hipError_t e = ensure_dynamic_lds(opt_in, reinterpret_cast<const void *>(kern), Q::LDS);
    if (e != hipSuccess) return e;
    hipLaunchKernelGGL(kern, dim3((unsigned)((size_t)p.nmt * p.ntt * p.B), (unsigned)p.nsplit), dim3(64 * kTermWaves), Q::LDS, s, p);
    return hipGetLastError();
}
template <bool FLIP, int KT>
hipError_t launch_conv_k(const F32ConvParams &p, int nt, hipStream_t s)
{
    if (nt == 1) return p.nsplit > 1 ? launch_conv_t<1, FLIP, KT, true>(p, s) : launch_conv_t<1, FLIP, KT, false>(p, s);
    if (nt == 2) return p.nsplit > 1 ? launch_conv_t<2, FLIP, KT, true>(p, s) : launch_conv_t<2, FLIP, KT, false>(p, s);
    return p.nsplit > 1 ? launch_conv_t<3, FLIP, KT, true>(p, s) : launch_conv_t<3, FLIP, KT, false>(p, s);
}

// ---- weight gradient (stride 1, dilation 1) -----------------------------------------------------------------------------
// A workgroup owns 32 output channels x 32 input channels x KG taps (12 at most) and every S-th unit of (batch item, 64 time
// steps).  Its wavefronts are four slices of 16 steps times two halves of the taps.  Both operands are split once, while they
// are staged, to rows of one channel, time innermost: a fragment is 16 bytes of such a row, and a tap is a shift by its number:
// a wavefront reads the words that all of its taps touch and shifts in registers, by naming them for even taps, by v_alignbit for
// odd ones (the second half begins with an even tap).  The next unit is held in registers meanwhile; two LDS buffers, one
// barrier per unit.  The slices are added through LDS at the end, tap by tap.
// An instruction that adds products to a much smaller accumulator (the corrections, here) cuts that towards minus infinity: 8e-9 of a sum of 16
// products, but of the same sign in all of them, 3.4e-7 of a gradient over 25600 steps.  So every other wavefront multiplies -dz and is
// subtracted, and the wavefronts of a pair change slices with every batch item, so that the steps of a row's end are shared too: error
// against 64 bits 3.7e-7 -> 1.5e-7 there (1.8e-7 to 2.0e-7 on the float32 instructions).
constexpr int kUnit = 64, kSlice = 16;
constexpr int kDzRow = 2 * kUnit + 16;          // bytes; an odd multiple of 16 (16-byte reads)
constexpr int kXWin = 80, kXRow = 2 * kXWin + 20;  // samples of a window; bytes, an odd multiple of 4 (4-byte reads)
constexpr int kDzBytes = 3 * kRows * kDzRow, kXBytes = 3 * kRows * kXRow, kUnitBytes = kDzBytes + kXBytes;
constexpr int kMostTaps = 6;                    // of a wavefront
constexpr int kRedRow = 36;                     // floats

struct TermsWgradParams {
    int B, Cin, Cout, T, To, K, pad;
    int ncot, ncit, ntg, KG, S, nchunk;
    int step_b, step_chunk;  // S units: items and chunks
    const float *x, *dz;
    const int *len;
    float *part;  // [S][K][Cout][Cin]
};

// products of one slice with TPW (even) taps; x: the first one's word
template <int TPW>
__device__ __forceinline__ void wgrad_slice(const unsigned char *dz, const unsigned char *x, f32x16 (&sum)[TPW])
{
    constexpr int kWords = (TPW - 1 + 8 + 1) / 2;
    static_assert(2 * (kSlice * 3 + 8 + kMostTaps + 2 * kWords) <= 2 * kXWin, "reads inside the window");
    bf16x8 fa[3];
    uint32_t xr[3][kWords];
#pragma unroll
    for (int q = 0; q < 3; ++q) {
        fa[q] = *reinterpret_cast<const bf16x8 *>(dz + q * kRows * kDzRow);
#pragma unroll
        for (int i = 0; i < kWords; ++i) xr[q][i] = *reinterpret_cast<const uint32_t *>(x + q * kRows * kXRow + 4 * i);
    }
    constexpr int ia[6] = {2, 0, 1, 1, 0, 0}, ib[6] = {0, 2, 1, 0, 1, 0};
#pragma unroll
    for (int j = 0; j < TPW; j += 2) {
        bf16x8 fb[2][3];
#pragma unroll
        for (int t = 0; t < 2; ++t)
#pragma unroll
            for (int q = 0; q < 3; ++q) {
                u32x4 v;
#pragma unroll
                for (int e = 0; e < 4; ++e) {
                    const int d = j / 2 + e;
                    v[e] = t == 0 ? xr[q][d] : __builtin_amdgcn_alignbit(xr[q][d + 1 < kWords ? d + 1 : d], xr[q][d], 16);
                }
                fb[t][q] = __builtin_bit_cast(bf16x8, v);
            }
        f32x16 z[2] = {};
#pragma unroll
        for (int i = 0; i < 6; ++i)
#pragma unroll
            for (int t = 0; t < 2; ++t) z[t] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(fa[ia[i]], fb[t][ib[i]], z[t], 0, 0, 0);
#pragma unroll
        for (int t = 0; t < 2; ++t) sum[j + t] += z[t];
    }
}

template <int TPW>
__global__ __launch_bounds__(64 * kTermWaves) __attribute__((amdgpu_waves_per_eu(2, 2))) void f32_wgrad_kernel(const TermsWgradParams p)
{
    __shared__ __align__(16) unsigned char smem[2 * kUnitBytes];
    const int tid = (int)threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    int v = (int)blockIdx.x;
    const int cit = v % p.ncit; v /= p.ncit;
    const int cot = v % p.ncot; v /= p.ncot;
    const int tg = v % p.ntg, sp = v / p.ntg;
    const int co0 = cot * kRows, ci0 = cit * kRows, k0 = tg * p.KG, kt = min(p.KG, p.K - k0);
    const int th = wave & 1, sl = wave >> 1;

    // a thread stages four steps of a row of dz and of x, those of the first two wavefronts also four of the window's end
    const int srow = tid >> 4, sq = 4 * (tid & 15), erow = tid >> 2, eq = kUnit + 4 * (tid & 3);
    const __amdgpu_buffer_rsrc_t rs_dz = rsrc(p.dz, (size_t)p.B * p.Cout * p.To);
    float dv[4], xv[2][4];
    struct Unit {
        int b, chunk;  // item; 64 steps of it
    };
    auto behind = [&](Unit u) {  // S units on
        u.b += p.step_b;
        u.chunk += p.step_chunk;
        if (u.chunk >= p.nchunk) {
            u.chunk -= p.nchunk;
            ++u.b;
        }
        return u;
    };
    auto load_unit = [&](Unit u) {
        if (u.b >= p.B) return;
        const int b = u.b, t0 = u.chunk * kUnit;
        int len = p.T;
        if (p.len) {
            const int l = p.len[b];
            len = l < 0 ? 0 : (l < len ? l : len);
        }
        const bool dz_ok = co0 + srow < p.Cout;
        const uint32_t drow = (uint32_t)(((size_t)b * p.Cout + co0 + srow) * p.To + t0 + sq) * 4u;
#pragma unroll
        for (int e = 0; e < 4; ++e) dv[e] = load1(rs_dz, dz_ok && t0 + sq + e < p.To ? drow + 4u * e : kFar);
        const __amdgpu_buffer_rsrc_t rs_x = rsrc(p.x + (size_t)b * p.Cin * p.T, (size_t)p.Cin * p.T);
        const int tau0 = t0 - p.pad + k0;
        auto load_x = [&](int row, int q, float(&to)[4]) {
            const bool ok = ci0 + row < p.Cin;
            const int tau = tau0 + q;
            const uint32_t at = (uint32_t)((ci0 + row) * p.T + tau) * 4u;
#pragma unroll
            for (int e = 0; e < 4; ++e) to[e] = load1(rs_x, ok && tau + e >= 0 && tau + e < len ? at + 4u * e : kFar);
        };
        load_x(srow, sq, xv[0]);
        if (wave < 2) load_x(erow, eq, xv[1]);
    };
    auto store_unit = [&](unsigned char *buf, Unit u) {
        const int minus = (sq / kSlice ^ u.b) & 1;
        const float dz_lift = __uint_as_float(__float_as_uint(kLift) | (uint32_t)minus << 31);
        auto put = [&](const float(&f)[4], float lift, unsigned char *to, int plane) {
            uint32_t a[3], b[3];
            split2(f[0] * lift, f[1] * lift, a[0], a[1], a[2]);
            split2(f[2] * lift, f[3] * lift, b[0], b[1], b[2]);
#pragma unroll
            for (int q = 0; q < 3; ++q) {
                reinterpret_cast<uint32_t *>(to + q * plane)[0] = a[q];
                reinterpret_cast<uint32_t *>(to + q * plane)[1] = b[q];
            }
        };
        put(dv, dz_lift, buf + srow * kDzRow + 2 * sq, kRows * kDzRow);
        put(xv[0], kLift, buf + kDzBytes + srow * kXRow + 2 * sq, kRows * kXRow);
        if (wave < 2) put(xv[1], kLift, buf + kDzBytes + erow * kXRow + 2 * eq, kRows * kXRow);
    };

    f32x16 sum[TPW];
#pragma unroll
    for (int j = 0; j < TPW; ++j)
#pragma unroll
        for (int r = 0; r < 16; ++r) sum[j][r] = 0.f;
    const int l32 = lane & 31, h = lane >> 5;
    const int a_off = l32 * kDzRow + 2 * (8 * h), x_off = kDzBytes + l32 * kXRow + 2 * (8 * h + TPW * th);
    Unit u = {sp / p.nchunk, sp % p.nchunk};
    if (u.b < p.B) {
        load_unit(u);
        store_unit(smem, u);
        load_unit(behind(u));
    }
    for (int par = 0; u.b < p.B; par ^= 1) {
        __syncthreads();  // this unit is in its buffer, the other buffer has been read
        const int slice = sl ^ (u.b & 1);  // the wavefront's; of -dz in odd ones
        const unsigned char *cur = smem + par * kUnitBytes + 2 * kSlice * slice;
        const Unit next = behind(u);
        auto stage = [&] {
            store_unit(smem + (par ^ 1) * kUnitBytes, next);
            load_unit(behind(next));
        };
        const bool more = next.b < p.B;
        if (wave < 4 && more) stage();  // (the wavefronts of a SIMD stage before and after their products)
        if (u.chunk * kUnit + kSlice * slice < p.To) wgrad_slice<TPW>(cur + a_off, cur + x_off, sum);
        if (wave >= 4 && more) stage();
        u = next;
    }

    // the four slices of a tap of either half, added in order
    float *red = reinterpret_cast<float *>(smem);
    constexpr int kTile = kRows * kRedRow;
    static_assert(kTermWaves * kTile * 4 <= (int)sizeof(smem), "sums fit");
#pragma unroll
    for (int j = 0; j < TPW; ++j) {
        __syncthreads();
#pragma unroll
        for (int r = 0; r < 16; ++r) red[(2 * sl + th) * kTile + (8 * (r >> 2) + 4 * h + (r & 3)) * kRedRow + l32] = sum[j][r];
        __syncthreads();
        const int half = tid >> 8, tap = half * TPW + j;
        if (tap < kt) {
#pragma unroll
            for (int i = 0; i < 4; ++i) {
                const int co = (tid >> 5 & 7) + 8 * i, at = co * kRedRow + l32;
                float z = red[half * kTile + at];
#pragma unroll
                for (int q = 1; q < 4; ++q) z += q & 1 ? -red[(2 * q + half) * kTile + at] : red[(2 * q + half) * kTile + at];
                if (co0 + co < p.Cout && ci0 + l32 < p.Cin)
                    p.part[(((size_t)sp * p.K + k0 + tap) * p.Cout + co0 + co) * p.Cin + ci0 + l32] = z * kDrop;
            }
        }
    }
}

struct TermsWgradPlan {
    int ntg, KG, TPW, S, nchunk, units, ncot, ncit;
    double cost;
};
// At most most_parts parts.  Estimated in microseconds: rounds of workgroups over the CUs (one each: the registers), their units, the sum of at most eight
// parts by their bytes.
TermsWgradPlan wgrad_plan(const Geom &g, int most_parts)
{
    TermsWgradPlan q = {};
    q.ntg = (g.K + 2 * kMostTaps - 1) / (2 * kMostTaps);
    q.KG = (g.K + q.ntg - 1) / q.ntg;
    q.TPW = (q.KG + 3) / 4 * 2;
    q.nchunk = (g.To + kUnit - 1) / kUnit;
    q.units = g.B * q.nchunk;
    q.ncot = (g.Cout + kRows - 1) / kRows;
    q.ncit = (g.Cin + kRows - 1) / kRows;
    const double tiles = (double)q.ncot * q.ncit * q.ntg, mb = 4e-6 * g.Cout * g.Cin * (double)g.K;
    for (int S = 1; S <= most_parts && S <= q.units; ++S) {
        const int each = (q.units + S - 1) / S;
        if (S > (q.units + each - 1) / each) continue;  // the last part of it would be empty
        const double rounds = (double)((long)(tiles * S + 255) / 256);
        const double cost = rounds * (5.0 + each * (0.6 + 0.19 * q.KG)) + 0.5 * mb * S;
        if (q.S == 0 || cost < q.cost) {
            q.cost = cost;
            q.S = S;
        }
    }
    return q;
}

}  // namespace

// The tap counts that have instances: 11 and 13, those of the encoder's first three blocks, whose layers the estimates below are fitted to.
// The LDS does not draw that line (3 to 14 taps fit with all three tiles, 15 with two, 17 with one): other counts have not been measured
// here and run on the float32 instructions.  And sums of no more links (products of a wavefront to one accumulator) than leave the error
// below that of those instructions' short sums: 42 of 384 channels, K=13, where it is the same (1.25e-7 against 64 bits; 20 to 35 %
// smaller with fewer).
bool f32_terms_conv_supported(int R, int K, int stride, int dil)
{
    const int links = ((R + 7) / 8 + kTermWaves - 1) / kTermWaves * ((K + 1) / 2);
    return (K == 11 || K == 13) && stride == 1 && dil == 1 && links <= 42;
}

// Tile and parts by estimate (us), fitted to 2600 calls (rms 5 %): a round of workgroups over the CUs (one each: the LDS) and
// the chunks of a SIMD; parts cost a launch and their bytes.
void f32_terms_plan(int B, int M, int R, int Tout, int K, int most_parts, int *nt, int *nsplit)
{
    const int chunks = (R + 7) / 8;
    double best = 0;
    *nt = 0;
    for (int t = 1; t <= 3; ++t)
        for (int n = 1; n <= most_parts && n <= chunks; ++n) {
            const size_t tiles = (size_t)((M + kRows - 1) / kRows) * ((Tout + 32 * t - 1) / (32 * t)) * B;
            const int each = ((chunks + n - 1) / n + 3) / 4;
            const double rounds = (double)((tiles * n + 255) / 256);
            const double cost = rounds * (1.07 + 0.61 * t + each * K * (0.052 + 0.042 * t)) + (n > 1 ? 1.8 + 1.84e-6 * n * B * M * (double)Tout : 0.0);
            if (*nt == 0 || cost < best) {
                best = cost;
                *nt = t;
                *nsplit = n;
            }
        }
}

hipError_t launch_f32_terms_conv(const F32ConvParams &p, bool flip, int nt, hipStream_t s)
{
    if (p.K == 11) return flip ? launch_conv_k<true, 11>(p, nt, s) : launch_conv_k<false, 11>(p, nt, s);
    return flip ? launch_conv_k<true, 13>(p, nt, s) : launch_conv_k<false, 13>(p, nt, s);
}

bool f32_terms_wgrad_supported(const Geom &g) { return g.stride == 1 && g.dil == 1; }
int f32_terms_wgrad_parts(const Geom &g, int most, double *cost)
{
    const TermsWgradPlan q = wgrad_plan(g, most);
    *cost = q.cost;
    return q.S;
}

// S: what f32_terms_wgrad_parts chose
hipError_t launch_f32_terms_wgrad(const Geom &g, int S, const float *x, const float *dz, float *part, hipStream_t s)
{
    const TermsWgradPlan q = wgrad_plan(g, 1);
    TermsWgradParams p = {};
    p.B = g.B; p.Cin = g.Cin; p.Cout = g.Cout; p.T = g.T; p.To = g.To; p.K = g.K; p.pad = g.pad;
    p.ncot = q.ncot; p.ncit = q.ncit; p.ntg = q.ntg; p.KG = q.KG; p.S = S; p.nchunk = q.nchunk;
    p.step_b = S / q.nchunk; p.step_chunk = S % q.nchunk;
    p.x = x; p.dz = dz; p.len = g.len; p.part = part;
    const unsigned grid = (unsigned)((size_t)p.ncot * p.ncit * p.ntg * p.S);
    auto go = [&](void (*kern)(const TermsWgradParams)) { hipLaunchKernelGGL(kern, dim3(grid), dim3(64 * kTermWaves), 0, s, p); };
    if (q.TPW == 2) go(f32_wgrad_kernel<2>);
    else if (q.TPW == 4) go(f32_wgrad_kernel<4>);
    else go(f32_wgrad_kernel<6>);
    return hipGetLastError();
}

}  // namespace nm
