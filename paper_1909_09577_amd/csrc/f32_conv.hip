// Float32 mode on the matrix cores: forward, input gradient (stride 1) and weight gradient with
// v_mfma_f32_32x32x2_f32 (exact float32 operands; A: row lane%32, k lane/32; B: column lane%32, k lane/32;
// D: row 8*(r/4) + 4*(lane/32) + r%4, column lane%32).
//
// Bound: the float32 matrix rate (64 flop per clock and SIMD; a large product reaches 153 TFLOP/s on this chip).
// One operand element serves 32 rows, so a pair of 4-byte LDS reads per 64-cycle MFMA is all the operand traffic and
// no vector layout is needed: weights stay in memory order and rows may have any length and alignment.
//
// The sums are kept as short as those of the plain kernels: the accumulators are added to a second set after every
// few staged chunks (at most 64 terms), and the partial sums of the wavefronts and of the splits are added last, in a
// fixed order.
//
// Convolutions of 11 and 13 taps and most weight gradients run on the bfloat16 instructions instead (f32_terms.hip, which has instances for
// no other taps, and says what these measured on the same call).  2732 us on the plain kernels, 141 here (4 x 256 -> 256 channels, K = 11, T = 400,
// forward and both gradients); relative error against 64 bits 1.3e-7, 1.6e-7 on those.  Of a 42 us convolution launch the
// products alone take 28 (19 at the full clock), the LDS reads 5 and the staging 9.
#include "f32_conv.h"

#include <algorithm>

namespace nm {
namespace {

constexpr int kTileM = 64;
constexpr int kConvWaves = 8;     // wavefronts of a workgroup: two per SIMD, one stages while the other multiplies
constexpr int kRun = 256;         // floats of a chunk's weight row: one 16-byte load per lane
constexpr int kXIter = 4;         // window columns per lane: windows of at most 256 samples
constexpr int kMaxLds = 160 * 1024;

// A workgroup owns 64 output channels x 32*NT time steps of one batch item.  The reduction channels are staged in chunks
// of CC (16 up to 16 taps, 8 up to 32) and split over the eight wavefronts in pairs (lane half h takes the pair's channel
// h, so that both operands of a tap are one LDS word at a fixed offset), with CC = 8 also by halves of the taps; their
// sums are added through LDS at the end.  NT = 1 doubles the workgroups where NT = 2 would leave CUs without one; NT = 2
// halves the weight traffic otherwise.  XN: window columns per lane.
// Two LDS buffers, one barrier per chunk; the next chunk is written while the current one is multiplied, by the wavefronts
// 0-3 before their products and by 4-7, the others of the same SIMDs, after them, so that a SIMD's matrix pipe has work
// while one of its two wavefronts stages (with two barriers around the writes the pipes were busy 41 % of the time).
template <int NT, bool FLIP, int CC, int XN, bool SPLIT>
__global__ __launch_bounds__(64 * kConvWaves) void f32_conv_kernel(const F32ConvParams p)
{
    extern __shared__ __align__(16) float lds[];
    constexpr int TN = 32 * NT;
    constexpr int kRowsPerWave = (FLIP ? CC : kTileM) / kConvWaves;  // weight rows a wavefront stages
    constexpr int kPieces = FLIP ? kTileM / CC : 1;                   // 256-float pieces of such a row (CC*K <= 256)
    constexpr int kWRegs = kRowsPerWave * kPieces;
    constexpr int kXRows = CC / kConvWaves;
    const int lane = threadIdx.x & 63;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int mt = (int)blockIdx.x % p.nmt, col = (int)blockIdx.x / p.nmt;
    // (an instance of its own: decided at run time, this cost the calls of many tiles 0.3 to 1 %)
    int r_first = 0, r_end = p.R;
    if constexpr (SPLIT) {
        const int split = (int)blockIdx.y, chunks = (p.R + CC - 1) / CC;
        r_first = split * chunks / p.nsplit * CC;
        r_end = min(p.R, (split + 1) * chunks / p.nsplit * CC);
    }
    const int b = col / p.ntt, t0 = (col - b * p.ntt) * TN;
    const int m0 = mt * kTileM;
    const int K = p.K;
    const int w_floats = (FLIP ? CC : kTileM) * p.w_stride, buf_floats = w_floats + CC * p.x_stride;

    int len = p.Tin;
    if (p.len_in) {
        const int l = p.len_in[b];
        len = l < 0 ? 0 : (l < len ? l : len);
    }
    const float *xb = p.in + (size_t)b * p.R * p.Tin;
    const __amdgpu_buffer_rsrc_t rs_w = rsrc(p.w, (size_t)p.M * p.R * p.K);
    const int tau0 = t0 * p.stride - p.padL;

    // what a wavefront has of a weight row: forward, the chunk's nr*K floats of one output channel; input gradient, the
    // floats of 64 output channels of one reduction channel
    const int m_have = min(kTileM, p.M - m0) * K;
    f32x4 wv[kWRegs];
    float xv[kXRows][XN];
    uint32_t xoff[kXRows][XN];  // inside a chunk's rows; rows beyond the last channel lie beyond the descriptor
#pragma unroll
    for (int i = 0; i < kXRows; ++i)
#pragma unroll
        for (int j = 0; j < XN; ++j) {
            const int c = j * 64 + lane, tau = tau0 + c;
            xoff[i][j] = c < p.W && tau >= 0 && tau < len ? (uint32_t)((wave * kXRows + i) * p.Tin + tau) * 4u : kFar;
        }
    auto load_chunk = [&](int r0) {
        if (r0 >= (SPLIT ? r_end : p.R)) return;
        const int nr = min(CC, p.R - r0);
#pragma unroll
        for (int i = 0; i < kRowsPerWave; ++i)
#pragma unroll
            for (int j = 0; j < kPieces; ++j) {
                const int row = wave * kRowsPerWave + i;
                const int have = (FLIP ? (row < nr ? m_have : 0) : (m0 + row < p.M ? nr * K : 0)) - 256 * j;
                const uint32_t base = (uint32_t)((FLIP ? (r0 + row) * p.M + m0 : (m0 + row) * p.R + r0) * K + 256 * j);
                wv[i * kPieces + j] = load4(rs_w, 4 * lane < have ? base * 4u + 16u * (uint32_t)lane : kFar);
            }
        const __amdgpu_buffer_rsrc_t rs_x = rsrc(xb + (size_t)r0 * p.Tin, (size_t)nr * p.Tin);
#pragma unroll
        for (int i = 0; i < kXRows; ++i)
#pragma unroll
            for (int j = 0; j < XN; ++j) xv[i][j] = load1(rs_x, xoff[i][j]);
    };
    auto store_chunk = [&](int r0, float *ws) {
        float *xs = ws + w_floats;
        // a load that straddles the end of what there is brought in elements of the next row: zeros instead
        const int end = FLIP ? m_have : min(CC, p.R - r0) * K;
        if ((FLIP ? kTileM : CC) * K != end) {
#pragma unroll
            for (int i = 0; i < kWRegs; ++i) {
                const int e = (i % kPieces) * 256 + 4 * lane;
#pragma unroll
                for (int q = 0; q < 4; ++q) wv[i][q] = e + q < end ? wv[i][q] : 0.f;
            }
        }
        if (FLIP && p.rscale) {
#pragma unroll
            for (int i = 0; i < kRowsPerWave; ++i) {
                const float f = p.rscale[min(r0 + wave * kRowsPerWave + i, p.R - 1)];
#pragma unroll
                for (int j = 0; j < kPieces; ++j) wv[i * kPieces + j] *= f;
            }
        }
#pragma unroll
        for (int j = 0; j < kPieces; ++j) {
            const int e = 256 * j + 4 * lane;
            if (e < p.w_stride) {  // (a multiple of four)
#pragma unroll
                for (int i = 0; i < kRowsPerWave; ++i)
                    *reinterpret_cast<f32x4 *>(ws + (wave * kRowsPerWave + i) * p.w_stride + e) = wv[i * kPieces + j];
            }
        }
#pragma unroll
        for (int j = 0; j < XN; ++j) {
            const int c = j * 64 + lane;
            if (c < p.W) {
#pragma unroll
                for (int i = 0; i < kXRows; ++i) xs[(wave * kXRows + i) * p.x_stride + c] = xv[i][j];
            }
        }
    };

    f32x16 acc[2][NT], sum[2][NT];
#pragma unroll
    for (int mi = 0; mi < 2; ++mi)
#pragma unroll
        for (int ni = 0; ni < NT; ++ni)
#pragma unroll
            for (int r = 0; r < 16; ++r) acc[mi][ni][r] = sum[mi][ni][r] = 0.f;

    const int l32 = lane & 31, h = lane >> 5;
    int since = 0;
    const int kh = (K + 1) / 2;  // CC = 8: taps of the first half
    const int klo = CC == 8 && wave >= 4 ? kh : 0, khi = CC == 8 && wave < 4 ? kh : K;
    auto multiply_chunk = [&](const float *ws, bool last) {
        const float *xs = ws + w_floats;
        {
            const int c = 2 * (CC == 8 ? wave & 3 : wave) + h;  // this lane's reduction channel
            const float *a = FLIP ? ws + c * p.w_stride + l32 * K + K - 1 : ws + l32 * p.w_stride + c * K;
            const int a_step = FLIP ? -1 : 1, a_m = FLIP ? 32 * K : 32 * p.w_stride;
            const float *x = xs + c * p.x_stride + l32 * p.stride;
            // four taps at a time, the next four read while these multiply
            float ra[2][2][4], rb[2][NT][4];
            auto read = [&](int k, int n, float(&fa)[2][4], float(&fb)[NT][4]) {
#pragma unroll
                for (int e = 0; e < 4; ++e)
                    if (e < n) {
                        fa[0][e] = a[(k + e) * a_step];
                        fa[1][e] = a[a_m + (k + e) * a_step];
#pragma unroll
                        for (int ni = 0; ni < NT; ++ni) fb[ni][e] = x[ni * 32 * p.stride + (k + e) * p.dil];
                    }
            };
            auto multiply = [&](int n, const float(&fa)[2][4], const float(&fb)[NT][4]) {
#pragma unroll
                for (int e = 0; e < 4; ++e)
                    if (e < n) {
#pragma unroll
                        for (int ni = 0; ni < NT; ++ni) {
                            acc[0][ni] = __builtin_amdgcn_mfma_f32_32x32x2f32(fa[0][e], fb[ni][e], acc[0][ni], 0, 0, 0);
                            acc[1][ni] = __builtin_amdgcn_mfma_f32_32x32x2f32(fa[1][e], fb[ni][e], acc[1][ni], 0, 0, 0);
                        }
                    }
            };
            int k = klo;
            if (k + 4 <= khi) read(k, 4, ra[0], rb[0]);
            for (; k + 8 <= khi; k += 8) {
                read(k + 4, 4, ra[1], rb[1]);
                multiply(4, ra[0], rb[0]);
                if (k + 12 <= khi) read(k + 8, 4, ra[0], rb[0]);
                multiply(4, ra[1], rb[1]);
            }
            if (k + 4 <= khi) {
                multiply(4, ra[0], rb[0]);
                k += 4;
            }
            const int rest = khi - k;  // 0 .. 3 (wave-uniform)
            if (rest > 0) {
                read(k, rest, ra[0], rb[0]);
                multiply(rest, ra[0], rb[0]);
            }
        }
        if (++since < p.flush && !last) return;
        since = 0;
#pragma unroll
        for (int mi = 0; mi < 2; ++mi)
#pragma unroll
            for (int ni = 0; ni < NT; ++ni)
#pragma unroll
                for (int r = 0; r < 16; ++r) {
                    sum[mi][ni][r] += acc[mi][ni][r];
                    acc[mi][ni][r] = 0.f;
                }
    };
    load_chunk(r_first);
    store_chunk(r_first, lds);
    load_chunk(r_first + CC);
    for (int r0 = r_first, par = 0; r0 < (SPLIT ? r_end : p.R); r0 += CC, par ^= 1) {
        __syncthreads();  // this chunk is in its buffer, the other buffer has been read
        const float *cur = lds + par * buf_floats;
        float *nxt = lds + (par ^ 1) * buf_floats;
        const bool more = r0 + CC < (SPLIT ? r_end : p.R);
        if (wave < 4 && more) {
            store_chunk(r0 + CC, nxt);
            load_chunk(r0 + 2 * CC);
        }
        multiply_chunk(cur, !more);
        if (wave >= 4 && more) {
            store_chunk(r0 + CC, nxt);
            load_chunk(r0 + 2 * CC);
        }
    }

    // the wavefronts' sums, added in order; one thread then finishes each output
    __syncthreads();
    float *red = lds + (size_t)wave * kTileM * TN;
#pragma unroll
    for (int mi = 0; mi < 2; ++mi)
#pragma unroll
        for (int ni = 0; ni < NT; ++ni)
#pragma unroll
            for (int r = 0; r < 16; ++r) red[(mi * 32 + 8 * (r >> 2) + 4 * h + (r & 3)) * TN + ni * 32 + l32] = sum[mi][ni][r];
    __syncthreads();
    int lim = p.Tout;
    if (p.len_out) {
        const int l = p.len_out[b];
        lim = l < 0 ? 0 : (l < lim ? l : lim);
    }
    for (int e = threadIdx.x; e < kTileM * TN; e += 64 * kConvWaves) {
        const int m = m0 + e / TN, t = t0 + e % TN;
        if (m >= p.M || t >= p.Tout) continue;
        float v = 0.f;
#pragma unroll
        for (int q = 0; q < kConvWaves; ++q) v += lds[(size_t)q * kTileM * TN + e];
        if constexpr (SPLIT) {
            p.part[(size_t)blockIdx.y * p.B * p.M * p.Tout + ((size_t)b * p.M + m) * p.Tout + t] = v;
        } else {
            if (v != v && t < lim) v = defined_sum<FLIP>(p, xb, len, m, t);
            finish_output(p, v, t < lim, m, ((size_t)b * p.M + m) * p.Tout + t);
        }
    }
}

// Adds the parts of an output in order and finishes it: a thread each.
template <bool FLIP>
__global__ __launch_bounds__(256) void f32_split_finish_kernel(const F32ConvParams p)
{
    const size_t n = (size_t)p.B * p.M * p.Tout, o = (size_t)blockIdx.x * 256 + threadIdx.x;
    if (o >= n) return;
    const int row = (int)(o / p.Tout), t = (int)(o - (size_t)row * p.Tout), b = row / p.M, m = row - b * p.M;
    float v = 0.f;
#pragma unroll 8
    for (int s = 0; s < p.nsplit; ++s) v += p.part[(size_t)s * n + o];
    auto limit = [&](const int *len_of, int most) {
        const int l = len_of ? len_of[b] : most;
        return l < 0 ? 0 : (l < most ? l : most);
    };
    const int lim = limit(p.len_out, p.Tout);
    if (made_again(v, p.infinities) && t < lim) v = defined_sum<FLIP>(p, p.in + (size_t)b * p.R * p.Tin, limit(p.len_in, p.Tin), m, t);
    finish_output(p, v, t < lim, m, o);
}

template <bool FLIP>
void launch_finish(const F32ConvParams &p, hipStream_t s)
{
    hipLaunchKernelGGL(f32_split_finish_kernel<FLIP>, dim3((unsigned)(((size_t)p.B * p.M * p.Tout + 255) / 256)), dim3(256), 0, s, p);
}

struct F32ConvPlan {
    bool ok;
    int cc, W, w_stride, x_stride;
    size_t lds;
};
F32ConvPlan f32_conv_plan(int K, int stride, int dil, int nt, bool flip)
{
    F32ConvPlan q = {};
    if (8 * K > kRun) return q;
    q.cc = 16 * K <= kRun ? 16 : 8;
    const long W = (long)(32 * nt - 1) * stride + (long)(K - 1) * dil + 1;
    if (W > 64 * kXIter) return q;
    q.W = (int)W;
    // rows are written 16 bytes at a time; a read touches 32 rows: four times an odd stride puts at most two in a bank
    // (input gradient: the read runs along a row, K apart)
    q.w_stride = flip ? kTileM * K : ((q.cc * K + 3) / 4 | 1) * 4;
    q.x_stride = q.W | 1;
    // (two buffers; the second one starts on 16 bytes: the strides' products are multiples of four)
    const size_t stage = 2 * ((size_t)(flip ? q.cc : kTileM) * q.w_stride + (size_t)q.cc * q.x_stride) * sizeof(float);
    const size_t red = (size_t)kConvWaves * kTileM * 32 * nt * sizeof(float);
    q.lds = stage > red ? stage : red;
    q.ok = q.lds <= (size_t)kMaxLds;
    return q;
}

template <int NT, bool FLIP, int CC, int XN, bool SPLIT>
hipError_t launch_f32_conv_t(F32ConvParams p, const F32ConvPlan &q, hipStream_t s)
{
    p.W = q.W; p.w_stride = q.w_stride; p.x_stride = q.x_stride;
    const int taps = CC == 8 ? (p.K + 1) / 2 : p.K;
    p.flush = 32 / taps;  // 64 products at most, two a tap and chunk
    p.nmt = (p.M + kTileM - 1) / kTileM;
    p.ntt = (p.Tout + 32 * NT - 1) / (32 * NT);
    auto kern = f32_conv_kernel<NT, FLIP, CC, XN, SPLIT>;
    static LdsOptIn opt_in;
    hipError_t e = ensure_dynamic_lds(opt_in, reinterpret_cast<const void *>(kern), kMaxLds);
    if (e != hipSuccess) return e;
    MainKernelTimer timer(s);  // (the sum of the parts counts with the kernel)
    hipLaunchKernelGGL(kern, dim3((unsigned)((size_t)p.nmt * p.ntt * p.B), (unsigned)p.nsplit), dim3(64 * kConvWaves), q.lds, s, p);
    if (SPLIT) launch_finish<FLIP>(p, s);
    return hipGetLastError();
}
template <int NT, bool FLIP, bool SPLIT>
hipError_t launch_f32_conv_nt(const F32ConvParams &p, const F32ConvPlan &q, hipStream_t s)
{
    if (q.cc == 16)
        return q.W <= 128 ? launch_f32_conv_t<NT, FLIP, 16, 2, SPLIT>(p, q, s) : launch_f32_conv_t<NT, FLIP, 16, kXIter, SPLIT>(p, q, s);
    return q.W <= 128 ? launch_f32_conv_t<NT, FLIP, 8, 2, SPLIT>(p, q, s) : launch_f32_conv_t<NT, FLIP, 8, kXIter, SPLIT>(p, q, s);
}
// Workgroups that share a tile's reduction channels where the tiles are too few to fill the chip (NT = 1 there) and that saves
// more than the second launch takes.  A chunk of channels takes 0.9 us and 0.15 a tap (with eight channels 1.1 and 0.065), the
// launch 1.8 and 0.7 per MB of parts (of 1587 calls 3 that share and 6 that do not are slower by 4 %, 13 at most).  Channels, K,
// B, T: 256 -> 384, 13, 1, 260 50.9 -> 20.7 us; 256, 11, 1, 60 46.5 -> 12.2; 256, 11, 4, 250 47.1 -> 29.7; but 32 -> 16, 1, 2, 165
// 7.0 -> 8.3, so in one part.  From half of the chip on there is nothing to share out.  (Times of this file's kernel; that of f32_terms.hip
// chooses again, at most as many parts as this: the room is asked for before it is known which of them runs.)
int f32_splits(int B, int M, int R, int Tout, int K)
{
    const size_t tiles = (size_t)((M + kTileM - 1) / kTileM) * ((Tout + 31) / 32) * B;
    const int cc = 16 * K <= kRun ? 16 : 8, chunks = (R + cc - 1) / cc;
    const int n = tiles > 128 ? 1 : std::max(1, std::min({(int)(256 / tiles), chunks, 8}));
    const double saved = (chunks - (chunks + n - 1) / n) * (cc == 16 ? 0.9 + 0.15 * K : 1.1 + 0.065 * K);
    return saved > 1.8 + 0.7 * 4e-6 * n * B * M * (double)Tout ? n : 1;
}
size_t f32_split_bytes(int B, int M, int R, int Tout, int K)
{
    const int n = f32_splits(B, M, R, Tout, K);
    return n > 1 ? align_up((size_t)n * B * M * Tout * sizeof(float), 256) : 0;
}

template <bool FLIP>
hipError_t launch_f32_conv(F32ConvParams p, void *part, size_t room, hipStream_t s)
{
    const size_t bytes = f32_split_bytes(p.B, p.M, p.R, p.Tout, p.K);
    p.nsplit = bytes > 0 && part && bytes <= room ? f32_splits(p.B, p.M, p.R, p.Tout, p.K) : 1;
    p.part = (float *)part;
    if (f32_terms_conv_supported(p.R, p.K, p.stride, p.dil)) {
        int nt;
        p.infinities = true;
        f32_terms_plan(p.B, p.M, p.R, p.Tout, p.K, p.nsplit, &nt, &p.nsplit);
        MainKernelTimer timer(s);
        const hipError_t e = launch_f32_terms_conv(p, FLIP, nt, s);
        if (e == hipSuccess && p.nsplit > 1) launch_finish<FLIP>(p, s);
        return e == hipSuccess ? hipGetLastError() : e;
    }
    // the wide tile from two workgroups per CU on (and where its window fits)
    const size_t wide = (size_t)((p.M + kTileM - 1) / kTileM) * ((p.Tout + 63) / 64) * p.B;
    const F32ConvPlan q2 = f32_conv_plan(p.K, p.stride, p.dil, 2, FLIP), q1 = f32_conv_plan(p.K, p.stride, p.dil, 1, FLIP);
    if (wide >= 512 && q2.ok) return launch_f32_conv_nt<2, FLIP, false>(p, q2, s);
    if (!q1.ok) return hipErrorInvalidValue;
    return p.nsplit > 1 ? launch_f32_conv_nt<1, FLIP, true>(p, q1, s) : launch_f32_conv_nt<1, FLIP, false>(p, q1, s);
}

// ---- weight gradient -------------------------------------------------------------------------------------------
// A workgroup owns 64 output channels x 32 input channels x up to 12 taps and every S-th unit of
// (batch item, 64 time steps); the 64 steps of a unit are the reduction: lane half h takes steps 32*h .. 32*h+31, so
// both operands are single LDS words in different banks.  Each of the eight wavefronts has 32 of the output channels and up
// to three taps.  The next unit is held in registers meanwhile.
struct F32WgradParams {
    int B, Cin, Cout, T, To, K, stride, dil, pad;
    int ncot, ncit, ntg, KG, S, nchunk, units;
    int W, x_stride;
    const float *x, *dz;
    const int *len;
    float *part;  // [S][K][Cout][Cin]
};
constexpr int kStep = 64;
constexpr int kTileCi = 32;
constexpr int kDzStride = kStep + 1;

template <int TPW, int XN>
__global__ __launch_bounds__(64 * kConvWaves) void f32_wgrad_kernel(const F32WgradParams p)
{
    extern __shared__ __align__(16) float lds[];
    const int lane = threadIdx.x & 63;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    int v = (int)blockIdx.x;
    const int cit = v % p.ncit; v /= p.ncit;
    const int cot = v % p.ncot; v /= p.ncot;
    const int tg = v % p.ntg;
    const int sp = v / p.ntg;
    const int co0 = cot * kTileM, ci0 = cit * kTileCi, k0 = tg * p.KG, kt = min(p.KG, p.K - k0);
    float *ds = lds, *xs = lds + kTileM * kDzStride;

    const __amdgpu_buffer_rsrc_t rs_dz = rsrc(p.dz, (size_t)p.B * p.Cout * p.To);
    // offsets inside a unit's rows; what lies beyond the tensor or the row is decided per unit
    float dv[8], xv[4][XN];
    const int srow_d = co0 + wave * 8, srow_x = ci0 + wave * 4;
    auto load_unit = [&](int u) {
        const int b = u / p.nchunk, t0 = (u - b * p.nchunk) * kStep;
        int len = p.T;
        if (p.len) {
            const int l = p.len[b];
            len = l < 0 ? 0 : (l < len ? l : len);
        }
        const uint32_t dcol = t0 + lane < p.To ? (uint32_t)(t0 + lane) * 4u : kFar;
#pragma unroll
        for (int i = 0; i < 8; ++i)  // (uniform row offsets; kFar stays beyond the tensor)
            dv[i] = load1(rs_dz, srow_d + i < p.Cout ? dcol + (dcol == kFar ? 0u : (uint32_t)((b * p.Cout + srow_d + i) * p.To) * 4u) : kFar);
        const __amdgpu_buffer_rsrc_t rs_x = rsrc(p.x + (size_t)b * p.Cin * p.T, (size_t)p.Cin * p.T);
        const int tau0 = t0 * p.stride - p.pad + k0 * p.dil;
#pragma unroll
        for (int j = 0; j < XN; ++j) {
            const int c = j * 64 + lane, tau = tau0 + c;
            const bool ok = c < p.W && tau >= 0 && tau < len;
#pragma unroll
            for (int i = 0; i < 4; ++i)
                xv[i][j] = load1(rs_x, ok && srow_x + i < p.Cin ? (uint32_t)((srow_x + i) * p.T + tau) * 4u : kFar);
        }
    };
    auto store_unit = [&]() {
#pragma unroll
        for (int i = 0; i < 8; ++i) ds[(wave * 8 + i) * kDzStride + lane] = dv[i];
#pragma unroll
        for (int j = 0; j < XN; ++j) {
            const int c = j * 64 + lane;
            if (c < p.W) {
#pragma unroll
                for (int i = 0; i < 4; ++i) xs[(wave * 4 + i) * p.x_stride + c] = xv[i][j];
            }
        }
    };

    f32x16 acc[TPW], sum[TPW];
#pragma unroll
    for (int j = 0; j < TPW; ++j)
#pragma unroll
        for (int r = 0; r < 16; ++r) acc[j][r] = sum[j][r] = 0.f;

    const int l32 = lane & 31, h = lane >> 5, wt = wave & 3, wm = wave >> 2;
    const float *a = ds + (32 * wm + l32) * kDzStride + 32 * h;
    int off[TPW];  // taps wt, wt + 4, ...; an absent one repeats the group's last tap and is not written
#pragma unroll
    for (int j = 0; j < TPW; ++j) off[j] = l32 * p.x_stride + 32 * h * p.stride + min(wt + 4 * j, kt - 1) * p.dil;
    if (sp < p.units) load_unit(sp);
    for (int u = sp; u < p.units; u += p.S) {
        __syncthreads();
        store_unit();
        __syncthreads();
        if (u + p.S < p.units) load_unit(u + p.S);
        float ra[2][4], rb[2][TPW][4];  // four steps at a time, the next four read while these multiply
        auto read = [&](int s, float(&fa)[4], float(&fb)[TPW][4]) {
#pragma unroll
            for (int e = 0; e < 4; ++e) {
                fa[e] = a[s + e];
#pragma unroll
                for (int j = 0; j < TPW; ++j) fb[j][e] = xs[off[j] + (s + e) * p.stride];
            }
        };
        auto multiply = [&](const float(&fa)[4], const float(&fb)[TPW][4]) {
#pragma unroll
            for (int e = 0; e < 4; ++e)
#pragma unroll
                for (int j = 0; j < TPW; ++j) acc[j] = __builtin_amdgcn_mfma_f32_32x32x2f32(fa[e], fb[j][e], acc[j], 0, 0, 0);
        };
        read(0, ra[0], rb[0]);
#pragma unroll
        for (int s = 0; s < 32; s += 8) {
            read(s + 4, ra[1], rb[1]);
            multiply(ra[0], rb[0]);
            if (s + 8 < 32) read(s + 8, ra[0], rb[0]);
            multiply(ra[1], rb[1]);
        }
#pragma unroll
        for (int j = 0; j < TPW; ++j)
#pragma unroll
            for (int r = 0; r < 16; ++r) {
                sum[j][r] += acc[j][r];
                acc[j][r] = 0.f;
            }
    }
    const int ci = ci0 + l32;
    if (ci >= p.Cin) return;
#pragma unroll
    for (int j = 0; j < TPW; ++j) {
        const int tap = wt + 4 * j;
        if (tap >= kt) continue;
#pragma unroll
        for (int r = 0; r < 16; ++r) {
            const int co = co0 + wm * 32 + 8 * (r >> 2) + 4 * h + (r & 3);
            if (co < p.Cout) p.part[(((size_t)sp * p.K + k0 + tap) * p.Cout + co) * p.Cin + ci] = sum[j][r];
        }
    }
}

struct F32WgradPlan {
    bool ok, terms;  // terms: on the kernel of f32_terms.hip
    int ntg, KG, TPW, S, nchunk, units, W, x_stride;
};
// most: parts that there is room for; fewer than this file's kernel takes are no reason to leave it (its parts are what is asked for at least)
F32WgradPlan f32_wgrad_plan(const Geom &g, long most = 8)
{
    F32WgradPlan q = {};
    if (g.K > 255) return q;  // the reduction kernel's LDS tile
    q.ntg = (g.K + 11) / 12;
    q.KG = (g.K + q.ntg - 1) / q.ntg;
    q.TPW = (q.KG + 3) / 4;
    const long W = (long)(kStep - 1) * g.stride + (long)(q.KG - 1) * g.dil + 1;
    if (W > 64 * kXIter) return q;
    q.W = (int)W;
    q.x_stride = (q.W + 31) / 32 * 32 + 1;  // 1 modulo 32: both lane halves of a stride-1 read hit different banks
    q.nchunk = (g.To + kStep - 1) / kStep;
    q.units = g.B * q.nchunk;
    const long tiles = (long)((g.Cout + kTileM - 1) / kTileM) * ((g.Cin + kTileCi - 1) / kTileCi) * q.ntg;
    // one workgroup per CU (256 of them), and no more than eight partial results to write and read back
    long S = 256 / tiles;
    if (S > 8) S = 8;
    if (S > q.units) S = q.units;
    if (S < 1) S = 1;
    const long each = (q.units + S - 1) / S;  // no split whose last round is nearly empty
    q.S = (int)((q.units + each - 1) / each);
    q.ok = true;
    if (f32_terms_wgrad_supported(g)) {
        // that kernel's tiles are half as large: where they take a round more for little work this one is faster (384 channels, K=13,
        // B=1, T=50: 20.0 us here, 23.3 there; T=300: 37.8, 35.1)
        double cost;
        const int parts = f32_terms_wgrad_parts(g, (int)std::max(most, (long)q.S), &cost);
        const double rounds = (double)((tiles * q.S + 255) / 256), mb = 4e-6 * g.Cout * g.Cin * (double)g.K;
        q.terms = cost < rounds * (8.2 + each * (0.8 + 1.8 * q.TPW)) + 0.5 * mb * q.S;
        if (q.terms) q.S = parts;
    }
    return q;
}

// The matrix cores pay from one block of rows, columns and reduction on; smaller layers are a launch either way.
// (And the staging loads have 32-bit offsets.)
bool worth_it(const Geom &g)
{
    const size_t lim = ((size_t)1 << 31) / sizeof(float);
    return g.Cout >= 16 && g.Cin >= 16 && g.To >= 16 && g.T >= 16 && (size_t)g.Cout * g.Cin * g.K < lim &&
           (size_t)g.Cin * g.T < lim && (size_t)g.B * g.Cout * g.To < lim;
}

}  // namespace

bool f32_fwd_supported(const Geom &g) { return worth_it(g) && f32_conv_plan(g.K, g.stride, g.dil, 1, false).ok; }
bool f32_dgrad_supported(const Geom &g) { return worth_it(g) && g.stride == 1 && f32_conv_plan(g.K, 1, g.dil, 1, true).ok; }
bool f32_wgrad_supported(const Geom &g) { return worth_it(g) && f32_wgrad_plan(g).ok; }

size_t f32_fwd_part_bytes(const Geom &g) { return f32_split_bytes(g.B, g.Cout, g.Cin, g.To, g.K); }
size_t f32_dgrad_part_bytes(const Geom &g) { return f32_split_bytes(g.B, g.Cin, g.Cout, g.T, g.K); }

hipError_t launch_f32_fwd(const Geom &g, const float *x, const float *w, const float *scale, const float *shift,
                          const float *res, float *y, bool relu, void *part, size_t room, hipStream_t s)
{
    F32ConvParams p = {};
    p.B = g.B; p.M = g.Cout; p.R = g.Cin; p.Tin = g.T; p.Tout = g.To;
    p.K = g.K; p.stride = g.stride; p.dil = g.dil; p.padL = g.pad;
    p.relu = relu ? 1 : 0;
    p.in = x; p.w = w; p.scale = scale; p.shift = shift; p.res = res; p.out = y;
    p.len_in = g.len;
    return launch_f32_conv<false>(p, part, room, s);
}

hipError_t launch_f32_dgrad(const Geom &g, const float *gy, const float *scale, const float *w, float *dx, bool accumulate,
                            void *part, size_t room, hipStream_t s)
{
    F32ConvParams p = {};
    p.B = g.B; p.M = g.Cin; p.R = g.Cout; p.Tin = g.To; p.Tout = g.T;
    p.K = g.K; p.stride = 1; p.dil = g.dil; p.padL = g.dil * (g.K - 1) - g.pad;
    p.in = gy; p.w = w; p.rscale = scale; p.out = dx;
    p.res = accumulate ? dx : nullptr;  // every thread reads the element it then writes
    p.len_out = g.len;
    return launch_f32_conv<true>(p, part, room, s);
}

namespace {
size_t wgrad_part(const Geom &g) { return (size_t)g.K * g.Cout * g.Cin * sizeof(float); }
// (the parts' room is rounded up to 256 bytes, so what there is counts rounded down)
F32WgradPlan wgrad_plan_within(const Geom &g, size_t room) { return f32_wgrad_plan(g, (long)std::min<size_t>(8, room / 256 * 256 / wgrad_part(g))); }
}  // namespace

size_t f32_wgrad_part_bytes(const Geom &g, size_t room) { return align_up(wgrad_plan_within(g, room).S * wgrad_part(g), 256); }

hipError_t launch_f32_wgrad(const Geom &g, const float *x, const float *dz, const float *scale, float *dw, bool accumulate,
                            void *part, size_t room, hipStream_t s)
{
    const F32WgradPlan q = wgrad_plan_within(g, room);
    if (!q.ok) return hipErrorInvalidValue;
    const DefinedDw fix = {true, x, dz, nullptr, q.terms};
    if (q.terms) {
        hipError_t e;
        {
            MainKernelTimer timer(s);
            e = launch_f32_terms_wgrad(g, q.S, x, dz, (float *)part, s);
        }
        return e == hipSuccess ? launch_wgrad_reduce(g, (const float *)part, dw, scale, q.S, accumulate, s, &g, &fix) : e;
    }
    F32WgradParams p = {};
    p.B = g.B; p.Cin = g.Cin; p.Cout = g.Cout; p.T = g.T; p.To = g.To;
    p.K = g.K; p.stride = g.stride; p.dil = g.dil; p.pad = g.pad;
    p.ncot = (g.Cout + kTileM - 1) / kTileM;
    p.ncit = (g.Cin + kTileCi - 1) / kTileCi;
    p.ntg = q.ntg; p.KG = q.KG; p.S = q.S; p.nchunk = q.nchunk; p.units = q.units;
    p.W = q.W; p.x_stride = q.x_stride;
    p.x = x; p.dz = dz; p.len = g.len; p.part = (float *)part;
    const unsigned grid = (unsigned)((size_t)p.ncot * p.ncit * p.ntg * p.S);
    const size_t lds = ((size_t)kTileM * kDzStride + (size_t)kTileCi * p.x_stride) * sizeof(float);
    {
        MainKernelTimer timer(s);
        auto go = [&](auto kern) { hipLaunchKernelGGL(kern, dim3(grid), dim3(64 * kConvWaves), lds, s, p); };
        if (q.W <= 128) {
            if (q.TPW == 1) go(f32_wgrad_kernel<1, 2>);
            else if (q.TPW == 2) go(f32_wgrad_kernel<2, 2>);
            else go(f32_wgrad_kernel<3, 2>);
        } else {
            if (q.TPW == 1) go(f32_wgrad_kernel<1, kXIter>);
            else if (q.TPW == 2) go(f32_wgrad_kernel<2, kXIter>);
            else go(f32_wgrad_kernel<3, kXIter>);
        }
        const hipError_t e = hipGetLastError();
        if (e != hipSuccess) return e;
    }
    return launch_wgrad_reduce(g, (const float *)part, dw, scale, q.S, accumulate, s, &g, &fix);
}

}  // namespace nm
