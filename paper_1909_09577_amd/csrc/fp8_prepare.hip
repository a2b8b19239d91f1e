// What an 8-bit call needs before its main kernels, in one launch: the weights in fragment order as codes, and the codes of one or
// two activation tensors.
//
// Bound: memory, and in small calls the latency of one block.  Packing a weight block was 15 to 30 us whatever the batch
// (768 channels, K=25: 18.8 forward, 29.5 flipped): bytes gathered one by one from LDS, an integer division per element, one
// workgroup of 102 KB of LDS per CU.  A thread now owns four channels of a row with all their taps: it reads them as whole
// words, makes four codes of a tap at a time and stores them straight to the fragments, where the threads of a wavefront
// have 256 contiguous bytes.  Measured, packing and passes over the activations together: 768 channels, K=25, B=32, T=800 forward 33 -> 24,
// backward 74.6 -> 47.6 (137 MB of activations); 512 -> 640, K=21, B=8, T=63 13.8 -> 6.4 and 28.3 -> 9.5.
#include "fp8_prepare.h"

namespace nm {
namespace {

typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));
typedef uint32_t u32x2 __attribute__((ext_vector_type(2)));

constexpr int kThreads = 256;
constexpr int kRowBytes = 80;    // LDS row of 64 codes: 64 B + 16 B pad
constexpr int kQuantT = 128;     // time steps of a block
constexpr int kPackRows = 16;    // rows (forward: output channels, flipped: input channels) of a block; 64 channels of the other side

struct QuantArgs {
    const bf16_t *src, *y;
    const float *scale;
    unsigned char *codes;
    bf16_t *copy;
    int C, T, Tp, pad, vec, nx;  // nx: blocks along time
};
struct PrepareArgs {
    unsigned npack, nfirst;
    const bf16_t *w;
    const float *scale, *row_scales;
    unsigned char *wq;
    int Cin, Cout;
    QuantArgs q[2];
};

// T % 8 == 0 and 16-byte aligned tensors: 16-byte loads along T, the transposition to time-major rows goes through LDS.  A block
// converts 64 channels x 128 time steps.  Thread (g, tv) loads 8 time steps of the four channels 4g .. 4g+3 and writes eight dwords
// (four channel codes of one time step each); then every thread copies 16-byte pieces of finished rows out.  The first and
// the last block of a row of blocks also write the zero rows before time 0 and behind time T.
__device__ __forceinline__ void quant_vec_block(const QuantArgs &q, int bx, int c, int b, unsigned char *tile)
{
    const int nck = q.C / 64, T = q.T;
    const int t0 = bx * kQuantT;
    const int g4 = threadIdx.x & 15, tv = threadIdx.x >> 4;
    const float inv = 1.0f / q.scale[0];
    const int t = t0 + tv * 8;
    if (t < T) {
        const size_t off = ((size_t)b * q.C + c * 64 + g4 * 4) * T + t;
        u32x4 raw[4];
#pragma unroll
        for (int j = 0; j < 4; ++j) raw[j] = *reinterpret_cast<const u32x4 *>(q.src + off + (size_t)j * T);
        if (q.y) {
            u32x4 yv[4];
#pragma unroll
            for (int j = 0; j < 4; ++j) yv[j] = *reinterpret_cast<const u32x4 *>(q.y + off + (size_t)j * T);
#pragma unroll
            for (int j = 0; j < 4; ++j) raw[j] = masked_grad8(raw[j], yv[j]);
        }
        if (q.copy) {
#pragma unroll
            for (int j = 0; j < 4; ++j) *reinterpret_cast<u32x4 *>(q.copy + off + (size_t)j * T) = raw[j];
        }
#pragma unroll
        for (int e = 0; e < 8; ++e) {
            float v[4];
#pragma unroll
            for (int j = 0; j < 4; ++j) v[j] = bf16_to_f32((bf16_t)((raw[j][e >> 1] >> (16 * (e & 1))) & 0xffffu)) * inv;
            *reinterpret_cast<uint32_t *>(tile + (tv * 8 + e) * kRowBytes + g4 * 4) = e4m3_pack4(v[0], v[1], v[2], v[3]);
        }
    }
    __syncthreads();
    unsigned char *const slab = q.codes + ((size_t)b * nck + c) * q.Tp * 64;
    const int rows = min(kQuantT, T - t0);
    for (int i = threadIdx.x; i < rows * 4; i += kThreads) {
        const int row = i >> 2, p = i & 3;
        *reinterpret_cast<u32x4 *>(slab + (size_t)(t0 + row + q.pad) * 64 + p * 16) = *reinterpret_cast<const u32x4 *>(tile + row * kRowBytes + p * 16);
    }
    const u32x4 zero = {0u, 0u, 0u, 0u};
    if (bx == 0)
        for (int i = threadIdx.x; i < q.pad * 4; i += kThreads) *reinterpret_cast<u32x4 *>(slab + (size_t)i * 16) = zero;
    if (bx == q.nx - 1)
        for (int i = threadIdx.x; i < (q.Tp - T - q.pad) * 4; i += kThreads)
            *reinterpret_cast<u32x4 *>(slab + (size_t)(T + q.pad) * 64 + (size_t)i * 16) = zero;
}

// The same element by element (any T and alignment): thread (tl, cg) has row 64*bx + tl, channels 16*cg .. 16*cg+15.
__device__ __forceinline__ void quant_block(const QuantArgs &q, int bx, int c, int b)
{
    const int tl = threadIdx.x & 63, cg = threadIdx.x >> 6;
    const int r = bx * 64 + tl;
    if (r >= q.Tp) return;
    const int t = r - q.pad;
    u32x4 out = {0u, 0u, 0u, 0u};
    if (t >= 0 && t < q.T) {
        const float inv = 1.0f / q.scale[0];
        const size_t off = ((size_t)b * q.C + c * 64 + cg * 16) * q.T + t;
        bf16_t g[16], yv[16];
#pragma unroll
        for (int j = 0; j < 16; ++j) g[j] = q.src[off + (size_t)j * q.T];
        if (q.y) {
#pragma unroll
            for (int j = 0; j < 16; ++j) yv[j] = q.y[off + (size_t)j * q.T];
#pragma unroll
            for (int j = 0; j < 16; ++j) g[j] = (uint32_t)yv[j] - 1u < 0x7f80u ? g[j] : (bf16_t)0;
        }
        if (q.copy) {
#pragma unroll
            for (int j = 0; j < 16; ++j) q.copy[off + (size_t)j * q.T] = g[j];
        }
#pragma unroll
        for (int j = 0; j < 4; ++j)
            out[j] = e4m3_pack4(bf16_to_f32(g[4 * j]) * inv, bf16_to_f32(g[4 * j + 1]) * inv, bf16_to_f32(g[4 * j + 2]) * inv,
                                bf16_to_f32(g[4 * j + 3]) * inv);
    }
    *reinterpret_cast<u32x4 *>(q.codes + (((size_t)b * (q.C / 64) + c) * q.Tp + r) * 64 + cg * 16) = out;
}

// A block packs 16 rows x 64 channels x K taps: the raw weights go to LDS as they lie in memory (forward: 16 rows of 64*K elements,
// flipped: 64 of 16*K), thread (channel quad of a half, row, half) takes four channels of its row.
template <int K, bool FLIP>
__device__ __forceinline__ void pack_block(const PrepareArgs &a, unsigned blk, unsigned char *raw)
{
    constexpr int kLines = FLIP ? 64 : kPackRows, kPieces = (FLIP ? 2 : 8) * K;  // 16-byte pieces of a line
    constexpr int kPitch = 16 * kPieces + 16;
    constexpr int kAll = kLines * kPieces, kLoads = (kAll + kThreads - 1) / kThreads;
    const int chunks = (FLIP ? a.Cout : a.Cin) / 64;
    const int c = (int)(blk % chunks), row0 = (int)(blk / chunks) * kPackRows;
    const bf16_t *base = FLIP ? a.w + ((size_t)c * 64 * a.Cin + row0) * K : a.w + ((size_t)row0 * a.Cin + c * 64) * K;
    u32x4 v[kLoads];
#pragma unroll
    for (int i = 0; i < kLoads; ++i) {
        const int p = min(i * kThreads + (int)threadIdx.x, kAll - 1), line = p / kPieces, at = p - line * kPieces;
        v[i] = *reinterpret_cast<const u32x4 *>(base + (size_t)line * a.Cin * K + at * 8);
    }
#pragma unroll
    for (int i = 0; i < kLoads; ++i) {
        const int p = min(i * kThreads + (int)threadIdx.x, kAll - 1), line = p / kPieces, at = p - line * kPieces;
        *reinterpret_cast<u32x4 *>(raw + line * kPitch + at * 16) = v[i];
    }
    const int quad = threadIdx.x & 7, r = (threadIdx.x >> 3) & 15, half = threadIdx.x >> 7;
    const int row = row0 + r, ch = 32 * half + 4 * quad;
    const float inv = 1.0f / a.row_scales[row];
    float f[4];
#pragma unroll
    for (int j = 0; j < 4; ++j) f[j] = FLIP && a.scale ? a.scale[c * 64 + ch + j] : 1.f;
    unsigned char *dst = a.wq + (((size_t)(row >> 6) * chunks + c) * K * 2 + ((row >> 5) & 1)) * 2048 + (32 * half + (row & 31)) * 32 + 4 * quad;
    __syncthreads();
    if constexpr (FLIP) {
        // K elements of a channel from an odd or even one on: whole words, moved down by the odd element
        constexpr int kWords = (K + 1) / 2;
        uint32_t d[4][kWords];
        const uint32_t odd = (uint32_t)(r * K & 1) * 16;
#pragma unroll
        for (int j = 0; j < 4; ++j) {
            const uint32_t *src = reinterpret_cast<const uint32_t *>(raw + (ch + j) * kPitch) + (r * K >> 1);
#pragma unroll
            for (int i = 0; i < kWords; ++i) d[j][i] = src[i];
#pragma unroll
            for (int i = 0; i < kWords; ++i) d[j][i] = __builtin_amdgcn_alignbit(i + 1 < kWords ? d[j][i + 1] : 0u, d[j][i], odd);
        }
#pragma unroll
        for (int k = 0; k < K; ++k) {
            float e[4];
#pragma unroll
            for (int j = 0; j < 4; ++j) e[j] = __uint_as_float(k & 1 ? d[j][k >> 1] & 0xffff0000u : d[j][k >> 1] << 16) * f[j] * inv;
            *reinterpret_cast<uint32_t *>(dst + (size_t)(K - 1 - k) * 4096) = e4m3_pack4(e[0], e[1], e[2], e[3]);
        }
    } else {
        u32x2 d[K];
#pragma unroll
        for (int i = 0; i < K; ++i) d[i] = *reinterpret_cast<const u32x2 *>(raw + r * kPitch + ch * K * 2 + 8 * i);
#pragma unroll
        for (int k = 0; k < K; ++k) {
            float e[4];
#pragma unroll
            for (int j = 0; j < 4; ++j) {
                const int x = j * K + k;
                const uint32_t word = d[x / 4][(x / 2) & 1];
                e[j] = __uint_as_float(x & 1 ? word & 0xffff0000u : word << 16) * inv;
            }
            *reinterpret_cast<uint32_t *>(dst + (size_t)k * 4096) = e4m3_pack4(e[0], e[1], e[2], e[3]);
        }
    }
}

template <int K, bool FLIP>
__global__ __launch_bounds__(kThreads) void fp8_prepare_kernel(const PrepareArgs a)
{
    extern __shared__ __align__(16) unsigned char smem[];
    unsigned blk = blockIdx.x;
    if (blk < a.npack) {
        if constexpr (K > 0) pack_block<K, FLIP>(a, blk, smem);
        return;
    }
    blk -= a.npack;
    const bool second = blk >= a.nfirst;
    const QuantArgs &q = second ? a.q[1] : a.q[0];
    blk -= second ? a.nfirst : 0;
    const int bx = (int)(blk % (unsigned)q.nx), slab = (int)(blk / (unsigned)q.nx), nck = q.C / 64, b = slab / nck, c = slab - b * nck;
    if (q.vec) quant_vec_block(q, bx, c, b, smem);
    else quant_block(q, bx, c, b);
}

QuantArgs quant_args(const Fp8Quant &q, unsigned *blocks)
{
    QuantArgs a = {};
    if (!q.src) {
        *blocks = 0;
        return a;
    }
    a.src = (const bf16_t *)q.src; a.y = (const bf16_t *)q.y; a.scale = q.scale; a.codes = q.codes; a.copy = (bf16_t *)q.copy;
    a.C = q.C; a.T = q.T; a.Tp = q.Tp; a.pad = q.pad;
    a.vec = q.T % 8 == 0 && !(((uintptr_t)q.src | (uintptr_t)q.y | (uintptr_t)q.copy) & 15);
    a.nx = a.vec ? (q.T + kQuantT - 1) / kQuantT : (q.Tp + 63) / 64;
    *blocks = (unsigned)a.nx * (unsigned)(q.C / 64) * (unsigned)q.B;
    return a;
}

template <int K, bool FLIP>
void launch(const PrepareArgs &a, unsigned blocks, hipStream_t s)
{
    constexpr size_t pack = K == 0 ? 0 : (FLIP ? 64 * (32 * K + 16) : kPackRows * (128 * K + 16)), quant = kQuantT * kRowBytes;
    static_assert(pack <= 64 * 1024, "LDS without an opt-in");
    hipLaunchKernelGGL((fp8_prepare_kernel<K, FLIP>), dim3(blocks), dim3(kThreads), pack > quant ? pack : quant, s, a);
}

}  // namespace

hipError_t fp8_prepare(const Fp8Pack &pack, const Fp8Quant &first, const Fp8Quant &second, hipStream_t s)
{
    PrepareArgs a = {};
    unsigned nsecond;
    a.q[0] = quant_args(first, &a.nfirst);
    a.q[1] = quant_args(second, &nsecond);
    if (pack.w) {
        a.w = (const bf16_t *)pack.w; a.scale = pack.scale; a.row_scales = pack.row_scales; a.wq = pack.out;
        a.Cin = pack.Cin; a.Cout = pack.Cout;
        a.npack = (unsigned)((pack.flip ? pack.Cin : pack.Cout) / kPackRows) * (unsigned)((pack.flip ? pack.Cout : pack.Cin) / 64);
    }
    const unsigned blocks = a.npack + a.nfirst + nsecond;
    if (blocks == 0) return hipSuccess;
    if (!pack.w) launch<0, false>(a, blocks, s);
    else if (pack.K == 17) pack.flip ? launch<17, true>(a, blocks, s) : launch<17, false>(a, blocks, s);
    else if (pack.K == 21) pack.flip ? launch<21, true>(a, blocks, s) : launch<21, false>(a, blocks, s);
    else if (pack.K == 25) pack.flip ? launch<25, true>(a, blocks, s) : launch<25, false>(a, blocks, s);
    else if (pack.K == 29) pack.flip ? launch<29, true>(a, blocks, s) : launch<29, false>(a, blocks, s);
    else return hipErrorInvalidValue;
    return hipGetLastError();
}

}  // namespace nm
