// Calls of few tiles on the weights as they lie in memory: forward pass and stride-1 input gradient, the encoder's filters.
//
// One utterance of 6 seconds at 768 channels, K=25 is 17.7 GFLOP and 29 MB of weights.  Packing those weights into
// fragment order first (prepack_kernel) reads and writes them once more and is a launch of its own: 15 us of the 42 us that
// such a call took on conv_split_kernel, 4 of the 19 us of 256 channels, K=11, 200 steps.  Here a workgroup cuts the
// fragments out of w itself:
//   * a chunk is 16 reduction channels, all taps, 64 output channels.  It is copied to LDS as it lies in memory, in whole
//     KiB per wavefront (buffer loads to LDS: no registers, requested a chunk ahead, between the taps).  From there a lane
//     takes four channels x all taps of a row (forward), resp. eight neighbouring (row, tap) elements of four channels
//     (input gradient, times scale), and writes them back in A-fragment order, four channels of a tap at a time.  (Cutting
//     them out of memory directly, 16 bytes per lane at 2-byte aligned addresses, kept the address unit busy for 92
//     cycles a load, and 64 with the rows in neighbouring lanes: 58 us at the sizes above.)
//   * the four wavefronts share the fragments; each has a column (NT*32 time steps of one batch item) of its own and
//     stages its window of the input: (8 time steps, octet of channels) per lane, eight loads of consecutive time steps
//     at any 2-byte aligned address (so rows of any length need no copy), an 8x8 transposition in registers, LDS rows of
//     [time][16 channels].  Eight time rows take 272 bytes, so that neighbouring lanes hit different banks.
//   * the reduction channels are split over nsplit >= 2 workgroups per tile; split_reduce_kernel adds the parts in a fixed
//     order and finishes.
// What bounds it: LDS reads (7 fragments per 10 MFMAs at NT = 5: 23 ns an MFMA against 15 at this clock), and latency in
// small calls.  The taps are unrolled, and the loads to LDS are buffer loads: behind one of the global form the
// compiler waits for all LDS reads in flight (28 ns an MFMA).  Measured, packing and all launches included, replayed in a
// graph, before -> now: 256 channels K=11, 200 steps 19.3 -> 10.9 us; 512 K=17, 600 steps 26 -> 21; 768 K=25, 600 steps 42 -> 35,
// its input gradient 53 -> 45; 384 -> 512 K=17, B=3, 72 steps 20 -> 16.
#include "../../include/nm_conv1d.h"
#include "conv_tile.h"

#include <string.h>

#include <algorithm>

namespace nm {
namespace {

constexpr int kUnpackedChunk = 16;       // reduction channels per chunk
constexpr int kGroupBytes = 272; // LDS bytes of eight time rows of a window

// an 8x8 block of 16-bit elements, rows in: column j comes out as one register quadruple
__device__ __forceinline__ u32x4 block_column(const u32x4 (&r)[8], int j)
{
    u32x4 c;
#pragma unroll
    for (int i = 0; i < 4; ++i)
        c[i] = j & 1 ? zip_hi16(r[2 * i][j >> 1], r[2 * i + 1][j >> 1]) : zip_lo16(r[2 * i][j >> 1], r[2 * i + 1][j >> 1]);
    return c;
}

// 16 bytes at a 2-byte aligned address, base uniform
__device__ __forceinline__ u32x4 load16_at(const bf16_t *base, uint32_t byte_off)
{
    u32x4 v;
    __builtin_memcpy(&v, reinterpret_cast<const unsigned char *>(base) + byte_off, 16);
    return v;
}

typedef uint32_t u32x2 __attribute__((ext_vector_type(2)));
typedef __attribute__((address_space(3))) uint32_t lds_u32;
constexpr int kTapBytes = 2048;      // fragments of one tap: 64 rows x 16 channels
constexpr int kAllVmem = 0x0f70;     // s_waitcnt: vmcnt(0) alone

struct UnpackedParams {
    ConvGemmParams c;     // nitems: 8-row groups of a window; ntt, nmt, nsplit, part as for conv_split_kernel; no packed weights
    const bf16_t *w;      // [M][R][K], of an input gradient [R][M][K]
    const float *rscale;  // factor of reduction channel r, folded into the weights (flipped ones only; NULL: 1)
    int ncolgroups;
};

template <int NT, int K, bool FLIP>
__global__ __launch_bounds__(kThreads, NT <= (FLIP ? 2 : 3) ? 2 : 1) void conv_unpacked_kernel(const UnpackedParams q)
{
    extern __shared__ __align__(16) unsigned char smem[];
    const ConvGemmParams &p = q.c;
    const int lane = threadIdx.x & 63;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    constexpr int TN = NT * 32;
    const int nch = p.R / kUnpackedChunk, ncols = p.B * p.ntt;
    // workgroups that read the same weights sit on one XCD (blockIdx % 8) where the counts divide
    const int ncombo = p.nmt * p.nsplit;
    int combo, group;
    if (ncombo % 8 == 0) {
        const int j = (int)blockIdx.x >> 3;
        group = j % q.ncolgroups;
        combo = (j / q.ncolgroups) * 8 + ((int)blockIdx.x & 7);
    } else {
        combo = (int)blockIdx.x % ncombo;
        group = (int)blockIdx.x / ncombo;
    }
    const int mt = combo / p.nsplit, split = combo - mt * p.nsplit;
    const int c0 = (int)((long)split * nch / p.nsplit), c1 = (int)((long)(split + 1) * nch / p.nsplit);
    const int col = group * kWaves + wave;
    const bool there = col < ncols;
    const int b = there ? col / p.ntt : 0, t0 = there ? (col - b * p.ntt) * TN : 0;

    const int ws = t0 - p.padL, ws_al = (ws >> 3) * 8;
    const int tlen = __builtin_amdgcn_readfirstlane(clipped_len(p.len_in, b, p.Tin));
    // a column that lies wholly in the padding of its batch item: its sums are zero
    const int out_end = __builtin_amdgcn_readfirstlane(clipped_len(p.len_out, b, p.Tout));
    const bool live = there && ws < tlen && t0 < out_end;

    unsigned char *const frags = smem;
    unsigned char *const raw = smem + K * kTapBytes;
    unsigned char *const xwin = smem + 2 * K * kTapBytes + (size_t)wave * p.nitems * kGroupBytes;

    // (input gradient) the factors of this workgroup's channels
    float *const factors = reinterpret_cast<float *>(smem + 2 * K * kTapBytes + (size_t)kWaves * p.nitems * kGroupBytes);
    if (FLIP && q.rscale)
        for (int i = (int)threadIdx.x; i < (c1 - c0) * kUnpackedChunk; i += kThreads) factors[i] = q.rscale[c0 * kUnpackedChunk + i];

    // ---- the window of the input: this lane's group of eight time steps and octet of channels
    const int grp = lane & 31, oct = lane >> 5;
    const bool mine = live && grp < p.nitems;
    const int t = ws_al + 8 * grp;
    // a group that runs over the end of the tensor is read from its last 16 bytes and shifted down
    const uint32_t tensor = (uint32_t)p.B * p.R * p.Tin;
    const bool tail = __builtin_amdgcn_readfirstlane(b == p.B - 1 && p.Tin % 8 != 0);
    u32x4 xr[8];
    auto x_at = [&](int c) {
        const uint32_t row = (uint32_t)b * p.R + c * kUnpackedChunk + oct * 8;
        return row * (uint32_t)p.Tin + (t < 0 || t >= tlen || !mine ? 0u : (uint32_t)t);
    };
    auto x_load = [&](uint32_t e0, int i) __attribute__((always_inline)) {  // channel i of the octet
        uint32_t e = e0 + (uint32_t)i * p.Tin;
        if (tail) e = min(e, tensor - 8);
        xr[i] = load16_at(p.in, e * 2);
    };
    auto x_write = [&](int c) __attribute__((always_inline)) {
        if (tail) {
            const uint32_t e0 = x_at(c);
#pragma unroll
            for (int i = 0; i < 8; ++i) {
                const uint32_t e = e0 + (uint32_t)i * p.Tin;
                const uint32_t sh = e + 8 > tensor ? e + 8 - tensor : 0;
                u32x4 v = xr[i];
                if (sh & 4) v = u32x4{v[2], v[3], 0u, 0u};
                if (sh & 2) v = u32x4{v[1], v[2], v[3], 0u};
                if (sh & 1) v = u32x4{(v[0] >> 16) | (v[1] << 16), (v[1] >> 16) | (v[2] << 16), (v[2] >> 16) | (v[3] << 16), v[3] >> 16};
                xr[i] = v;
            }
        }
        if (!mine) return;
        const int nv = t < 0 ? 0 : tlen - t;  // valid steps of the group
#pragma unroll
        for (int j = 0; j < 8; ++j) {
            u32x4 v = block_column(xr, j);
            if (j >= nv) v = u32x4{0u, 0u, 0u, 0u};
            *reinterpret_cast<u32x4 *>(xwin + grp * kGroupBytes + j * 32 + oct * 16) = v;
        }
    };

    // ---- the weights
    const __amdgpu_buffer_rsrc_t rs_w = __builtin_amdgcn_make_buffer_rsrc((void *)q.w, 0, (int)((size_t)p.M * p.R * K * 2), 0x00020000);
    const int rows = p.M - mt * kTileM < kTileM ? p.M - mt * kTileM : kTileM;
    // A chunk goes to LDS as it lies in memory: 64 rows of 16*K contiguous elements, of an input gradient 16 of 64*K.
    auto raw_request = [&](int c, int i) __attribute__((always_inline)) {  // the wavefront's i-th KiB
        const int n = i * kWaves + wave;
        if (n >= 2 * K) return;
        constexpr int pieces = FLIP ? 8 * K : 2 * K;  // 16-byte pieces of a row
        const int piece = n * 64 + lane, row = piece / pieces, at = piece - row * pieces;
        uint32_t base, off;
        if (FLIP) {
            base = (uint32_t)(c * kUnpackedChunk * p.M + mt * kTileM) * (uint32_t)(2 * K);
            off = (uint32_t)row * (uint32_t)(p.M * K * 2) + (uint32_t)min(at, rows * K / 8 - 1) * 16u;
        } else {
            base = (uint32_t)(mt * kTileM * p.R + c * kUnpackedChunk) * (uint32_t)(2 * K);
            off = (uint32_t)min(row, rows - 1) * (uint32_t)(p.R * K * 2) + (uint32_t)at * 16u;
        }
        __builtin_amdgcn_raw_ptr_buffer_load_lds(rs_w, (lds_u32 *)(raw + n * 1024), 16, off, base, 0, 0);
    };
    // Forward: it comes back four channels x all taps per lane, and each tap's four channels go to the fragments.
    auto raw_to_frags = [&]() {
        const int item = (int)threadIdx.x, row = item >> 2, o = (item >> 1) & 1;
        const unsigned char *src = raw + item * (8 * K);
        u32x2 d[K];
#pragma unroll
        for (int j = 0; j < K; ++j) d[j] = *reinterpret_cast<const u32x2 *>(src + 8 * j);
        const int at = (row >> 5) * 1024 + o * 512 + (((row & 31) ^ (o << 3)) * 16) + (item & 1) * 8;
        auto half = [&](int f) { return d[f / 4][(f / 2) & 1]; };  // the register that element f of the 4*K lies in
        auto pair = [&](int f0, int f1) {
            const uint32_t sel = (f0 & 1 ? 0x0302u : 0x0100u) | (f1 & 1 ? 0x07060000u : 0x05040000u);
            return __builtin_amdgcn_perm(half(f1), half(f0), sel);
        };
#pragma unroll
        for (int k = 0; k < K; ++k)
            *reinterpret_cast<u32x2 *>(frags + k * kTapBytes + at) = u32x2{pair(k, K + k), pair(2 * K + k, 3 * K + k)};
    };
    // Input gradient: a lane owns eight neighbouring (row, tap) elements of four channels.
    constexpr int kItems = (32 * K + kThreads - 1) / kThreads;
    auto flip_to_frags = [&](int c) __attribute__((always_inline)) {
#pragma unroll
        for (int it = 0; it < kItems; ++it) {
            const int idx = (int)threadIdx.x + kThreads * it, quad = idx / (8 * K), g = idx - quad * (8 * K);
            if (quad >= 4) break;
            u32x4 v[4];
#pragma unroll
            for (int i = 0; i < 4; ++i) v[i] = *reinterpret_cast<const u32x4 *>(raw + ((quad * 4 + i) * (8 * K) + g) * 16);
            if (q.rscale) {
#pragma unroll
                for (int i = 0; i < 4; ++i) {
                    const float f = factors[(c - c0) * kUnpackedChunk + 4 * quad + i];
#pragma unroll
                    for (int d = 0; d < 4; ++d)
                        v[i][d] = pack_bf16x2(__uint_as_float(v[i][d] << 16) * f, __uint_as_float(v[i][d] & 0xffff0000u) * f);
                }
            }
            const int o = quad >> 1;
            int row = 8 * g / K, k = K - 1 - (8 * g - row * K);
#pragma unroll
            for (int j = 0; j < 8; ++j) {
                const int slot = (row & 31) ^ (o << 3);
                const uint32_t a = j & 1 ? zip_hi16(v[0][j >> 1], v[1][j >> 1]) : zip_lo16(v[0][j >> 1], v[1][j >> 1]);
                const uint32_t e = j & 1 ? zip_hi16(v[2][j >> 1], v[3][j >> 1]) : zip_lo16(v[2][j >> 1], v[3][j >> 1]);
                *reinterpret_cast<u32x2 *>(frags + k * kTapBytes + (row >> 5) * 1024 + o * 512 + slot * 16 + (quad & 1) * 8) = u32x2{a, e};
                row = k == 0 ? row + 1 : row;
                k = k == 0 ? K - 1 : k - 1;
            }
        }
    };

    f32x16 acc[2][NT];
#pragma unroll
    for (int mi = 0; mi < 2; ++mi)
#pragma unroll
        for (int ni = 0; ni < NT; ++ni)
#pragma unroll
            for (int r = 0; r < 16; ++r) acc[mi][ni][r] = 0.f;

    const int row0 = (lane & 31) + ws - ws_al, a_at = oct * 512 + ((lane & 31) ^ (oct << 3)) * 16;
    auto read_frags = [&](int k, bf16x8(&a)[2], bf16x8(&bf)[NT]) __attribute__((always_inline)) {
        const int r = row0 + k * p.dil;
        const unsigned char *bp = xwin + r * 32 + (r >> 3) * 16 + oct * 16;
        const unsigned char *ap = frags + k * kTapBytes + a_at;
#pragma unroll
        for (int mi = 0; mi < 2; ++mi) a[mi] = *reinterpret_cast<const bf16x8 *>(ap + mi * 1024);
#pragma unroll
        for (int ni = 0; ni < NT; ++ni) bf[ni] = *reinterpret_cast<const bf16x8 *>(bp + ni * 32 * 34);
    };
    auto multiply = [&](const bf16x8(&a)[2], const bf16x8(&bf)[NT]) __attribute__((always_inline)) {
#pragma unroll
        for (int mi = 0; mi < 2; ++mi)
#pragma unroll
            for (int ni = 0; ni < NT; ++ni) acc[mi][ni] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(a[mi], bf[ni], acc[mi][ni], 0, 0, 0);
    };

    constexpr int kRequests = (2 * K + kWaves - 1) / kWaves;  // of the weights, per chunk and wavefront
    auto request_x = [&](int c) __attribute__((always_inline)) {
        const uint32_t e0 = x_at(c);
#pragma unroll
        for (int i = 0; i < 8; ++i) x_load(e0, i);
    };
    auto request_all = [&](int c) {
#pragma unroll
        for (int i = 0; i < kRequests; ++i) raw_request(c, i);
        request_x(c);
    };
    request_all(c0);
    for (int c = c0; c < c1; ++c) {
        __builtin_amdgcn_s_waitcnt(kAllVmem);
        __syncthreads();
        if constexpr (FLIP) flip_to_frags(c);
        else raw_to_frags();
        x_write(c);
        __syncthreads();
        const bool more = c + 1 < c1;
        if (!live) {
            if (more) request_all(c + 1);
            continue;
        }
        bf16x8 a[2][2], bf[2][NT];
        read_frags(0, a[0], bf[0]);
        for_each_index([&](auto tap) __attribute__((always_inline)) {  // (a loop of this size is not unrolled for every K)
            constexpr int k = decltype(tap)::value;
            if (k + 1 < K) read_frags(k + 1, a[(k + 1) & 1], bf[(k + 1) & 1]);
            if (more) {
                if (k < kRequests) raw_request(c + 1, k);
                if (k == kRequests) request_x(c + 1);
            }
            __builtin_amdgcn_sched_barrier(0);
            multiply(a[k & 1], bf[k & 1]);
            __builtin_amdgcn_sched_barrier(0);
        }, std::make_integer_sequence<int, K>{});
    }

    if (!there) return;
    // the layout split_reduce_kernel reads: quarter g of a tile holds accumulator rows 4g .. 4g+3 of every block
    f32x4 *dst = p.part + (((size_t)split * ncols + col) * p.nmt + mt) * kWaves * (2 * NT) * 64 + lane;
#pragma unroll
    for (int g = 0; g < 4; ++g)
#pragma unroll
        for (int mi = 0; mi < 2; ++mi)
#pragma unroll
            for (int ni = 0; ni < NT; ++ni)
                dst[((size_t)g * 2 * NT + mi * NT + ni) * 64] =
                    f32x4{acc[mi][ni][4 * g], acc[mi][ni][4 * g + 1], acc[mi][ni][4 * g + 2], acc[mi][ni][4 * g + 3]};
}

template <int NT, int K, bool FLIP>
hipError_t launch_t(const UnpackedParams &q, unsigned grid, size_t lds, hipStream_t s)
{
    auto kern = conv_unpacked_kernel<NT, K, FLIP>;
    static LdsOptIn opt_in;
    hipError_t e = ensure_dynamic_lds(opt_in, reinterpret_cast<const void *>(kern), kMaxLds);
    if (e != hipSuccess) return e;
    hipLaunchKernelGGL(kern, dim3(grid), dim3(kThreads), lds, s, q);
    return hipGetLastError();
}
template <int NT, bool FLIP>
hipError_t launch_taps(const UnpackedParams &q, unsigned grid, size_t lds, hipStream_t s)
{
    if constexpr (NT < 5) {
        switch (q.c.K) {
        case 11: return launch_t<NT, 11, FLIP>(q, grid, lds, s);
        case 13: return launch_t<NT, 13, FLIP>(q, grid, lds, s);
        case 17: return launch_t<NT, 17, FLIP>(q, grid, lds, s);
        default: break;
        }
    }
    switch (q.c.K) {
    case 21: return launch_t<NT, 21, FLIP>(q, grid, lds, s);
    case 25: return launch_t<NT, 25, FLIP>(q, grid, lds, s);
    case 29:
        if constexpr (!FLIP) return launch_t<NT, 29, FLIP>(q, grid, lds, s);
        return hipErrorInvalidValue;
    default: return hipErrorInvalidValue;
    }
}
template <bool FLIP>
hipError_t launch_columns(int nt, const UnpackedParams &q, unsigned grid, size_t lds, hipStream_t s)
{
    switch (nt) {
    case 2: return launch_taps<2, FLIP>(q, grid, lds, s);
    case 3: return launch_taps<3, FLIP>(q, grid, lds, s);
    case 5: return launch_taps<5, FLIP>(q, grid, lds, s);
    default: return hipErrorInvalidValue;
    }
}

int window_groups(int nt, int K, int dil) { return ((nt * 32 - 1) + (K - 1) * dil + 1 + 7 + 7) / 8; }

// The best tile and split by the time estimated for them on the device, in microseconds: fitted to 11600 measurements (plans x
// 345 geometries of 256 to 896 channels, 48 to 3000 time steps in all, both directions, replayed in a graph with cold
// weights; rms of the fit 8 %, the plan taken is 4 % from the best one on average, 21 % at most).  A chunk is staged
// and multiplied in turn; where two workgroups fit a CU one does the one while the other does the other.
UnpackedPlan make_unpacked_plan(int B, int M, int R, int Tout, int K, int dil, bool flip, size_t part_limit)
{
    UnpackedPlan best = {};
    const int nmt = (M + kTileM - 1) / kTileM, nch = R / kUnpackedChunk;
    for (const int nt : {2, 3, 5}) {
        const int ngroups = window_groups(nt, K, dil);
        if (ngroups > 32 || (nt == 5 && K < 21)) continue;  // a lane for each group and octet; (short filters never took the widest)
        const long cols = (long)B * ((Tout + nt * 32 - 1) / (nt * 32));
        if (cols > 4096) break;
        for (const int ns : {2, 3, 4, 6, 8, 12, 16, 24}) {
            if (ns > nch) break;
            const int chunks = (nch + ns - 1) / ns;
            const size_t lds = (size_t)2 * K * kTapBytes + (size_t)kWaves * ngroups * kGroupBytes + (size_t)chunks * kUnpackedChunk * sizeof(float);
            const size_t part = (size_t)cols * nmt * ns * kTileM * nt * 32 * sizeof(float);
            if (lds > (size_t)kMaxLds || part > part_limit) continue;
            const long wgs = nmt * ((cols + kWaves - 1) / kWaves) * ns, per_cu = (wgs + 255) / 256;
            const int resident = std::min(nt <= (flip ? 2 : 3) ? 2 : 1, (int)(kMaxLds / lds));
            const double stage = 0.034 + (flip ? 0.047 * K : 0.0), multiply = K * (0.0176 + 0.0444 * nt);
            const double alone = chunks * (stage + multiply), pair = chunks * std::max(stage + multiply, 1.39 * multiply + 1.16 * stage);
            const double cost = 10.7 + (resident == 2 ? per_cu / 2 * pair + per_cu % 2 * alone : per_cu * alone) +
                                0.36e-6 * 4 * ns * M * (double)cols * nt * 32 + 0.01e-6 * M * R * K;
            if (best.nt && cost >= best.cost) continue;
            // (forward calls on the plans taken, 6164 of them: rms 8 %; two workgroups on a CU overlap far less there than the fit above has it)
            const double mult = K * (0.036 + 0.0337 * nt), one = chunks * (0.4 + mult);
            best.device = 8.4 + per_cu % 2 * one + per_cu / 2 * (resident == 2 ? std::max(one, 1.86 * chunks * mult) : 2 * one) +
                          0.576e-6 * 4 * ns * M * (double)cols * nt * 32 + 0.5e-6 * B * M * (double)Tout;
            best.nt = nt;
            best.nsplit = ns;
            best.ngroups = ngroups;
            best.lds = lds;
            best.part_bytes = part;
            best.cost = cost;
        }
    }
    return best;
}

}  // namespace

bool unpacked_supported(int M, int R, int K, int stride, bool flip)
{
    if (K != 11 && K != 13 && K != 17 && K != 21 && K != 25 && K != 29) return false;
    if (K == 29 && flip) return false;  // (the compiler keeps that instance's arrays in scratch: 146 us where the other engines take 50)
    // whole chunks, eight of them at least (with fewer there is nothing to share out), a whole tile of output channels, and
    // rows of w that start at 16-byte addresses
    return stride == 1 && M >= kTileM && R % kUnpackedChunk == 0 && R >= 8 * kUnpackedChunk && (!flip || M % 8 == 0);
}

UnpackedPlan unpacked_plan(int B, int M, int R, int Tout, int K, int dil, bool flip, size_t part_limit)
{
    // remembered: a call asks several times (workspace query, checks, launch)
    struct Entry {
        int key[8];
        UnpackedPlan plan;
    };
    static thread_local Entry table[16] = {};  // (no call has B = 0)
    part_limit = std::min(part_limit, (size_t)1 << 38) >> 8 << 8;
    const int key[8] = {B, M, R, Tout, K, dil, flip, (int)(part_limit >> 8)};
    unsigned h = 0;
    for (int k : key) h = h * 31u + (unsigned)k;
    Entry &e = table[(h ^ (h >> 7) ^ (h >> 15)) % 16];
    if (memcmp(e.key, key, sizeof key) != 0) {
        e.plan = make_unpacked_plan(B, M, R, Tout, K, dil, flip, part_limit);
        memcpy(e.key, key, sizeof key);
    }
    return e.plan;
}

hipError_t launch_unpacked_conv(const UnpackedPlan &plan, const ConvGemmParams &p, const void *w, bool flip, const float *rscale,
                                void *part, hipStream_t s, SplitSum *later)
{
    UnpackedParams q = {};
    q.c = p;
    q.c.ntt = (p.Tout + plan.nt * 32 - 1) / (plan.nt * 32);
    q.c.nsplit = plan.nsplit;
    q.c.nitems = plan.ngroups;
    q.c.part = (f32x4 *)part;
    q.c.col0 = 0;
    q.c.ncols = q.c.ntt * p.B;
    q.w = (const bf16_t *)w;
    q.rscale = rscale;
    q.ncolgroups = (q.c.ncols + kWaves - 1) / kWaves;
    const unsigned grid = (unsigned)(p.nmt * plan.nsplit * q.ncolgroups);
    MainKernelTimer timer(s);
    const hipError_t e = flip ? launch_columns<true>(plan.nt, q, grid, plan.lds, s) : launch_columns<false>(plan.nt, q, grid, plan.lds, s);
    return e != hipSuccess ? e : launch_split_reduce(q.c, plan.nt, s, timer.stop ? nullptr : later);
}
}  // namespace nm
