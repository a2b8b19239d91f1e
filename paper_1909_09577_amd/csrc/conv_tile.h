// What the convolution engines share (mfma_conv.hip, unpacked_conv.hip): vector types, tile constants, launch parameters and
// the epilogue that takes a tile from the accumulators to memory.
#pragma once

#include "nm_common.h"

#include <type_traits>
#include <utility>

namespace nm {

typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef float f32x16 __attribute__((ext_vector_type(16)));
typedef float f32x4 __attribute__((ext_vector_type(4)));
typedef float f32x2 __attribute__((ext_vector_type(2)));
typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));

constexpr int kWaves = 4;
constexpr int kThreads = 64 * kWaves;
constexpr int kTileM = 64;       // output channels per tile
constexpr int kChunk = 32;       // reduction channels per staged chunk
constexpr int kRowBytes = 80;    // LDS row: 32 channels * 2 B + 16 B pad (bank-conflict-free 16 B reads)
constexpr int kRowDwords = kRowBytes / 4;
constexpr int kDumpRows = 8;     // rows at the end of a staging buffer that absorb idle staging writes
constexpr int kMaxLds = 160 * 1024;

struct ConvGemmParams {
    int B, M, R, Tin, Tout, K, Kp, dil, padL;  // Kp: K rounded up to even (packed weights)
    int nmt, nch, ntt, num_tiles;
    int nitems;      // staging items per lane and chunk = ceil(rows/8 * 16 / 64)
    int buf_bytes;   // bytes of one staging buffer: (nitems*32 + kDumpRows) rows of kRowBytes
    int overlap;     // the next tile's first chunk is staged during the current tile
    int full;        // tiles every wavefront computes on its own, over the whole reduction, before the shared ones
    int relu;
    const bf16_t *in;       // [B][R][Tin]
    const int *len_in;      // [B] valid input lengths (samples beyond read as zero) or NULL
    const int *len_out;     // [B] lengths beyond which the output is written as zero, or NULL; the limit of
    int len_out_div;        // batch item b is ceil(len_out[b] / div) (2: both parities of a strided gradient)
    const bf16x8 *wp;       // packed weights
    size_t wp_bytes;        // size of the packed weights including the zero pair (< 2 GiB)
    size_t wp_zero;         // offset (in fragments of 16 bytes) of one tap pair of zero weights
    const float *scale;     // epilogue (may be NULL)
    const float *shift;     // epilogue (may be NULL)
    const bf16_t *res;      // epilogue (may be NULL)
    bf16_t *out;            // [B][M][Tout]
    int nsplit;             // conv_split_kernel: parts the reduction channels are split into
    f32x4 *part;            // their partial sums (nsplit > 1)
    double *stats;          // optional [B*ntt][M][3]: count, mean and centred second moment of the stored outputs of
                            // every (batch item, time tile, channel) -- the partial statistics of a BatchNorm over out
    int col0, ncols;        // conv_split_kernel: the columns (time tiles of all batch items) of this launch
    int odd_rows;           // rows of in or out are no multiple of 16 bytes long (host: which instances serve the call)
};

__device__ __forceinline__ void wave_lds_fence()
{
    // LDS operations of one wavefront execute in order; this only stops the compiler from
    // moving LDS accesses across the point where other lanes' data must be visible.
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}

// Buffer offset beyond any tensor this engine accepts (the host limits them to 1 GiB): the load
// returns zeros.  Small additions to it neither wrap nor come back into range.
constexpr uint32_t kOutOfRange = 0x80000000u;

// The lane number, recomputed where it is needed.  The staging code runs once per chunk inside a
// loop whose registers are all taken; values derived from a long-lived lane id would be spilled
// and their reload would wait for every load in flight.  Two ALU operations avoid that.
__device__ __forceinline__ int fresh_lane()
{
    int l = (int)__builtin_amdgcn_mbcnt_hi(~0u, __builtin_amdgcn_mbcnt_lo(~0u, 0u));
    asm volatile("" : "+v"(l));
    return l;
}

// f(integral_constant<0>), f(integral_constant<1>), ... in order
template <class F, int... Is>
__device__ __forceinline__ void for_each_index(F &&f, std::integer_sequence<int, Is...>)
{
    (f(std::integral_constant<int, Is>{}), ...);
}

// Staging items the unrolled kernel built for K taps keeps in registers; 0: no such kernel.
__host__ __device__ constexpr int unrolled_slots(int K) { return K == 29 ? 7 : (K == 11 || K == 13 || K == 17 || K == 21 || K == 25) ? 6 : 0; }

// ---- epilogue shared by the engines of this file ------------------------------------------------
// The sums leave the accumulators through a wave-private LDS tile [16 rows][NT*32] (float32) so that
// each lane finishes 8 consecutive time steps of one channel: one 16-byte residual load, one scale,
// one shift, one 16-byte store per item.  All of these are buffer accesses without branches: absent
// operands have empty descriptors and read zeros, masked lanes go out of range.  That needs 16-byte
// aligned rows of out and res; the ANYROW instances also serve rows of any length (`anyrow`): the same
// items through 16-byte global accesses at 2-byte aligned addresses, element by element for the group
// that holds the end of a row.
template <int NT>
struct Epilogue {
    static constexpr int TN = NT * 32;
    static constexpr int kItems = NT;  // 16 rows * (TN/8) groups / 64 lanes
    __amdgpu_buffer_rsrc_t rs_out, rs_res, rs_scale, rs_shift;
    int M, Tout;
    bool has_scale, relu, anyrow;
    bf16_t *out_p;        // (anyrow) the tensors themselves
    const bf16_t *res_p;
    const int *len_out;  // optional [B]: outputs at t >= ceil(len_out[b] / div) are written as zero
    int len_div;
    double *stats;       // see ConvGemmParams::stats (used by the STATS instances only)
    static constexpr int kStatsOffset = 16 * TN;  // float2 [16 rows][TN/8] behind the tile (in floats)
    static constexpr int kTileBytesWithStats = 16 * TN * (int)sizeof(float) + 16 * (TN / 8) * 2 * (int)sizeof(float);

    struct RowLoads {
        u32x4 rvec[kItems];
        float scv[kItems], shv[kItems];
        uint32_t ooff[kItems];
        int tlim_rel;  // output limit of the batch item relative to the tile's first time step (wave-uniform)
        int tout_rel;  // the same of the row's end
    };
    // first time step of batch item b that is written as zero (Tout without lengths)
    __device__ __forceinline__ int out_limit(int b) const
    {
        if (!len_out) return Tout;
        const int n = (len_out[b] + len_div - 1) / len_div;
        return n < 0 ? 0 : (n > Tout ? Tout : n);
    }

    __device__ __forceinline__ void init(const bf16_t *out, const bf16_t *res, const float *scale, const float *shift, int B,
                                         int M_, int Tout_, int relu_, const int *len_out_ = nullptr, int div = 1,
                                         double *stats_ = nullptr)
    {
        stats = stats_;
        len_out = len_out_;
        len_div = div < 1 ? 1 : div;
        const int out_bytes = (int)((size_t)B * M_ * Tout_ * 2);
        M = M_;
        Tout = Tout_;
        has_scale = scale != nullptr;
        relu = relu_ != 0;
        anyrow = Tout_ % 8 != 0;
        out_p = const_cast<bf16_t *>(out);
        res_p = res;
        rs_out = __builtin_amdgcn_make_buffer_rsrc((void *)out, 0, out_bytes, 0x00020000);
        rs_res = __builtin_amdgcn_make_buffer_rsrc((void *)res, 0, res ? out_bytes : 0, 0x00020000);
        rs_scale = __builtin_amdgcn_make_buffer_rsrc((void *)scale, 0, scale ? M_ * 4 : 0, 0x00020000);
        rs_shift = __builtin_amdgcn_make_buffer_rsrc((void *)shift, 0, shift ? M_ * 4 : 0, 0x00020000);
    }
    // operands of the 16 tile rows whose first channel is m0 (tile row r is channel m0 + r, or
    // m0 + 32*(r/8) + r%8 when `split`: eight rows from each row of blocks); el: the lane number
    template <bool ANYROW = false>
    __device__ __forceinline__ RowLoads request_rows(int el, int b, int t0, int m0, bool split) const
    {
        RowLoads ld;
        ld.tlim_rel = out_limit(b) - t0;
        ld.tout_rel = Tout - t0;
#pragma unroll
        for (int q = 0; q < kItems; ++q) {
            const int idx = el + 64 * q;
            const int r = idx / (TN / 8), c8 = idx - r * (TN / 8);
            const int m = m0 + (split ? (r >> 3) * 32 + (r & 7) : r);
            const int t = t0 + c8 * 8;
            const bool ok = m < M && t < Tout;
            ld.ooff[q] = ok ? (uint32_t)((((size_t)b * M + m) * Tout + t) * 2) : kOutOfRange;
            const uint32_t moff = ok ? (uint32_t)m * 4u : kOutOfRange;
            if (ANYROW && anyrow) {
                if (!res_p) ld.rvec[q] = u32x4{0u, 0u, 0u, 0u};
                else if (Tout >= 8) ld.rvec[q] = load8_row(res_p + ((size_t)b * M + min(m, M - 1)) * Tout, t, Tout);  // moved down in finish_rows
                else ld.rvec[q] = load8_any(res_p + ld.ooff[q] / 2, ok ? Tout - t : 0);
            } else
                ld.rvec[q] = __builtin_amdgcn_raw_buffer_load_b128(rs_res, ld.ooff[q], 0, 0);
            ld.scv[q] = __uint_as_float(__builtin_amdgcn_raw_buffer_load_b32(rs_scale, moff, 0, 0));
            ld.shv[q] = __uint_as_float(__builtin_amdgcn_raw_buffer_load_b32(rs_shift, moff, 0, 0));
        }
        return ld;
    }
    // affine, residual, ReLU, rounding and the stores of the 16 rows that sit in the LDS tile tp
    template <bool STATS = false, bool ANYROW = false>
    __device__ __forceinline__ void finish_rows(int el, float *tp, const RowLoads &ld) const
    {
#pragma unroll
        for (int q = 0; q < kItems; ++q) {
            const int idx = el + 64 * q;
            const int r = idx / (TN / 8), c8 = idx - r * (TN / 8);
            const f32x4 lo = *reinterpret_cast<const f32x4 *>(tp + r * TN + c8 * 8);
            const f32x4 hi = *reinterpret_cast<const f32x4 *>(tp + r * TN + c8 * 8 + 4);
            const float sc = has_scale ? ld.scv[q] : 1.f;
            u32x4 rv = ld.rvec[q], o;
            if (ANYROW && anyrow && res_p && Tout >= 8) rv = shift8_down(rv, c8 * 8, ld.tout_rel);
#pragma unroll
            for (int e = 0; e < 4; ++e) {
                const float a0 = (e < 2 ? lo[2 * e] : hi[2 * e - 4]), a1 = (e < 2 ? lo[2 * e + 1] : hi[2 * e - 3]);
                float v0 = a0 * sc + ld.shv[q] + __uint_as_float(rv[e] << 16);
                float v1 = a1 * sc + ld.shv[q] + __uint_as_float(rv[e] & 0xffff0000u);
                if (relu) {
                    v0 = v0 > 0.f ? v0 : 0.f;
                    v1 = v1 > 0.f ? v1 : 0.f;
                }
                o[e] = pack_bf16x2(v0, v1);
            }
            if (len_out) {  // zeros from the output limit on (a uniform branch: nothing to do without lengths)
                const int nvalid = ld.tlim_rel - c8 * 8;
#pragma unroll
                for (int e = 0; e < 4; ++e) o[e] &= nvalid >= 2 * e + 2 ? 0xffffffffu : (nvalid == 2 * e + 1 ? 0x0000ffffu : 0u);
            }
            if (ANYROW && anyrow)
                store8_any(out_p + ld.ooff[q] / 2, o, ld.ooff[q] != kOutOfRange ? ld.tout_rel - c8 * 8 : 0);
            else
                __builtin_amdgcn_raw_buffer_store_b128(o, rs_out, ld.ooff[q], 0, 0);
            if constexpr (STATS) {  // sums of the eight stored (rounded) values; an item outside the tensor adds nothing
                float s1 = 0.f, s2 = 0.f;
                if (ld.ooff[q] != kOutOfRange) {
#pragma unroll
                    for (int e = 0; e < 4; ++e) {
                        const float v0 = __uint_as_float(o[e] << 16), v1 = __uint_as_float(o[e] & 0xffff0000u);
                        s1 += v0 + v1;
                        s2 = fmaf(v0, v0, fmaf(v1, v1, s2));
                    }
                }
                reinterpret_cast<f32x2 *>(tp + kStatsOffset)[idx] = f32x2{s1, s2};
            }
        }
    }
    // (STATS instances) after finish_rows<true> and a fence: lane r < 16 adds the TN/8 partial sums of tile row r in
    // order and writes count, mean and centred second moment of that row's part of channel m_of_row
    __device__ __forceinline__ void emit_row_stats(int el, const float *tp, int m_of_row, int part, int t0) const
    {
        if (el >= 16 || m_of_row >= M) return;
        const f32x2 *sp = reinterpret_cast<const f32x2 *>(tp + kStatsOffset) + el * (TN / 8);
        double a = 0.0, b2 = 0.0;
#pragma unroll
        for (int i = 0; i < TN / 8; ++i) {
            const f32x2 v = sp[i];
            a += (double)v[0];
            b2 += (double)v[1];
        }
        const int left = Tout - t0;
        const double n = (double)(left < TN ? (left > 0 ? left : 0) : TN);
        double *o = stats + ((size_t)part * M + m_of_row) * 3;
        o[0] = n;
        o[1] = n > 0 ? a / n : 0.0;
        o[2] = n > 0 ? b2 - a * a / n : 0.0;
    }
    // the 16 rows of a wavefront's quarter of a tile (eight from each row of blocks) to the LDS tile
    __device__ __forceinline__ void put_quarter(float *tp, int el, const f32x4 (&own)[2][NT]) const
    {
#pragma unroll
        for (int mi = 0; mi < 2; ++mi)
#pragma unroll
            for (int j = 0; j < 4; ++j)
#pragma unroll
                for (int ni = 0; ni < NT; ++ni) tp[(mi * 8 + 4 * (el >> 5) + j) * TN + ni * 32 + (el & 31)] = own[mi][ni][j];
    }
    // A whole 64-row tile held by one wavefront (rows m_first .. m_first+63): four rounds of 16 rows
    // (row of blocks mi, accumulator registers 8*gp .. 8*gp+7) through tp; the operands of a round
    // are requested two rounds ahead.
    template <bool STATS = false, bool ANYROW = false>
    __device__ __forceinline__ void store_private_tile(const f32x16 (&acc)[2][NT], float *tp, int el, int b, int t0,
                                                       int m_first, int part = 0) const
    {
        const int tcol = el & 31, thalf = el >> 5;
        RowLoads ld[2] = {request_rows<ANYROW>(el, b, t0, m_first, false), request_rows<ANYROW>(el, b, t0, m_first + 16, false)};
#pragma unroll
        for (int rd = 0; rd < 4; ++rd) {
            const int mi = rd >> 1, gp = rd & 1;
#pragma unroll
            for (int g = 0; g < 2; ++g)
#pragma unroll
                for (int j = 0; j < 4; ++j) {
                    const int r = g * 8 + 4 * thalf + j;
#pragma unroll
                    for (int ni = 0; ni < NT; ++ni) tp[r * TN + ni * 32 + tcol] = acc[mi][ni][4 * (2 * gp + g) + j];
                }
            wave_lds_fence();
            finish_rows<STATS, ANYROW>(el, tp, ld[rd & 1]);
            if (rd + 2 < 4) ld[rd & 1] = request_rows<ANYROW>(el, b, t0, m_first + (rd + 2) * 16, false);
            wave_lds_fence();
            if constexpr (STATS) emit_row_stats(el, tp, m_first + rd * 16 + el, part, t0);
        }
    }
};

// Adds the nsplit parts of 16 rows x 32 steps in order and finishes them: one wavefront's work, tp its LDS tile of 16 x 32 floats.
__device__ __forceinline__ void split_reduce_piece(const ConvGemmParams &p, int nt, int piece, int lane, float *tp)
{
    const int ni = piece % nt, quarter = piece / nt;
    const int wave = quarter & 3, tile = quarter >> 2;
    const int col = tile / p.nmt, mt = tile - col * p.nmt;
    const int b = (p.col0 + col) / p.ntt, t0 = ((p.col0 + col - b * p.ntt) * nt + ni) * 32;
    Epilogue<1> epi;
    epi.init(p.out, p.res, p.scale, p.shift, p.B, p.M, p.Tout, p.relu, p.len_out, p.len_out_div);
    const auto ld = epi.template request_rows<true>(lane, b, t0, mt * kTileM + 8 * wave, true);
    const size_t pitch = (size_t)p.nmt * p.ncols * kWaves * 2 * nt * 64;
    const f32x4 *src = p.part + ((size_t)quarter * 2 * nt + ni) * 64 + lane;
    f32x4 own[2][1] = {};
#pragma unroll 8
    for (int s = 0; s < p.nsplit; ++s) {
        own[0][0] += src[(size_t)s * pitch];
        own[1][0] += src[(size_t)s * pitch + (size_t)nt * 64];
    }
    epi.put_quarter(tp, lane, own);
    wave_lds_fence();
    epi.template finish_rows<false, true>(lane, tp, ld);
}

// Such a sum that is still to be launched.
struct SplitSum {
    bool set = false;
    ConvGemmParams p;
    int nt;
    unsigned pieces() const { return (unsigned)(p.nmt * p.ncols * kWaves * nt); }
};

// valid length of batch item b from an optional device array, clipped to [0, T]
__device__ __forceinline__ int clipped_len(const int *len, int b, int T)
{
    if (!len) return T;
    const int n = len[b];
    return n < 0 ? 0 : (n > T ? T : n);
}

// ---- unpacked_conv.hip: calls of few tiles on the weights as they lie in memory ------------------
struct UnpackedPlan {
    int nt, nsplit, ngroups;  // nt = 0: none
    size_t lds, part_bytes;
    double cost;              // estimated time on the device (us), by which plans are compared
    double device;            // the same, fitted to forward calls on the plans taken
};
bool unpacked_supported(int M, int R, int K, int stride, bool flip);
UnpackedPlan unpacked_plan(int B, int M, int R, int Tout, int K, int dil, bool flip, size_t part_limit);
// p: as for the other engines, without the packed weights; w 16-byte aligned; part: plan.part_bytes of scratch
hipError_t launch_unpacked_conv(const UnpackedPlan &plan, const ConvGemmParams &p, const void *w, bool flip, const float *rscale,
                                void *part, hipStream_t s, SplitSum *later = nullptr);
// adds p.nsplit parts in a fixed order and finishes the tiles (mfma_conv.hip); later: leaves that to the caller
hipError_t launch_split_reduce(const ConvGemmParams &p, int nt, hipStream_t s, SplitSum *later = nullptr);

}  // namespace nm
