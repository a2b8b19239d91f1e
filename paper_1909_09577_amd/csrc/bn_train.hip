// Training-mode BatchNorm of the conv1d sub-block: batch statistics over (batch, time) of the stored
// pre-activation z, the normalise + affine + residual + ReLU pass, and the backward pass through the
// statistics (dgamma, dbeta and the corrected dz that the two convolution gradients then contract).
//
//   mean[c] = (1/N) sum z,  var[c] = (1/N) sum (z-mean)^2,  invstd = 1/sqrt(var+eps),  zhat = (z-mean)*invstd
//   y  = relu?( gamma*zhat + beta + residual )
//   g  = dy*[y>0];  dbeta = sum g;  dgamma = sum g*zhat;  dz = gamma*invstd*( g - dbeta/N - zhat*dgamma/N )
//
// All of these are bandwidth-bound passes over [B][C][T] tensors.  Sums are deterministic: every block
// owns one channel and a fixed subset of the batch items, reduces in a fixed tree (in double, so that
// var = M2/N does not cancel), and the per-block results are combined in a fixed order (block means and
// centred second moments, merged pairwise as in a streaming variance).
// Elements move in groups of 16 bytes, 8 bf16 or 4 float, whatever the row length and the address: the last
// group of a row ends with the row and begins inside the one before it (the elements that both hold are
// counted once, and written twice with the same value); rows shorter than a group go element by element.
// Rows that are no multiple of a group used to go element by element throughout: 384 channels, B=10, T=711 six launches of 41.8 us,
// 24.4 in four now (640 channels, B=16, T=800, where nothing but the last merge went: 47.1 and 43.4).
#include "nm_common.h"

#include <type_traits>

namespace nm {
namespace {

constexpr int kThreads = 256;
constexpr int kMaxParts = 8;  // of a channel, where a pass over the tensor makes them
template <int N>
using Vec = std::integral_constant<int, N>;

// Group i of the rows of channel c that a block handles: row i / ng of them, first element at(..), of which the first `skip`
// belong to the group before.
struct Rows {
    int C, T, ng;
    __device__ __forceinline__ size_t at(int vec, unsigned i, int c, int b0, int step, int &skip) const
    {
        const unsigned r = i / (unsigned)ng;
        const int t = (int)(i - r * (unsigned)ng) * vec, from = min(t, T - vec);
        skip = t - from;
        return ((size_t)(b0 + (int)r * step) * C + c) * T + from;
    }
};

template <typename TS, int VEC>
struct Group {
    TS raw[VEC] __attribute__((aligned(VEC > 1 ? 16 : sizeof(TS))));
    __device__ __forceinline__ void load(const TS *p) { __builtin_memcpy(raw, p, sizeof raw); }
    __device__ __forceinline__ float operator[](int e) const { return load_as_f32(raw, e); }
};
template <typename TS, int VEC>
__device__ __forceinline__ void store_group(TS *p, const float *v)
{
    if constexpr (sizeof(TS) == 2 && VEC == 8) {
        u32x4_t raw;
#pragma unroll
        for (int j = 0; j < 4; ++j) raw[j] = pack_bf16x2(v[2 * j], v[2 * j + 1]);
        __builtin_memcpy(p, &raw, 16);
    } else {
        TS raw[VEC] __attribute__((aligned(16)));
#pragma unroll
        for (int e = 0; e < VEC; ++e) store_from_f32(raw, e, v[e]);
        __builtin_memcpy(p, raw, sizeof raw);
    }
}

// Sum of `a` and of `b` over the block, in a fixed tree, returned to thread 0.
__device__ __forceinline__ void block_sum2(double &a, double &b)
{
    __shared__ double red[2][kThreads / 64];
    for (int off = 32; off > 0; off >>= 1) {
        a += __shfl_down(a, off, 64);
        b += __shfl_down(b, off, 64);
    }
    const int wave = threadIdx.x >> 6;
    if ((threadIdx.x & 63) == 0) {
        red[0][wave] = a;
        red[1][wave] = b;
    }
    __syncthreads();
    a = (red[0][0] + red[0][1]) + (red[0][2] + red[0][3]);
    b = (red[1][0] + red[1][1]) + (red[1][2] + red[1][3]);
}

// Block (c, g): batch items g, g+G, ... of channel c -> part[(g*C + c)*3] = {count, mean, centred second moment}.
template <typename TS, int VEC>
__global__ __launch_bounds__(kThreads) void bn_stats_kernel(const TS *__restrict__ z, int B, Rows rows, int G,
                                                            double *__restrict__ part)
{
    const int c = blockIdx.x, g = blockIdx.y;
    const int nrows = (B - g + G - 1) / G;
    const unsigned n = (unsigned)nrows * rows.ng;
    double a = 0.0, q = 0.0;
    for (unsigned i = threadIdx.x; i < n; i += kThreads) {
        int skip;
        Group<TS, VEC> v;
        v.load(z + rows.at(VEC, i, c, g, G, skip));
        float s1 = 0.f, s2 = 0.f;
#pragma unroll
        for (int e = 0; e < VEC; ++e) {
            const float f = e < skip ? 0.f : v[e];
            s1 += f;
            s2 = fmaf(f, f, s2);
        }
        a += s1;
        q += s2;
    }
    block_sum2(a, q);
    if (threadIdx.x == 0) {
        const double cnt = (double)nrows * rows.T;
        double *o = part + ((size_t)g * rows.C + c) * 3;
        o[0] = cnt;
        o[1] = cnt > 0 ? a / cnt : 0.0;
        o[2] = cnt > 0 ? q - a * a / cnt : 0.0;
    }
}

struct BnFinal {
    const double *part;
    int G;
    const float *gamma, *beta;
    float eps;
    float *mean, *invstd, *scale, *shift;
};

// A wavefront's merge of the parts of channel c: lane l merges parts l, l+64, ... in order (Chan's update), then the lanes
// merge in a fixed tree; lane 0 has the mean, 1/std and the affine that they imply.
__device__ __forceinline__ void bn_merge(const BnFinal &f, int C, int c, int lane, float (&out)[4])
{
    double n = 0.0, mu = 0.0, m2 = 0.0;
    auto merge = [&](double nb, double mb, double qb) {
        if (nb <= 0.0) return;
        const double delta = mb - mu, tot = n + nb;
        mu += delta * nb / tot;
        m2 += qb + delta * delta * n * nb / tot;
        n = tot;
    };
    for (int g = lane; g < f.G; g += 64) {
        const double *p = f.part + ((size_t)g * C + c) * 3;
        merge(p[0], p[1], p[2]);
    }
    for (int off = f.G > kMaxParts ? 32 : kMaxParts / 2; off > 0; off >>= 1) {
        const double nb = __shfl_down(n, off, 64), mb = __shfl_down(mu, off, 64), qb = __shfl_down(m2, off, 64);
        if (lane < off) merge(nb, mb, qb);
    }
    const double var = n > 0 ? (m2 > 0 ? m2 / n : 0.0) : 0.0;
    const double is = 1.0 / sqrt(var + (double)f.eps);
    const double ga = f.gamma ? (double)f.gamma[c] : 1.0, be = f.beta ? (double)f.beta[c] : 0.0;
    out[0] = (float)mu;
    out[1] = (float)is;
    out[2] = (float)(ga * is);
    out[3] = (float)(be - mu * ga * is);
}

// One wavefront per channel.
__global__ __launch_bounds__(64) void bn_finalize_kernel(BnFinal f, int C)
{
    float o[4];
    bn_merge(f, C, blockIdx.x, threadIdx.x, o);
    if (threadIdx.x != 0) return;
    f.mean[blockIdx.x] = o[0];
    f.invstd[blockIdx.x] = o[1];
    f.scale[blockIdx.x] = o[2];
    f.shift[blockIdx.x] = o[3];
}

// Block j*C + c: groups j*per, ... of channel c: y = relu?(scale[c]*z + shift[c] + residual).  MERGE: the parts of the statistics are
// merged here while z and the residual are under way, by the block's first wavefront, and block c writes mean and invstd.
// That goes for the at most eight parts of bn_stats_kernel (a launch of 4.9 us before); the parts that
// a convolution's epilogue writes are one per tile of time, some hundred, and merging them is longer than a launch.
constexpr int kApplyGroups = 2;  // a thread's, read at once (four: 5.9 -> 7.0 us at 384 channels, B=10, T=711)
template <typename TS, int VEC, bool MERGE>
__global__ __launch_bounds__(kThreads) void bn_apply_fwd_kernel(unsigned n, unsigned per, Rows rows, const TS *__restrict__ z,
                                                                BnFinal f, const TS *__restrict__ res, int relu,
                                                                TS *__restrict__ y)
{
    const int c = blockIdx.x % (unsigned)rows.C;
    const unsigned j = blockIdx.x / (unsigned)rows.C, first = j * per, last = min(n, first + per);
    Group<TS, VEC> zv[kApplyGroups], rv[kApplyGroups];
    size_t at[kApplyGroups];
#pragma unroll
    for (int u = 0; u < kApplyGroups; ++u) {
        const unsigned i = first + u * kThreads + threadIdx.x;
        int skip;
        at[u] = rows.at(VEC, min(i, n - 1), c, 0, 1, skip);
        if (i < last) {
            zv[u].load(z + at[u]);
            if (res) rv[u].load(res + at[u]);
        }
    }
    float sc, sh;
    if constexpr (MERGE) {
        __shared__ float affine[2];
        if (threadIdx.x < 64) {
            float o[4];
            bn_merge(f, rows.C, c, threadIdx.x, o);
            if (threadIdx.x == 0) {
                affine[0] = o[2];
                affine[1] = o[3];
                if (j == 0) {
                    f.mean[c] = o[0];
                    f.invstd[c] = o[1];
                }
            }
        }
        __syncthreads();
        sc = affine[0];
        sh = affine[1];
    } else {
        sc = f.scale[c];
        sh = f.shift[c];
    }
#pragma unroll
    for (int u = 0; u < kApplyGroups; ++u) {
        if (first + u * kThreads + threadIdx.x >= last) break;
        float out[VEC];
#pragma unroll
        for (int e = 0; e < VEC; ++e) {
            out[e] = fmaf(zv[u][e], sc, sh);
            if (res) out[e] += rv[u][e];
            if (relu) out[e] = out[e] > 0.f ? out[e] : 0.f;
        }
        store_group<TS, VEC>(y + at[u], out);
    }
}

// Block (c, g): part[(g*C + c)*2] = {sum g, sum g*zhat} over its batch items, g = dy*[y>0].
template <typename TS, int VEC>
__global__ __launch_bounds__(kThreads) void bn_bwd_stats_kernel(const TS *__restrict__ dy, const TS *__restrict__ y,
                                                                const TS *__restrict__ z, const float *__restrict__ mean,
                                                                const float *__restrict__ invstd, int relu, int B, Rows rows,
                                                                int G, double *__restrict__ part)
{
    const int c = blockIdx.x, g = blockIdx.y;
    const unsigned n = (unsigned)((B - g + G - 1) / G) * rows.ng;
    const float mu = mean[c], is = invstd[c];
    double a = 0.0, q = 0.0;
    for (unsigned i = threadIdx.x; i < n; i += kThreads) {
        int skip;
        const size_t at = rows.at(VEC, i, c, g, G, skip);
        Group<TS, VEC> dv, zv, yv;
        dv.load(dy + at);
        zv.load(z + at);
        if (relu) yv.load(y + at);
        float s1 = 0.f, s2 = 0.f;
#pragma unroll
        for (int e = 0; e < VEC; ++e) {
            const bool counts = e >= skip;
            const float gv = counts && (!relu || yv[e] > 0.f) ? dv[e] : 0.f;
            s1 += gv;
            s2 = fmaf(gv, counts ? (zv[e] - mu) * is : 0.f, s2);
        }
        a += s1;
        q += s2;
    }
    block_sum2(a, q);
    if (threadIdx.x == 0) {
        double *o = part + ((size_t)g * rows.C + c) * 2;
        o[0] = a;
        o[1] = q;
    }
}

struct BnBwdFinal {
    const double *part;
    int G;
    double N;
    const float *gamma, *mean, *invstd;
    float *dgamma, *dbeta;
    int accumulate;
};

// Block j*C + c: groups j*per, ... of channel c: dz = gamma*invstd*(g - dbeta/N - zhat*dgamma/N) in the storage type; dres = g
// (optional).  Every block adds up the at most eight parts of its channel itself, behind its loads; block c also writes dbeta and
// dgamma (added to the old values when accumulating).  A launch of its own took 4.8 us for that.
template <typename TS, int VEC>
__global__ __launch_bounds__(kThreads) void bn_bwd_apply_kernel(unsigned n, unsigned per, Rows rows, const TS *__restrict__ dy,
                                                                const TS *__restrict__ y, const TS *__restrict__ z,
                                                                BnBwdFinal f, int relu, TS *__restrict__ dz,
                                                                TS *__restrict__ dres)
{
    const int c = blockIdx.x % (unsigned)rows.C;
    const unsigned j = blockIdx.x / (unsigned)rows.C, first = j * per, last = min(n, first + per);
    Group<TS, VEC> dv[kApplyGroups], zv[kApplyGroups], yv[kApplyGroups];
    size_t at[kApplyGroups];
#pragma unroll
    for (int u = 0; u < kApplyGroups; ++u) {
        const unsigned i = first + u * kThreads + threadIdx.x;
        int skip;
        at[u] = rows.at(VEC, min(i, n - 1), c, 0, 1, skip);
        if (i < last) {
            dv[u].load(dy + at[u]);
            zv[u].load(z + at[u]);
            if (relu) yv[u].load(y + at[u]);
        }
    }
    double sb = 0.0, sg = 0.0;
    double pb[kMaxParts], pg[kMaxParts];
#pragma unroll
    for (int g = 0; g < kMaxParts; ++g) {
        const double *o = f.part + ((size_t)min(g, f.G - 1) * rows.C + c) * 2;
        pb[g] = o[0];
        pg[g] = o[1];
    }
#pragma unroll
    for (int g = 0; g < kMaxParts; ++g) {
        if (g < f.G) sb += pb[g], sg += pg[g];
    }
    if (threadIdx.x == 0 && j == 0) {
        if (f.dbeta) f.dbeta[c] = f.accumulate ? f.dbeta[c] + (float)sb : (float)sb;
        if (f.dgamma) f.dgamma[c] = f.accumulate ? f.dgamma[c] + (float)sg : (float)sg;
    }
    const float mu = f.mean[c], is = f.invstd[c];
    const float k0 = (f.gamma ? f.gamma[c] : 1.f) * is, k1 = (float)(sb / f.N), k2 = (float)(sg / f.N);
#pragma unroll
    for (int u = 0; u < kApplyGroups; ++u) {
        if (first + u * kThreads + threadIdx.x >= last) break;
        float gout[VEC], zout[VEC];
#pragma unroll
        for (int e = 0; e < VEC; ++e) {
            const float gv = (!relu || yv[u][e] > 0.f) ? dv[u][e] : 0.f;
            gout[e] = gv;
            zout[e] = k0 * (gv - k1 - (zv[u][e] - mu) * is * k2);
        }
        store_group<TS, VEC>(dz + at[u], zout);
        if (dres) store_group<TS, VEC>(dres + at[u], gout);
    }
}

int batch_groups(int B) { return B < kMaxParts ? B : kMaxParts; }

// elements of a group: 16 bytes, one in rows that are shorter
int group_size(bool is_bf16, int T)
{
    const int vec = is_bf16 ? 8 : 4;
    return T >= vec ? vec : 1;
}

// The groups of a channel in as many blocks as a thread's kApplyGroups need, of equal work.
struct ApplySplit {
    unsigned n, per, blocks;
    ApplySplit(int B, int ng)
    {
        n = (unsigned)B * ng;
        blocks = (n + kApplyGroups * kThreads - 1) / (kApplyGroups * kThreads);
        per = (n + blocks - 1) / blocks;
    }
};

// parts of a channel's statistics: the groups of batch items of bn_stats_kernel, or one per (batch item, 160-step
// time tile) when the convolution kernel writes them from its epilogue
size_t bn_parts_cap(int B, int T)
{
    const size_t tiles = (size_t)B * ((T + 159) / 160);
    return tiles > (size_t)batch_groups(B) ? tiles : (size_t)batch_groups(B);
}

}  // namespace

size_t bn_fwd_scratch_bytes(int B, int C, int T)
{
    return align_up(bn_parts_cap(B, T) * C * 3 * sizeof(double), 256) + 2 * align_up((size_t)C * sizeof(float), 256);
}

size_t bn_bwd_scratch_bytes(int B, int C) { return align_up((size_t)batch_groups(B) * C * 2 * sizeof(double), 256); }

namespace {

template <typename TS, int VEC>
hipError_t fwd_passes(int B, int C, int T, const TS *z, const BnFinal &f, bool given, const TS *res, bool relu, TS *y, hipStream_t s)
{
    const Rows rows{C, T, (T + VEC - 1) / VEC};
    if (given)
        hipLaunchKernelGGL(bn_finalize_kernel, dim3(C), dim3(64), 0, s, f, C);
    else
        hipLaunchKernelGGL((bn_stats_kernel<TS, VEC>), dim3(C, f.G), dim3(kThreads), 0, s, z, B, rows, f.G, (double *)f.part);
    const hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
    const ApplySplit a(B, rows.ng);
    const dim3 grid(C * a.blocks);
    if (given)
        hipLaunchKernelGGL((bn_apply_fwd_kernel<TS, VEC, false>), grid, dim3(kThreads), 0, s, a.n, a.per, rows, z, f, res,
                           relu ? 1 : 0, y);
    else
        hipLaunchKernelGGL((bn_apply_fwd_kernel<TS, VEC, true>), grid, dim3(kThreads), 0, s, a.n, a.per, rows, z, f, res,
                           relu ? 1 : 0, y);
    return hipGetLastError();
}

template <typename TS, int VEC>
hipError_t bwd_passes(int B, int C, int T, const TS *dy, const TS *y, const TS *z, const BnBwdFinal &f, bool relu, TS *dz, TS *dres,
                      hipStream_t s)
{
    const Rows rows{C, T, (T + VEC - 1) / VEC};
    hipLaunchKernelGGL((bn_bwd_stats_kernel<TS, VEC>), dim3(C, f.G), dim3(kThreads), 0, s, dy, y, z, f.mean, f.invstd, relu ? 1 : 0,
                       B, rows, f.G, (double *)f.part);
    const hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
    const ApplySplit a(B, rows.ng);
    hipLaunchKernelGGL((bn_bwd_apply_kernel<TS, VEC>), dim3(C * a.blocks), dim3(kThreads), 0, s, a.n, a.per, rows, dy, y, z, f,
                       relu ? 1 : 0, dz, dres);
    return hipGetLastError();
}

}  // namespace

// Statistics of z [B][C][T], then y = relu?(gamma*zhat + beta + residual).  scratch: bn_fwd_scratch_bytes.
hipError_t launch_bn_fwd(int B, int C, int T, bool is_bf16, const void *z, const float *gamma, const float *beta, float eps,
                         const void *residual, bool relu, void *y, float *mean, float *invstd, void *scratch, hipStream_t s,
                         int given_parts)
{
    // given_parts > 0: the part array already holds that many parts per channel (written by the convolution kernel)
    const int G = given_parts > 0 ? given_parts : batch_groups(B);
    float *scale = (float *)((unsigned char *)scratch + align_up(bn_parts_cap(B, T) * C * 3 * sizeof(double), 256));
    float *shift = (float *)((unsigned char *)scale + align_up((size_t)C * sizeof(float), 256));
    const BnFinal f{(const double *)scratch, G, gamma, beta, eps, mean, invstd, scale, shift};
    auto run = [&](auto type, auto vec) {
        using TS = decltype(type);
        return fwd_passes<TS, decltype(vec)::value>(B, C, T, (const TS *)z, f, given_parts > 0, (const TS *)residual, relu, (TS *)y, s);
    };
    const bool whole = group_size(is_bf16, T) > 1;
    if (is_bf16) return whole ? run(bf16_t{}, Vec<8>{}) : run(bf16_t{}, Vec<1>{});
    return whole ? run(float{}, Vec<4>{}) : run(float{}, Vec<1>{});
}

// dgamma, dbeta, dres and the corrected dz (storage type) from dy, the saved y and z and the saved statistics.
hipError_t launch_bn_bwd(int B, int C, int T, bool is_bf16, const void *dy, const void *y, const void *z, const float *gamma,
                         const float *mean, const float *invstd, bool relu, void *dz, void *dres, float *dgamma,
                         float *dbeta, bool accumulate, void *scratch, hipStream_t s)
{
    const BnBwdFinal f{(const double *)scratch, batch_groups(B), (double)B * T, gamma, mean, invstd, dgamma, dbeta, accumulate ? 1 : 0};
    auto run = [&](auto type, auto vec) {
        using TS = decltype(type);
        return bwd_passes<TS, decltype(vec)::value>(B, C, T, (const TS *)dy, (const TS *)y, (const TS *)z, f, relu, (TS *)dz, (TS *)dres,
                                                    s);
    };
    const bool whole = group_size(is_bf16, T) > 1;
    if (is_bf16) return whole ? run(bf16_t{}, Vec<8>{}) : run(bf16_t{}, Vec<1>{});
    return whole ? run(float{}, Vec<4>{}) : run(float{}, Vec<1>{});
}

}  // namespace nm
