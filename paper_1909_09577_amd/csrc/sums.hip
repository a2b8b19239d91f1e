// The last launch of a backward call of few tiles: the sum of the input gradient's parts and that of the weight gradient's, which do not
// depend on each other, side by side.  Each is bound by latency (4 to 5 us for a few MB on a chip that reads 20 in that time).
// 3 x 256 channels, K = 11, T = 48: 4.0 and 4.2 us one after the other, 4.9 together; steps of few tiles 3 to 8 % shorter.
#include "conv_tile.h"
#include "wgrad_reduce.h"

namespace nm {
namespace {

struct BothArgs {
    ConvGemmParams conv;
    int nt;
    unsigned pieces, nred, ncb;  // wavefronts' pieces of the first sum; blocks of the second, per output channel
    const float *part, *scale;
    float *dw;
    int S, K, Cout, Cin, accumulate;
    Geom own;
    DefinedDw defined;
};

template <bool MEND, bool MANY>
__global__ __launch_bounds__(256) void both_sums_kernel(const BothArgs a)
{
    extern __shared__ __align__(16) unsigned char smem[];
    unsigned blk = blockIdx.x;
    if (blk < a.nred) {  // (the longer ones first)
        reduce4_block<MEND, MANY>(reinterpret_cast<float *>(smem), (int)(blk % a.ncb), (int)(blk / a.ncb), a.part, a.dw, a.scale, a.S, a.K, a.Cout,
                                  a.Cin, a.accumulate, a.own, a.defined);
        return;
    }
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const unsigned piece = (blk - a.nred) * 4 + wave;
    if (piece < a.pieces) split_reduce_piece(a.conv, a.nt, (int)piece, threadIdx.x & 63, reinterpret_cast<float *>(smem) + wave * 16 * 32);
}

}  // namespace

hipError_t launch_split_sum(const SplitSum &sum, hipStream_t s) { return sum.set ? launch_split_reduce(sum.p, sum.nt, s) : hipSuccess; }

hipError_t launch_both_sums(const SplitSum &first, const float *part, float *dw, const float *scale, int S, int K, int Cout, int Cin,
                            bool accumulate, bool mend, const Geom &own, const DefinedDw &defined, hipStream_t s)
{
    BothArgs a = {};
    if (first.set) {
        a.conv = first.p;
        a.nt = first.nt;
        a.pieces = first.pieces();
    }
    a.ncb = (unsigned)(Cin + kReduce4Ci - 1) / kReduce4Ci;
    a.nred = a.ncb * (unsigned)Cout;
    a.part = part; a.dw = dw; a.scale = scale;
    a.S = S; a.K = K; a.Cout = Cout; a.Cin = Cin; a.accumulate = accumulate ? 1 : 0;
    a.own = own; a.defined = defined;
    const size_t tile = (size_t)kReduce4Ci * (K + 1) * sizeof(float), pieces = 4 * 16 * 32 * sizeof(float);
    auto kern = S >= 8 ? (mend ? both_sums_kernel<true, true> : both_sums_kernel<false, true>)
                       : (mend ? both_sums_kernel<true, false> : both_sums_kernel<false, false>);
    hipLaunchKernelGGL(kern, dim3(a.nred + (a.pieces + 3) / 4), dim3(256), tile > pieces ? tile : pieces, s, a);
    return hipGetLastError();
}

}  // namespace nm
