// Host side of the C ABI declared in include/nm_conv1d.h: argument validation,
// choice between the matrix-core kernels and the plain kernels, workspace carving,
// launches.  Validation never touches the HIP runtime, so it behaves the same on a
// host without a device.
#include "../../include/nm_conv1d.h"
#include "conv_tile.h"

#include <stdio.h>

#include <initializer_list>

#include <mutex>

using namespace nm;

// Scratch of nm_conv1d_block_fwd_static.  The name is a host-side handle only: device code and
// launches use the address hipGetSymbolAddress returns for the current device (static_scratch()).
static __device__ __align__(256) unsigned char scratch[NM_STATIC_SCRATCH_BYTES];

namespace {
// Address of `scratch` on the current device, looked up once per device.
std::mutex g_scratch_mutex;
void *g_scratch_ptr[kMaxDevices] = {};
hipError_t static_scratch(void **out)
{
    int dev = 0;
    hipError_t e = hipGetDevice(&dev);
    if (e != hipSuccess) return e;
    if (dev < 0 || dev >= kMaxDevices) return hipErrorInvalidDevice;
    std::lock_guard<std::mutex> lock(g_scratch_mutex);
    if (!g_scratch_ptr[dev]) {
        void *ptr = nullptr;
        e = hipGetSymbolAddress(&ptr, HIP_SYMBOL(scratch));
        if (e != hipSuccess) return e;
        if (!ptr) return hipErrorInvalidSymbol;
        g_scratch_ptr[dev] = ptr;
    }
    *out = g_scratch_ptr[dev];
    return hipSuccess;
}

thread_local hipEvent_t t_start_event = nullptr;
thread_local hipEvent_t t_stop_event = nullptr;
thread_local int t_timed_op = -1;    // pass whose main kernel the armed pair is for (-1: the first one launched)
thread_local int t_current_op = -1;  // pass the calling entry point is launching right now
}  // namespace

namespace nm {
DeviceInfo current_device_info()
{
    static int cached_cus[kMaxDevices] = {};  // 0: not asked yet
    DeviceInfo d = {-1, 256};
    int dev = 0;
    if (hipGetDevice(&dev) != hipSuccess) return d;
    d.dev = dev;
    if (dev < 0 || dev >= kMaxDevices) return d;
    if (cached_cus[dev] == 0) {
        int v = 0;
        cached_cus[dev] =
            (hipDeviceGetAttribute(&v, hipDeviceAttributeMultiprocessorCount, dev) == hipSuccess && v > 0) ? v : 256;
    }
    d.cus = cached_cus[dev];
    return d;
}

hipError_t ensure_dynamic_lds(LdsOptIn &state, const void *fn, int bytes)
{
    const DeviceInfo d = current_device_info();
    const bool known = d.dev >= 0 && d.dev < kMaxDevices;
    if (known && state.done[d.dev]) return hipSuccess;
    const hipError_t e = hipFuncSetAttribute(fn, hipFuncAttributeMaxDynamicSharedMemorySize, bytes);
    if (e == hipSuccess && known) state.done[d.dev] = 1;
    return e;
}

MainKernelTimer::MainKernelTimer(hipStream_t s) : stream(s), stop(nullptr)
{
    if (!(t_start_event && t_stop_event)) return;
    if (t_timed_op >= 0 && t_timed_op != t_current_op) return;  // armed for another pass of this call
    (void)hipEventRecord(t_start_event, s);
    stop = t_stop_event;
    t_start_event = nullptr;
    t_stop_event = nullptr;
}
MainKernelTimer::~MainKernelTimer()
{
    if (stop) (void)hipEventRecord(stop, stream);
}
}  // namespace nm

namespace {

constexpr unsigned kAllFlags = NM_RELU | NM_ACCUM_DW | NM_FORCE_DIRECT | NM_ACCUM_DX;
constexpr size_t kWsAlign = 256;
constexpr long long kMaxElems = (1LL << 31) - 1;

int out_len(int T, int K, int stride, int dil, int pad)
{
    if (T <= 0 || K <= 0 || stride <= 0 || dil <= 0 || pad < 0) return NM_ERR_BAD_ARG;
    const long long span = (long long)T + 2LL * pad - (long long)dil * (K - 1) - 1;
    if (span < 0) return NM_ERR_BAD_ARG;
    const long long to = span / stride + 1;
    if (to > kMaxElems) return NM_ERR_BAD_ARG;
    return (int)to;
}

// Fills g; returns NM_OK or the status to hand back.
int check_geometry(int B, int Cin, int Cout, int T, int K, int stride, int dil, int pad, int dtype,
                   unsigned flags, unsigned allowed_flags, Geom *g)
{
    if (B <= 0 || Cin <= 0 || Cout <= 0) return NM_ERR_BAD_ARG;
    const int to = out_len(T, K, stride, dil, pad);
    if (to <= 0) return NM_ERR_BAD_ARG;
    if (dtype != NM_BF16 && dtype != NM_F32) return NM_ERR_BAD_ARG;
    if (flags & ~allowed_flags) return NM_ERR_BAD_ARG;
    if ((long long)B * Cin * T > kMaxElems || (long long)B * Cout * to > kMaxElems ||
        (long long)Cout * Cin * K > kMaxElems)
        return NM_ERR_UNSUPPORTED;
    if (B > 65535 || Cout > 65535 || Cin > 65535) return NM_ERR_UNSUPPORTED;  // grid y/z limits
    if ((long long)pad + (long long)dil * K > (1 << 28) || stride > (1 << 20)) return NM_ERR_UNSUPPORTED;
    g->B = B; g->Cin = Cin; g->Cout = Cout; g->T = T; g->K = K;
    g->stride = stride; g->dil = dil; g->pad = pad; g->To = to;
    g->len = nullptr;
    return NM_OK;
}

bool overlap(const void *a, size_t na, const void *b, size_t nb)
{
    if (!a || !b) return false;
    const char *pa = (const char *)a, *pb = (const char *)b;
    return pa < pb + nb && pb < pa + na;
}

size_t elt(int dtype) { return dtype == NM_BF16 ? 2 : 4; }

// Calls so small that a thread of the plain kernel is through before the two or three launches of the matrix-core kernels are:
// its time is that of its chain of products, one after the other (0.3 to 0.4 us each, 0.08 in the weight gradient), as long
// as there are not too many of them in all.  Only float32 weight gradients and rows that are no multiple of eight long take
// this way (the others have run on the matrix-core kernels from the start).  Measured, plain / matrix cores: forward, chain
// Cin*K, 8 6.7 / 10.2 us, 22 10.8 / 8.3, K=1 in the GEMM kernel 24 13.4 / 24.8; input gradient, chain Cout*K, 6 8.0 / 11.4,
// 12 10.8 / 9.8, K=11 11 9.5 / 12.4, 22 13.1 / 12.0, stride 2 22 9.1 / 15.0; weight gradient, chain B*To, K=11 44 10.6 / 21.2,
// 90 13.7 / 21.9, K=1 82 15.6 / 12.3; float32 K=11 44 8.9 / 18.4, K=1 66 14.4 / 12.5.
bool tiny(int op, const Geom &g, int dtype)
{
    const bool wgrad = op == NM_OP_BWD_WEIGHT;
    if (dtype == NM_F32 ? !wgrad : rows16(g)) return false;
    const double products = (double)g.B * g.Cout * g.To * g.Cin * g.K;
    if (products > 1.2e7) return false;
    if (wgrad) {
        const double plain = 7.0 + 0.08 * g.B * g.To + 0.6e-6 * products;
        const bool gemm = g.K == 1 && g.stride == 1 && g.Cin >= 64 && g.Cout >= 64;
        const double base = dtype == NM_F32 ? 10.5 : gemm ? 17.0 : g.stride == 1 ? 13.0 : 12.0;
        const int most_taps = dtype == NM_F32 ? 24 : 14;  // what a tap adds to the matrix-core kernels' time, up to here
        return plain < base + 0.7 * (g.K < most_taps ? g.K : most_taps);
    }
    const long chain = (long)(op == NM_OP_FWD ? g.Cin : g.Cout) * g.K;
    const int rows = op == NM_OP_FWD ? g.Cout : g.Cin;
    if (g.K == 1 && g.stride == 1 && g.pad == 0 && rows > 64 && g.To > 64) return chain <= (op == NM_OP_FWD ? 40 : 24);  // the GEMM kernel
    if (op == NM_OP_FWD) return 5.0 + 0.3 * chain + 0.4e-6 * products < (g.K == 1 && g.stride == 1 && g.To > 64 ? 12.5 : 9.3);
    return chain <= (g.stride == 2 ? 22 : g.K == 1 ? 12 : g.K >= 11 ? 16 : 10);
}

bool use_mfma(int op, const Geom &g, int dtype, unsigned flags)
{
    if (dtype != NM_BF16 || (flags & NM_FORCE_DIRECT)) return false;
    if (tiny(op, g, dtype)) return false;
    switch (op) {
    case NM_OP_FWD: return mfma_fwd_supported(g);
    case NM_OP_BWD_DATA: return mfma_dgrad_supported(g);
    case NM_OP_BWD_WEIGHT: return mfma_wgrad_supported(g);
    default: return false;
    }
}

// Whether dz = dy*[y>0]*scale differs from dy (the plain input-gradient kernel contracts a materialised dz;
// the plain weight-gradient kernel contracts dy*[y>0] and applies scale to its sums).
bool needs_dz(unsigned flags, const float *scale) { return (flags & NM_RELU) || scale != nullptr; }

// float32 storage on the matrix cores (no copies, any alignment)
bool use_f32(int op, const Geom &g, int dtype, unsigned flags)
{
    if (dtype != NM_F32 || (flags & NM_FORCE_DIRECT) || tiny(op, g, dtype)) return false;
    return op == NM_OP_FWD ? f32_fwd_supported(g) : op == NM_OP_BWD_DATA ? f32_dgrad_supported(g) : f32_wgrad_supported(g);
}

// g = dy*[y>0] of a float32 call, written once: into dres when that is wanted, else (with a ReLU) into buf
hipError_t f32_mask_pass(const Geom &g, const void *dy, const void *y, bool relu, void *buf, void *dres, const void **gy,
                         hipStream_t s)
{
    *gy = dy;
    if (!relu && !dres) return hipSuccess;
    if (relu) *gy = dres ? dres : buf;
    return launch_epilogue_bwd(g, false, dy, y, nullptr, relu, dres ? nullptr : buf, dres, s);
}

bool aligned16(const void *p) { return ((uintptr_t)p % 16) == 0; }

// Whether a call with per-sample lengths may take the matrix-core kernels: the forward pass, the input
// gradient and the stride-1 weight-gradient kernels apply them; the general weight-gradient kernel
// does not (lengths then go to the plain kernel), unless x is copied for it, with zeros for the padding.
bool masked_on_mfma(const Geom &g, int op = NM_OP_FWD)
{
    return g.len == nullptr || op != NM_OP_BWD_WEIGHT || mfma_wgrad_fast_supported(g) || g.T % 8 != 0;
}

// Scratch need of one operation on one path (mfma: matrix-core kernels, else plain kernels).
// least: without room for the partial sums of the split engine and for as many parts of a weight gradient as are fastest.
size_t workspace_for(int op, const Geom &g, int dtype, bool mfma, bool scale_or_relu, bool least = false)
{
    if (mfma) {
        if (op == NM_OP_FWD) return least ? mfma_fwd_workspace_least(g) : mfma_fwd_workspace(g);
        if (op == NM_OP_BWD_DATA) return least ? mfma_dgrad_workspace_least(g) : mfma_dgrad_workspace(g);
        return mfma_wgrad_workspace(g, scale_or_relu, least ? 1 : kAllParts);
    }
    if (op == NM_OP_FWD) return 0;
    return scale_or_relu ? align_up((size_t)g.B * g.Cout * g.To * elt(dtype), kWsAlign) : 0;
}

// Room that a float32 forward pass or input gradient of few tiles asks for and does without (parts of
// nm_conv1d_block_fwd_static, which gives the bits of the ordinary call, fit its array).
size_t f32_conv_room(int op, const Geom &g)
{
    const size_t n = op == NM_OP_FWD ? f32_fwd_part_bytes(g) : f32_dgrad_part_bytes(g);
    return n <= NM_STATIC_SCRATCH_BYTES ? n : 0;
}
// That room inside a workspace, behind the `used` bytes: none where it is not there, or where a tensor of the call lies in it.
struct Tensor {
    const void *p;
    size_t bytes;
};
void *f32_conv_part(int op, const Geom &g, void *ws, size_t have, size_t used, std::initializer_list<Tensor> tensors)
{
    const size_t n = f32_conv_room(op, g);
    if (n == 0 || !ws || ((uintptr_t)ws % kWsAlign) != 0 || have < used + n) return nullptr;
    unsigned char *at = (unsigned char *)ws + used;
    for (const Tensor &t : tensors)
        if (overlap(at, n, t.p, t.bytes)) return nullptr;
    return at;
}

// What nm_conv1d_workspace_bytes answers for one pass.  The query sees neither the scale pointer nor the
// alignment of the tensors (misaligned tensors take the plain kernels); it sizes for the larger of the cases.
size_t asked_workspace(int op, const Geom &g, int dtype, unsigned flags, bool least = false)
{
    const size_t plain = workspace_for(op, g, dtype, false, true);
    const size_t fast = use_mfma(op, g, dtype, flags) ? workspace_for(op, g, dtype, true, true, least) : 0;
    if (use_f32(op, g, dtype, flags))
        return plain + (op == NM_OP_BWD_WEIGHT ? f32_wgrad_part_bytes(g) : f32_conv_room(op, g));
    return plain > fast ? plain : fast;
}
// The smallest workspace a pass of this geometry is served with: rows that are no multiple of eight long are served
// without room for their copies too, and float32 weight gradients without room for partial sums, by the plain kernels, so are stride-2 input gradients;
// calls of few tiles without room for the split engine's partial sums with fewer parts or by the other engines, weight gradients with fewer parts.
size_t least_workspace(int op, const Geom &g, int dtype, unsigned flags)
{
    const bool strided = op == NM_OP_BWD_DATA && g.stride == 2;
    return rows16(g) && dtype != NM_F32 && !strided ? asked_workspace(op, g, dtype, flags, true) : workspace_for(op, g, dtype, false, true);
}

int check_workspace(const void *ws, size_t have, size_t need)
{
    if (need == 0) return NM_OK;
    if (!ws || have < need || ((uintptr_t)ws % kWsAlign) != 0) return NM_ERR_WORKSPACE;
    return NM_OK;
}

int dev(hipError_t e) { return e == hipSuccess ? NM_OK : NM_ERR_DEVICE; }

// Which kernels serve one pass, and the workspace they use.
struct Route {
    bool mfma, f32;
    size_t need;     // bytes of workspace in use
    size_t part_at;  // float32 weight gradient: where the partial sums lie (behind the masked gradient)
    int status;      // NM_ERR_WORKSPACE: the workspace is too small for all of them
};
// aligned: the tensors and the way dx is accumulated allow the matrix-core kernels
Route route_pass(int op, const Geom &g, int dtype, unsigned flags, bool aligned, bool dzneeded, const void *ws, size_t have)
{
    Route r = {};
    r.mfma = use_mfma(op, g, dtype, flags) && aligned && masked_on_mfma(g, op);
    auto room = [&](bool least) {
        // (a weight gradient's copy of x lies behind room for g whether g is formed or not)
        const bool dz = op == NM_OP_FWD || dzneeded || (op == NM_OP_BWD_WEIGHT && r.mfma && !rows16(g));
        return workspace_for(op, g, dtype, r.mfma, dz, least);
    };
    r.need = room(false);
    if (r.mfma && have < r.need) {
        r.need = room(true);
        if (op == NM_OP_BWD_WEIGHT && have > r.need) {  // more than one part
            const bool dz = dzneeded || !rows16(g);
            r.need = mfma_wgrad_workspace(g, dz, mfma_wgrad_parts(g, dz, have));
        }
    }
    const bool plain_too = !rows16(g) || (op == NM_OP_BWD_DATA && g.stride == 2);
    if (r.mfma && plain_too && check_workspace(ws, have, r.need) != NM_OK) {
        r.mfma = false;  // no room for the copies
        r.need = room(false);
    }
    r.part_at = r.need;
    r.f32 = use_f32(op, g, dtype, flags);
    if (r.f32 && op == NM_OP_BWD_WEIGHT) {
        const size_t part = f32_wgrad_part_bytes(g, have > r.part_at ? have - r.part_at : 0);
        r.f32 = check_workspace(ws, have, r.need + part) == NM_OK;
        if (r.f32) r.need += part;
    }
    r.status = check_workspace(ws, have, r.need);
    return r;
}
bool accumulates_on_mfma(const Geom &g, unsigned flags) { return !((flags & NM_ACCUM_DX) && (g.stride != 1 || g.len)); }

// Consumes the armed event pair when an entry point returns without launching its main kernel.
struct DisarmOnExit {
    ~DisarmOnExit()
    {
        t_start_event = nullptr;
        t_stop_event = nullptr;
        t_current_op = -1;
    }
};

}  // namespace

extern "C" {

int nm_conv1d_out_len(int T, int K, int stride, int dilation, int pad)
{
    return out_len(T, K, stride, dilation, pad);
}

size_t nm_conv1d_workspace_bytes(int op, int B, int Cin, int Cout, int T, int K, int stride, int dilation,
                                 int pad, int dtype, unsigned flags)
{
    Geom g;
    if (op != NM_OP_FWD && op != NM_OP_BWD_DATA && op != NM_OP_BWD_WEIGHT && op != NM_OP_BWD && op != NM_OP_BN_FWD &&
        op != NM_OP_BN_BWD)
        return 0;
    if (check_geometry(B, Cin, Cout, T, K, stride, dilation, pad, dtype, flags, kAllFlags, &g) != NM_OK)
        return 0;
    // the BatchNorm calls keep their own scratch (and, backward, the dz tensor) in front of the inner call's workspace
    if (op == NM_OP_BN_FWD)
        return bn_fwd_scratch_bytes(g.B, g.Cout, g.To) +
               nm_conv1d_workspace_bytes(NM_OP_FWD, B, Cin, Cout, T, K, stride, dilation, pad, dtype, flags);
    if (op == NM_OP_BN_BWD)
        return bn_bwd_scratch_bytes(g.B, g.Cout) + align_up((size_t)g.B * g.Cout * g.To * elt(dtype), kWsAlign) +
               nm_conv1d_workspace_bytes(NM_OP_BWD, B, Cin, Cout, T, K, stride, dilation, pad, dtype, flags);
    // the fused backward keeps the two gradients' workspaces side by side
    if (op == NM_OP_BWD)
        return asked_workspace(NM_OP_BWD_DATA, g, dtype, flags) + asked_workspace(NM_OP_BWD_WEIGHT, g, dtype, flags);
    return asked_workspace(op, g, dtype, flags);
}

int nm_conv1d_time_next_main_kernel(void *start_event, void *stop_event)
{
    t_start_event = (start_event && stop_event) ? (hipEvent_t)start_event : nullptr;
    t_stop_event = (start_event && stop_event) ? (hipEvent_t)stop_event : nullptr;
    t_timed_op = -1;
    return NM_OK;
}

int nm_conv1d_time_next_kernel_of(void *start_event, void *stop_event, int op)
{
    if (op != NM_OP_FWD && op != NM_OP_BWD_DATA && op != NM_OP_BWD_WEIGHT) return NM_ERR_BAD_ARG;
    nm_conv1d_time_next_main_kernel(start_event, stop_event);
    t_timed_op = op;
    return NM_OK;
}

int nm_conv1d_kernel_name(int op, int B, int Cin, int Cout, int T, int K, int stride, int dilation, int pad, int dtype,
                          unsigned flags, int masked, size_t workspace_bytes, char *name, size_t name_bytes)
{
    static const int some_length = 0;
    const bool bn = op == NM_OP_BN_FWD;
    if (bn) op = NM_OP_FWD;
    if ((op != NM_OP_FWD && op != NM_OP_BWD_DATA && op != NM_OP_BWD_WEIGHT) || !name || name_bytes == 0) return NM_ERR_BAD_ARG;
    Geom g;
    const int st = check_geometry(B, Cin, Cout, T, K, stride, dilation, pad, dtype, flags, kAllFlags, &g);
    if (st != NM_OK) return st;
    g.len = masked ? &some_length : nullptr;
    const void *ws = (const void *)(uintptr_t)(workspace_bytes ? kWsAlign : 0);
    const Route r = route_pass(op, g, dtype, flags, op != NM_OP_BWD_DATA || accumulates_on_mfma(g, flags), true, ws, workspace_bytes);
    if (r.status != NM_OK) return r.status;
    const char *pass = op == NM_OP_FWD ? "fwd" : op == NM_OP_BWD_DATA ? "dgrad" : "wgrad";
    if (r.mfma && op == NM_OP_FWD) name_mfma_fwd(g, bn, workspace_bytes, name, name_bytes);
    else if (r.mfma && op == NM_OP_BWD_DATA) name_mfma_dgrad(g, (flags & NM_ACCUM_DX) != 0, workspace_bytes, name, name_bytes);
    else if (r.mfma) name_mfma_wgrad(g, (flags & NM_RELU) != 0, workspace_bytes, name, name_bytes);
    else if (r.f32) snprintf(name, name_bytes, "%s", op == NM_OP_BWD_WEIGHT ? "f32_wgrad_kernel" : "f32_conv_kernel");
    else snprintf(name, name_bytes, "direct_%s_kernel", pass);
    return NM_OK;
}

const char *nm_strerror(int status)
{
    switch (status) {
    case NM_OK: return "ok";
    case NM_ERR_BAD_ARG: return "invalid argument";
    case NM_ERR_UNSUPPORTED: return "unsupported size";
    case NM_ERR_WORKSPACE: return "workspace missing, misaligned or too small";
    case NM_ERR_DEVICE: return "HIP runtime error";
    case NM_ERR_SCRATCH_LIMIT: return "geometry needs more scratch than the fixed array of the no-allocation entry point";
    default: return "unknown status";
    }
}

static int block_fwd_impl(int B, int Cin, int Cout, int T, int K, int stride, int dilation, int pad, const int *lengths,
                          const void *x, const void *w, const float *scale, const float *shift,
                          const void *residual, void *y, unsigned flags, int dtype, void *workspace,
                          size_t workspace_bytes, void *hip_stream, double *stats = nullptr, int *stats_parts = nullptr,
                          bool in_rounds = false)
{
    // stats / stats_parts (the BatchNorm entry point): where the kernel that runs can write the partial statistics of
    // its outputs it does, and *stats_parts says into how many parts per channel (0: it did not)
    DisarmOnExit disarm;
    if (stats_parts) *stats_parts = 0;
    Geom g;
    int st = check_geometry(B, Cin, Cout, T, K, stride, dilation, pad, dtype, flags,
                            NM_RELU | NM_FORCE_DIRECT, &g);
    if (st != NM_OK) return st;
    if (!x || !w || !y) return NM_ERR_BAD_ARG;
    g.len = lengths;
    const size_t e = elt(dtype);
    const size_t ny = (size_t)g.B * g.Cout * g.To * e;
    if (overlap(y, ny, x, (size_t)g.B * g.Cin * g.T * e) || overlap(y, ny, w, (size_t)g.Cout * g.Cin * g.K * e) ||
        overlap(y, ny, residual, ny))
        return NM_ERR_BAD_ARG;
    const Route r = route_pass(NM_OP_FWD, g, dtype, flags, aligned16(x) && aligned16(y) && aligned16(residual), true, workspace, workspace_bytes);
    if (r.status != NM_OK) return r.status;
    if (overlap(y, ny, workspace, r.need)) return NM_ERR_BAD_ARG;
    hipStream_t s = (hipStream_t)hip_stream;
    const bool relu = (flags & NM_RELU) != 0;
    t_current_op = NM_OP_FWD;
    if (r.mfma) {
        const int parts = (stats && stats_parts) ? mfma_fwd_stats_parts(g, w, workspace_bytes) : 0;
        const hipError_t err = launch_mfma_fwd(g, x, w, scale, shift, residual, y, relu, workspace, workspace_bytes, s, parts > 0 ? stats : nullptr, in_rounds);
        if (err == hipSuccess && parts > 0) *stats_parts = parts;
        return dev(err);
    }
    if (r.f32) {
        const size_t nc = (size_t)g.Cout * sizeof(float);
        void *part = f32_conv_part(NM_OP_FWD, g, workspace, workspace_bytes, 0,
                                   {{x, (size_t)g.B * g.Cin * g.T * e}, {w, (size_t)g.Cout * g.Cin * g.K * e}, {residual, ny}, {y, ny},
                                    {scale, nc}, {shift, nc}, {lengths, (size_t)g.B * sizeof(int)}});
        return dev(launch_f32_fwd(g, (const float *)x, (const float *)w, scale, shift, (const float *)residual, (float *)y, relu, part,
                                  part ? f32_conv_room(NM_OP_FWD, g) : 0, s));
    }
    MainKernelTimer timer(s);
    return dev(launch_direct_fwd(g, dtype == NM_BF16, x, w, scale, shift, residual, y, relu, s));
}

static int bwd_data_impl(int B, int Cin, int Cout, int T, int K, int stride, int dilation, int pad, const int *lengths,
                         const void *dy, const void *y, const float *scale, const void *w, void *dx,
                         void *dres, unsigned flags, int dtype, void *workspace, size_t workspace_bytes,
                         void *hip_stream)
{
    DisarmOnExit disarm;
    Geom g;
    int st = check_geometry(B, Cin, Cout, T, K, stride, dilation, pad, dtype, flags,
                            NM_RELU | NM_FORCE_DIRECT | NM_ACCUM_DX, &g);
    if (st != NM_OK) return st;
    if (!dy || !w || !dx) return NM_ERR_BAD_ARG;
    g.len = lengths;
    const bool relu = (flags & NM_RELU) != 0;
    if (relu && !y) return NM_ERR_BAD_ARG;
    const size_t e = elt(dtype);
    const size_t ndy = (size_t)g.B * g.Cout * g.To * e, ndx = (size_t)g.B * g.Cin * g.T * e;
    if (overlap(dx, ndx, dy, ndy) || overlap(dx, ndx, y, ndy) || overlap(dx, ndx, w, (size_t)g.Cout * g.Cin * g.K * e) ||
        overlap(dx, ndx, dres, ndy) || overlap(dres, ndy, dy, ndy) || overlap(dres, ndy, y, ndy))
        return NM_ERR_BAD_ARG;
    const bool accum = (flags & NM_ACCUM_DX) != 0;
    // accumulation into dx: the matrix-core engine adds the old value in its epilogue (stride 1, no lengths)
    const bool dzneeded = needs_dz(flags, scale);
    const Route r = route_pass(NM_OP_BWD_DATA, g, dtype, flags,
                               aligned16(dy) && aligned16(dx) && (!relu || aligned16(y)) && accumulates_on_mfma(g, flags), dzneeded,
                               workspace, workspace_bytes);
    if (r.status != NM_OK) return r.status;
    const size_t need = r.need;
    if (overlap(dx, ndx, workspace, need) || overlap(dres, ndy, workspace, need)) return NM_ERR_BAD_ARG;
    hipStream_t s = (hipStream_t)hip_stream;
    t_current_op = NM_OP_BWD_DATA;
    if (r.mfma) return dev(launch_mfma_dgrad(g, dy, y, scale, w, dx, dres, relu, accum, workspace, workspace_bytes, s));
    if (r.f32) {
        const void *gy = dy;
        hipError_t err = f32_mask_pass(g, dy, y, relu, workspace, dres, &gy, s);
        if (err != hipSuccess) return NM_ERR_DEVICE;
        void *part = f32_conv_part(NM_OP_BWD_DATA, g, workspace, workspace_bytes, align_up(need, kWsAlign),
                                   {{dy, ndy}, {y, ndy}, {w, (size_t)g.Cout * g.Cin * g.K * e}, {dx, ndx}, {dres, ndy},
                                    {scale, (size_t)g.Cout * sizeof(float)}, {lengths, (size_t)g.B * sizeof(int)}});
        return dev(launch_f32_dgrad(g, (const float *)gy, scale, (const float *)w, (float *)dx, accum, part,
                                    part ? f32_conv_room(NM_OP_BWD_DATA, g) : 0, s));
    }
    const bool bf = dtype == NM_BF16;
    const void *dz = dy;
    if (dzneeded || dres) {
        hipError_t err = launch_epilogue_bwd(g, bf, dy, y, scale, relu, dzneeded ? workspace : nullptr, dres, s);
        if (err != hipSuccess) return NM_ERR_DEVICE;
        if (dzneeded) dz = workspace;
    }
    MainKernelTimer timer(s);
    return dev(launch_direct_dgrad(g, bf, dz, w, dx, accum, s));
}

static int bwd_weight_impl(int B, int Cin, int Cout, int T, int K, int stride, int dilation, int pad, const int *lengths,
                           const void *x, const void *dy, const void *y, const float *scale, float *dw,
                           unsigned flags, int dtype, void *workspace, size_t workspace_bytes,
                           void *hip_stream)
{
    DisarmOnExit disarm;
    Geom g;
    int st = check_geometry(B, Cin, Cout, T, K, stride, dilation, pad, dtype, flags,
                            NM_RELU | NM_ACCUM_DW | NM_FORCE_DIRECT, &g);
    if (st != NM_OK) return st;
    if (!x || !dy || !dw) return NM_ERR_BAD_ARG;
    g.len = lengths;
    const bool relu = (flags & NM_RELU) != 0;
    if (relu && !y) return NM_ERR_BAD_ARG;
    const size_t e = elt(dtype);
    const size_t ndy = (size_t)g.B * g.Cout * g.To * e, ndw = (size_t)g.Cout * g.Cin * g.K * sizeof(float);
    if (overlap(dw, ndw, dy, ndy) || overlap(dw, ndw, y, ndy) || overlap(dw, ndw, x, (size_t)g.B * g.Cin * g.T * e))
        return NM_ERR_BAD_ARG;
    const Route r = route_pass(NM_OP_BWD_WEIGHT, g, dtype, flags, aligned16(x) && aligned16(dy) && (!relu || aligned16(y)),
                               needs_dz(flags, scale), workspace, workspace_bytes);
    if (r.status != NM_OK) return r.status;
    const size_t need = r.need;
    if (overlap(dw, ndw, workspace, need)) return NM_ERR_BAD_ARG;
    hipStream_t s = (hipStream_t)hip_stream;
    const bool accum = (flags & NM_ACCUM_DW) != 0;
    t_current_op = NM_OP_BWD_WEIGHT;
    if (r.mfma) return dev(launch_mfma_wgrad(g, x, dy, y, scale, dw, relu, accum, workspace, workspace_bytes, s));
    const bool bf = dtype == NM_BF16;
    const void *dz = dy;
    if (relu) {  // the kernel contracts dy*[y>0]; scale multiplies its float32 sums
        hipError_t err = launch_epilogue_bwd(g, bf, dy, y, nullptr, relu, workspace, nullptr, s);
        if (err != hipSuccess) return NM_ERR_DEVICE;
        dz = workspace;
    }
    if (r.f32)
        return dev(launch_f32_wgrad(g, (const float *)x, (const float *)dz, scale, dw, accum, (unsigned char *)workspace + r.part_at,
                                    workspace_bytes - r.part_at, s));
    MainKernelTimer timer(s);
    return dev(launch_direct_wgrad(g, bf, x, dz, scale, dw, accum, s));
}

int nm_conv1d_block_fwd(int B, int Cin, int Cout, int T, int K, int stride, int dilation, int pad, const void *x,
                        const void *w, const float *scale, const float *shift, const void *residual, void *y,
                        unsigned flags, int dtype, void *workspace, size_t workspace_bytes, void *hip_stream)
{
    return block_fwd_impl(B, Cin, Cout, T, K, stride, dilation, pad, nullptr, x, w, scale, shift, residual, y, flags, dtype,
                          workspace, workspace_bytes, hip_stream);
}

int nm_conv1d_block_fwd_static(int B, int Cin, int Cout, int T, int K, int stride, int dilation, int pad, const void *x,
                               const void *w, const float *scale, const float *shift, const void *residual, void *y,
                               unsigned flags, int dtype, void *hip_stream)
{
    // Size the scratch like nm_conv1d_workspace_bytes does (0 for invalid arguments: the shared
    // implementation below then reports them, before any device call).  Where the weights fit but not the split
    // engine's partial sums, those are made in rounds: the plan allows for this array, so the bits stay the same.
    const size_t need = nm_conv1d_workspace_bytes(NM_OP_FWD, B, Cin, Cout, T, K, stride, dilation, pad, dtype, flags);
    if (need > NM_STATIC_SCRATCH_BYTES) {
        Geom g;  // (need > 0: the arguments are valid)
        check_geometry(B, Cin, Cout, T, K, stride, dilation, pad, dtype, flags, kAllFlags, &g);
        if (least_workspace(NM_OP_FWD, g, dtype, flags) > NM_STATIC_SCRATCH_BYTES) {
            DisarmOnExit disarm;
            return NM_ERR_SCRATCH_LIMIT;
        }
    }
    void *ptr = nullptr;
    if (need > 0 && x && w && y) {  // (missing tensors: no device call before the argument error)
        if (static_scratch(&ptr) != hipSuccess) {
            DisarmOnExit disarm;
            return NM_ERR_DEVICE;
        }
    }
    return block_fwd_impl(B, Cin, Cout, T, K, stride, dilation, pad, nullptr, x, w, scale, shift, residual, y, flags, dtype,
                          ptr, ptr ? (size_t)NM_STATIC_SCRATCH_BYTES : 0, hip_stream, nullptr, nullptr, true);
}

int nm_conv1d_bwd_data(int B, int Cin, int Cout, int T, int K, int stride, int dilation, int pad, const void *dy,
                       const void *y, const float *scale, const void *w, void *dx, void *dres, unsigned flags, int dtype,
                       void *workspace, size_t workspace_bytes, void *hip_stream)
{
    return bwd_data_impl(B, Cin, Cout, T, K, stride, dilation, pad, nullptr, dy, y, scale, w, dx, dres, flags, dtype,
                         workspace, workspace_bytes, hip_stream);
}

int nm_conv1d_bwd_weight(int B, int Cin, int Cout, int T, int K, int stride, int dilation, int pad, const void *x,
                         const void *dy, const void *y, const float *scale, float *dw, unsigned flags, int dtype,
                         void *workspace, size_t workspace_bytes, void *hip_stream)
{
    return bwd_weight_impl(B, Cin, Cout, T, K, stride, dilation, pad, nullptr, x, dy, y, scale, dw, flags, dtype, workspace,
                           workspace_bytes, hip_stream);
}

int nm_conv1d_block_fwd_masked(int B, int Cin, int Cout, int T, int K, int stride, int dilation, int pad,
                               const int *lengths, const void *x, const void *w, const float *scale, const float *shift,
                               const void *residual, void *y, unsigned flags, int dtype, void *workspace,
                               size_t workspace_bytes, void *hip_stream)
{
    if (!lengths) return NM_ERR_BAD_ARG;
    return block_fwd_impl(B, Cin, Cout, T, K, stride, dilation, pad, lengths, x, w, scale, shift, residual, y, flags, dtype,
                          workspace, workspace_bytes, hip_stream);
}

int nm_conv1d_bwd_data_masked(int B, int Cin, int Cout, int T, int K, int stride, int dilation, int pad,
                              const int *lengths, const void *dy, const void *y, const float *scale, const void *w,
                              void *dx, void *dres, unsigned flags, int dtype, void *workspace, size_t workspace_bytes,
                              void *hip_stream)
{
    if (!lengths) return NM_ERR_BAD_ARG;
    return bwd_data_impl(B, Cin, Cout, T, K, stride, dilation, pad, lengths, dy, y, scale, w, dx, dres, flags, dtype,
                         workspace, workspace_bytes, hip_stream);
}

int nm_conv1d_bwd_weight_masked(int B, int Cin, int Cout, int T, int K, int stride, int dilation, int pad,
                                const int *lengths, const void *x, const void *dy, const void *y, const float *scale,
                                float *dw, unsigned flags, int dtype, void *workspace, size_t workspace_bytes,
                                void *hip_stream)
{
    if (!lengths) return NM_ERR_BAD_ARG;
    return bwd_weight_impl(B, Cin, Cout, T, K, stride, dilation, pad, lengths, x, dy, y, scale, dw, flags, dtype, workspace,
                           workspace_bytes, hip_stream);
}

static int bwd_impl(int B, int Cin, int Cout, int T, int K, int stride, int dilation, int pad, const int *lengths,
                    const void *x, const void *dy, const void *y, const float *scale, const void *w, void *dx, void *dres,
                    float *dw, unsigned flags, int dtype, void *workspace, size_t workspace_bytes, void *hip_stream)
{
    Geom g;
    int st = check_geometry(B, Cin, Cout, T, K, stride, dilation, pad, dtype, flags, kAllFlags, &g);
    if (st == NM_OK && (!x || !dy || !w || !dx || !dw)) st = NM_ERR_BAD_ARG;
    if (st == NM_OK && (flags & NM_RELU) && !y) st = NM_ERR_BAD_ARG;
    const size_t need =
        st == NM_OK ? nm_conv1d_workspace_bytes(NM_OP_BWD, B, Cin, Cout, T, K, stride, dilation, pad, dtype, flags) : 0;
    bool whole = true;  // the workspace has the size nm_conv1d_workspace_bytes asks for
    if (st == NM_OK) {
        st = check_workspace(workspace, workspace_bytes, need);
        whole = st == NM_OK;
        if (!whole)
            st = check_workspace(workspace, workspace_bytes, least_workspace(NM_OP_BWD_DATA, g, dtype, flags) +
                                                                 least_workspace(NM_OP_BWD_WEIGHT, g, dtype, flags));
    }
    if (st != NM_OK) {
        DisarmOnExit disarm;  // an armed timer is consumed by this call whatever happens
        return st;
    }
    const bool relu = (flags & NM_RELU) != 0;
    g.len = lengths;
    const size_t e = elt(dtype);
    const size_t ndy = (size_t)g.B * g.Cout * g.To * e, nx = (size_t)g.B * g.Cin * g.T * e;
    const size_t nw = (size_t)g.Cout * g.Cin * g.K * e, ndw = (size_t)g.Cout * g.Cin * g.K * sizeof(float);
    const size_t used = need < workspace_bytes ? need : workspace_bytes;
    const bool clash = overlap(dx, nx, dy, ndy) || overlap(dx, nx, y, ndy) || overlap(dx, nx, w, nw) || overlap(dx, nx, x, nx) ||
                       overlap(dres, ndy, dy, ndy) || overlap(dres, ndy, y, ndy) || overlap(dres, ndy, dx, nx) ||
                       overlap(dw, ndw, dy, ndy) || overlap(dw, ndw, y, ndy) || overlap(dw, ndw, x, nx) || overlap(dw, ndw, dx, nx) ||
                       overlap(dw, ndw, dres, ndy) || overlap(dx, nx, workspace, used) || overlap(dres, ndy, workspace, used) ||
                       overlap(dw, ndw, workspace, used);
    // the geometries that once were two calls keep those calls' own checks where tensors overlap
    const bool own_checks = clash && (dtype == NM_F32 || !rows16(g));
    whole = whole && !own_checks;
    // the matrix-core kernels of both gradients, and the workspace they can do with: what is more goes to the input gradient
    const bool both_mfma = use_mfma(NM_OP_BWD_DATA, g, dtype, flags) && use_mfma(NM_OP_BWD_WEIGHT, g, dtype, flags);
    const size_t dgrad_least = both_mfma ? mfma_dgrad_workspace_least(g) : 0;
    const int most = !both_mfma ? 0 : whole ? kAllParts : workspace_bytes < dgrad_least ? 0 : mfma_wgrad_parts(g, true, workspace_bytes - dgrad_least);
    const bool fits = whole || (both_mfma && !own_checks && most > 0);
    const bool fused = fits && both_mfma && !(lengths && (flags & NM_ACCUM_DX)) && g.stride == 1 && mfma_wgrad_fast_supported(g) &&
                       !wgrad_k1_supported(pitched(g)) && aligned16(x) && aligned16(dy) && aligned16(dx) && (!relu || aligned16(y)) &&
                       (!dres || aligned16(dres));
    // only meaningful when fused
    const size_t ws_data = whole ? mfma_dgrad_workspace(g) : fits ? (workspace_bytes - mfma_wgrad_workspace(g, true, most)) / kWsAlign * kWsAlign : 0;
    // pointwise layers: the input gradient's masked g = dy*[y>0] also feeds the K=1 weight-gradient GEMM
    const bool fused_k1 = fits && both_mfma && !lengths && g.stride == 1 && wgrad_k1_supported(pitched(g)) && aligned16(x) &&
                          aligned16(dy) && aligned16(dx) && (!relu || aligned16(y));
    SplitSum dx_sum;  // of the input gradient's parts: launched with the weight gradient's
    if (fused_k1) {
        DisarmOnExit disarm;
        if (clash) return NM_ERR_BAD_ARG;
        hipStream_t s = (hipStream_t)hip_stream;
        const void *g_plain = nullptr;
        hipError_t err;
        if (!rows16(g)) {  // (K = 1 without padding: To == T)
            unsigned char *ws_w = (unsigned char *)workspace + ws_data;
            void *xp = ws_w + mfma_wgrad_x_offset(g, most);
            const DzfLayout none = {};
            err = launch_bwd_prepare(g, dy, y, scale, w, true, relu, workspace, nullptr, none, dres, &g_plain, s, x, xp);
            if (err != hipSuccess) return NM_ERR_DEVICE;
            t_current_op = NM_OP_BWD_DATA;
            err = launch_mfma_dgrad_prepared(g, g_plain, scale, w, dx, (flags & NM_ACCUM_DX) != 0, workspace, ws_data, s, &dx_sum);
            if (err != hipSuccess) return NM_ERR_DEVICE;
            t_current_op = NM_OP_BWD_WEIGHT;
            return dev(launch_wgrad_k1(pitched(g), xp, g_plain, scale, dw, (flags & NM_ACCUM_DW) != 0, ws_w, s, dx_sum.set ? &dx_sum : nullptr));
        }
        t_current_op = NM_OP_BWD_DATA;
        err = launch_mfma_dgrad(g, dy, y, scale, w, dx, dres, relu, (flags & NM_ACCUM_DX) != 0, workspace, ws_data, s, &g_plain, &dx_sum);
        if (err != hipSuccess || !g_plain) return NM_ERR_DEVICE;
        t_current_op = NM_OP_BWD_WEIGHT;
        return dev(launch_wgrad_k1(g, x, g_plain, scale, dw, (flags & NM_ACCUM_DW) != 0, (unsigned char *)workspace + ws_data, s,
                                   dx_sum.set ? &dx_sum : nullptr));
    }
    // stride 2: the input gradient's g is plain too, and what the general weight-gradient kernel reads
    const bool fused_s2 = fits && both_mfma && !clash && g.stride == 2 && rows16(g) && !(flags & NM_ACCUM_DX) && masked_on_mfma(g, NM_OP_BWD_WEIGHT) && aligned16(x) &&
                          aligned16(dy) && aligned16(dx) && (!relu || aligned16(y));
    if (fused_s2) {
        DisarmOnExit disarm;
        hipStream_t s = (hipStream_t)hip_stream;
        const void *g_plain = nullptr;
        t_current_op = NM_OP_BWD_DATA;
        hipError_t err = launch_mfma_dgrad(g, dy, y, scale, w, dx, dres, relu, false, workspace, ws_data, s, &g_plain);
        if (err != hipSuccess || !g_plain) return NM_ERR_DEVICE;
        t_current_op = NM_OP_BWD_WEIGHT;
        return dev(launch_mfma_wgrad(g, x, g_plain, nullptr, scale, dw, false, (flags & NM_ACCUM_DW) != 0,
                                     (unsigned char *)workspace + ws_data, workspace_bytes - ws_data, s));
    }
    // float32 on the matrix cores: the masked gradient is formed once for both
    // (a workspace without room for the input gradient's parts serves it too)
    const size_t f32_taken = dtype == NM_F32 ? workspace_for(NM_OP_BWD_DATA, g, dtype, false, true) + workspace_for(NM_OP_BWD_WEIGHT, g, dtype, false, true) : 0;
    const size_t f32_parts_room = workspace_bytes > f32_taken ? workspace_bytes - f32_taken : 0;
    const bool f32_room = whole || (!own_checks && dtype == NM_F32 &&
                                    check_workspace(workspace, workspace_bytes, f32_taken + f32_wgrad_part_bytes(g, f32_parts_room)) == NM_OK);
    const bool fused_f32 = f32_room && use_f32(NM_OP_BWD_DATA, g, dtype, flags) && use_f32(NM_OP_BWD_WEIGHT, g, dtype, flags);
    if (fused_f32) {
        DisarmOnExit disarm;
        hipStream_t s = (hipStream_t)hip_stream;
        const void *gy = dy;
        hipError_t err = f32_mask_pass(g, dy, y, relu, workspace, dres, &gy, s);
        if (err != hipSuccess) return NM_ERR_DEVICE;
        t_current_op = NM_OP_BWD_DATA;
        // (the weight gradient's parts come to lie where the input gradient's were)
        const size_t behind = workspace_for(NM_OP_BWD_DATA, g, dtype, false, true);
        void *part = f32_conv_part(NM_OP_BWD_DATA, g, workspace, workspace_bytes, behind,
                                   {{x, nx}, {dy, ndy}, {y, ndy}, {w, nw}, {dx, nx}, {dres, ndy}, {dw, ndw},
                                    {scale, (size_t)g.Cout * sizeof(float)}, {lengths, (size_t)g.B * sizeof(int)}});
        err = launch_f32_dgrad(g, (const float *)gy, scale, (const float *)w, (float *)dx, (flags & NM_ACCUM_DX) != 0, part,
                               part ? f32_conv_room(NM_OP_BWD_DATA, g) : 0, s);
        if (err != hipSuccess) return NM_ERR_DEVICE;
        t_current_op = NM_OP_BWD_WEIGHT;
        return dev(launch_f32_wgrad(g, (const float *)x, (const float *)gy, scale, dw, (flags & NM_ACCUM_DW) != 0,
                                    (unsigned char *)workspace + behind, f32_parts_room, s));
    }
    if (!fused) {
        // two calls sharing the workspace one after the other (their own argument checks apply)
        const size_t w1 = whole ? nm_conv1d_workspace_bytes(NM_OP_BWD_DATA, B, Cin, Cout, T, K, stride, dilation, pad, dtype, flags)
                                : workspace_bytes;
        // a timer armed for the weight-gradient kernel outlives the first of the two calls
        hipEvent_t keep_start = t_start_event, keep_stop = t_stop_event;
        const bool keep = t_timed_op == NM_OP_BWD_WEIGHT;
        st = bwd_data_impl(B, Cin, Cout, T, K, stride, dilation, pad, lengths, dy, y, scale, w, dx, dres, flags & ~NM_ACCUM_DW,
                           dtype, workspace, w1, hip_stream);
        if (st != NM_OK) return st;
        if (keep) {
            t_start_event = keep_start;
            t_stop_event = keep_stop;
        }
        return bwd_weight_impl(B, Cin, Cout, T, K, stride, dilation, pad, lengths, x, dy, y, scale, dw, flags & ~NM_ACCUM_DX,
                               dtype, workspace, workspace_bytes, hip_stream);
    }
    DisarmOnExit disarm;
    if (clash) return NM_ERR_BAD_ARG;
    hipStream_t s = (hipStream_t)hip_stream;
    void *ws_w = (unsigned char *)workspace + ws_data;  // the weight gradient's workspace: partials, then dz fragments
    const DzfLayout layout = mfma_wgrad_dzf_layout(g, most);
    const void *g_plain = nullptr;
    void *xp = g.T % 8 == 0 ? nullptr : (unsigned char *)ws_w + mfma_wgrad_x_offset(g, most);  // pitched copy of x
    hipError_t err = launch_bwd_prepare(g, dy, y, scale, w, !mfma_dgrad_unpacked(g, w, ws_data), relu, workspace, (unsigned char *)ws_w + layout.offset, layout,
                                        dres, &g_plain, s, x, xp);
    if (err != hipSuccess) return NM_ERR_DEVICE;
    t_current_op = NM_OP_BWD_DATA;
    err = launch_mfma_dgrad_prepared(g, g_plain, scale, w, dx, (flags & NM_ACCUM_DX) != 0, workspace, ws_data, s, &dx_sum);
    if (err != hipSuccess) return NM_ERR_DEVICE;
    t_current_op = NM_OP_BWD_WEIGHT;
    const DefinedDw defined = {false, x, dy, relu ? y : nullptr};
    return dev(launch_mfma_wgrad_prepared(g, xp ? xp : x, scale, dw, (flags & NM_ACCUM_DW) != 0, ws_w, s, most, rows16(g) ? nullptr : &defined,
                                          dx_sum.set ? &dx_sum : nullptr));
}

int nm_conv1d_bwd(int B, int Cin, int Cout, int T, int K, int stride, int dilation, int pad, const void *x,
                  const void *dy, const void *y, const float *scale, const void *w, void *dx, void *dres, float *dw,
                  unsigned flags, int dtype, void *workspace, size_t workspace_bytes, void *hip_stream)
{
    return bwd_impl(B, Cin, Cout, T, K, stride, dilation, pad, nullptr, x, dy, y, scale, w, dx, dres, dw, flags, dtype,
                    workspace, workspace_bytes, hip_stream);
}

int nm_conv1d_bwd_masked(int B, int Cin, int Cout, int T, int K, int stride, int dilation, int pad, const int *lengths,
                         const void *x, const void *dy, const void *y, const float *scale, const void *w, void *dx,
                         void *dres, float *dw, unsigned flags, int dtype, void *workspace, size_t workspace_bytes,
                         void *hip_stream)
{
    if (!lengths) return NM_ERR_BAD_ARG;
    return bwd_impl(B, Cin, Cout, T, K, stride, dilation, pad, lengths, x, dy, y, scale, w, dx, dres, dw, flags, dtype,
                    workspace, workspace_bytes, hip_stream);
}

int nm_conv1d_bn_fwd(int B, int Cin, int Cout, int T, int K, int stride, int dilation, int pad, const void *x,
                     const void *w, const float *gamma, const float *beta, float eps, const void *residual, void *z,
                     void *y, float *mean, float *invstd, unsigned flags, int dtype, void *workspace,
                     size_t workspace_bytes, void *hip_stream)
{
    Geom g;
    int st = check_geometry(B, Cin, Cout, T, K, stride, dilation, pad, dtype, flags, NM_RELU | NM_FORCE_DIRECT, &g);
    if (st == NM_OK && (!x || !w || !z || !y || !mean || !invstd || !(eps >= 0.f))) st = NM_ERR_BAD_ARG;
    const size_t e = st == NM_OK ? elt(dtype) : 0;
    const size_t ny = st == NM_OK ? (size_t)g.B * g.Cout * g.To * e : 0;
    if (st == NM_OK && (overlap(y, ny, z, ny) || overlap(y, ny, residual, ny) || overlap(z, ny, residual, ny) ||
                        overlap(y, ny, x, (size_t)g.B * g.Cin * g.T * e) || overlap(y, ny, w, (size_t)g.Cout * g.Cin * g.K * e)))
        st = NM_ERR_BAD_ARG;
    const size_t need =
        st == NM_OK ? nm_conv1d_workspace_bytes(NM_OP_BN_FWD, B, Cin, Cout, T, K, stride, dilation, pad, dtype, flags) : 0;
    if (st == NM_OK && check_workspace(workspace, workspace_bytes, need) != NM_OK)
        st = check_workspace(workspace, workspace_bytes, bn_fwd_scratch_bytes(g.B, g.Cout, g.To) + least_workspace(NM_OP_FWD, g, dtype, flags));
    if (st == NM_OK && (overlap(y, ny, workspace, need < workspace_bytes ? need : workspace_bytes) ||
                        overlap(z, ny, workspace, need < workspace_bytes ? need : workspace_bytes)))
        st = NM_ERR_BAD_ARG;
    if (st != NM_OK) {
        DisarmOnExit disarm;
        return st;
    }
    const size_t own = bn_fwd_scratch_bytes(g.B, g.Cout, g.To);
    // the convolution itself: z = conv(x, w), no epilogue (its own argument checks apply once more); the unrolled
    // matrix-core kernels write the partial statistics of z from their epilogue, for the others a pass over z follows
    int parts = 0;
    st = block_fwd_impl(B, Cin, Cout, T, K, stride, dilation, pad, nullptr, x, w, nullptr, nullptr, nullptr, z,
                        flags & NM_FORCE_DIRECT, dtype, (unsigned char *)workspace + own, workspace_bytes - own, hip_stream,
                        (double *)workspace, &parts);
    if (st != NM_OK) return st;
    return dev(launch_bn_fwd(g.B, g.Cout, g.To, dtype == NM_BF16, z, gamma, beta, eps, residual, (flags & NM_RELU) != 0, y, mean,
                             invstd, workspace, (hipStream_t)hip_stream, parts));
}

int nm_conv1d_bn_bwd(int B, int Cin, int Cout, int T, int K, int stride, int dilation, int pad, const void *x,
                     const void *w, const float *gamma, const void *z, const void *y, const float *mean,
                     const float *invstd, const void *dy, void *dx, void *dres, float *dw, float *dgamma, float *dbeta,
                     unsigned flags, int dtype, void *workspace, size_t workspace_bytes, void *hip_stream)
{
    Geom g;
    int st = check_geometry(B, Cin, Cout, T, K, stride, dilation, pad, dtype, flags, kAllFlags, &g);
    if (st == NM_OK && (!x || !w || !z || !mean || !invstd || !dy || !dx || !dw)) st = NM_ERR_BAD_ARG;
    if (st == NM_OK && (flags & NM_RELU) && !y) st = NM_ERR_BAD_ARG;
    const size_t e = st == NM_OK ? elt(dtype) : 0;
    const size_t ny = st == NM_OK ? (size_t)g.B * g.Cout * g.To * e : 0;
    if (st == NM_OK && (overlap(dres, ny, dy, ny) || overlap(dres, ny, y, ny) || overlap(dres, ny, z, ny))) st = NM_ERR_BAD_ARG;
    const size_t need =
        st == NM_OK ? nm_conv1d_workspace_bytes(NM_OP_BN_BWD, B, Cin, Cout, T, K, stride, dilation, pad, dtype, flags) : 0;
    if (st == NM_OK && check_workspace(workspace, workspace_bytes, need) != NM_OK)
        st = check_workspace(workspace, workspace_bytes, bn_bwd_scratch_bytes(g.B, g.Cout) + align_up(ny, kWsAlign) +
                                                             least_workspace(NM_OP_BWD_DATA, g, dtype, flags) +
                                                             least_workspace(NM_OP_BWD_WEIGHT, g, dtype, flags));
    if (st == NM_OK && overlap(dres, ny, workspace, need < workspace_bytes ? need : workspace_bytes)) st = NM_ERR_BAD_ARG;
    if (st != NM_OK) {
        DisarmOnExit disarm;
        return st;
    }
    const size_t own = bn_bwd_scratch_bytes(g.B, g.Cout);
    void *dz = (unsigned char *)workspace + own;
    const size_t used = own + align_up(ny, kWsAlign);
    const bool relu = (flags & NM_RELU) != 0;
    hipError_t err = launch_bn_bwd(g.B, g.Cout, g.To, dtype == NM_BF16, dy, y, z, gamma, mean, invstd, relu, dz, dres, dgamma,
                                   dbeta, (flags & NM_ACCUM_DW) != 0, workspace, (hipStream_t)hip_stream);
    if (err != hipSuccess) {
        DisarmOnExit disarm;
        return NM_ERR_DEVICE;
    }
    // both convolution gradients of the corrected dz (no mask, no scale left to apply)
    return nm_conv1d_bwd(B, Cin, Cout, T, K, stride, dilation, pad, x, dz, nullptr, nullptr, w, dx, nullptr, dw,
                         flags & (NM_ACCUM_DW | NM_ACCUM_DX | NM_FORCE_DIRECT), dtype, (unsigned char *)workspace + used,
                         workspace_bytes - used, hip_stream);
}

}  // extern "C"
