// hexconv_abi.hip -- the extern "C" entry points declared in hexconv.h:
// argument validation (host only, before anything is enqueued), choice of
// kernel per shape regime, and launch-status mapping.
#include <atomic>
#include <math.h>
#include <mutex>
#include <stdint.h>
#include <string>
#include <vector>
#include <stdlib.h>
#include <string.h>

#include "../../include/hexconv.h"
#include "hexgeom.h"
#include "kernels.h"

namespace hexk {

int device_cus()
{
    constexpr int kMaxDev = 64;
    static std::atomic<int> cache[kMaxDev];
    int dev = 0;
    if (hipGetDevice(&dev) != hipSuccess || dev < 0)
        return 256;
    if (dev < kMaxDev) {
        const int c = cache[dev].load(std::memory_order_relaxed);
        if (c > 0)
            return c;
    }
    int cus = 0;
    if (hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess ||
        cus <= 0)
        cus = 256;
    if (dev < kMaxDev)
        cache[dev].store(cus, std::memory_order_relaxed);
    return cus;
}

// ---- per-launch timing --------------------------------------------------

namespace {

std::atomic<bool> g_timing{false};
std::mutex g_timing_mu;

struct TimedLaunch {
    std::string name;
    hipEvent_t a, b;
};
std::vector<TimedLaunch> g_timed;

// "(name<args>)" or "name<args>" -> "name"
std::string kernel_base_name(const char *s)
{
    std::string n;
    for (; *s == '(' || *s == ' '; ++s) {
    }
    for (; *s != '\0' && *s != '<' && *s != '(' && *s != ')' && *s != ' ' && *s != ','; ++s)
        n.push_back(*s);
    return n;
}

} // namespace

KTimer::KTimer(const char *kernel) : name_(kernel), a_(nullptr), b_(nullptr)
{
    if (!g_timing.load(std::memory_order_relaxed))
        return;
    if (hipEventCreate(&a_) != hipSuccess) {
        a_ = nullptr;
        return;
    }
    if (hipEventCreate(&b_) != hipSuccess) {
        (void)hipEventDestroy(a_);
        a_ = nullptr;
        return;
    }
    // the launch itself records the pair (see HEX_LAUNCH)
}

KTimer::~KTimer()
{
    if (a_ == nullptr)
        return;
    std::lock_guard<std::mutex> lock(g_timing_mu);
    g_timed.push_back(TimedLaunch{kernel_base_name(name_), a_, b_});
}

} // namespace hexk

namespace {

using hexk::ConvShape;
using hexk::Dtype;
using hexk::Tried;

constexpr long kMaxElems = (1L << 31) - 1; // per tensor, int32-indexable planes

bool aligned16(const void *p) { return (reinterpret_cast<uintptr_t>(p) & 15u) == 0; }

bool dtype_ok(int dt) { return dt == HEX_F32 || dt == HEX_BF16; }

size_t dtype_bytes(int dt) { return dt == HEX_F32 ? 4 : 2; }

// Shape checks shared by every op.  Fills `sh`.  C_in/C_out both = C for pools.
int check_shape(int N, int Ci, int Co, int H, int W, int k, int stride, int dt, ConvShape &sh)
{
    if (N < 0 || Ci < 1 || Co < 1 || H < 1 || W < 1)
        return HEX_ERR_INVALID_ARG;
    if (k < 0 || k > HEX_MAX_K || stride < 1 || stride > HEX_MAX_STRIDE)
        return HEX_ERR_INVALID_ARG;
    if (!dtype_ok(dt))
        return HEX_ERR_INVALID_ARG;
    if (H > 65535 || W > 65535 || N > 65535 || Ci > 65535 || Co > 65535)
        return HEX_ERR_UNSUPPORTED;
    const long hw = static_cast<long>(H) * W;
    if (hw * N > kMaxElems / Ci || hw * N > kMaxElems / Co)
        return HEX_ERR_UNSUPPORTED;
    if (static_cast<long>(Co) * Ci * hexgeom::num_taps(k) > kMaxElems)
        return HEX_ERR_UNSUPPORTED;
    sh.N = N;
    sh.Ci = Ci;
    sh.Co = Co;
    sh.H = H;
    sh.W = W;
    sh.k = k;
    sh.s = stride;
    sh.T = hexgeom::num_taps(k);
    hexgeom::out_shape(H, W, stride, sh.Ho, sh.Wo);
    sh.D = sh.Do = sh.Z = sh.sz = 1;
    sh.kz = 0;
    return HEX_OK;
}

// Shape checks of the three-dimensional entry points: the 2-D checks of the
// plane, then the planes (D), the window depth (kz) and the plane stride.
int check_shape3d(int N, int Ci, int Co, int D, int H, int W, int k, int kz, int stride,
                  int stride_z, int dt, ConvShape &sh)
{
    if (D < 1 || kz < 0 || kz > HEX_MAX_KZ || stride_z < 1 || stride_z > HEX_MAX_STRIDE)
        return HEX_ERR_INVALID_ARG;
    int rc = check_shape(N, Ci, Co, H, W, k, stride, dt, sh);
    if (rc != HEX_OK)
        return rc;
    if (D > 65535)
        return HEX_ERR_UNSUPPORTED;
    const long dhw = static_cast<long>(D) * H * W;
    if (dhw * N > kMaxElems / Ci || dhw * N > kMaxElems / Co)
        return HEX_ERR_UNSUPPORTED;
    if (static_cast<long>(Co) * Ci * (2 * kz + 1) * sh.T > kMaxElems)
        return HEX_ERR_UNSUPPORTED;
    sh.D = D;
    sh.kz = kz;
    sh.Z = 2 * kz + 1;
    sh.sz = stride_z;
    sh.Do = (D - 1) / stride_z + 1;
    return HEX_OK;
}

int ptrs_ok(std::initializer_list<const void *> required, std::initializer_list<const void *> optional)
{
    for (const void *p : required)
        if (p == nullptr || !aligned16(p))
            return HEX_ERR_INVALID_ARG;
    for (const void *p : optional)
        if (p != nullptr && !aligned16(p))
            return HEX_ERR_INVALID_ARG;
    return HEX_OK;
}

// HIP status of the last failed launch on this thread (hex_last_launch_error)
thread_local hipError_t g_last_launch_error = hipSuccess;

int launched(hipError_t e)
{
    if (e == hipSuccess)
        return HEX_OK;
    g_last_launch_error = e;
    return HEX_ERR_LAUNCH;
}

// HEXCONV_PATH puts one family of kernels before the choice by size, for
// tests that compare the families on small tensors: "generic" takes nothing
// else; "any" (planes of any size, k_conv_any, k_conv_f32, k_wgrad_any), "few"
// (few input channels) and "rows" (bf16 rows of whole 16-byte vectors,
// k_mfma_gen, k_wgrad_bf16) where the family takes the shape at all.
enum class Force { None, Generic, Any, Few, Rows };

Force forced()
{
    const char *v = getenv("HEXCONV_PATH");
    if (v == nullptr)
        return Force::None;
    return strcmp(v, "generic") == 0 ? Force::Generic
           : strcmp(v, "any") == 0   ? Force::Any
           : strcmp(v, "few") == 0   ? Force::Few
           : strcmp(v, "rows") == 0  ? Force::Rows
                                     : Force::None;
}

bool force_generic() { return forced() == Force::Generic; }

// Estimated time of a call's other choice as offered to the kernels for any
// shape: strided = that choice is a kernel of the family "rows".
double other_us(Force f, double us, bool strided)
{
    if (f == Force::Any)
        return HUGE_VAL;
    return strided && f == Force::Rows ? 0.0 : us;
}

// Weight-gradient kernel family for a shape, its workspace and, for the
// kernel for any shape, its plan; the workspace query and the call must
// agree, so both go through this choice.
enum class WgradPath { Generic, Fused, Small, Bf16Mfma32, Bf16Mfma, Any };

struct WgradPick {
    WgradPath path = WgradPath::Generic;
    size_t ws = 0;
    hexk::WAnyPlan any;
};

WgradPath wgrad_path(const ConvShape &sh, Dtype d, hexk::WAnyPlan &any)
{
    const Force f = forced();
    if (f == Force::Generic)
        return WgradPath::Generic;
    if (f == Force::Any && hexk::wgrad_any_plan(sh, d, any))
        return WgradPath::Any;
    // where the fused backward applies, it is also the fastest weight
    // gradient with its data-gradient waves off (fp32 1 -> 16 channels, 40x40,
    // k = 2: 18 -> 13 us; bf16 1 -> 32 channels, 48x48, N = 512: 69 -> 59 us
    // at k = 2, 66 -> 38 us at k = 1)
    if (hexk::smallc_bwd_fused_ok(sh, d))
        return WgradPath::Fused;
    const bool small = hexk::smallc_wgrad_ok(sh);
    if (small && f == Force::Few)
        return WgradPath::Small;
    // few channels on rows of whole 4-column groups: float32 (43 shapes, all
    // faster than generic); bf16, for which the small-channel kernel stages x
    // once per 16 output channels, with one such block at k <= 2 (1 -> 16
    // channels, 40x40, N = 256: 27 -> 18 us at k = 1, 26 -> 23 us at k = 2; 32
    // or 64 output channels and k = 3 favour the bf16 kernels)
    if (small && sh.W % 4 == 0 && (d == hexk::F32 || (sh.Co <= 16 && sh.k <= 2)))
        return WgradPath::Small;
    int passes = 0;
    if (d == hexk::BF16) {
        // one pass of the tuned kernel (64 -> 64 channels, 128 x 128, N = 64:
        // 98 us against 149 on the kernel for any shape); several passes
        // re-read x, and the kernel for any shape wins (64 -> 128 channels, 12
        // x 12, N = 512: 59 -> 35 us; 64 -> 96, 45 x 48, N = 96: 114 -> 56)
        passes = hexk::bf16_wgrad32_passes(sh);
        if (passes == 1)
            return WgradPath::Bf16Mfma32;
    }
    // else the bf16 kernel for whole 16-byte rows, the small-channel kernel on
    // rows of whole 4-column groups or the generic one, unless the estimates
    // put another kernel clearly below it
    const bool mfma = d == hexk::BF16 && hexk::bf16_wgrad_ok(sh);
    if (mfma && f == Force::Rows)
        return WgradPath::Bf16Mfma;
    WgradPath best = WgradPath::Generic;
    double us = hexk::wgrad_generic_us(sh, d);
    const auto offer = [&](WgradPath path, double t) {
        if (t < us) {
            us = t;
            best = path;
        }
    };
    if (mfma) {
        const double t = hexk::bf16_wgrad_us(sh) * hexk::kClearly;
        offer(WgradPath::Bf16Mfma, t);
    } else if (small && sh.W % 4 == 0) {
        best = WgradPath::Small;
        us = hexk::smallc_wgrad_us(sh, d) * hexk::kClearly;
    } else {
        us *= hexk::kClearly;
        if (small)
            offer(WgradPath::Small, hexk::smallc_wgrad_us(sh, d));
    }
    if (hexk::wgrad_any_plan(sh, d, any))
        offer(WgradPath::Any, any.us);
    else if (passes > 1 && !mfma)
        return WgradPath::Bf16Mfma32;
    return best;
}

WgradPick wgrad_pick(const ConvShape &sh, Dtype d)
{
    WgradPick p;
    p.path = wgrad_path(sh, d, p.any);
    switch (p.path) {
    case WgradPath::Fused:
        p.ws = hexk::smallc_bwd_fused_workspace(sh);
        break;
    case WgradPath::Small:
        p.ws = hexk::smallc_wgrad_workspace(sh);
        break;
    case WgradPath::Bf16Mfma32:
        p.ws = hexk::bf16_wgrad32_workspace(sh);
        break;
    case WgradPath::Bf16Mfma:
        p.ws = hexk::bf16_wgrad_workspace(sh);
        break;
    case WgradPath::Any:
        p.ws = p.any.ws;
        break;
    default:
        p.ws = hexk::wgrad_generic_workspace(sh);
    }
    return p;
}

// 3-D weight gradient: the small-channel kernel with the planes around each
// output plane staged as channels (on rows of whole 4-column groups always),
// the matrix-core kernel for any size or the generic one, by their estimates
WgradPick wgrad3d_pick(const ConvShape &sh, Dtype d)
{
    WgradPick p;
    p.ws = hexk::wgrad_generic_workspace(sh);
    const Force f = forced();
    if (f == Force::Generic)
        return p;
    const double us = hexk::wgrad_generic_us(sh, d) * hexk::kClearly;
    if (hexk::smallc_wgrad_ok(sh)) {
        if (sh.W % 4 == 0 || f == Force::Few || hexk::smallc_wgrad_us(sh, d) < us) {
            p.path = WgradPath::Small;
            p.ws = hexk::smallc_wgrad_workspace(sh);
        }
        return p;
    }
    if (hexk::wgrad_any_plan(sh, d, p.any) && (p.any.us < us || f == Force::Any)) {
        p.path = WgradPath::Any;
        p.ws = p.any.ws;
    }
    return p;
}

hipError_t wgrad_run(const WgradPick &p, const void *x, const void *dy, float *dw, float *db,
                     void *ws, const ConvShape &sh, Dtype d, hipStream_t st)
{
    switch (p.path) {
    case WgradPath::Fused: // no data gradient: w is not read
        return hexk::smallc_bwd_fused(x, dy, nullptr, nullptr, dw, db, ws, sh, d, st);
    case WgradPath::Small:
        return hexk::smallc_wgrad(x, dy, dw, db, ws, sh, d, st);
    case WgradPath::Bf16Mfma32:
        return hexk::bf16_wgrad32(x, dy, dw, db, ws, sh, st);
    case WgradPath::Bf16Mfma:
        return hexk::bf16_wgrad(x, dy, dw, db, ws, sh, st);
    case WgradPath::Any:
        return hexk::wgrad_any(x, dy, dw, db, ws, sh, d, p.any, st);
    default:
        return hexk::wgrad_generic(x, dy, dw, db, ws, sh, d, st);
    }
}

// Estimated time of the generic forward / data gradient, where it runs at all.
double fwd_generic_us(const ConvShape &sh, Dtype d)
{
    return hexk::conv_fwd_generic_ok(sh) ? hexk::conv_fwd_generic_us(sh, d) : HUGE_VAL;
}

double bwd_data_generic_us(const ConvShape &sh, Dtype d)
{
    return hexk::conv_bwd_data_generic_ok(sh) ? hexk::conv_bwd_data_generic_us(sh, d) : HUGE_VAL;
}

// Every check of hexconv_bwd's arguments but the workspace, so that a bad
// argument enqueues nothing; `pick` receives the weight-gradient kernel and
// its workspace (none for an empty batch).
int bwd_check(const void *x, const void *dy, const void *w, const void *dx, const float *dw,
              const float *db, int N, int Ci, int Co, int H, int W, int k, int stride, int dt,
              ConvShape &sh, WgradPick &pick)
{
    int rc = check_shape(N, Ci, Co, H, W, k, stride, dt, sh);
    if (rc != HEX_OK)
        return rc;
    if ((rc = ptrs_ok({dw}, {x, dy, w, dx, db})) != HEX_OK)
        return rc;
    const bool empty = (N == 0 || sh.Ho == 0);
    if (!empty && (x == nullptr || dy == nullptr))
        return HEX_ERR_INVALID_ARG;
    if (dx != nullptr && w == nullptr)
        return HEX_ERR_INVALID_ARG;
    if (!empty)
        pick = wgrad_pick(sh, static_cast<Dtype>(dt));
    return HEX_OK;
}

} // namespace

// Scratch memory of hexconv_bwd_noalloc: one copy of this array per GPU,
// held until the process ends, shared by every such call on that GPU.  On
// the host the name only stands for the symbol: host code uses the device
// address of the current GPU's copy, obtained once per device by
// scratch_ptr(), never the name itself.
static __device__ __align__(256) unsigned char scratch[HEX_NOALLOC_SCRATCH_BYTES];

namespace {

constexpr int kMaxScratchDevices = 64;
std::mutex g_scratch_mu;
void *g_scratch_dev[kMaxScratchDevices];

// Device address of the current GPU's scratch array (looked up on the
// first call on each device), or nullptr if it cannot be obtained.
void *scratch_ptr()
{
    int dev = -1;
    if (hipGetDevice(&dev) != hipSuccess || dev < 0 || dev >= kMaxScratchDevices)
        return nullptr;
    std::lock_guard<std::mutex> lock(g_scratch_mu);
    if (g_scratch_dev[dev] == nullptr) {
        void *p = nullptr;
        if (hipGetSymbolAddress(&p, HIP_SYMBOL(scratch)) != hipSuccess || p == nullptr)
            return nullptr;
        g_scratch_dev[dev] = p;
    }
    return g_scratch_dev[dev];
}

} // namespace

extern "C" {

int hex_num_taps(int k)
{
    if (k < 0 || k > HEX_MAX_K)
        return HEX_ERR_INVALID_ARG;
    return hexgeom::num_taps(k);
}

int hex_out_shape(int H, int W, int k, int stride, int *H_out, int *W_out)
{
    if (H < 1 || W < 1 || k < 0 || k > HEX_MAX_K || stride < 1 || stride > HEX_MAX_STRIDE ||
        H_out == nullptr || W_out == nullptr)
        return HEX_ERR_INVALID_ARG;
    int ho = 0, wo = 0;
    hexgeom::out_shape(H, W, stride, ho, wo);
    *H_out = ho;
    *W_out = wo;
    return HEX_OK;
}

int hex_tap_table(int k, int parity, int *dcol, int *drow)
{
    if (k < 0 || k > HEX_MAX_K || (parity != 0 && parity != 1) || dcol == nullptr ||
        drow == nullptr)
        return HEX_ERR_INVALID_ARG;
    const int T = hexgeom::num_taps(k);
    for (int t = 0; t < T; ++t) {
        int dq = 0, ds = 0;
        hexgeom::tap_axial(k, t, dq, ds);
        dcol[t] = dq;
        drow[t] = hexgeom::tap_drow(dq, ds, parity);
    }
    return HEX_OK;
}

int hexconv_fwd(const void *x, const void *w, const void *bias, void *y, int N, int C_in,
                int C_out, int H, int W, int k, int stride, hex_dtype dt, int flags, void *stream)
{
    ConvShape sh;
    int rc = check_shape(N, C_in, C_out, H, W, k, stride, dt, sh);
    if (rc != HEX_OK)
        return rc;
    if ((flags & ~HEX_FLAG_RELU) != 0)
        return HEX_ERR_INVALID_ARG;
    if (N == 0)
        return HEX_OK; // empty batch: buffers may be NULL
    if ((rc = ptrs_ok({x, w, y}, {bias})) != HEX_OK)
        return rc;
    if (sh.Ho == 0)
        return HEX_OK;
    hipStream_t st = static_cast<hipStream_t>(stream);
    const bool relu = (flags & HEX_FLAG_RELU) != 0;
    const Dtype d = static_cast<Dtype>(dt);
    const Force f = forced();
    if (f != Force::Generic) {
        const bool any = f == Force::Any;
        if (!any && hexk::smallc_fwd_ok(sh))
            return launched(hexk::smallc_fwd(x, w, bias, y, sh, d, relu, st));
        // the tuned bf16 stride-1 kernels where they win, then the kernels
        // for any shape or, where the work is little, the generic one; the
        // strided bf16 kernel only where the any-shape window does not fit
        if (d == hexk::BF16 && !any && hexk::bf16_wide_first(sh, sh.Ci, sh.Co, false))
            return launched(hexk::bf16_wide_conv(x, w, bias, y, sh, false, relu, st));
        hipError_t e = hipSuccess;
        const bool strided = d == hexk::BF16 && hexk::bf16_gen_fwd_ok(sh);
        const double other =
            other_us(f, strided ? HUGE_VAL : fwd_generic_us(sh, d), strided);
        const Tried t = d == hexk::F32
                            ? hexk::conv_f32_fwd(x, w, bias, y, sh, relu, st, other, e)
                            : hexk::conv_any(x, w, bias, y, sh, d, false, relu, st, other, e);
        if (t == Tried::Ran)
            return launched(e);
        if (strided)
            return launched(hexk::bf16_gen_fwd(x, w, bias, y, sh, relu, st));
    }
    if (!hexk::conv_fwd_generic_ok(sh))
        return HEX_ERR_UNSUPPORTED;
    return launched(hexk::conv_fwd_generic(x, w, bias, y, sh, d, relu, st));
}

int hexconv_bwd_data(const void *dy, const void *w, void *dx, int N, int C_in, int C_out, int H,
                     int W, int k, int stride, hex_dtype dt, void *stream)
{
    ConvShape sh;
    int rc = check_shape(N, C_in, C_out, H, W, k, stride, dt, sh);
    if (rc != HEX_OK)
        return rc;
    if (N == 0)
        return HEX_OK; // empty batch: buffers may be NULL
    if ((rc = ptrs_ok({w, dx}, {dy})) != HEX_OK)
        return rc;
    if (dy == nullptr && sh.Ho > 0)
        return HEX_ERR_INVALID_ARG;
    hipStream_t st = static_cast<hipStream_t>(stream);
    const Dtype d = static_cast<Dtype>(dt);
    const Force f = forced();
    if (f != Force::Generic && sh.Ho > 0) {
        // bf16 on the matrix cores, by the tuned kernels where they win, unless
        // the work is little (64 images of 41 x 43, 4 -> 32 channels, k = 1:
        // 52 us on the small-channel kernel, whose fp32 arithmetic runs on
        // the vector units, 10 us here; 170 of 46 x 18, 5 -> 2: 8.6 on the
        // generic one, 13.4); fp32 of few channels on the vector units first
        const bool any = f == Force::Any;
        if (d == hexk::BF16 && !any && hexk::bf16_wide_first(sh, sh.Co, sh.Ci, true))
            return launched(hexk::bf16_wide_conv(dy, w, nullptr, dx, sh, true, false, st));
        const bool small = hexk::smallc_bwd_data_ok(sh);
        if (small && (f == Force::Few || (d == hexk::F32 && !any)))
            return launched(hexk::smallc_bwd_data(dy, w, dx, sh, d, st));
        hipError_t e = hipSuccess;
        // bf16 on rows of whole 16-byte vectors: one walk over dy for all
        // classes of pixels is the faster one for many output channels (3 ->
        // 192 channels, 112 x 96, N = 2, k = 1, stride 2: 23 us, 50 here; 128
        // -> 96, 64 x 80, N = 9, k = 2: 112, 56)
        const bool strided = d == hexk::BF16 && !small && hexk::bf16_gen_dgrad_ok(sh);
        const double other = other_us(f,
                                      small     ? hexk::smallc_bwd_data_us(sh)
                                      : strided ? hexk::bf16_gen_dgrad_us(sh)
                                                : bwd_data_generic_us(sh, d),
                                      strided);
        const Tried t = hexk::conv_any(dy, w, nullptr, dx, sh, d, true, false, st, other, e);
        if (t == Tried::Ran)
            return launched(e);
        if (small)
            return launched(hexk::smallc_bwd_data(dy, w, dx, sh, d, st));
        if (strided)
            return launched(hexk::bf16_gen_dgrad(dy, w, dx, sh, st));
    }
    if (!hexk::conv_bwd_data_generic_ok(sh))
        return HEX_ERR_UNSUPPORTED;
    return launched(hexk::conv_bwd_data_generic(dy, w, dx, sh, d, st));
}

size_t hexconv_bwd_weight_workspace(int N, int C_in, int C_out, int H, int W, int k, int stride,
                                    hex_dtype dt)
{
    ConvShape sh;
    if (check_shape(N, C_in, C_out, H, W, k, stride, dt, sh) != HEX_OK)
        return 0;
    if (N == 0 || sh.Ho == 0)
        return 0;
    return wgrad_pick(sh, static_cast<Dtype>(dt)).ws;
}

int hexconv_bwd_weight(const void *x, const void *dy, float *dw, float *db, void *ws,
                       size_t ws_bytes, int N, int C_in, int C_out, int H, int W, int k,
                       int stride, hex_dtype dt, void *stream)
{
    ConvShape sh;
    int rc = check_shape(N, C_in, C_out, H, W, k, stride, dt, sh);
    if (rc != HEX_OK)
        return rc;
    if ((rc = ptrs_ok({dw}, {x, dy, db, ws})) != HEX_OK)
        return rc;
    const bool empty = (N == 0 || sh.Ho == 0);
    if (!empty && (x == nullptr || dy == nullptr))
        return HEX_ERR_INVALID_ARG;
    const Dtype d = static_cast<Dtype>(dt);
    WgradPick pick;
    if (!empty)
        pick = wgrad_pick(sh, d);
    if (pick.ws > 0 && (ws == nullptr || ws_bytes < pick.ws))
        return HEX_ERR_INVALID_ARG;
    hipStream_t st = static_cast<hipStream_t>(stream);
    if (empty)
        return launched(hexk::fill_zero_f32(dw, db, sh, st));
    return launched(wgrad_run(pick, x, dy, dw, db, ws, sh, d, st));
}

size_t hexconv_bwd_workspace(int N, int C_in, int C_out, int H, int W, int k, int stride,
                             hex_dtype dt)
{
    ConvShape sh;
    if (check_shape(N, C_in, C_out, H, W, k, stride, dt, sh) != HEX_OK)
        return 0;
    if (N == 0 || sh.Ho == 0)
        return 0;
    return wgrad_pick(sh, static_cast<Dtype>(dt)).ws;
}

// hexconv_bwd after its checks: ws holds at least pick.ws bytes.
static int bwd_run(const WgradPick &pick, const void *x, const void *dy, const void *w, void *dx,
                   float *dw, float *db, void *ws, const ConvShape &sh, hex_dtype dt, void *stream)
{
    hipStream_t st = static_cast<hipStream_t>(stream);
    const Dtype d = static_cast<Dtype>(dt);
    const bool empty = (sh.N == 0 || sh.Ho == 0);
    if (!empty && pick.path == WgradPath::Fused)
        return launched(hexk::smallc_bwd_fused(x, dy, w, dx, dw, db, ws, sh, d, st));
    if (dx != nullptr && sh.N > 0) {
        const int rc = hexconv_bwd_data(dy, w, dx, sh.N, sh.Ci, sh.Co, sh.H, sh.W, sh.k, sh.s, dt,
                                        stream);
        if (rc != HEX_OK)
            return rc;
    }
    if (empty)
        return launched(hexk::fill_zero_f32(dw, db, sh, st));
    return launched(wgrad_run(pick, x, dy, dw, db, ws, sh, d, st));
}

int hexconv_bwd(const void *x, const void *dy, const void *w, void *dx, float *dw, float *db,
                void *ws, size_t ws_bytes, int N, int C_in, int C_out, int H, int W, int k,
                int stride, hex_dtype dt, void *stream)
{
    ConvShape sh;
    WgradPick pick;
    int rc = bwd_check(x, dy, w, dx, dw, db, N, C_in, C_out, H, W, k, stride, dt, sh, pick);
    if (rc != HEX_OK)
        return rc;
    if ((rc = ptrs_ok({}, {ws})) != HEX_OK)
        return rc;
    if (pick.ws > 0 && (ws == nullptr || ws_bytes < pick.ws))
        return HEX_ERR_INVALID_ARG;
    return bwd_run(pick, x, dy, w, dx, dw, db, ws, sh, dt, stream);
}

int hexconv_bwd_noalloc(const void *x, const void *dy, const void *w, void *dx, float *dw,
                        float *db, int N, int C_in, int C_out, int H, int W, int k, int stride,
                        hex_dtype dt, void *stream)
{
    ConvShape sh;
    WgradPick pick;
    int rc = bwd_check(x, dy, w, dx, dw, db, N, C_in, C_out, H, W, k, stride, dt, sh, pick);
    if (rc != HEX_OK)
        return rc;
    if (pick.ws > HEX_NOALLOC_SCRATCH_BYTES)
        return HEX_ERR_UNSUPPORTED;
    void *ws = nullptr;
    if (pick.ws > 0 && (ws = scratch_ptr()) == nullptr)
        return HEX_ERR_LAUNCH;
    return bwd_run(pick, x, dy, w, dx, dw, db, ws, sh, dt, stream);
}

int hexpool_fwd(const void *x, void *y, uint8_t *argmax_tap, int N, int C, int H, int W, int k,
                int stride, hex_pool_mode mode, hex_dtype dt, void *stream)
{
    ConvShape sh;
    int rc = check_shape(N, C, C, H, W, k, stride, dt, sh);
    if (rc != HEX_OK)
        return rc;
    if (mode != HEX_POOL_MAX && mode != HEX_POOL_AVG)
        return HEX_ERR_INVALID_ARG;
    if (N == 0)
        return HEX_OK; // empty batch: buffers may be NULL
    if ((rc = ptrs_ok({x, y}, {argmax_tap})) != HEX_OK)
        return rc;
    if (sh.Ho == 0)
        return HEX_OK;
    hipStream_t st = static_cast<hipStream_t>(stream);
    const Dtype d = static_cast<Dtype>(dt);
    uint8_t *am = mode == HEX_POOL_MAX ? argmax_tap : nullptr;
    if (!force_generic() && hexk::pool_fast_ok(sh, d))
        return launched(hexk::pool_fwd_fast(x, y, am, sh, mode, d, st));
    if (!force_generic() && hexk::pool_any_ok(sh, d, false, false, mode))
        return launched(hexk::pool_any_fwd(x, y, am, sh, mode, d, false, st));
    return launched(hexk::pool_fwd_generic(x, y, am, sh, mode, d, false, st));
}

int hexpool_bwd(const void *dy, const uint8_t *argmax_tap, const void *relu_y, void *dx, int N,
                int C, int H, int W, int k, int stride, hex_pool_mode mode, hex_dtype dt,
                void *stream)
{
    ConvShape sh;
    int rc = check_shape(N, C, C, H, W, k, stride, dt, sh);
    if (rc != HEX_OK)
        return rc;
    if (mode != HEX_POOL_MAX && mode != HEX_POOL_AVG)
        return HEX_ERR_INVALID_ARG;
    if (N == 0)
        return HEX_OK; // empty batch: buffers may be NULL
    if ((rc = ptrs_ok({dx}, {dy, argmax_tap, relu_y})) != HEX_OK)
        return rc;
    if (sh.Ho > 0 && (dy == nullptr || (mode == HEX_POOL_MAX && argmax_tap == nullptr)))
        return HEX_ERR_INVALID_ARG;
    hipStream_t st = static_cast<hipStream_t>(stream);
    const Dtype d = static_cast<Dtype>(dt);
    // The mean's gradient at stride 1 gathers (512 x 32 planes of 48 x 48,
    // bf16, k = 2: 1306 -> 218 us), and so does the one-tap pool.  At k = 1 by
    // phases it is the faster where a block holds a few outputs per thread
    // (160 shapes, with a mask: planes of up to 1024 pixels 0.73 to 1.06 times
    // the gather's time, larger ones 0.82 to 1.08), but for small calls of
    // more than 1024 pixels a plane (1.0 to 1.38) and past 2048 (1.3 to 1.95;
    // 512 x 32 of 48 x 48 228 -> 113 us).  Every other shape of whole rows is
    // at least as fast by phases (stride 2, max, 256 x 64 of 40 x 40: 21 us
    // against 28).
    const long hw = static_cast<long>(sh.H) * sh.W;
    const bool gather = sh.k != 1 || hw > 2048 || (hw > 1024 && hw * sh.N * sh.Ci <= 3L << 20);
    if (!force_generic() && sh.Ho > 0 && mode == HEX_POOL_AVG && sh.s == 1 && gather &&
        hexk::pool_any_ok(sh, d, false, true, mode))
        return launched(hexk::pool_any_bwd(dy, argmax_tap, relu_y, dx, sh, mode, d, false, st));
    if (!force_generic() && sh.Ho > 0 && hexk::pool_fast_ok(sh, d))
        return launched(hexk::pool_bwd_fast(dy, argmax_tap, relu_y, dx, sh, mode, d, st));
    if (!force_generic() && hexk::pool_any_ok(sh, d, false, true, mode))
        return launched(hexk::pool_any_bwd(dy, argmax_tap, relu_y, dx, sh, mode, d, false, st));
    return launched(hexk::pool_bwd_generic(dy, argmax_tap, relu_y, dx, sh, mode, d, false, st));
}

// ------------------------------------------------------- three dimensions

int hex_out_shape3d(int D, int H, int W, int k, int kz, int stride, int stride_z, int *D_out,
                    int *H_out, int *W_out)
{
    if (D < 1 || kz < 0 || kz > HEX_MAX_KZ || stride_z < 1 || stride_z > HEX_MAX_STRIDE ||
        D_out == nullptr)
        return HEX_ERR_INVALID_ARG;
    const int rc = hex_out_shape(H, W, k, stride, H_out, W_out);
    if (rc != HEX_OK)
        return rc;
    *D_out = (D - 1) / stride_z + 1;
    return HEX_OK;
}

int hexconv3d_fwd(const void *x, const void *w, const void *bias, void *y, int N, int C_in,
                  int C_out, int D, int H, int W, int k, int kz, int stride, int stride_z,
                  hex_dtype dt, int flags, void *stream)
{
    ConvShape sh;
    int rc = check_shape3d(N, C_in, C_out, D, H, W, k, kz, stride, stride_z, dt, sh);
    if (rc != HEX_OK)
        return rc;
    if ((flags & ~HEX_FLAG_RELU) != 0)
        return HEX_ERR_INVALID_ARG;
    if (N == 0)
        return HEX_OK;
    if ((rc = ptrs_ok({x, w, y}, {bias})) != HEX_OK)
        return rc;
    if (sh.Ho == 0)
        return HEX_OK;
    const Dtype d = static_cast<Dtype>(dt);
    const bool relu = (flags & HEX_FLAG_RELU) != 0;
    hipStream_t st = static_cast<hipStream_t>(stream);
    const Force f = forced();
    if (f != Force::Generic) {
        // few input channels: the small-channel forward with the 2kz + 1
        // planes around each output plane staged as extra input channels
        if (hexk::smallc_fwd_ok(sh))
            return launched(hexk::smallc_fwd(x, w, bias, y, sh, d, relu, st));
        hipError_t e = hipSuccess;
        const double gen = other_us(f, fwd_generic_us(sh, d), false);
        const Tried t = d == hexk::F32
                            ? hexk::conv_f32_fwd(x, w, bias, y, sh, relu, st, gen, e)
                            : hexk::conv_any(x, w, bias, y, sh, d, false, relu, st, gen, e);
        if (t == Tried::Ran)
            return launched(e);
    }
    if (!hexk::conv_fwd_generic_ok(sh))
        return HEX_ERR_UNSUPPORTED;
    return launched(hexk::conv_fwd_generic(x, w, bias, y, sh, d, relu, st));
}

int hexconv3d_bwd_data(const void *dy, const void *w, void *dx, int N, int C_in, int C_out, int D,
                       int H, int W, int k, int kz, int stride, int stride_z, hex_dtype dt,
                       void *stream)
{
    ConvShape sh;
    int rc = check_shape3d(N, C_in, C_out, D, H, W, k, kz, stride, stride_z, dt, sh);
    if (rc != HEX_OK)
        return rc;
    if (N == 0)
        return HEX_OK;
    if ((rc = ptrs_ok({w, dx}, {dy})) != HEX_OK)
        return rc;
    if (dy == nullptr && sh.Ho > 0)
        return HEX_ERR_INVALID_ARG;
    const Dtype d = static_cast<Dtype>(dt);
    hipStream_t st = static_cast<hipStream_t>(stream);
    const Force f = forced();
    if (f != Force::Generic && sh.Ho > 0) {
        if (hexk::smallc3d_bwd_data_ok(sh))
            return launched(hexk::smallc3d_bwd_data(dy, w, dx, sh, d, st));
        hipError_t e = hipSuccess;
        if (hexk::conv_any(dy, w, nullptr, dx, sh, d, true, false, st,
                           other_us(f, bwd_data_generic_us(sh, d), false), e) == Tried::Ran)
            return launched(e);
    }
    if (!hexk::conv_bwd_data_generic_ok(sh))
        return HEX_ERR_UNSUPPORTED;
    return launched(hexk::conv_bwd_data_generic(dy, w, dx, sh, d, st));
}

size_t hexconv3d_bwd_weight_workspace(int N, int C_in, int C_out, int D, int H, int W, int k,
                                      int kz, int stride, int stride_z, hex_dtype dt)
{
    ConvShape sh;
    if (check_shape3d(N, C_in, C_out, D, H, W, k, kz, stride, stride_z, dt, sh) != HEX_OK)
        return 0;
    if (N == 0 || sh.Ho == 0)
        return 0;
    return wgrad3d_pick(sh, static_cast<Dtype>(dt)).ws;
}

int hexconv3d_bwd_weight(const void *x, const void *dy, float *dw, float *db, void *ws,
                         size_t ws_bytes, int N, int C_in, int C_out, int D, int H, int W, int k,
                         int kz, int stride, int stride_z, hex_dtype dt, void *stream)
{
    ConvShape sh;
    int rc = check_shape3d(N, C_in, C_out, D, H, W, k, kz, stride, stride_z, dt, sh);
    if (rc != HEX_OK)
        return rc;
    if ((rc = ptrs_ok({dw}, {x, dy, db, ws})) != HEX_OK)
        return rc;
    const bool empty = (N == 0 || sh.Ho == 0);
    if (!empty && (x == nullptr || dy == nullptr))
        return HEX_ERR_INVALID_ARG;
    const Dtype d = static_cast<Dtype>(dt);
    WgradPick pick;
    if (!empty)
        pick = wgrad3d_pick(sh, d);
    if (pick.ws > 0 && (ws == nullptr || ws_bytes < pick.ws))
        return HEX_ERR_INVALID_ARG;
    hipStream_t st = static_cast<hipStream_t>(stream);
    if (empty)
        return launched(hexk::fill_zero_f32(dw, db, sh, st));
    return launched(wgrad_run(pick, x, dy, dw, db, ws, sh, d, st));
}

int hexpool3d_fwd(const void *x, void *y, uint16_t *argmax, int N, int C, int D, int H, int W,
                  int k, int kz, int stride, int stride_z, hex_pool_mode mode, hex_dtype dt,
                  void *stream)
{
    ConvShape sh;
    int rc = check_shape3d(N, C, C, D, H, W, k, kz, stride, stride_z, dt, sh);
    if (rc != HEX_OK)
        return rc;
    if (mode != HEX_POOL_MAX && mode != HEX_POOL_AVG)
        return HEX_ERR_INVALID_ARG;
    if (N == 0)
        return HEX_OK;
    if ((rc = ptrs_ok({x, y}, {argmax})) != HEX_OK)
        return rc;
    if (sh.Ho == 0)
        return HEX_OK;
    const Dtype d = static_cast<Dtype>(dt);
    hipStream_t st = static_cast<hipStream_t>(stream);
    uint16_t *am = mode == HEX_POOL_MAX ? argmax : nullptr;
    if (!force_generic() && hexk::pool_any_ok(sh, d, true, false, mode))
        return launched(hexk::pool_any_fwd(x, y, am, sh, mode, d, true, st));
    return launched(hexk::pool_fwd_generic(x, y, am, sh, mode, d, true, st));
}

int hexpool3d_bwd(const void *dy, const uint16_t *argmax, const void *relu_y, void *dx, int N,
                  int C, int D, int H, int W, int k, int kz, int stride, int stride_z,
                  hex_pool_mode mode, hex_dtype dt, void *stream)
{
    ConvShape sh;
    int rc = check_shape3d(N, C, C, D, H, W, k, kz, stride, stride_z, dt, sh);
    if (rc != HEX_OK)
        return rc;
    if (mode != HEX_POOL_MAX && mode != HEX_POOL_AVG)
        return HEX_ERR_INVALID_ARG;
    if (N == 0)
        return HEX_OK;
    if ((rc = ptrs_ok({dx}, {dy, argmax, relu_y})) != HEX_OK)
        return rc;
    if (sh.Ho > 0 && (dy == nullptr || (mode == HEX_POOL_MAX && argmax == nullptr)))
        return HEX_ERR_INVALID_ARG;
    const Dtype d = static_cast<Dtype>(dt);
    hipStream_t st = static_cast<hipStream_t>(stream);
    if (!force_generic() && hexk::pool_any_ok(sh, d, true, true, mode))
        return launched(hexk::pool_any_bwd(dy, argmax, relu_y, dx, sh, mode, d, true, st));
    return launched(hexk::pool_bwd_generic(dy, argmax, relu_y, dx, sh, mode, d, true, st));
}

int hexconv_timing_begin(void)
{
    std::lock_guard<std::mutex> lock(hexk::g_timing_mu);
    for (auto &t : hexk::g_timed) {
        (void)hipEventDestroy(t.a);
        (void)hipEventDestroy(t.b);
    }
    hexk::g_timed.clear();
    hexk::g_timing.store(true);
    return HEX_OK;
}

int hexconv_timing_end(int max_kernels, char *names, int *counts, double *total_ms,
                       int *n_kernels)
{
    hexk::g_timing.store(false);
    if (max_kernels < 1 || names == nullptr || counts == nullptr || total_ms == nullptr ||
        n_kernels == nullptr)
        return HEX_ERR_INVALID_ARG;
    std::lock_guard<std::mutex> lock(hexk::g_timing_mu);
    std::vector<std::string> order;
    int rc = HEX_OK;
    *n_kernels = 0;
    for (auto &t : hexk::g_timed) {
        float ms = 0.f;
        if (hipEventSynchronize(t.b) != hipSuccess || hipEventElapsedTime(&ms, t.a, t.b) != hipSuccess)
            rc = HEX_ERR_LAUNCH;
        (void)hipEventDestroy(t.a);
        (void)hipEventDestroy(t.b);
        int i = 0;
        while (i < static_cast<int>(order.size()) && order[i] != t.name)
            ++i;
        if (i == static_cast<int>(order.size())) {
            if (i >= max_kernels)
                continue;
            order.push_back(t.name);
            char *dst = names + static_cast<size_t>(i) * HEX_TIMING_NAME_LEN;
            strncpy(dst, t.name.c_str(), HEX_TIMING_NAME_LEN - 1);
            dst[HEX_TIMING_NAME_LEN - 1] = '\0';
            counts[i] = 0;
            total_ms[i] = 0.0;
        }
        counts[i] += 1;
        total_ms[i] += ms;
    }
    hexk::g_timed.clear();
    *n_kernels = static_cast<int>(order.size());
    return rc;
}

const char *hex_last_launch_error(void)
{
    return g_last_launch_error == hipSuccess ? "" : hipGetErrorString(g_last_launch_error);
}

const char *hex_status_string(int status)
{
    switch (status) {
    case HEX_OK:
        return "HEX_OK";
    case HEX_ERR_INVALID_ARG:
        return "HEX_ERR_INVALID_ARG: invalid argument";
    case HEX_ERR_UNSUPPORTED:
        return "HEX_ERR_UNSUPPORTED: valid request not implemented by the library";
    case HEX_ERR_LAUNCH:
        return "HEX_ERR_LAUNCH: kernel launch failed";
    default:
        return "unknown hex_status";
    }
}

} // extern "C"
