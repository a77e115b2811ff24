// k_pool_any.hip -- hexagonal max / mean pooling, forward and backward, on
// planes of any size and in three dimensions, kernel sizes 1 to 3, strides 1
// to 3 in the plane and any stride along z (Sec. 2.4).  Takes the shapes that
// the whole-row kernels of k_pool.hip do not.
//
// Both directions move little more than their bytes, so the work is to keep
// loads wide and in flight and the arithmetic per element short.  Planes that
// lie one after the other in memory are staged flat into LDS by 16-byte
// copies (no row pitch, so a row of any length costs nothing), and borders are
// tested per tap.  A 2-D pool is a single volume of N*C planes with kz = 0.
//
// Forward: a block stages the input planes that a few output planes need and
// each thread reduces whole outputs.
//
// Backward: a gather by lattice cells.  The pixels of axial coordinates
// (s Q + a, s S + b), 0 <= a, b < s, form the cell (Q, S): tap (dq, ds) sends
// to exactly one class, a = dq mod s, b = ds mod s, and reads the output
// (Q + (a - dq) / s, S + (b - ds) / s).  So a thread that owns a cell reads
// each of the few distinct outputs once (3 for k = 1, s = 2), and every
// (output, tap) pair is looked at exactly once -- no scan over taps per pixel,
// no atomics and no barriers between taps; a pixel's terms are added in tap
// order, dz first.  96 x 48 planes of 45 x 51, k = 1, stride 2, float32, max:
// 195 us on the generic kernels (a lattice test with divisions per pixel and
// tap).
#include <algorithm>
#include <type_traits>

#include "hexdev.h"
#include "kernels.h"
#include "shear.h" // FastDiv

namespace hexk {
namespace {

using namespace hexgeom;

constexpr int kPaThreads = 256;

struct PoolAnyArgs {
    int D, H, W, Do, Ho, Wo; // planes of a volume, input and output sizes
    int kz, sz, Z;
    int ch, nch;      // planes (forward: output, backward: input) per block, chunks per volume
    int rows, cols;   // backward: cell rows and columns
    FastDiv f0, f1;   // forward: by Wo and Ho * Wo; backward: by cols and rows * cols
};

// n elements of src (any element alignment) to the 16-byte aligned LDS dst
template <typename T>
__device__ __forceinline__ void copy_flat(T *__restrict__ dst, const T *__restrict__ src, int n)
{
    constexpr int V = 16 / sizeof(T);
    constexpr int U = 4;
    const int nv = n / V;
    for (int i0 = threadIdx.x; i0 < nv; i0 += U * kPaThreads) {
        uint4 q[U];
#pragma unroll
        for (int u = 0; u < U; ++u)
            __builtin_memcpy(&q[u], src + static_cast<size_t>(min(i0 + u * kPaThreads, nv - 1)) * V,
                             16);
#pragma unroll
        for (int u = 0; u < U; ++u)
            if (i0 + u * kPaThreads < nv)
                *reinterpret_cast<uint4 *>(dst + (i0 + u * kPaThreads) * V) = q[u];
    }
    for (int i = nv * V + threadIdx.x; i < n; i += kPaThreads)
        dst[i] = src[i];
}

template <typename TT, int MODE, int K, int S, typename AM>
__global__ __launch_bounds__(kPaThreads) void pool_any_fwd_k(const TT *__restrict__ x,
                                                             TT *__restrict__ y,
                                                             AM *__restrict__ am, PoolAnyArgs a)
{
    constexpr int T = num_taps(K);
    constexpr TapTable<K> tab{};
    extern __shared__ __align__(16) unsigned char smem[];
    TT *lds = reinterpret_cast<TT *>(smem);
    const int vol = blockIdx.x / a.nch;
    const int l0 = (blockIdx.x - vol * a.nch) * a.ch;
    const int l1 = min(a.Do, l0 + a.ch);
    const int z0 = max(0, a.sz * l0 - a.kz), z1 = min(a.D, a.sz * (l1 - 1) + a.kz + 1);
    const int HW = a.H * a.W, HWo = a.Ho * a.Wo;
    copy_flat(lds, x + (static_cast<size_t>(vol) * a.D + z0) * HW, (z1 - z0) * HW);
    __syncthreads();

    const size_t o0 = (static_cast<size_t>(vol) * a.Do + l0) * HWo;
    const int total = (l1 - l0) * HWo;
    for (int e = threadIdx.x; e < total; e += kPaThreads) {
        const int ll = static_cast<int>(fdiv(static_cast<uint32_t>(e), a.f1));
        const int o = e - ll * HWo;
        const int i = static_cast<int>(fdiv(static_cast<uint32_t>(o), a.f0));
        const int j = o - i * a.Wo;
        const int rc = S * i + (j & 1) * (S / 2), cc = S * j;
        const int par = (S % 2 == 0) ? 0 : (cc & 1);
        bool colok[2 * K + 1];
#pragma unroll
        for (int q = -K; q <= K; ++q)
            colok[q + K] = static_cast<uint32_t>(cc + q) < static_cast<uint32_t>(a.W);
        float best = 0.f, sum = 0.f;
        int arg = 0;
        for (int dzi = 0; dzi < a.Z; ++dzi) {
            const int z = a.sz * (l0 + ll) + dzi - a.kz;
            const bool zin = z >= 0 && z < a.D;
            const int base = (z - z0) * HW + rc * a.W + cc;
#pragma unroll
            for (int t = 0; t < T; ++t) {
                const int dq = tab.dq[t];
                const int dr = tap_drow(dq, tab.ds[t], 0) + ((dq & 1) ? par : 0);
                const bool ok = zin && colok[dq + K] &&
                                static_cast<uint32_t>(rc + dr) < static_cast<uint32_t>(a.H);
                const float raw = to_f(lds[ok ? base + dr * a.W + dq : 0]);
                const float v = ok ? raw : 0.f;
                if (MODE == 0) {
                    if ((dzi == 0 && t == 0) || v > best) {
                        best = v;
                        arg = dzi * T + t;
                    }
                } else {
                    sum += v;
                }
            }
        }
        if (MODE == 0) {
            y[o0 + e] = from_f<TT>(best);
            if (am != nullptr)
                am[o0 + e] = static_cast<AM>(arg);
        } else {
            y[o0 + e] = from_f<TT>(sum / static_cast<float>(a.Z * T));
        }
    }
}

// floor division and residue of a tap offset by the stride (compile time)
constexpr int fmod_(int v, int s) { return ((v % s) + s) % s; }

template <typename TT, int MODE, int K, int S, typename AM, bool D3, bool RELU>
__global__ __launch_bounds__(kPaThreads) void pool_any_bwd_k(const TT *__restrict__ dy,
                                                             const AM *__restrict__ am,
                                                             const TT *__restrict__ relu_y,
                                                             TT *__restrict__ dx, PoolAnyArgs a,
                                                             int am_off)
{
    constexpr int T = num_taps(K);
    extern __shared__ __align__(16) unsigned char smem[];
    TT *dyl = reinterpret_cast<TT *>(smem);
    AM *aml = reinterpret_cast<AM *>(smem + am_off);
    const int vol = blockIdx.x / a.nch;
    const int z0 = (blockIdx.x - vol * a.nch) * a.ch;
    const int z1 = min(a.D, z0 + a.ch);
    const int HW = a.H * a.W, HWo = a.Ho * a.Wo;
    // output planes whose windows reach these input planes
    const int l0 = D3 ? max(0, (z0 - a.kz + a.sz - 1) / a.sz) : z0;
    const int l1 = D3 ? min(a.Do, (z1 - 1 + a.kz) / a.sz + 1) : z1;
    const size_t go = (static_cast<size_t>(vol) * a.Do + l0) * HWo;
    if (l1 > l0) {
        copy_flat(dyl, dy + go, (l1 - l0) * HWo);
        if (MODE == 0)
            copy_flat(aml, am + go, (l1 - l0) * HWo);
    }
    __syncthreads();

    const int cells = a.rows * a.cols;
    const int nz = D3 ? 1 : z1 - z0; // planes walked by the threads together
    for (int zb = z0; zb < (D3 ? z1 : z0 + 1); ++zb) {
        for (int e = threadIdx.x; e < nz * cells; e += kPaThreads) {
            const int zi = D3 ? 0 : static_cast<int>(fdiv(static_cast<uint32_t>(e), a.f1));
            const int z = zb + zi;
            const int ce = e - zi * cells;
            const int ip = static_cast<int>(fdiv(static_cast<uint32_t>(ce), a.f0));
            const int Q = ce - ip * a.cols;
            const int Sx = ip - 1 - (Q >> 1); // axial row of the cell
            const size_t pl = (static_cast<size_t>(vol) * a.D + z) * HW;
            float acc[S][S];
            bool keep[S][S]; // the mask's reads are in flight during the sums
#pragma unroll
            for (int ca = 0; ca < S; ++ca)
#pragma unroll
                for (int b = 0; b < S; ++b) {
                    acc[ca][b] = 0.f;
                    keep[ca][b] = true;
                    if (RELU) {
                        const int c = S * Q + ca, r = S * Sx + b + (c >> 1);
                        const bool in = static_cast<uint32_t>(r) < static_cast<uint32_t>(a.H) &&
                                        c < a.W;
                        keep[ca][b] = to_f(relu_y[in ? pl + static_cast<size_t>(r) * a.W + c
                                                     : pl]) > 0.f;
                    }
                }
            for (int dzi = 0; dzi < (D3 ? a.Z : 1); ++dzi) {
                int l = z;
                if (D3) {
                    const int zc = z - (dzi - a.kz); // the same for the whole block
                    if (zc < 0 || zc % a.sz != 0 || zc / a.sz >= a.Do)
                        continue;
                    l = zc / a.sz;
                }
                const int pbase = (l - l0) * HWo;
                // the distinct outputs (Q + oq, Sx + os) reached by the taps
                constexpr int OR = (K + S - 1) / S; // largest |oq|, |os|
                float gv[2 * OR + 1][2 * OR + 1];
                int tv[2 * OR + 1][2 * OR + 1];
#pragma unroll
                for (int oq = -OR; oq <= OR; ++oq)
#pragma unroll
                    for (int os = -OR; os <= OR; ++os) {
                        const int j = Q + oq, i = Sx + os + (j >> 1);
                        const bool ok = static_cast<uint32_t>(j) < static_cast<uint32_t>(a.Wo) &&
                                        static_cast<uint32_t>(i) < static_cast<uint32_t>(a.Ho);
                        const int at = ok ? pbase + i * a.Wo + j : 0;
                        const float g = to_f(dyl[at]);
                        gv[oq + OR][os + OR] = ok ? g : 0.f;
                        if (MODE == 0) {
                            const int tp = aml[at];
                            tv[oq + OR][os + OR] = ok ? tp - dzi * T : -1;
                        }
                    }
#pragma unroll
                for (int t = 0; t < T; ++t) {
                    constexpr TapTable<K> tb{};
                    const int ca = fmod_(tb.dq[t], S), cb = fmod_(tb.ds[t], S);
                    const int oq = (ca - tb.dq[t]) / S, os = (cb - tb.ds[t]) / S;
                    const float g = gv[oq + OR][os + OR];
                    if (MODE == 0)
                        acc[ca][cb] += tv[oq + OR][os + OR] == t ? g : 0.f;
                    else
                        acc[ca][cb] += g;
                }
            }
            auto value = [&](int ca, int b) {
                float v = acc[ca][b];
                if (MODE == 1)
                    v = v / static_cast<float>(a.Z * T);
                return from_f<TT>(keep[ca][b] ? v : 0.f);
            };
#pragma unroll
            for (int b = 0; b < S; ++b) {
                if constexpr (S == 2) {
                    // the two columns of a cell share their rows
                    const int r = 2 * Sx + b + Q, c = 2 * Q;
                    if (static_cast<uint32_t>(r) >= static_cast<uint32_t>(a.H))
                        continue;
                    const size_t at = pl + static_cast<size_t>(r) * a.W + c;
                    if (c + 1 < a.W) {
                        const TT v[2] = {value(0, b), value(1, b)};
                        uint32_t u[sizeof(v) / 4];
                        __builtin_memcpy(u, v, sizeof(v));
                        // keeps the pair one store (the compiler would share
                        // the first element's store with the other branch)
                        asm volatile("" : "+v"(u[0]));
                        __builtin_memcpy(dx + at, u, sizeof(v));
                    } else {
                        dx[at] = value(0, b);
                    }
                } else {
#pragma unroll
                    for (int ca = 0; ca < S; ++ca) {
                        const int c = S * Q + ca, r = S * Sx + b + (c >> 1);
                        if (static_cast<uint32_t>(r) < static_cast<uint32_t>(a.H) && c < a.W)
                            dx[pl + static_cast<size_t>(r) * a.W + c] = value(ca, b);
                    }
                }
            }
        }
    }
}

// Gradient of the one-tap mean pool (k = 0, stride 1): dx = dy, or dy where
// the mask is positive -- the backward of a ReLU.  Flat over the tensor, 16
// bytes a lane (32 x 32 x 8 planes of 20 x 20, float32: 22.8 us as a gather
// per pixel).
template <typename TT>
__global__ __launch_bounds__(kPaThreads) void mask_k(const TT *__restrict__ dy,
                                                     const TT *__restrict__ relu_y,
                                                     TT *__restrict__ dx, size_t n)
{
    constexpr int V = 16 / sizeof(TT);
    const size_t i = (static_cast<size_t>(blockIdx.x) * kPaThreads + threadIdx.x) * V;
    if (i + V <= n) {
        TT g[V], m[V];
        *reinterpret_cast<uint4 *>(g) = *reinterpret_cast<const uint4 *>(dy + i);
        if (relu_y != nullptr) {
            *reinterpret_cast<uint4 *>(m) = *reinterpret_cast<const uint4 *>(relu_y + i);
#pragma unroll
            for (int e = 0; e < V; ++e)
                g[e] = to_f(m[e]) > 0.f ? g[e] : TT(0);
        }
        *reinterpret_cast<uint4 *>(dx + i) = *reinterpret_cast<uint4 *>(g);
    } else {
        for (size_t e = i; e < n; ++e)
            dx[e] = (relu_y == nullptr || to_f(relu_y[e]) > 0.f) ? dy[e] : TT(0);
    }
}

inline int cdiv(long a, long b) { return static_cast<int>((a + b - 1) / b); }

constexpr size_t kPaLds = 64 * 1024;    // most that one plane's work may need
constexpr size_t kPaTarget = 20 * 1024; // staged per block: eight blocks per compute unit

struct PoolAnyPlan {
    PoolAnyArgs a;
    size_t lds;
    long grid;
    int am_off;
};

// A 2-D call is one volume of N * C planes; d3 keeps the planes of a sample.
bool plan(const ConvShape &sh, Dtype dt, bool d3, bool bwd, int amb, PoolAnyPlan &p)
{
    if (sh.k < 1 || sh.k > 3 || sh.s < 1 || sh.s > 3 || sh.Ho < 1)
        return false;
    const int es = dt == F32 ? 4 : 2;
    PoolAnyArgs &a = p.a;
    a = PoolAnyArgs{};
    const long planes = static_cast<long>(sh.N) * sh.Ci;
    const long nvol = d3 ? planes : 1;
    const long D = d3 ? sh.D : planes, Do = d3 ? sh.Do : planes;
    a.D = static_cast<int>(D);
    a.Do = static_cast<int>(Do);
    a.H = sh.H;
    a.W = sh.W;
    a.Ho = sh.Ho;
    a.Wo = sh.Wo;
    a.kz = sh.kz;
    a.sz = sh.sz;
    a.Z = sh.Z;
    const size_t plane_i = static_cast<size_t>(sh.H) * sh.W * es;
    const size_t plane_o = static_cast<size_t>(sh.Ho) * sh.Wo;
    // LDS for ch planes of work
    auto need = [&](long ch) -> size_t {
        if (!bwd)
            return plane_i * std::min<long>(D, a.sz * (ch - 1) + 2 * a.kz + 1) + 16;
        const long l = d3 ? std::min<long>(Do, (ch - 1 + 2 * a.kz) / a.sz + 1) : ch;
        const size_t g = (plane_o * es * l + 15) & ~static_cast<size_t>(15);
        return g + plane_o * amb * l + 16;
    };
    const long most = bwd ? D : Do;
    if (need(1) > kPaLds || most < 1)
        return false;
    // about the target staged and enough outputs (cells) for every thread;
    // in 3-D a longer run of planes re-reads fewer of its neighbours'
    const long work = bwd ? static_cast<long>(cdiv(sh.H, sh.s) + 1) * cdiv(sh.W, sh.s)
                          : static_cast<long>(plane_o);
    long ch = 1;
    while (ch < most && need(ch + 1) <= kPaTarget && ch * work < 16 * kPaThreads)
        ++ch;
    // at least four blocks per compute unit where there is that much work
    const long want = 4L * device_cus();
    while (ch > 1 && nvol * cdiv(most, ch) < want)
        --ch;
    a.ch = static_cast<int>(ch);
    a.nch = cdiv(most, ch);
    p.lds = need(ch);
    p.grid = nvol * a.nch;
    if (p.grid > (1L << 31) - 1)
        return false;
    a.rows = (sh.H - 1) / sh.s + 2;
    a.cols = (sh.W + sh.s - 1) / sh.s;
    const long l = d3 ? std::min<long>(Do, (ch - 1 + 2 * a.kz) / a.sz + 1) : ch;
    p.am_off = static_cast<int>((plane_o * es * l + 15) & ~static_cast<size_t>(15));
    a.f0 = make_fastdiv(static_cast<uint32_t>(bwd ? a.cols : sh.Wo));
    a.f1 = make_fastdiv(static_cast<uint32_t>(bwd ? a.rows * a.cols : sh.Ho * sh.Wo));
    return true;
}

template <typename TT, int MODE, int K, int S, typename AM>
hipError_t launch_fwd(const PoolAnyPlan &p, const void *x, void *y, void *am, hipStream_t st)
{
    HEX_LAUNCH((pool_any_fwd_k<TT, MODE, K, S, AM>), dim3(static_cast<uint32_t>(p.grid)),
               dim3(kPaThreads), p.lds, st, static_cast<const TT *>(x), static_cast<TT *>(y),
               static_cast<AM *>(am), p.a);
    return hipGetLastError();
}

template <typename TT, int MODE, int K, int S, typename AM, bool D3>
hipError_t launch_bwd(const PoolAnyPlan &p, const void *dy, const void *am, const void *relu_y,
                      void *dx, hipStream_t st)
{
    const dim3 grid(static_cast<uint32_t>(p.grid));
    const TT *dyt = static_cast<const TT *>(dy), *rt = static_cast<const TT *>(relu_y);
    if (relu_y != nullptr)
        HEX_LAUNCH((pool_any_bwd_k<TT, MODE, K, S, AM, D3, true>), grid, dim3(kPaThreads), p.lds,
                   st, dyt, static_cast<const AM *>(am), rt, static_cast<TT *>(dx), p.a, p.am_off);
    else
        HEX_LAUNCH((pool_any_bwd_k<TT, MODE, K, S, AM, D3, false>), grid, dim3(kPaThreads), p.lds,
                   st, dyt, static_cast<const AM *>(am), rt, static_cast<TT *>(dx), p.a, p.am_off);
    return hipGetLastError();
}

// f(integral constants of K and S)
template <int V> using IC = std::integral_constant<int, V>;
template <typename F> hipError_t by_size(int k, int s, F &&f)
{
    auto stride = [&](auto kc) {
        return s == 1 ? f(kc, IC<1>{}) : s == 2 ? f(kc, IC<2>{}) : f(kc, IC<3>{});
    };
    return k == 1 ? stride(IC<1>{}) : k == 2 ? stride(IC<2>{}) : stride(IC<3>{});
}

bool is_mask(const ConvShape &sh, int mode)
{
    return mode == 1 && sh.k == 0 && sh.s == 1 && sh.kz == 0 && sh.sz == 1;
}

} // namespace

bool pool_any_ok(const ConvShape &sh, Dtype dt, bool d3, bool bwd, int mode)
{
    PoolAnyPlan p;
    return (bwd && is_mask(sh, mode)) || plan(sh, dt, d3, bwd, d3 ? 2 : 1, p);
}

hipError_t pool_any_fwd(const void *x, void *y, void *am, const ConvShape &sh, int mode, Dtype dt,
                        bool d3, hipStream_t st)
{
    PoolAnyPlan p;
    if (!plan(sh, dt, d3, false, d3 ? 2 : 1, p))
        return hipErrorInvalidValue;
    return by_size(sh.k, sh.s, [&](auto kc, auto sc) {
        constexpr int K = decltype(kc)::value, S = decltype(sc)::value;
        if (mode != 0)
            return dt == F32 ? launch_fwd<float, 1, K, S, uint8_t>(p, x, y, nullptr, st)
                             : launch_fwd<bf16raw, 1, K, S, uint8_t>(p, x, y, nullptr, st);
        if (d3)
            return dt == F32 ? launch_fwd<float, 0, K, S, uint16_t>(p, x, y, am, st)
                             : launch_fwd<bf16raw, 0, K, S, uint16_t>(p, x, y, am, st);
        return dt == F32 ? launch_fwd<float, 0, K, S, uint8_t>(p, x, y, am, st)
                         : launch_fwd<bf16raw, 0, K, S, uint8_t>(p, x, y, am, st);
    });
}

hipError_t pool_any_bwd(const void *dy, const void *am, const void *relu_y, void *dx,
                        const ConvShape &sh, int mode, Dtype dt, bool d3, hipStream_t st)
{
    if (is_mask(sh, mode)) {
        const size_t n = static_cast<size_t>(sh.N) * sh.Ci * sh.D * sh.H * sh.W;
        const int V = dt == F32 ? 4 : 8;
        const dim3 grid(static_cast<uint32_t>((n + V * kPaThreads - 1) / (V * kPaThreads)));
        if (dt == F32)
            HEX_LAUNCH(mask_k<float>, grid, dim3(kPaThreads), 0, st,
                       static_cast<const float *>(dy), static_cast<const float *>(relu_y),
                       static_cast<float *>(dx), n);
        else
            HEX_LAUNCH(mask_k<bf16raw>, grid, dim3(kPaThreads), 0, st,
                       static_cast<const bf16raw *>(dy), static_cast<const bf16raw *>(relu_y),
                       static_cast<bf16raw *>(dx), n);
        return hipGetLastError();
    }
    PoolAnyPlan p;
    if (!plan(sh, dt, d3, true, d3 ? 2 : 1, p))
        return hipErrorInvalidValue;
    return by_size(sh.k, sh.s, [&](auto kc, auto sc) {
        constexpr int K = decltype(kc)::value, S = decltype(sc)::value;
        auto go = [&](auto m, auto *t) {
            constexpr int M = decltype(m)::value;
            using TT = std::remove_pointer_t<decltype(t)>;
            return d3 ? launch_bwd<TT, M, K, S, uint16_t, true>(p, dy, am, relu_y, dx, st)
                      : launch_bwd<TT, M, K, S, uint8_t, false>(p, dy, am, relu_y, dx, st);
        };
        float *f = nullptr;
        bf16raw *h = nullptr;
        if (mode == 0)
            return dt == F32 ? go(IC<0>{}, f) : go(IC<0>{}, h);
        return dt == F32 ? go(IC<1>{}, f) : go(IC<1>{}, h);
    });
}

} // namespace hexk
