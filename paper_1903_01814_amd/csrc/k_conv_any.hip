// k_conv_any.hip -- convolution on the matrix cores for planes of odd sizes
// and any channel count, k = 1 to 3: the bfloat16 forward at any stride and the data
// gradient (at stride 1 the same sum with the reflected kernel) in bfloat16
// and float32, two- and three-dimensional.  (The float32 forward keeps the
// order of its sums: k_conv_f32.hip.)  The tuned bfloat16 kernels of
// k_mfma_bf16.hip need rows of whole 16-byte vectors and whole 32-channel
// blocks; this one takes what they do not, and what it does faster.  Rows
// have 4 (float32) or 8 (bfloat16) pixels and more, and the window of one
// destination row fits LDS beside a chunk's weights: at stride 1 rows to 512 /
// 307 / 149 pixels in bfloat16 and 341 / 204 / 146 in float32 at k = 1 / 2 /
// 3, in the bfloat16 forward at stride 2 464 / 254 / 130.  The data gradient
// at a stride stages the window of all its source channels: at k = 1 and
// stride 2 1024 pixels with 32 bfloat16 channels, 318 with 128, 158 with 256.
//
// Implicit GEMM on 32x32 tiles.  A block (8 waves) computes a tile of whole
// output rows of one plane (up to 256 MG pixels, groups of 32, MG per wave)
// times NB = 32 NT destination channels.  The contraction runs over chunks
// of 64 bytes of source channels (32 bfloat16 or 16 float32) and, in 3-D,
// the 2kz+1 source planes; per chunk the source rows are staged channel-last
// in LDS (chanlast.h), 80 bytes per slot (an odd multiple of 16: 16-byte
// reads of consecutive slots do not conflict).  A 16-byte operand feeds one
// 32x32x16 bfloat16 product or four 32x32x2 float32 products (lane half h
// holds channels 4h .. 4h+3 of a group of 8, product i taking channels i and
// 4 + i: the order of the contraction is free as long as both operands agree).
//
// A destination pixel's taps are fixed slot offsets from its centre's slot;
// for odd tap columns the centre column's parity adds one row, so each pixel
// keeps two base addresses and a tap costs one add.  Tiles hold whole rows
// and start at column 0, so the bases are the same for every tile.
//
// Weights sit in LDS as [tap][destination channel][64 bytes], the four
// 16-byte vectors of a row swizzled by the row (no padding, no conflicts):
// for the block's life where all chunks fit, else staged with each chunk.
// The next chunk's rows are loaded into registers during the products.
//
// float32 results leave from the accumulators, 32 pixels (128 bytes) per
// channel and instruction; bfloat16 results go through LDS, one 32-channel
// tile at a time, and leave as 16-byte vectors.
#include <algorithm>
#include <cmath>
#include <type_traits>

#include "chanlast.h"
#include "kernels.h"
#include "shear.h" // FastDiv

namespace hexk {
namespace {

using namespace hexgeom;

typedef float floatx16 __attribute__((ext_vector_type(16)));
typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));

constexpr int kAThreads = 512;
constexpr int kAWaves = kAThreads / 64;
constexpr int kSB = 80;      // bytes per window slot: 64 of channels and a pad
constexpr int kMaxTaps = 37; // k <= 3

struct AnyArgs {
    int Cs, Cd;          // source and destination channels
    int Ds, Hs, Ws;      // source planes
    int Dd, Hd, Wd;      // destination planes
    int s, sz, kz, Z;    // strides, half-depth, window planes
    int sD, sS;          // weight elements between destination / source channels
    int J;               // weight elements per channel pair (Z * taps)
    int reflect;         // data gradient: taps in reverse order
    int TR, tiles;       // destination rows per tile, tiles per plane
    int rows, RP, WCs;   // window
    int nch;             // source-channel chunks
    int nblk;            // destination-channel blocks
    int ntot;            // tiles of the batch
    int resident;
    int relu;
    int win_off;         // window (and bfloat16 result tile) after the weights
    int OP;              // result tile: bfloat16 per channel
    FastDiv fper, ftiles; // by tiles per image (all planes) and per plane
    int toff[kMaxTaps];  // byte offset of each tap from its centre's slot
};

template <typename E> struct Frag;
template <> struct Frag<bf16raw> {
    using T = bf16x8;
};
template <> struct Frag<float> {
    typedef float T __attribute__((ext_vector_type(4)));
};

// Weights of one chunk -- source channels [c0, c0 + 64 bytes), window plane
// z -- for destination channels d0 .. d0 + NB - 1; zero past Cs and Cd.
template <typename E, int T, int NB>
__device__ __forceinline__ void stage_weights(unsigned char *__restrict__ wl,
                                              const E *__restrict__ w, const AnyArgs &a, int d0,
                                              int c0, int z)
{
    constexpr int PX = AnyE<E>::PX;
    constexpr int WT = NB * 64 + 16;
    constexpr int N = T * NB * 4; // 16-byte vectors
    constexpr int UW = 4;
    using I = std::conditional_t<sizeof(E) == 4, uint32_t, uint16_t>;
    const I *wi = reinterpret_cast<const I *>(w);
    // Loads without conditions (clamped, then masked), UW vectors at a time,
    // all issued before the first is used: with a condition on each value
    // the compiler made every one of the 2-byte loads a branch with its own
    // wait, and a block spent tens of microseconds on its weights.
    for (int i0 = threadIdx.x; i0 < N; i0 += UW * kAThreads) {
        uint32_t v[UW][PX];
        int at[UW], live[UW];
#pragma unroll
        for (int u = 0; u < UW; ++u) {
            const int i = min(i0 + u * kAThreads, N - 1);
            const int t = i % T, r = i / T;
            const int o = r & 3, n = r >> 2;
            const int c = c0 + o * PX, d = d0 + n;
            const int j = a.reflect ? a.J - 1 - (z * T + t) : z * T + t;
            const I *p = wi + static_cast<size_t>(min(d, a.Cd - 1)) * a.sD + j;
            live[u] = d < a.Cd ? a.Cs - c : 0; // channels that exist
            at[u] = t * WT + n * 64 + ((o ^ ((n >> 1) & 3)) << 4);
#pragma unroll
            for (int e = 0; e < PX; ++e)
                v[u][e] = p[static_cast<size_t>(min(c + e, a.Cs - 1)) * a.sS];
        }
        __builtin_amdgcn_sched_barrier(0);
#pragma unroll
        for (int u = 0; u < UW; ++u) {
#pragma unroll
            for (int e = 0; e < PX; ++e)
                v[u][e] &= e < live[u] ? ~0u : 0u;
            uint4 q;
            if constexpr (PX == 4)
                q = make_uint4(v[u][0], v[u][1], v[u][2], v[u][3]);
            else
                q = make_uint4(v[u][0] | (v[u][1] << 16), v[u][2] | (v[u][3] << 16),
                               v[u][PX - 4] | (v[u][PX - 3] << 16),
                               v[u][PX - 2] | (v[u][PX - 1] << 16));
            if (i0 + u * kAThreads < N)
                *reinterpret_cast<uint4 *>(wl + at[u]) = q;
        }
    }
}

// HS: 32-byte halves of a chunk that are contracted (1 where every source
// channel fits the first)
template <typename E, int K, int NT, int MG, int U, int HS, bool MIS>
__global__ __launch_bounds__(kAThreads) void conv_any_k(const E *x, // not restrict: the loads ahead stay where they are
                                                        const E *__restrict__ w,
                                                        const E *__restrict__ bias,
                                                        E *__restrict__ y, AnyArgs a)
{
    constexpr bool F32 = sizeof(E) == 4;
    constexpr int PX = AnyE<E>::PX;
    constexpr int CK = 64 / sizeof(E);
    constexpr int T = num_taps(K);
    constexpr TapTable<K> tab{};
    constexpr int NB = 32 * NT;
    constexpr int WT = NB * 64 + 16;
    using F = typename Frag<E>::T;
    extern __shared__ __align__(16) unsigned char smem[];
    unsigned char *win = smem + a.win_off;
    E *outl = reinterpret_cast<E *>(win);

    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const int n32 = lane & 31, kh = lane >> 5;
    const int db = blockIdx.x % a.nblk, tstep = gridDim.x / a.nblk;
    const int d0 = db * NB;
    const size_t HWs = static_cast<size_t>(a.Hs) * a.Ws, HWd = static_cast<size_t>(a.Hd) * a.Wd;
    const size_t cs_src = HWs * a.Ds, cs_dst = HWd * a.Dd; // between channels
    const WinGeom wg{a.rows, a.RP, a.WCs, a.s, K, a.Ws};
    const int Q = a.Z * a.nch;

    // the lane's pixel per group: byte address of its centre slot, and the
    // same one row further where the centre column is odd
    int be[MG], bo[MG];
#pragma unroll
    for (int m = 0; m < MG; ++m) {
        const int p = min((wave + kAWaves * m) * 32 + n32, a.TR * a.Wd - 1);
        const int i = p / a.Wd, j = p - i * a.Wd;
        // window column s j + K + dq: residue and quotient of K + dq (toff) plus j
        be[m] = ((a.s * i + (j & 1) * (a.s >> 1) + K) * a.RP + j) * kSB + 16 * kh;
        bo[m] = be[m] + (((a.s * j) & 1) ? a.RP * kSB : 0);
    }
    // B rows (destination channel n32 of each 32): swizzled 16-byte vectors
    const int wb0 = n32 * 64 + (((0 + kh) ^ ((n32 >> 1) & 3)) << 4);
    const int wb1 = n32 * 64 + (((2 + kh) ^ ((n32 >> 1) & 3)) << 4);

    if (a.resident)
        for (int q = 0; q < Q; ++q)
            stage_weights<E, T, NB>(smem + q * T * WT, w, a, d0, (q % a.nch) * CK, q / a.nch);

    // Position: tile, window plane, chunk of channels.  Planes outside the
    // volume are passed over; the centre plane never is.
    struct Pos {
        int tb, zi, cc; // tile, window plane, channel chunk
        int n, l, i0;   // image, destination plane, first row
        int first;      // first chunk of its tile
    };
    auto place = [&](Pos &p) {
        const uint32_t per = static_cast<uint32_t>(a.Dd) * a.tiles;
        p.n = static_cast<int>(fdiv(static_cast<uint32_t>(p.tb), a.fper));
        const uint32_t r = p.tb - p.n * per;
        p.l = static_cast<int>(fdiv(r, a.ftiles));
        p.i0 = (r - p.l * a.tiles) * a.TR;
    };
    auto settle = [&](Pos &p) { // first plane from p.zi on that exists
        for (; p.zi < a.Z; ++p.zi) {
            const int zs = a.sz * p.l + p.zi - a.kz;
            if (zs >= 0 && zs < a.Ds)
                return true;
        }
        return false;
    };
    AnyItem<E, MIS> it[U];
    auto span = [&](const Pos &p, int &lo, int &run) { // existing rows of the window
        const int r_lo = a.s * p.i0 - K;
        lo = max(0, -r_lo);
        const int hi = min(a.rows, a.Hs - r_lo);
        run = (hi - lo) * a.Ws;
        return hi;
    };
    auto source = [&](const Pos &p, int lo) { // first pixel of the window's rows
        const int c0 = p.cc * CK;
        return x + (static_cast<size_t>(p.n) * a.Cs + c0) * cs_src +
                       static_cast<size_t>(a.sz * p.l + p.zi - a.kz) * HWs +
                       static_cast<size_t>(a.s * p.i0 - K + lo) * a.Ws;
    };
    auto load = [&](const Pos &p) {
        int lo, run;
        span(p, lo, run);
        const E *src = source(p, lo);
#pragma unroll
        for (int u = 0; u < U; ++u) {
            const int i = threadIdx.x + u * kAThreads;
            const int f = min((i >> 2) * PX, run - PX);
            it[u].load(src, cs_src, (i & 3) * PX, a.Cs - p.cc * CK, f);
        }
    };
    auto commit = [&](const Pos &p) {
        int lo, run;
        const int hi = span(p, lo, run);
        const int left = a.Cs - p.cc * CK; // source channels from this chunk on
#pragma unroll
        for (int u = 0; u < U; ++u) {
            const int i = threadIdx.x + u * kAThreads;
            const int f = min((i >> 2) * PX, run - PX);
            it[u].align(source(p, lo), cs_src, (i & 3) * PX, left, f);
            if (left < CK)
                it[u].drop((i & 3) * PX, left);
            if ((i >> 2) * PX < run)
                it[u].template commit<kSB>(win, wg, lo, f, i & 3);
        }
        if (p.first)
            zero_border<kSB, 4, kAThreads>(win, wg, lo, hi);
    };

    Pos cur{static_cast<int>(blockIdx.x) / a.nblk, 0, 0, 0, 0, 0, 1};
    if (cur.tb >= a.ntot)
        return;
    place(cur);
    settle(cur);
    load(cur);
    floatx16 acc[MG][NT];
    while (true) {
        // the chunk after this one, in this tile or the block's next
        Pos nxt = cur;
        nxt.first = 0;
        bool more = true, last = false;
        if (++nxt.cc == a.nch) {
            nxt.cc = 0;
            ++nxt.zi;
            last = !settle(nxt);
        }
        if (last) {
            nxt.tb += tstep;
            nxt.zi = 0;
            nxt.first = 1;
            more = nxt.tb < a.ntot;
            if (more) {
                place(nxt);
                settle(nxt);
            }
        }
        if (cur.first) {
#pragma unroll
            for (int m = 0; m < MG; ++m)
#pragma unroll
                for (int j = 0; j < NT; ++j)
                    acc[m][j] = floatx16{};
        }
        __syncthreads(); // the previous chunk's (or tile's) readers are done
        commit(cur);
        if (!a.resident)
            stage_weights<E, T, NB>(smem, w, a, d0, cur.cc * CK, cur.zi);
        __syncthreads();
        if (more)
            load(nxt);

        const int rows = min(a.TR, a.Hd - cur.i0);
        const int M = rows * a.Wd;
        if (wave * 32 < M) {
            const unsigned char *wq = smem + (a.resident ? (cur.zi * a.nch + cur.cc) * T * WT : 0);
            F fa[2][MG], fb[2][NT];
            auto read = [&](int i, F(&ra)[MG], F(&rb)[NT]) {
                const int t = i / HS, h = i % HS;
#pragma unroll
                for (int m = 0; m < MG; ++m)
                    ra[m] = *reinterpret_cast<const F *>(
                        win + ((tab.dq[t] & 1) ? bo[m] : be[m]) + a.toff[t] + 32 * h);
#pragma unroll
                for (int j = 0; j < NT; ++j)
                    rb[j] = *reinterpret_cast<const F *>(wq + (h ? wb1 : wb0) + t * WT +
                                                         j * 32 * 64);
            };
            read(0, fa[0], fb[0]);
#pragma unroll
            for (int i = 0; i < HS * T; ++i) {
                // the next step's operands are requested before this step's
                // products (left alone, the scheduler sinks them to their use)
                if (i + 1 < HS * T)
                    read(i + 1, fa[(i + 1) & 1], fb[(i + 1) & 1]);
                __builtin_amdgcn_sched_barrier(0);
#pragma unroll
                for (int j = 0; j < NT; ++j)
#pragma unroll
                    for (int m = 0; m < MG; ++m) {
                        if constexpr (F32) {
#pragma unroll
                            for (int e = 0; e < 4; ++e)
                                acc[m][j] = __builtin_amdgcn_mfma_f32_32x32x2f32(
                                    fb[i & 1][j][e], fa[i & 1][m][e], acc[m][j], 0, 0, 0);
                        } else {
                            acc[m][j] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(
                                fa[i & 1][m], fb[i & 1][j], acc[m][j], 0, 0, 0);
                        }
                    }
                __builtin_amdgcn_sched_barrier(0);
            }
        }

        if (last) {
            E *yb = y + (static_cast<size_t>(cur.n) * a.Cd + d0) * cs_dst +
                    static_cast<size_t>(cur.l) * HWd + static_cast<size_t>(cur.i0) * a.Wd;
            const int nd = min(NB, a.Cd - d0);
            if constexpr (F32) {
                // row r of D: channel 8 (r / 4) + 4 kh + r % 4; column: pixel
#pragma unroll
                for (int m = 0; m < MG; ++m) {
                    const int p = (wave + kAWaves * m) * 32 + n32;
                    if (p >= M)
                        continue;
#pragma unroll
                    for (int j = 0; j < NT; ++j)
#pragma unroll
                        for (int r = 0; r < 16; ++r) {
                            const int d = j * 32 + 8 * (r >> 2) + 4 * kh + (r & 3);
                            if (d < nd) {
                                float v = acc[m][j][r] + (bias != nullptr ? bias[d0 + d] : 0.f);
                                yb[d * cs_dst + p] = a.relu ? fmaxf(v, 0.f) : v;
                            }
                        }
                }
            } else {
#pragma unroll
                for (int j = 0; j < NT; ++j) {
                    const int ndj = min(32, nd - 32 * j);
                    if (ndj <= 0)
                        break;
                    const float bv =
                        (bias != nullptr && n32 < ndj) ? to_f(bias[d0 + 32 * j + n32]) : 0.f;
                    __syncthreads();
#pragma unroll
                    for (int m = 0; m < MG; ++m) {
                        const int g = wave + kAWaves * m;
                        if (g * 32 >= M)
                            break;
                        E *orow = outl + n32 * a.OP + g * 32 + 4 * kh;
#pragma unroll
                        for (int q = 0; q < 4; ++q) {
                            E o[4];
#pragma unroll
                            for (int r = 0; r < 4; ++r) {
                                const float v = acc[m][j][4 * q + r] + bv;
                                o[r] = from_f<E>(a.relu ? fmaxf(v, 0.f) : v);
                            }
                            uint2 u;
                            __builtin_memcpy(&u, o, 8);
                            *reinterpret_cast<uint2 *>(orow + 8 * q) = u;
                        }
                    }
                    __syncthreads();
                    const int nv = (M + 7) >> 3;
                    for (int e = threadIdx.x; e < ndj * nv; e += kAThreads) {
                        const int d = e / nv, v = e - d * nv;
                        const E *src = outl + d * a.OP + 8 * v;
                        E *dst = yb + (32 * j + d) * cs_dst + 8 * v;
                        if (8 * v + 8 <= M) {
                            const uint2 lo = *reinterpret_cast<const uint2 *>(src);
                            const uint2 hi = *reinterpret_cast<const uint2 *>(src + 4);
                            const uint4 u = make_uint4(lo.x, lo.y, hi.x, hi.y);
                            __builtin_memcpy(dst, &u, 16);
                        } else {
                            for (int p = 8 * v; p < M; ++p)
                                dst[p - 8 * v] = src[p - 8 * v];
                        }
                    }
                }
            }
        }
        if (!more)
            break;
        cur = nxt;
    }
}

// ------------------------------------------- data gradient at strides above 1
// dx pixel p = (r, c) of axial class (a, b) = (c mod s, (r - floor(c/2)) mod s)
// receives from the taps with dq = a, ds = b (mod s), and tap (dq, ds) reads
// the output at the axial offset ((a - dq) / s, (b - ds) / s) from the pixel's
// lattice cell: within a class a dense convolution of dy with a few taps.  A
// block takes s TR rows of dx; each class holds TR pixels of every column
// c = a (mod s), so the pixels of a class are the TR x ceil(W / s) elements
// (u, Q) whatever the class.  The dy rows of the tile are staged once, every
// channel of them (nch windows), and the classes take turns on them; weights
// as in the forward (all taps for the block's life where they fit, else a
// class's taps chunk by chunk).  Results leave straight from the accumulators
// (32 pixels s apart per channel; the classes that fill the gaps follow within
// the block, so the lines meet in its L2).  64 x 64 -> 64 channels, 128 x 128,
// k = 1, stride 2, bfloat16, 134 MB of dx: 161 us with the pixels sorted
// through LDS, 1020 us on the generic kernel (rows of odd length).
constexpr int kMaxCls = 64; // strides up to 8

struct DgsArgs {
    int Cs, Cd;         // dy and dx channels
    int Hs, Ws, Hd, Wd; // dy and dx planes
    int s;
    int sD, sS;         // weight elements between dx / dy channels
    int TR, tiles;      // rows of each class per tile, tiles per image
    int Qn;             // columns of a class
    int rows, RP;       // window
    int rlo, coff;      // first row offset of a tap, window column of dy column 0
    int nch, nblk, ntot, resident;
    int win_off, win_bytes; // first window, bytes per window
    FastDiv ftiles;
    int cstart[kMaxCls + 1];
    int toff[kMaxTaps]; // by class: byte offset, odd column, tap
    int todd[kMaxTaps];
    int tap[kMaxTaps];
};

template <typename E, int K, int NT, int MG, bool MIS>
__global__ __launch_bounds__(kAThreads) void conv_any_dgs_k(const E *dy, const E *__restrict__ w,
                                                            E *__restrict__ dx, DgsArgs a)
{
    constexpr bool F32 = sizeof(E) == 4;
    constexpr int PX = AnyE<E>::PX;
    constexpr int CK = 64 / sizeof(E);
    constexpr int T = num_taps(K);
    constexpr int NB = 32 * NT;
    constexpr int WT = NB * 64 + 16;
    constexpr int U = 2;
    using F = typename Frag<E>::T;
    extern __shared__ __align__(16) unsigned char smem[];
    __shared__ int tlist[kMaxTaps];

    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const int n32 = lane & 31, kh = lane >> 5;
    const int db = blockIdx.x % a.nblk, tstep = gridDim.x / a.nblk;
    const int d0 = db * NB;
    const int s = a.s;
    const uint32_t HWs = static_cast<uint32_t>(a.Hs) * a.Ws;
    const size_t HWd = static_cast<size_t>(a.Hd) * a.Wd;
    const WinGeom wg{a.rows, a.RP, a.RP, 1, a.coff, a.Ws};
    const int wb0 = n32 * 64 + (((0 + kh) ^ ((n32 >> 1) & 3)) << 4);
    const int wb1 = n32 * 64 + (((2 + kh) ^ ((n32 >> 1) & 3)) << 4);
    if (threadIdx.x < T)
        tlist[threadIdx.x] = a.tap[threadIdx.x];
    __syncthreads();

    // weights of the taps k0 .. k0 + nt - 1 (in class order) and chunk q
    auto stage_w = [&](unsigned char *wl, int k0, int nt, int q) {
        using I = std::conditional_t<F32, uint32_t, uint16_t>;
        const I *wi = reinterpret_cast<const I *>(w);
        constexpr int UW = 2;
        const int n_items = nt * NB * 4;
        for (int i0 = threadIdx.x; i0 < n_items; i0 += UW * kAThreads) {
            uint32_t v[UW][PX];
            int at[UW], live[UW];
#pragma unroll
            for (int u = 0; u < UW; ++u) {
                const int i = min(i0 + u * kAThreads, n_items - 1);
                const int t = i % nt, r = i / nt;
                const int o = r & 3, n = r >> 2;
                const int c = q * CK + o * PX, d = d0 + n;
                const I *p = wi + static_cast<size_t>(min(d, a.Cd - 1)) * a.sD + tlist[k0 + t];
                live[u] = d < a.Cd ? a.Cs - c : 0;
                at[u] = t * WT + n * 64 + ((o ^ ((n >> 1) & 3)) << 4);
#pragma unroll
                for (int e = 0; e < PX; ++e)
                    v[u][e] = p[static_cast<size_t>(min(c + e, a.Cs - 1)) * a.sS];
            }
            __builtin_amdgcn_sched_barrier(0);
#pragma unroll
            for (int u = 0; u < UW; ++u) {
#pragma unroll
                for (int e = 0; e < PX; ++e)
                    v[u][e] &= e < live[u] ? ~0u : 0u;
                uint4 q4;
                if constexpr (PX == 4)
                    q4 = make_uint4(v[u][0], v[u][1], v[u][2], v[u][3]);
                else
                    q4 = make_uint4(v[u][0] | (v[u][1] << 16), v[u][2] | (v[u][3] << 16),
                                    v[u][PX - 4] | (v[u][PX - 3] << 16),
                                    v[u][PX - 2] | (v[u][PX - 1] << 16));
                if (i0 + u * kAThreads < n_items)
                    *reinterpret_cast<uint4 *>(wl + at[u]) = q4;
            }
        }
    };
    if (a.resident)
        for (int q = 0; q < a.nch; ++q)
            stage_w(smem + q * T * WT, 0, T, q);

    for (int tb = blockIdx.x / a.nblk; tb < a.ntot; tb += tstep) {
        const int n = static_cast<int>(fdiv(static_cast<uint32_t>(tb), a.ftiles));
        const int i0 = (tb - n * a.tiles) * a.TR; // r0 = s i0
        // window row 0 is dy row i0 - 1 + rlo
        const int r_lo = i0 - 1 + a.rlo;
        const int lo = min(a.rows, max(0, -r_lo));
        const int hi = max(lo, min(a.rows, a.Hs - r_lo));
        const int run = (hi - lo) * a.Ws;
        __syncthreads(); // the previous tile's readers are done
        for (int q = 0; q < a.nch; ++q) {
            unsigned char *win = smem + a.win_off + q * a.win_bytes;
            if (run > 0) {
                const int left = a.Cs - q * CK;
                const E *src = dy + (static_cast<size_t>(n) * a.Cs + q * CK) * HWs +
                               static_cast<size_t>(r_lo + lo) * a.Ws;
                AnyItem<E, MIS> it[U];
#pragma unroll
                for (int u = 0; u < U; ++u) {
                    const int i = threadIdx.x + u * kAThreads;
                    it[u].load(src, HWs, (i & 3) * PX, left, min((i >> 2) * PX, run - PX));
                }
#pragma unroll
                for (int u = 0; u < U; ++u) {
                    const int i = threadIdx.x + u * kAThreads;
                    const int f = min((i >> 2) * PX, run - PX);
                    it[u].align(src, HWs, (i & 3) * PX, left, f);
                    if (left < CK)
                        it[u].drop((i & 3) * PX, left);
                    if ((i >> 2) * PX < run)
                        it[u].template commit<kSB>(win, wg, lo, f, i & 3);
                }
            }
            zero_border<kSB, 4, kAThreads>(win, wg, lo, hi);
        }
        __syncthreads();

        const int M = a.TR * a.Qn;
        for (int cl = 0; cl < s * s; ++cl) {
            const int ca = cl / s, cb = cl - ca * s;
            const int k0 = a.cstart[cl], nt = a.cstart[cl + 1] - k0;
            int be[MG], bo[MG], at[MG];
#pragma unroll
            for (int m = 0; m < MG; ++m) {
                const int e = min((wave + kAWaves * m) * 32 + n32, M - 1);
                const int u = e / a.Qn, Q = e - u * a.Qn;
                const int c = ca + s * Q, h = c >> 1;
                const int rr = (cb + h) % s + s * u;             // row of the tile
                const int i = (rr - cb - (h - s * (Q >> 1))) / s; // exact; its cell's row - i0
                be[m] = ((i + 1 - a.rlo) * a.RP + Q + a.coff) * kSB + 16 * kh;
                bo[m] = be[m] + ((Q & 1) ? a.RP * kSB : 0);
                const int r = s * i0 + rr;
                at[m] = (wave + kAWaves * m) * 32 + n32 < M && r < a.Hd && c < a.Wd
                            ? r * a.Wd + c
                            : -1;
            }
            floatx16 acc[MG][NT];
#pragma unroll
            for (int m = 0; m < MG; ++m)
#pragma unroll
                for (int j = 0; j < NT; ++j)
                    acc[m][j] = floatx16{};
            for (int q = 0; q < a.nch; ++q) {
                if (!a.resident) {
                    __syncthreads();
                    stage_w(smem, k0, nt, q);
                    __syncthreads();
                }
                const unsigned char *wq = smem + (a.resident ? (q * T + k0) * WT : 0);
                const unsigned char *win = smem + a.win_off + q * a.win_bytes;
                if (wave * 32 >= M)
                    continue;
                F fa[2][MG], fb[2][NT];
                auto read = [&](int t, int h) {
#pragma unroll
                    for (int m = 0; m < MG; ++m)
                        fa[h][m] = *reinterpret_cast<const F *>(
                            win + (a.todd[k0 + t] ? bo[m] : be[m]) + a.toff[k0 + t] + 32 * h);
#pragma unroll
                    for (int j = 0; j < NT; ++j)
                        fb[h][j] = *reinterpret_cast<const F *>(wq + (h ? wb1 : wb0) + t * WT +
                                                                j * 32 * 64);
                };
                auto mul = [&](int h) {
#pragma unroll
                    for (int j = 0; j < NT; ++j)
#pragma unroll
                        for (int m = 0; m < MG; ++m) {
                            if constexpr (F32) {
#pragma unroll
                                for (int e = 0; e < 4; ++e)
                                    acc[m][j] = __builtin_amdgcn_mfma_f32_32x32x2f32(
                                        fb[h][j][e], fa[h][m][e], acc[m][j], 0, 0, 0);
                            } else {
                                acc[m][j] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(
                                    fb[h][j], fa[h][m], acc[m][j], 0, 0, 0);
                            }
                        }
                };
                if (nt > 0)
                    read(0, 0);
                for (int t = 0; t < nt; ++t) {
                    read(t, 1);
                    __builtin_amdgcn_sched_barrier(0);
                    mul(0);
                    __builtin_amdgcn_sched_barrier(0);
                    if (t + 1 < nt)
                        read(t + 1, 0);
                    __builtin_amdgcn_sched_barrier(0);
                    mul(1);
                    __builtin_amdgcn_sched_barrier(0);
                }
            }
            // row r of D: channel 8 (r / 4) + 4 kh + r % 4; column: pixel
            const int nd = min(NB, a.Cd - d0);
            E *xb = dx + (static_cast<size_t>(n) * a.Cd + d0) * HWd;
#pragma unroll
            for (int m = 0; m < MG; ++m) {
                if (at[m] < 0)
                    continue;
#pragma unroll
                for (int j = 0; j < NT; ++j)
#pragma unroll
                    for (int r = 0; r < 16; ++r) {
                        const int d = j * 32 + 8 * (r >> 2) + 4 * kh + (r & 3);
                        if (d < nd)
                            xb[d * HWd + at[m]] = from_f<E>(acc[m][j][r]);
                    }
            }
        }
    }
}

// ------------------------------------------------------------------- host

constexpr size_t kAnyLds = 160 * 1024;

struct AnyPlan {
    AnyArgs a;
    int NT, MG, U, HS, grid;
    size_t lds;
    double cost;
};

// Tile of TR rows at NT x MG (of plan_any's `pl`, which holds the rest); false
// if it does not fit.  The cost counts, in clocks of a compute unit, the
// rounds of tiles times products (or the LDS reads that feed them, about 6.5
// clocks per 16-byte wave read), staging and results.
bool plan_tile(const ConvShape &sh, Dtype d, int cus, AnyPlan &pl)
{
    const int es = d == F32 ? 4 : 2, PX = 16 / es;
    const int K = sh.k, T = sh.T, NT = pl.NT, MG = pl.MG;
    AnyArgs &a = pl.a;
    const int NB = 32 * NT, WT = NB * 64 + 16;
    const int maxM = 32 * kAWaves * MG;
    if (a.Wd > maxM)
        return false;
    a.nblk = (a.Cd + NB - 1) / NB;
    const int per = (a.Ws + 2 * K + a.s - 1) / a.s; // slots per class of columns
    const int Q = a.Z * a.nch;
    const size_t wchunk = static_cast<size_t>(T) * WT;
    // three tiles of channels leave no registers for two items of two groups
    const int most = NT == 3 && MG == 2 ? 1 : 2;
    // the rows that the items and the LDS allow at best
    const int fixed = (a.Wd > 1 ? a.s / 2 : 0) + 2 * K + 1;
    int rows = static_cast<int>((kAnyLds - std::min(wchunk, kAnyLds)) /
                                (static_cast<size_t>(a.s) * per * kSB));
    if (a.Hs * a.Ws > most * kAThreads / 4 * PX)
        rows = std::min(rows, most * kAThreads / 4 * PX / a.Ws);
    if (rows < fixed)
        return false;
    int items = 0, M = 0;
    bool ok = false;
    for (int TR = std::min({maxM / a.Wd, a.Hd, (rows - fixed) / a.s + 1}); TR >= 1 && !ok; --TR) {
        a.tiles = (a.Hd + TR - 1) / TR;
        a.TR = (a.Hd + a.tiles - 1) / a.tiles;
        M = a.TR * a.Wd;
        a.OP = ((M + 31) & ~31) + 4;
        a.rows = a.s * (a.TR - 1) + fixed;
        items = 4 * ((std::min(a.rows, a.Hs) * a.Ws + PX - 1) / PX);
        pl.U = (items + kAThreads - 1) / kAThreads;
        if (pl.U > most)
            continue;
        const size_t outb = d == F32 ? 0 : static_cast<size_t>(32) * a.OP * 2;
        // weights resident, else streamed; window rows of a multiple of 8
        // slots per class of columns (odd tap columns at odd centres then
        // keep the banks' phase), else unpadded
        for (int pass = 0; pass < 4 && !ok; ++pass) {
            a.resident = pass < 2;
            a.WCs = (pass & 1) ? per : (per + 7) & ~7;
            a.RP = a.s * a.WCs;
            const size_t winb = static_cast<size_t>(a.rows) * a.RP * kSB;
            size_t wts = a.resident ? wchunk * Q : wchunk;
            wts = (wts + 255) & ~static_cast<size_t>(255);
            pl.lds = wts + std::max(winb, outb);
            a.win_off = static_cast<int>(wts);
            ok = pl.lds <= kAnyLds;
        }
    }
    if (!ok)
        return false;
    const long ntot = static_cast<long>(sh.N) * a.Dd * a.tiles;
    if (ntot > (1L << 30))
        return false;
    a.ntot = static_cast<int>(ntot);
    const int blocks = std::min(a.ntot, std::max(1, cus / a.nblk));
    pl.grid = blocks * a.nblk;
    const double mf = 2.0 * T * pl.HS * MG * NT * (d == F32 ? 256 : 32);
    const double rd = 8.0 * T * pl.HS * (MG + NT) * 6.5;
    const double stage = 800 + items * 1.5 + (a.resident ? 0 : T * NB * 4 * 2.0);
    const double waves = std::min(1.0, (M + 31) / 32 / static_cast<double>(kAWaves * MG));
    const double out = static_cast<double>(M) * NB * es / 12;
    const int rounds = (a.ntot + blocks - 1) / blocks;
    const int serial = (a.nblk * blocks + cus - 1) / cus;
    pl.cost = serial * (rounds * (Q * (std::max(mf * std::max(0.5, waves), rd) + stage) + out) +
                        (a.resident ? Q * T * NB * 4 * 2.0 : 0.0));
    return true;
}

bool plan_any(const ConvShape &sh, Dtype d, bool dgrad, AnyPlan &best)
{
    if (sh.k < 1 || sh.k > 3)
        return false;
    if (dgrad && (sh.s != 1 || sh.sz != 1))
        return false;
    // a run of rows has to hold one whole item
    if (sh.W < (d == F32 ? 4 : 8) || sh.Ho < 1)
        return false;
    const int es = d == F32 ? 4 : 2, CK = 64 / es;
    const int K = sh.k, T = sh.T;
    AnyPlan pl;
    AnyArgs &a = pl.a;
    a.Cs = dgrad ? sh.Co : sh.Ci;
    a.Cd = dgrad ? sh.Ci : sh.Co;
    a.Ds = dgrad ? sh.Do : sh.D;
    a.Hs = dgrad ? sh.Ho : sh.H;
    a.Ws = dgrad ? sh.Wo : sh.W;
    a.Dd = dgrad ? sh.D : sh.Do;
    a.Hd = dgrad ? sh.H : sh.Ho;
    a.Wd = dgrad ? sh.W : sh.Wo;
    a.s = sh.s;
    a.sz = sh.sz;
    a.kz = sh.kz;
    a.Z = sh.Z;
    a.J = sh.Z * T;
    a.sD = dgrad ? a.J : sh.Ci * a.J;
    a.sS = dgrad ? sh.Ci * a.J : a.J;
    a.reflect = dgrad;
    a.relu = 0;
    a.nch = (a.Cs + CK - 1) / CK;
    pl.HS = a.Cs <= CK / 2 ? 1 : 2;
    if (static_cast<long>(a.Ds) * a.Hs * a.Ws * CK * es >= kAnyMaxSpan)
        return false;
    const int cus = device_cus();
    bool found = false;
    // no more tiles of channels than there are channels, no second group of
    // pixels where a plane has none
    for (pl.NT = 1; pl.NT <= std::min(3, (a.Cd + 31) / 32); ++pl.NT)
        for (pl.MG = 1; pl.MG <= (a.Hd * a.Wd > 32 * kAWaves ? 2 : 1); ++pl.MG) {
            if (d == F32 && pl.NT == 3 && pl.MG == 2)
                continue; // does not fit the registers
            if (plan_tile(sh, d, cus, pl) && (!found || pl.cost < best.cost)) {
                best = pl;
                found = true;
            }
        }
    if (!found)
        return false;
    AnyArgs &b = best.a;
    b.fper = make_fastdiv(static_cast<uint32_t>(b.Dd) * b.tiles);
    b.ftiles = make_fastdiv(static_cast<uint32_t>(b.tiles));
    int t = 0;
    for (int dq = -K; dq <= K; ++dq)
        for (int i = 0; i < col_len(K, dq); ++i, ++t) {
            const int ds = col_ds_lo(K, dq) + i;
            const int c = K + dq;
            b.toff[t] = ((ds + floor_half(dq)) * b.RP + (c % b.s) * b.WCs + c / b.s) * kSB;
        }
    return true;
}

template <typename E, int K, int NT, int MG, int U, int HS, bool MIS>
hipError_t launch_h(const AnyPlan &pl, const void *x, const void *w, const void *b, void *y,
                  hipStream_t st)
{
    HEX_LAUNCH((conv_any_k<E, K, NT, MG, U, HS, MIS>), dim3(pl.grid), dim3(kAThreads), pl.lds, st,
               static_cast<const E *>(x), static_cast<const E *>(w), static_cast<const E *>(b),
               static_cast<E *>(y), pl.a);
    return hipGetLastError();
}

template <typename E, int K, int NT, int MG, int U>
hipError_t launch(const AnyPlan &pl, const void *x, const void *w, const void *b, void *y,
                  hipStream_t st)
{
    if constexpr (sizeof(E) == 2)
        if (pl.a.Ws & 1) // some runs start at an odd element
            return pl.HS == 1 ? launch_h<E, K, NT, MG, U, 1, true>(pl, x, w, b, y, st)
                              : launch_h<E, K, NT, MG, U, 2, true>(pl, x, w, b, y, st);
    return pl.HS == 1 ? launch_h<E, K, NT, MG, U, 1, false>(pl, x, w, b, y, st)
                      : launch_h<E, K, NT, MG, U, 2, false>(pl, x, w, b, y, st);
}

template <typename E, int K, int NT>
hipError_t dispatch_m(const AnyPlan &pl, const void *x, const void *w, const void *b, void *y,
                      hipStream_t st)
{
    if (pl.MG == 1 || (sizeof(E) == 4 && NT == 3))
        return pl.U == 1 ? launch<E, K, NT, 1, 1>(pl, x, w, b, y, st)
                         : launch<E, K, NT, 1, 2>(pl, x, w, b, y, st);
    if constexpr (sizeof(E) == 2 && NT == 3)
        return launch<E, K, NT, 2, 1>(pl, x, w, b, y, st);
    else if constexpr (NT < 3)
        return pl.U == 1 ? launch<E, K, NT, 2, 1>(pl, x, w, b, y, st)
                         : launch<E, K, NT, 2, 2>(pl, x, w, b, y, st);
    return hipErrorInvalidValue;
}

template <typename E, int K>
hipError_t dispatch_n(const AnyPlan &pl, const void *x, const void *w, const void *b, void *y,
                      hipStream_t st)
{
    switch (pl.NT) {
    case 1:
        return dispatch_m<E, K, 1>(pl, x, w, b, y, st);
    case 2:
        return dispatch_m<E, K, 2>(pl, x, w, b, y, st);
    default:
        return dispatch_m<E, K, 3>(pl, x, w, b, y, st);
    }
}

template <typename E>
hipError_t dispatch_k(const AnyPlan &pl, int k, const void *x, const void *w, const void *b,
                      void *y, hipStream_t st)
{
    switch (k) {
    case 1:
        return dispatch_n<E, 1>(pl, x, w, b, y, st);
    case 2:
        return dispatch_n<E, 2>(pl, x, w, b, y, st);
    default:
        return dispatch_n<E, 3>(pl, x, w, b, y, st);
    }
}

struct DgsPlan {
    DgsArgs a;
    int NT, MG, grid;
    size_t lds;
    double cost;
};

bool plan_dgs(const ConvShape &sh, Dtype d, DgsPlan &best)
{
    if (sh.k < 1 || sh.k > 3 || sh.s < 2 || sh.s * sh.s > kMaxCls || sh.Z != 1 || sh.D != 1 ||
        sh.Wo < (d == F32 ? 4 : 8) || sh.Ho < 1)
        return false;
    const int es = d == F32 ? 4 : 2, PX = 16 / es, CK = 64 / es;
    const int K = sh.k, T = sh.T, s = sh.s;
    DgsArgs a;
    a.Cs = sh.Co;
    a.Cd = sh.Ci;
    a.Hs = sh.Ho;
    a.Ws = sh.Wo;
    a.Hd = sh.H;
    a.Wd = sh.W;
    a.s = s;
    a.sD = T;
    a.sS = sh.Ci * T;
    a.nch = (a.Cs + CK - 1) / CK;
    a.Qn = (sh.W + s - 1) / s;
    if (static_cast<long>(sh.Ho) * sh.Wo * CK * es >= kAnyMaxSpan ||
        static_cast<long>(sh.H) * sh.W >= (1L << 30))
        return false;
    // taps by class, with their offsets on the output lattice
    int oq[kMaxTaps], os[kMaxTaps], cls[kMaxTaps], count[kMaxCls + 1] = {};
    int rlo = 0, rhi = 0, clo = 0, chi = 0, most = 0, n = 0;
    for (int dq = -K; dq <= K; ++dq)
        for (int i = 0; i < col_len(K, dq); ++i, ++n) {
            const int ds = col_ds_lo(K, dq) + i;
            const int ra = ((dq % s) + s) % s, rb = ((ds % s) + s) % s;
            cls[n] = ra * s + rb;
            oq[n] = (ra - dq) / s;
            os[n] = (rb - ds) / s;
            most = std::max(most, ++count[cls[n]]);
            for (int par = 0; par < 2; ++par) {
                const int row = tap_drow(oq[n], os[n], par);
                rlo = std::min(rlo, row);
                rhi = std::max(rhi, row);
            }
            clo = std::min(clo, oq[n]);
            chi = std::max(chi, oq[n]);
        }
    a.rlo = rlo;
    a.coff = -clo;
    // columns of the window: cells reach column Qn - 1, taps chi beyond
    const int cols = a.coff + std::max(a.Ws, a.Qn + chi);
    a.RP = (cols + 7) & ~7;
    const int cus = device_cus();
    const int all = (sh.H + s - 1) / s; // rows of each class in a plane
    const int fixed = 1 + rhi - rlo;    // window rows beside the tile's
    bool found = false;
    for (int NT = 1; NT <= std::min(2, (a.Cd + 31) / 32); ++NT)
        for (int MG = 1; MG <= (all * a.Qn > 32 * kAWaves ? 2 : 1); ++MG)
            for (int resident = 1; resident >= 0; --resident) {
                const int NB = 32 * NT, WT = NB * 64 + 16;
                const int maxM = 32 * kAWaves * MG;
                if (a.Qn > maxM)
                    continue;
                a.resident = resident;
                a.nblk = (a.Cd + NB - 1) / NB;
                const size_t wts = (static_cast<size_t>(resident ? T * a.nch : most) * WT + 255) &
                                   ~static_cast<size_t>(255);
                if (wts >= kAnyLds - 256)
                    continue;
                // the rows that the LDS and two items per thread allow
                int rows = static_cast<int>((kAnyLds - 256 - wts) /
                                            (static_cast<size_t>(a.RP) * kSB * a.nch));
                if (a.Hs * a.Ws > kAThreads / 2 * PX)
                    rows = std::min(rows, kAThreads / 2 * PX / a.Ws);
                const int TR = std::min({maxM / a.Qn, all, rows - fixed});
                if (TR < 1)
                    continue;
                a.tiles = (all + TR - 1) / TR;
                a.TR = (all + a.tiles - 1) / a.tiles;
                a.rows = a.TR + fixed;
                a.win_bytes = a.rows * a.RP * kSB;
                const size_t lds = wts + static_cast<size_t>(a.win_bytes) * a.nch;
                const long ntot = static_cast<long>(sh.N) * a.tiles;
                if (ntot > (1L << 30))
                    continue;
                a.win_off = static_cast<int>(wts);
                a.ntot = static_cast<int>(ntot);
                const int blocks = std::min(a.ntot, std::max(1, cus / a.nblk));
                const int rounds = (a.ntot + blocks - 1) / blocks;
                const double M = static_cast<double>(a.TR) * a.Qn;
                const double mf = a.nch * 2.0 * T * 2 * MG * NT * (d == F32 ? 256 : 32);
                const double st = a.nch * 1600.0 + s * s * M * NB / 64 * 12 +
                                  (resident ? 0 : a.nch * (s * s * 2500.0 + T * NB * 8.0));
                const double v =
                    rounds * (mf + st) + (resident ? a.nch * T * NB * 8.0 : 0.0);
                if (!found || v < best.cost) {
                    best.a = a;
                    best.NT = NT;
                    best.MG = MG;
                    best.grid = blocks * a.nblk;
                    best.lds = lds;
                    best.cost = v;
                    found = true;
                }
            }
    if (!found)
        return false;
    DgsArgs &b = best.a;
    b.ftiles = make_fastdiv(static_cast<uint32_t>(b.tiles));
    b.cstart[0] = 0;
    for (int cl = 0; cl < s * s; ++cl)
        b.cstart[cl + 1] = b.cstart[cl] + count[cl];
    int at[kMaxCls];
    std::copy(b.cstart, b.cstart + s * s, at);
    for (int t = 0; t < T; ++t) {
        const int i = at[cls[t]]++;
        b.tap[i] = t;
        b.todd[i] = oq[t] & 1;
        b.toff[i] = ((os[t] + floor_half(oq[t])) * b.RP + oq[t]) * kSB;
    }
    return true;
}

// Estimated time: products, staging, results, weights (once, or per class) and
// the classes' turns.
double dgs_us(const DgsPlan &pl, const ConvShape &sh, Dtype d)
{
    static const double c[2][8] = {{3.6, 1.11, 1.23, 1.19, -0.56, 0.29, 0.59, 0.45},
                                   {2.0, 2.61, 4.65, 0.39, 3.03, 0.48, 4.21, 0.77}};
    const DgsArgs &a = pl.a;
    const double blocks = pl.grid / a.nblk, classes = a.s * a.s;
    const double rounds = std::ceil(a.ntot / blocks) * std::max(1.0, pl.grid / 256.0);
    const double wts = a.nch * sh.T * 32.0 * pl.NT / 1000;
    const double *k = c[d];
    return k[0] + (a.resident ? k[4] * wts : 0) +
           rounds * (k[1] * a.nch * sh.T * pl.MG * pl.NT * (d == F32 ? 1024 : 128) / 2400 +
                     k[2] * a.nch + k[3] * classes * a.TR * a.Qn * 32 * pl.NT / 1e4 +
                     (a.resident ? 0 : k[5] * a.nch * classes + k[6] * wts) + k[7] * classes);
}

template <typename E, int K, int NT, int MG>
hipError_t launch_dgs(const DgsPlan &pl, const void *dy, const void *w, void *dx, hipStream_t st)
{
    const E *g = static_cast<const E *>(dy), *we = static_cast<const E *>(w);
    if constexpr (sizeof(E) == 2)
        if (pl.a.Ws & 1) {
            HEX_LAUNCH((conv_any_dgs_k<E, K, NT, MG, true>), dim3(pl.grid), dim3(kAThreads),
                       pl.lds, st, g, we, static_cast<E *>(dx), pl.a);
            return hipGetLastError();
        }
    HEX_LAUNCH((conv_any_dgs_k<E, K, NT, MG, false>), dim3(pl.grid), dim3(kAThreads), pl.lds, st, g,
               we, static_cast<E *>(dx), pl.a);
    return hipGetLastError();
}

template <typename E, int K>
hipError_t dispatch_dgs(const DgsPlan &pl, const void *dy, const void *w, void *dx, hipStream_t st)
{
    if (pl.NT == 1)
        return pl.MG == 1 ? launch_dgs<E, K, 1, 1>(pl, dy, w, dx, st)
                          : launch_dgs<E, K, 1, 2>(pl, dy, w, dx, st);
    return pl.MG == 1 ? launch_dgs<E, K, 2, 1>(pl, dy, w, dx, st)
                      : launch_dgs<E, K, 2, 2>(pl, dy, w, dx, st);
}

} // namespace

Tried conv_any(const void *in, const void *w, const void *bias, void *out, const ConvShape &sh,
               Dtype d, bool dgrad, bool relu, hipStream_t st, double other_us, hipError_t &e)
{
    // One source channel in bfloat16, two in float32 leave nearly all of a
    // chunk empty (64 images of 41 x 43, k = 1, us here against generic: bf16
    // 1 -> 16 9.9 / 10.8; 8 volumes of 12 planes of 37 x 41, kz = 1: bf16
    // 1 -> 16 25 / 20).
    if ((dgrad ? sh.Co : sh.Ci) < (d == F32 ? 3 : 2))
        return Tried::No;
    if (dgrad && sh.s > 1) {
        DgsPlan dp;
        if (!plan_dgs(sh, d, dp))
            return Tried::No;
        if (dgs_us(dp, sh, d) > kClearly * other_us)
            return Tried::Slower;
        auto go = [&](auto *p) {
            using E = std::remove_pointer_t<decltype(p)>;
            return sh.k == 1   ? dispatch_dgs<E, 1>(dp, in, w, out, st)
                   : sh.k == 2 ? dispatch_dgs<E, 2>(dp, in, w, out, st)
                               : dispatch_dgs<E, 3>(dp, in, w, out, st);
        };
        e = d == F32 ? go(static_cast<float *>(nullptr)) : go(static_cast<bf16raw *>(nullptr));
        return Tried::Ran;
    }
    AnyPlan pl;
    if (!plan_any(sh, d, dgrad, pl))
        return Tried::No;
    if ((d == F32 ? 4.8 + 1.19 * pl.cost / 2400 : 5.8 + 1.32 * pl.cost / 2400) > other_us)
        return Tried::Slower;
    pl.a.relu = relu;
    e = d == F32 ? dispatch_k<float>(pl, sh.k, in, w, bias, out, st)
                 : dispatch_k<bf16raw>(pl, sh.k, in, w, bias, out, st);
    return Tried::Ran;
}

} // namespace hexk
