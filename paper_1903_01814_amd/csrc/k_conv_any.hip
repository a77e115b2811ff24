// k_conv_any.hip -- convolution on the matrix cores for planes of any size
// and any channel count: forward at any stride and, at stride 1, the data
// gradient (the same sum with the reflected kernel), in bfloat16 and in
// float32, two- and three-dimensional.  The tuned bfloat16 kernels
// (k_mfma_bf16.hip, k_mfma_gen.hip) need rows of whole 16-byte vectors and
// whole 32-channel blocks; this one takes what they do not: odd rows, other
// channel counts, float32 layers with more than a few channels, 3-D layers.
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

#include "chanlast.h"
#include "kernels.h"

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
    for (int i = threadIdx.x; i < T * NB * 4; i += kAThreads) {
        const int t = i % T, r = i / T;
        const int o = r & 3, n = r >> 2;
        const int c = c0 + o * PX, d = d0 + n;
        const int j = a.reflect ? a.J - 1 - (z * T + t) : z * T + t;
        E v[PX];
        const bool dok = d < a.Cd;
        const E *p = w + static_cast<size_t>(min(d, a.Cd - 1)) * a.sD + j;
#pragma unroll
        for (int e = 0; e < PX; ++e) {
            const E q = p[static_cast<size_t>(min(c + e, a.Cs - 1)) * a.sS];
            v[e] = (dok && c + e < a.Cs) ? q : E(0);
        }
        uint4 u;
        __builtin_memcpy(&u, v, 16);
        *reinterpret_cast<uint4 *>(wl + t * WT + n * 64 + ((o ^ ((n >> 1) & 3)) << 4)) = u;
    }
}

// HS: 32-byte halves of a chunk that are contracted (1 where every source
// channel fits the first)
template <typename E, int K, int NT, int MG, int U, int HS>
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

    // Position: tile, chunk.  Chunks whose source plane lies outside are
    // passed over; the centre plane never does.
    struct Pos {
        int tb, q;         // tile, chunk
        int n, l, i0;      // image, destination plane, first row
        int zs;            // source plane of the chunk
        int first;         // first chunk of its tile
    };
    auto place = [&](Pos &p) {
        const int per = a.Dd * a.tiles;
        p.n = p.tb / per;
        const int r = p.tb - p.n * per;
        p.l = r / a.tiles;
        p.i0 = (r - p.l * a.tiles) * a.TR;
    };
    auto settle = [&](Pos &p) { // first chunk from p.q on with its plane inside
        for (; p.q < Q; ++p.q) {
            p.zs = a.sz * p.l + p.q / a.nch - a.kz;
            if (p.zs >= 0 && p.zs < a.Ds)
                return true;
        }
        return false;
    };
    AnyItem<E> it[U];
    auto span = [&](const Pos &p, int &lo, int &run) { // existing rows of the window
        const int r_lo = a.s * p.i0 - K;
        lo = max(0, -r_lo);
        const int hi = min(a.rows, a.Hs - r_lo);
        run = (hi - lo) * a.Ws;
        return hi;
    };
    auto load = [&](const Pos &p) {
        int lo, run;
        span(p, lo, run);
        const int c0 = (p.q % a.nch) * CK;
        const E *src = x + (static_cast<size_t>(p.n) * a.Cs + c0) * cs_src +
                       static_cast<size_t>(p.zs) * HWs +
                       static_cast<size_t>(a.s * p.i0 - K + lo) * a.Ws;
#pragma unroll
        for (int u = 0; u < U; ++u) {
            const int i = threadIdx.x + u * kAThreads;
            const int f = min((i >> 2) * PX, run - PX);
            it[u].load(src, cs_src, (i & 3) * PX, a.Cs - c0, f);
        }
    };
    auto commit = [&](const Pos &p) {
        int lo, run;
        const int hi = span(p, lo, run);
#pragma unroll
        for (int u = 0; u < U; ++u) {
            const int i = threadIdx.x + u * kAThreads;
            if ((i >> 2) * PX < run)
                it[u].template commit<kSB>(win, wg, lo, min((i >> 2) * PX, run - PX), i & 3);
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
        ++nxt.q;
        bool more = true, last = false;
        if (!settle(nxt)) {
            last = true;
            nxt.tb += tstep;
            nxt.q = 0;
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
            stage_weights<E, T, NB>(smem, w, a, d0, (cur.q % a.nch) * CK, cur.q / a.nch);
        __syncthreads();
        if (more)
            load(nxt);

        const int rows = min(a.TR, a.Hd - cur.i0);
        const int M = rows * a.Wd;
        if (wave * 32 < M) {
            const unsigned char *wq = smem + (a.resident ? cur.q * T * WT : 0);
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
                if (i + 1 < HS * T)
                    read(i + 1, fa[(i + 1) & 1], fb[(i + 1) & 1]);
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

// ------------------------------------------------------------------- host

constexpr size_t kAnyLds = 160 * 1024;

struct AnyPlan {
    AnyArgs a;
    int NT, MG, U, HS, grid;
    size_t lds;
    double cost;
};

// Tile of TR rows at NT x MG; false if it does not fit.  The cost counts, in
// clocks of a compute unit, the rounds of tiles times products (or the LDS
// reads that feed them, about 6.5 clocks per 16-byte wave read), staging and
// results.
bool plan_tile(const ConvShape &sh, Dtype d, bool dgrad, int NT, int MG, AnyPlan &pl)
{
    const int es = d == F32 ? 4 : 2, PX = 16 / es, CK = 64 / es;
    const int K = sh.k, T = sh.T;
    AnyArgs &a = pl.a;
    a = AnyArgs{};
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
    if (static_cast<long>(a.Ds) * a.Hs * a.Ws * CK * es >= kAnyMaxSpan)
        return false;
    const int NB = 32 * NT, WT = NB * 64 + 16;
    const int maxM = 32 * kAWaves * MG;
    if (a.Wd > maxM)
        return false;
    a.TR = std::min(maxM / a.Wd, a.Hd);
    a.tiles = (a.Hd + a.TR - 1) / a.TR;
    a.TR = (a.Hd + a.tiles - 1) / a.tiles;
    a.nch = (a.Cs + CK - 1) / CK;
    a.nblk = (a.Cd + NB - 1) / NB;
    const long ntot = static_cast<long>(sh.N) * a.Dd * a.tiles;
    if (ntot > (1L << 30))
        return false;
    a.ntot = static_cast<int>(ntot);
    const int M = a.TR * a.Wd;
    a.OP = ((M + 31) & ~31) + 4;
    a.rows = a.s * (a.TR - 1) + (a.Wd > 1 ? a.s / 2 : 0) + 2 * K + 1;
    const int cols = a.Ws + 2 * K; // one class of columns: rows of a multiple of 8 slots where it fits
    const int items = 4 * ((std::min(a.rows, a.Hs) * a.Ws + PX - 1) / PX);
    pl.U = (items + kAThreads - 1) / kAThreads;
    if (pl.U > 2)
        return false;
    const int Q = a.Z * a.nch;
    const size_t wchunk = static_cast<size_t>(T) * WT;
    const size_t outb = d == F32 ? 0 : static_cast<size_t>(32) * a.OP * 2;
    bool ok = false;
    for (int pass = 0; pass < 4 && !ok; ++pass) { // resident padded, unpadded, then streamed
        a.resident = pass < 2;
        const int per = (cols + a.s - 1) / a.s;
        a.WCs = (pass & 1) ? per : (per + 7) & ~7;
        a.RP = a.s * a.WCs;
        // the padded columns of the last slots are reached by no tap, only staged as zeros
        const size_t winb = (static_cast<size_t>(a.rows) * a.RP * kSB + 15) & ~static_cast<size_t>(15);
        size_t wts = a.resident ? wchunk * Q : wchunk;
        wts = (wts + 255) & ~static_cast<size_t>(255);
        pl.lds = wts + std::max(winb, outb);
        a.win_off = static_cast<int>(wts);
        ok = pl.lds <= kAnyLds;
    }
    if (!ok)
        return false;
    int t = 0;
    for (int dq = -K; dq <= K; ++dq)
        for (int i = 0; i < col_len(K, dq); ++i, ++t) {
            const int ds = col_ds_lo(K, dq) + i;
            const int c = K + dq;
            a.toff[t] = ((ds + floor_half(dq)) * a.RP + (c % a.s) * a.WCs + c / a.s) * kSB;
        }
    pl.NT = NT;
    pl.MG = MG;
    const int cus = device_cus();
    const int per = std::max(1, cus / a.nblk);
    const int blocks = std::min(a.ntot, per);
    pl.grid = blocks * a.nblk;
    pl.HS = a.Cs <= CK / 2 ? 1 : 2;
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
    if (sh.W < 8 || sh.Wo < 8 || sh.Ho < 1)
        return false;
    bool found = false;
    for (int NT = 1; NT <= 3; ++NT)
        for (int MG = 1; MG <= 2; ++MG) {
            if (d == F32 && NT == 3 && MG == 2)
                continue; // does not fit the registers
            AnyPlan pl;
            if (!plan_tile(sh, d, dgrad, NT, MG, pl))
                continue;
            if (!found || pl.cost < best.cost) {
                best = pl;
                found = true;
            }
        }
    return found;
}

template <typename E, int K, int NT, int MG, int U, int HS>
hipError_t launch_h(const AnyPlan &pl, const void *x, const void *w, const void *b, void *y,
                  hipStream_t st)
{
    HEX_LAUNCH((conv_any_k<E, K, NT, MG, U, HS>), dim3(pl.grid), dim3(kAThreads), pl.lds, st,
               static_cast<const E *>(x), static_cast<const E *>(w), static_cast<const E *>(b),
               static_cast<E *>(y), pl.a);
    return hipGetLastError();
}

template <typename E, int K, int NT, int MG, int U>
hipError_t launch(const AnyPlan &pl, const void *x, const void *w, const void *b, void *y,
                  hipStream_t st)
{
    return pl.HS == 1 ? launch_h<E, K, NT, MG, U, 1>(pl, x, w, b, y, st)
                      : launch_h<E, K, NT, MG, U, 2>(pl, x, w, b, y, st);
}

template <typename E, int K, int NT>
hipError_t dispatch_m(const AnyPlan &pl, const void *x, const void *w, const void *b, void *y,
                      hipStream_t st)
{
    if (pl.MG == 1 || (sizeof(E) == 4 && NT == 3))
        return pl.U == 1 ? launch<E, K, NT, 1, 1>(pl, x, w, b, y, st)
                         : launch<E, K, NT, 1, 2>(pl, x, w, b, y, st);
    if constexpr (sizeof(E) == 2 || NT < 3)
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

} // namespace

bool conv_any_ok(const ConvShape &sh, Dtype d, bool dgrad)
{
    // Few source channels leave most of a chunk empty; then the generic
    // kernel is the faster one.  64 images of 41 x 43, k = 1, us here against
    // generic: fp32 3 -> 16 channels 13.4 / 18.0, 2 -> 16 18.5 / 15.4; bf16
    // 3 -> 16 8.6 / 17.7, 1 -> 16 9.9 / 10.8; 8 volumes of 12 planes of
    // 37 x 41, kz = 1: fp32 4 -> 16 38 / 54, 3 -> 16 38 / 43; bf16 2 -> 16
    // 25 / 32, 1 -> 16 25 / 20.
    const int Cs = dgrad ? sh.Co : sh.Ci;
    if (Cs < (d == F32 ? 3 : 2))
        return false;
    AnyPlan pl;
    return plan_any(sh, d, dgrad, pl);
}

hipError_t conv_any(const void *in, const void *w, const void *bias, void *out,
                    const ConvShape &sh, Dtype d, bool dgrad, bool relu, hipStream_t st)
{
    AnyPlan pl;
    if (!plan_any(sh, d, dgrad, pl))
        return hipErrorInvalidValue;
    pl.a.relu = relu;
    return d == F32 ? dispatch_k<float>(pl, sh.k, in, w, bias, out, st)
                    : dispatch_k<bf16raw>(pl, sh.k, in, w, bias, out, st);
}

} // namespace hexk
