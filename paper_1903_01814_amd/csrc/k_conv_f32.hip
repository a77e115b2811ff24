// k_conv_f32.hip -- float32 forward convolution on the matrix cores for planes
// of any size, any channel count and any stride, two- and three-dimensional,
// k = 1 to 3.
//
// The sums are those of the generic kernel bit for bit: v_mfma_f32_32x32x2f32
// adds its two products to the accumulator one after the other like two fused
// multiply-adds, so an accumulator that starts from the bias and takes the
// products in the weight's own order (channel, window plane, tap) goes
// through the same roundings as a loop over them.  Results that a ReLU or a
// maximum decides on (a pre-activation within an ulp of 0) therefore do not
// depend on which kernel ran.
//
// Implicit GEMM: the 32 columns of a product are 32 output pixels, the rows 32
// output channels, the contraction the products above in pairs, lane half h
// taking the pair's element h.  A block (8 waves) computes a tile of whole
// output rows (up to 256 MG pixels) times NB = 32 NT channels.  The source
// planes are staged as they are, G planes (channel, window plane) at a time,
// rows of RP floats with the border as zeros: lanes read consecutive pixels,
// so plain rows do not conflict, and a tap is a fixed offset (one row more
// for odd tap columns at odd centre columns).  T is odd, so the pattern of
// pairs repeats every two planes: a lane keeps the T addresses of its element
// of each pair and moves them on by two planes.  Weights sit in LDS as
// [product][channel] (pitch 33 mod 64 floats: the two halves read different
// banks), for the block's life where all fit, else per stage.  The next
// stage's rows are loaded into registers during the products.
//
// Bound by the turns of staging and products, which a barrier parts: at 32 ->
// 64 channels, 40 x 40, N = 128, k = 1 the matrix cores are busy 0.37 of the
// time (64 clocks per 32x32x2 product and SIMD; a pair costs MG + NT four-byte
// reads for MG NT products), LDS 0.15 and the vector units 0.07.  32 -> 64 channels,
// 40 x 40, N = 128, k = 1: 356 us on the generic kernel, 101 here, 39 at the
// matrix rate; 48 -> 96, 46 x 45, N = 15, k = 2: 370, 98, 36.  (Items' places
// worked out once instead of per stage: 101 -> 115 us, the registers spill.)
#include <algorithm>
#include <cmath>

#include "chanlast.h"
#include "kernels.h"
#include "shear.h" // FastDiv

namespace hexk {
namespace {

using namespace hexgeom;

typedef float floatx16 __attribute__((ext_vector_type(16)));

constexpr int kFThreads = 512;
constexpr int kFWaves = kFThreads / 64;
constexpr int kMaxTaps = 37;

struct F32Args {
    int Cs, Cd;
    int Ds, Hs, Ws, Dd, Hd, Wd;
    int s, sz, kz, Z;
    int J;                 // weights per channel pair (Z * taps)
    int TR, tiles, ntot;
    int rows, RP, WCs, PL; // window rows, floats per row, per class of columns, per plane
    int P, G, nst;         // planes (channel, window plane), per stage (even), stages
    int nblk, resident, relu;
    int win_off, bias_off; // bytes; weights at 0
    FastDiv fper, ftiles, fw, fz;
    int toff[kMaxTaps]; // floats
};

template <int K, int NT, int MG, int U>
__global__ __launch_bounds__(kFThreads) void conv_f32_k(const float *x, const float *__restrict__ w,
                                                        const float *__restrict__ bias,
                                                        float *__restrict__ y, F32Args a)
{
    constexpr int T = num_taps(K);
    constexpr TapTable<K> tab{};
    constexpr int NB = 32 * NT;
    constexpr int WP = NT == 1 ? 33 : 97;
    extern __shared__ __align__(16) unsigned char smem[];
    float *wl = reinterpret_cast<float *>(smem);
    float *win = reinterpret_cast<float *>(smem + a.win_off);
    float *bl = reinterpret_cast<float *>(smem + a.bias_off);

    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const int n32 = lane & 31, kh = lane >> 5;
    const int db = blockIdx.x % a.nblk, tstep = gridDim.x / a.nblk;
    const int d0 = db * NB;
    const size_t HWs = static_cast<size_t>(a.Hs) * a.Ws, HWd = static_cast<size_t>(a.Hd) * a.Wd;
    const size_t cs_src = HWs * a.Ds, cs_dst = HWd * a.Dd;

    // weights of the planes p0 .. p0 + np - 1, products in order
    auto stage_w = [&](float *dst, int p0, int np) {
        const int nk = np * T;
        constexpr int UW = 8;
        for (int i0 = threadIdx.x; i0 < nk * NB; i0 += UW * kFThreads) {
            float v[UW];
            int at[UW];
#pragma unroll
            for (int u = 0; u < UW; ++u) {
                const int i = min(i0 + u * kFThreads, nk * NB - 1);
                const int n = i / nk, kk = i - n * nk;
                const int pl = kk / T, t = kk - pl * T;
                const int c = static_cast<int>(fdiv(static_cast<uint32_t>(p0 + pl), a.fz));
                const int zt = (p0 + pl - c * a.Z) * T + t;
                const int d = d0 + n;
                v[u] = w[(static_cast<size_t>(min(d, a.Cd - 1)) * a.Cs + c) * a.J + zt];
                at[u] = d < a.Cd ? kk * WP + n : ~(kk * WP + n);
            }
            __builtin_amdgcn_sched_barrier(0);
#pragma unroll
            for (int u = 0; u < UW; ++u)
                if (i0 + u * kFThreads < nk * NB)
                    dst[at[u] < 0 ? ~at[u] : at[u]] = at[u] < 0 ? 0.f : v[u];
        }
    };
    if (a.resident)
        stage_w(wl, 0, a.P);
    for (int i = threadIdx.x; i < NB; i += kFThreads)
        bl[i] = (bias != nullptr && d0 + i < a.Cd) ? bias[d0 + i] : 0.f;
    // the window's border columns, once; rows outside are written per stage
    for (int i = threadIdx.x; i < a.G * a.PL; i += kFThreads)
        win[i] = 0.f;

    // this lane's address (floats) of its element of each pair, per group
    int ad[T][MG];
#pragma unroll
    for (int m = 0; m < MG; ++m) {
        const int p = min((wave + kFWaves * m) * 32 + n32, a.TR * a.Wd - 1);
        const int i = p / a.Wd, j = p - i * a.Wd;
        const int be = (a.s * i + (j & 1) * (a.s >> 1) + K) * a.RP + j;
        const int odd = ((a.s * j) & 1) ? a.RP : 0;
#pragma unroll
        for (int q = 0; q < T; ++q) {
            // products 2q and 2q + 1 of two planes
            const int t0 = (2 * q) % T, t1 = (2 * q + 1) % T;
            const int o0 = a.toff[t0] + (2 * q >= T ? a.PL : 0) + ((tab.dq[t0] & 1) ? odd : 0);
            const int o1 = a.toff[t1] + (2 * q + 1 >= T ? a.PL : 0) + ((tab.dq[t1] & 1) ? odd : 0);
            ad[q][m] = be + (kh ? o1 : o0);
        }
    }

    struct Pos {
        int tb, st, n, l, i0;
    };
    auto place = [&](Pos &p) {
        const uint32_t per = static_cast<uint32_t>(a.Dd) * a.tiles;
        p.n = static_cast<int>(fdiv(static_cast<uint32_t>(p.tb), a.fper));
        const uint32_t r = p.tb - p.n * per;
        p.l = static_cast<int>(fdiv(r, a.ftiles));
        p.i0 = (r - p.l * a.tiles) * a.TR;
    };
    // item i of a stage: plane i / ipp, flat pixels 4 (i % ipp) .. of the run
    // of existing rows (the last moved back to end with it)
    float4 v[U];
    int pg[U], pf[U]; // plane within the stage (-1: none, or zeros: ~plane), flat pixel
    auto load = [&](const Pos &p) {
        const int r_lo = a.s * p.i0 - K;
        const int lo = max(0, -r_lo), hi = min(a.rows, a.Hs - r_lo);
        const int run = (hi - lo) * a.Ws, ipp = (run + 3) >> 2;
        const int np = min(a.G, a.P - p.st * a.G);
        const float rcp = 1.0f / static_cast<float>(ipp);
        const float *img = x + static_cast<size_t>(p.n) * a.Cs * cs_src +
                           static_cast<size_t>(r_lo + lo) * a.Ws;
#pragma unroll
        for (int u = 0; u < U; ++u) {
            const int i = threadIdx.x + u * kFThreads;
            // i / ipp (i < 2^13: the rounded quotient is off by at most one)
            int g = static_cast<int>(static_cast<float>(i) * rcp);
            int f = i - g * ipp;
            if (f < 0) {
                --g;
                f += ipp;
            } else if (f >= ipp) {
                ++g;
                f -= ipp;
            }
            const int gg = min(g, np - 1);
            const int pi = p.st * a.G + gg;
            const int c = static_cast<int>(fdiv(static_cast<uint32_t>(pi), a.fz));
            const int z = a.sz * p.l + (pi - c * a.Z) - a.kz;
            const bool in = z >= 0 && z < a.Ds;
            pf[u] = min(4 * f, run - 4);
            pg[u] = g < np ? (in ? g : ~g - 1) : -1;
            __builtin_memcpy(&v[u], img + c * cs_src + (in ? z : 0) * HWs + pf[u], 16);
        }
    };
    auto commit = [&](const Pos &p) {
        const int r_lo = a.s * p.i0 - K;
        const int lo = max(0, -r_lo), hi = min(a.rows, a.Hs - r_lo);
#pragma unroll
        for (int u = 0; u < U; ++u) {
            if (pg[u] == -1)
                continue;
            const int g = pg[u] >= 0 ? pg[u] : ~(pg[u] + 1);
            const bool in = pg[u] >= 0;
            const float e[4] = {in ? v[u].x : 0.f, in ? v[u].y : 0.f, in ? v[u].z : 0.f,
                                in ? v[u].w : 0.f};
            const int row = static_cast<int>(fdiv(static_cast<uint32_t>(pf[u]), a.fw));
            int col = pf[u] - row * a.Ws;
            float *d = win + g * a.PL + (lo + row) * a.RP;
            if (a.s == 1) {
                d += col + K;
#pragma unroll
                for (int q = 0; q < 4; ++q) {
                    *d++ = e[q];
                    if (++col == a.Ws) {
                        col = 0;
                        d += a.RP - a.Ws;
                    }
                }
            } else {
#pragma unroll
                for (int q = 0; q < 4; ++q) {
                    const int cq = (col + K) / a.s;
                    d[(col + K - cq * a.s) * a.WCs + cq] = e[q];
                    if (++col == a.Ws) {
                        col = 0;
                        d += a.RP;
                    }
                }
            }
        }
        // rows outside the plane (whole rows, every plane of the stage)
        const int bad = lo + a.rows - hi;
        if (bad > 0) {
            const int n = bad * a.RP;
            for (int i = threadIdx.x; i < n * a.G; i += kFThreads) {
                const int g = i / n, r = i - g * n;
                win[g * a.PL + (r < lo * a.RP ? r : r - lo * a.RP + hi * a.RP)] = 0.f;
            }
        }
    };

    Pos cur{static_cast<int>(blockIdx.x) / a.nblk, 0, 0, 0, 0};
    if (cur.tb >= a.ntot)
        return;
    place(cur);
    load(cur);
    floatx16 acc[MG][NT];
    while (true) {
        Pos nxt = cur;
        bool more = true;
        const bool last = ++nxt.st == a.nst;
        if (last) {
            nxt.st = 0;
            nxt.tb += tstep;
            more = nxt.tb < a.ntot;
            if (more)
                place(nxt);
        }
        const int p0 = cur.st * a.G, np = min(a.G, a.P - p0);
        __syncthreads(); // the previous stage's readers are done
        commit(cur);
        if (!a.resident)
            stage_w(wl, p0, np);
        __syncthreads();
        if (cur.st == 0) {
#pragma unroll
            for (int j = 0; j < NT; ++j)
#pragma unroll
                for (int r = 0; r < 16; ++r) {
                    const float b = bl[j * 32 + 8 * (r >> 2) + 4 * kh + (r & 3)];
#pragma unroll
                    for (int m = 0; m < MG; ++m)
                        acc[m][j][r] = b;
                }
        }
        if (more)
            load(nxt);

        const int M = min(a.TR, a.Hd - cur.i0) * a.Wd;
        if (wave * 32 < M) {
            // B (pixels) and A (weights) of the pairs, one pair ahead
            const float *wq = wl + ((a.resident ? p0 * T : 0) + kh) * WP + n32;
            float fp[2][MG], fw[2][NT];
            int base = 0; // floats: two planes per round
            auto read = [&](int q, int b) {
#pragma unroll
                for (int m = 0; m < MG; ++m)
                    fp[b][m] = win[ad[q][m] + base];
#pragma unroll
                for (int j = 0; j < NT; ++j)
                    fw[b][j] = wq[2 * q * WP + 32 * j];
            };
            auto mul = [&](int b) {
#pragma unroll
                for (int j = 0; j < NT; ++j)
#pragma unroll
                    for (int m = 0; m < MG; ++m)
                        acc[m][j] = __builtin_amdgcn_mfma_f32_32x32x2f32(fw[b][j], fp[b][m],
                                                                         acc[m][j], 0, 0, 0);
            };
            for (int g = 0; g + 1 < np; g += 2) {
                read(0, 0);
#pragma unroll
                for (int q = 0; q < T; ++q) {
                    if (q + 1 < T)
                        read(q + 1, (q + 1) & 1);
                    __builtin_amdgcn_sched_barrier(0);
                    mul(q & 1);
                    __builtin_amdgcn_sched_barrier(0);
                }
                base += 2 * a.PL;
                wq += 2 * T * WP;
            }
            if (np & 1) { // one plane: T products, the last pair half empty
#pragma unroll
                for (int q = 0; q < (T + 1) / 2; ++q) {
                    if (2 * q + 1 < T) {
                        read(q, 0);
                    } else {
#pragma unroll
                        for (int m = 0; m < MG; ++m) {
                            const float e = win[kh ? 0 : ad[q][m] + base];
                            fp[0][m] = kh ? 0.f : e;
                        }
#pragma unroll
                        for (int j = 0; j < NT; ++j) {
                            const float e = wq[(kh ? 2 * q - 1 : 2 * q) * WP + 32 * j];
                            fw[0][j] = kh ? 0.f : e;
                        }
                    }
                    mul(0);
                }
            }
        }

        if (last) {
            float *yb = y + (static_cast<size_t>(cur.n) * a.Cd + d0) * cs_dst +
                        static_cast<size_t>(cur.l) * HWd + static_cast<size_t>(cur.i0) * a.Wd;
            const int nd = min(NB, a.Cd - d0);
            // row r of D: channel 8 (r / 4) + 4 kh + r % 4; column: pixel
#pragma unroll
            for (int m = 0; m < MG; ++m) {
                const int p = (wave + kFWaves * m) * 32 + n32;
                if (p >= M)
                    continue;
#pragma unroll
                for (int j = 0; j < NT; ++j)
#pragma unroll
                    for (int r = 0; r < 16; ++r) {
                        const int d = j * 32 + 8 * (r >> 2) + 4 * kh + (r & 3);
                        if (d < nd) {
                            const float o = acc[m][j][r];
                            yb[d * cs_dst + p] = a.relu ? fmaxf(o, 0.f) : o;
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

constexpr size_t kF32Lds = 160 * 1024;

struct F32Plan {
    F32Args a;
    int NT, MG, U, grid;
    size_t lds;
    double cost;
};

// Items per thread that fit the registers beside the sums (16 NT MG) and the
// pairs' addresses (T MG); 0: the combination does not.
constexpr int max_items(int K, int NT, int MG)
{
    if (NT == 1 && MG == 1)
        return 8;
    if (MG == 1 && NT == 2)
        return K < 3 ? 8 : 4;
    if (NT == 3)
        return MG == 2 || K == 3 ? 0 : K == 1 ? 4 : 2;
    if (NT == 1)
        return K < 3 ? 8 : 0;
    return K == 1 ? 4 : 0;
}

// The largest stage (and the tallest tile) that fits at NT x MG.  The cost
// counts, in clocks of a compute unit, rounds of tiles times products,
// staging and results.
// `pl` holds the rest.
bool plan_tile(const ConvShape &sh, int cus, F32Plan &pl)
{
    const int K = sh.k, T = sh.T, NT = pl.NT, MG = pl.MG;
    F32Args &a = pl.a;
    const int NB = 32 * NT, WP = NT == 1 ? 33 : 97;
    const int maxM = 32 * kFWaves * MG;
    const int most = max_items(K, NT, MG);
    if (a.Wd > maxM || most == 0)
        return false;
    a.nblk = (a.Cd + NB - 1) / NB;
    const int Pe = (a.P + 1) & ~1;
    // the rows of which a stage holds two planes at best
    const int fixed_rows = (a.Wd > 1 ? a.s / 2 : 0) + 2 * K + 1;
    int rows = static_cast<int>((kF32Lds - 256) / (8 * static_cast<size_t>(a.RP)));
    if (a.Hs * a.Ws > 2 * most * kFThreads)
        rows = std::min(rows, 2 * most * kFThreads / a.Ws);
    if (rows < fixed_rows)
        return false;
    int ipp = 0;
    bool any = false;
    for (int TR = std::min({maxM / a.Wd, a.Hd, (rows - fixed_rows) / a.s + 1}); TR >= 1 && !any;
         --TR) {
        a.tiles = (a.Hd + TR - 1) / TR;
        a.TR = (a.Hd + a.tiles - 1) / a.tiles;
        a.rows = a.s * (a.TR - 1) + fixed_rows;
        a.PL = a.rows * a.RP;
        ipp = (std::min(a.rows, a.Hs) * a.Ws + 3) / 4;
        for (int res = 1; res >= 0 && !any; --res) {
            const size_t fixed = NB * 4 + (res ? static_cast<size_t>(a.P) * T * WP * 4 : 0);
            const size_t per = static_cast<size_t>(a.PL) * 4 + (res ? 0 : static_cast<size_t>(T) * WP * 4);
            if (fixed + 2 * per + 256 > kF32Lds)
                continue;
            int G = static_cast<int>((kF32Lds - fixed - 256) / per);
            G = std::min(G, most * kFThreads / ipp) & ~1;
            G = std::min(G, Pe);
            if (G < 2)
                continue;
            const int nst = (a.P + G - 1) / G; // balanced stages, an even number of planes each
            G = std::min(G, ((a.P + nst - 1) / nst + 1) & ~1);
            a.G = G;
            a.nst = (a.P + G - 1) / G;
            a.resident = res;
            const size_t wts = static_cast<size_t>(res ? a.P : G) * T * WP * 4;
            a.bias_off = static_cast<int>((wts + 15) & ~static_cast<size_t>(15));
            a.win_off = a.bias_off + NB * 4;
            any = true;
        }
    }
    if (!any)
        return false;
    const long ntot = static_cast<long>(sh.N) * a.Dd * a.tiles;
    if (ntot > (1L << 30))
        return false;
    a.ntot = static_cast<int>(ntot);
    const int blocks = std::min(a.ntot, std::max(1, cus / a.nblk));
    const int rounds = (a.ntot + blocks - 1) / blocks;
    const int serial = (a.nblk * blocks + cus - 1) / cus;
    const int M = a.TR * a.Wd;
    const double busy = (M + 31) / 32 > kFWaves ? 1.0 : std::max(0.5, (M + 31) / 32 / 8.0);
    const double mf = 2.0 * busy * a.P * T / 2 * MG * NT * 66;
    const double stg = a.nst * 1200.0 + a.P * ipp * 0.6 + (a.resident ? 0 : a.P * T * NB * 0.3);
    const double out = M * NB * 4 / 12.0;
    pl.cost = serial * (rounds * (mf + stg + out) + (a.resident ? a.P * T * NB * 0.3 : 0));
    const int u = (a.G * ipp + kFThreads - 1) / kFThreads;
    pl.U = u <= 2 ? 2 : u <= 4 ? 4 : 8;
    pl.grid = blocks * a.nblk;
    pl.lds = static_cast<size_t>(a.win_off) + static_cast<size_t>(a.G) * a.PL * 4;
    return true;
}

bool plan_f32(const ConvShape &sh, F32Plan &best)
{
    if (sh.k < 1 || sh.k > 3 || sh.W < 4 || sh.Ho < 1)
        return false;
    const int K = sh.k, T = sh.T;
    F32Plan pl;
    F32Args &a = pl.a;
    a.Cs = sh.Ci;
    a.Cd = sh.Co;
    a.Ds = sh.D;
    a.Hs = sh.H;
    a.Ws = sh.W;
    a.Dd = sh.Do;
    a.Hd = sh.Ho;
    a.Wd = sh.Wo;
    a.s = sh.s;
    a.sz = sh.sz;
    a.kz = sh.kz;
    a.Z = sh.Z;
    a.J = sh.Z * T;
    a.P = a.Cs * a.Z;
    a.relu = 0;
    a.WCs = (a.Ws + 2 * K + a.s - 1) / a.s;
    a.RP = a.s * a.WCs;
    const int cus = device_cus();
    bool found = false;
    // no more tiles of channels than there are channels, no second group of
    // pixels where a plane has none
    for (pl.NT = 1; pl.NT <= std::min(3, (a.Cd + 31) / 32); ++pl.NT)
        for (pl.MG = 1; pl.MG <= (a.Hd * a.Wd > 32 * kFWaves ? 2 : 1); ++pl.MG)
            if (plan_tile(sh, cus, pl) && (!found || pl.cost < best.cost)) {
                best = pl;
                found = true;
            }
    if (!found)
        return false;
    F32Args &b = best.a;
    b.fper = make_fastdiv(static_cast<uint32_t>(b.Dd) * b.tiles);
    b.ftiles = make_fastdiv(static_cast<uint32_t>(b.tiles));
    b.fw = make_fastdiv(static_cast<uint32_t>(b.Ws));
    b.fz = make_fastdiv(static_cast<uint32_t>(b.Z));
    int t = 0;
    for (int dq = -K; dq <= K; ++dq)
        for (int i = 0; i < col_len(K, dq); ++i, ++t) {
            const int c = K + dq;
            b.toff[t] =
                (col_ds_lo(K, dq) + i + floor_half(dq)) * b.RP + (c % b.s) * b.WCs + c / b.s;
        }
    return true;
}

// Estimated time: rounds, products, staging, results, weights.
double f32_us(const F32Plan &pl, const ConvShape &sh)
{
    const F32Args &a = pl.a;
    const double blocks = pl.grid / a.nblk, M = a.TR * a.Wd;
    const double rounds = std::ceil(a.ntot / blocks) * std::max(1.0, pl.grid / 256.0);
    const double busy = M > 32 * kFWaves ? 1.0 : std::max(0.5, std::ceil(M / 32) / kFWaves);
    const double pt = static_cast<double>(a.P) * sh.T;
    const double items = static_cast<double>(a.P) * ((std::min(a.rows, a.Hs) * a.Ws + 3) / 4);
    return 2.6 + rounds * (2.87 + (0.93 * 66 * busy * pt * pl.MG * pl.NT + 3.79 * items +
                                   0.80 * M * 32 * pl.NT / 3) / 2400) +
           6.26 * 0.3 * pt * 32 * pl.NT / 2400;
}

template <int K, int NT, int MG>
hipError_t launch(const F32Plan &pl, const float *x, const float *w, const float *b, float *y,
                  hipStream_t st)
{
    constexpr int most = max_items(K, NT, MG);
    const dim3 grid(pl.grid), block(kFThreads);
    if (pl.U == 2)
        HEX_LAUNCH((conv_f32_k<K, NT, MG, 2>), grid, block, pl.lds, st, x, w, b, y, pl.a);
    else if (pl.U == 4 || most < 8)
        HEX_LAUNCH((conv_f32_k<K, NT, MG, (most < 4 ? 2 : 4)>), grid, block, pl.lds, st, x, w, b, y,
                   pl.a);
    else
        HEX_LAUNCH((conv_f32_k<K, NT, MG, (most < 8 ? 2 : 8)>), grid, block, pl.lds, st, x, w, b, y,
                   pl.a);
    return hipGetLastError();
}

template <int K>
hipError_t dispatch(const F32Plan &pl, const float *x, const float *w, const float *b, float *y,
                    hipStream_t st)
{
    if (pl.MG == 1) {
        if (pl.NT == 1)
            return launch<K, 1, 1>(pl, x, w, b, y, st);
        if (pl.NT == 2)
            return launch<K, 2, 1>(pl, x, w, b, y, st);
        if constexpr (max_items(K, 3, 1) > 0)
            return launch<K, 3, 1>(pl, x, w, b, y, st);
    } else {
        if constexpr (max_items(K, 1, 2) > 0)
            if (pl.NT == 1)
                return launch<K, 1, 2>(pl, x, w, b, y, st);
        if constexpr (max_items(K, 2, 2) > 0)
            if (pl.NT == 2)
                return launch<K, 2, 2>(pl, x, w, b, y, st);
    }
    return hipErrorInvalidValue;
}

} // namespace

Tried conv_f32_fwd(const void *in, const void *w, const void *bias, void *out, const ConvShape &sh,
                   bool relu, hipStream_t st, double other_us, hipError_t &e)
{
    // One input plane (at a stride; the few-channel kernel has the others) is
    // too short a contraction to pay for staging and weights: stride 2, us
    // here against generic, 2 x 1 -> 15 channels, 33 x 48, k = 2 7.3 / 6.1;
    // 4 x 1 -> 4, 24 x 30, k = 1 5.3 / 4.6.
    if (sh.Ci * sh.Z == 1)
        return Tried::No;
    F32Plan pl;
    if (!plan_f32(sh, pl))
        return Tried::No;
    if (f32_us(pl, sh) > other_us)
        return Tried::Slower;
    pl.a.relu = relu;
    const float *x = static_cast<const float *>(in), *wf = static_cast<const float *>(w);
    const float *b = static_cast<const float *>(bias);
    float *y = static_cast<float *>(out);
    e = sh.k == 1   ? dispatch<1>(pl, x, wf, b, y, st)
        : sh.k == 2 ? dispatch<2>(pl, x, wf, b, y, st)
                    : dispatch<3>(pl, x, wf, b, y, st);
    return Tried::Ran;
}

} // namespace hexk
