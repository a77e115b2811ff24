// k_wgrad_any.hip -- weight and bias gradient on the matrix cores for planes
// of odd sizes, any channel count and any stride, k = 1 to 3, in bfloat16 and
// float32, two- and three-dimensional: output rows of 4 (float32) or 8
// (bfloat16) pixels and more whose x window and dy row fit LDS (x rows to
// 170 / 102 / 73 pixels in float32 and 624 / 409 / 292 in bfloat16 at k = 1 /
// 2 / 3 and stride 1, 128 / 85 / 64 and 512 / 341 / 256 at stride 2).  Takes
// what the tuned bfloat16 kernels (k_wgrad32.hip, k_wgrad_bf16.hip: whole
// 16-byte rows) and the small-channel kernels do not.
//
//   D_t[co][ci] = sum over output pixels p of dy[co][p] x[ci][p + tap t]
//
// one 32x32 product per tap with the pixels as the contraction.  A block (8
// waves) holds up to 64 output channels, up to 64 input channels and one
// window plane dz, and walks tiles of whole output rows: dy as a list of
// pixels and x as a window, both channel-last in LDS (chanlast.h).  Any
// pixel-to-slot map then serves as the contraction's index: a table in LDS
// gives each output pixel's centre slot, a tap adds a fixed offset (one row
// more for odd tap columns at odd centre columns), so odd row lengths,
// strides and parities cost nothing.
//  - bfloat16: an operand holds 8 pixels of one channel; the transposing LDS
//    read (ds_read_b64_tr_b16: 16 lanes read four slots of 16 channels, lane
//    i receives channel i of the four) gathers it from channel-last slots.
//    32x32x16 products.
//  - float32: an operand is one 4-byte read, lanes 0-31 the channels of one
//    pixel and lanes 32-63 of the next. 32x32x2 products.
// The bias gradient is one more "tap" whose x operand is all ones.
//
// Wave roles: G groups of TPW taps (T + 1 of them with the bias), A blocks of
// 32 input channels, and the rest splits the pixels (KS); each wave holds
// TPW x NCO accumulators, so a dy operand serves TPW products and an x
// operand NCO.  The pixel splits are added through LDS at the end, the
// block's sums go to a slot of the workspace and reduce_any_k adds the slots
// in order (deterministic).
//
// float32 sums: a chain of n additions of independent terms is off by about
// 2.5e-8 sqrt(n / 2) of the sum, and a block's run of tiles is long.  So the
// matrix cores add 16 pixels at a time, from zero, eight of these sums (or
// the root of their number, which makes the two chains equal, where that is
// more: 512 -> 512 channels, k = 3, 16 of 57 x 57, whose one slot a type has
// 3 600 of them: dw 3.9e-7 with eight, 2.1e-7 now, generic kernel 2.6e-7)
// are added up, and those are added over the run: three short chains.  Off the
// sum in 64 bits (generic kernel, one chain, now): 4 -> 8 channels, k = 2, 227
// images of 41 x 39, dw 1.1e-7, 1.8e-7, 0.85e-7, db 1.8e-7, 4.4e-7, 1.4e-7; 64
// -> 96, 28 x 29 x 33, dw 1.4e-7, 2.1e-7, 1.0e-7; 22 volumes of 12 -> 32, dw
// 1.1e-7, 2.7e-7, 1.1e-7.  The two sums kept of a tap take 32 registers, so a block holds one 32 x 32
// tile of channels (at k = 1 two of output channels, a tap a wave), which
// costs little, the products being the slow part (64 clocks each).  (64-bit sums of the 16 pixels: the conversions made k = 2
// 1.3 times as slow.)
//
// Pixels past a tile's end: both operands are zeroed (by masks), so that no
// product of a stray infinity reaches a sum.
#include <algorithm>
#include <cmath>
#include <type_traits>

#include "../../include/hexconv.h"
#include "chanlast.h"
#include "kernels.h"

namespace hexk {
namespace {

using namespace hexgeom;

typedef float floatx16 __attribute__((ext_vector_type(16)));
typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef short shortx4 __attribute__((ext_vector_type(4)));

constexpr int kWThreads = 512;

// Taps per wave and tap groups: T + 1 columns (the taps and the bias)
constexpr int role_tpw(bool f32, int k, int nco) { return k > 1 ? 5 : f32 ? 2 / nco : 4; }
constexpr int role_g(bool f32, int k, int nco) { return k == 3 ? 8 : k == 2 ? 4 : f32 ? 4 * nco : 2; }
constexpr int kRunSteps = 8; // float32: least steps of 16 pixels per chain of step sums

// Four pixels of a channel from a0 and four from a1, transposed (see above)
__device__ __forceinline__ bf16x8 tr_read(unsigned char *a0, unsigned char *a1)
{
    using lp = __attribute__((address_space(3))) shortx4 *;
    const shortx4 lo = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lp)a0);
    const shortx4 hi = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lp)a1);
    typedef short shortx8 __attribute__((ext_vector_type(8)));
    const shortx8 v = __builtin_shufflevector(lo, hi, 0, 1, 2, 3, 4, 5, 6, 7);
    return __builtin_bit_cast(bf16x8, v);
}

// NCO: 32-channel tiles of output channels (1 or 2); A: of input channels
// U: items of x and of dy per thread.  PF: the next tile's items are loaded
// during the products (where the registers hold them beside the sums).
template <typename E, int K, int NCO, int A, int U, bool PF, bool MIS>
__global__ __launch_bounds__(kWThreads) void wgrad_any_k(const E *x, const E *dy,
                                                         float *__restrict__ part, WAnyArgs a)
{
    constexpr bool F32 = sizeof(E) == 4;
    constexpr int PX = AnyE<E>::PX;
    constexpr int T = num_taps(K);
    constexpr TapTable<K> tab{};
    constexpr int TPW = role_tpw(F32, K, NCO), G = role_g(F32, K, NCO);
    constexpr int KS = 8 / (G * A);
    constexpr int CB = 32 * sizeof(E);      // bytes of 32 channels
    constexpr int XB = A * CB, DB = NCO * CB; // bytes per slot
    constexpr int XG = XB / 16, DG = DB / 16; // 16-byte vectors per slot
    extern __shared__ __align__(16) unsigned char smem[];
    unsigned char *dyl = smem, *win = smem + a.x_off;
    int *ptab = reinterpret_cast<int *>(smem + a.tab_off);

    const int lane = threadIdx.x & 63;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int grp = wave % G, ai = (wave / G) % A, ks = wave / (G * A);
    const int types = a.Z * a.nci * a.nco;
    const int type = blockIdx.x % types, slot = blockIdx.x / types;
    const int cob = type % a.nco, cib = (type / a.nco) % a.nci, dz = type / (a.nco * a.nci);
    const int co0 = cob * 32 * NCO, ci0 = cib * 32 * A;
    const size_t HWx = static_cast<size_t>(a.H) * a.W, HWy = static_cast<size_t>(a.Ho) * a.Wo;
    const size_t csx = HWx * a.D, csy = HWy * a.Do;
    const WinGeom wg{a.rows, a.RP, a.WCs, a.s, K, a.W};

    // byte address of every tile pixel's centre slot; bit 0: odd centre column
    for (int p = threadIdx.x; p < a.npix; p += kWThreads) {
        const int q = min(p, a.TR * a.Wo - 1);
        const int i = q / a.Wo, j = q - i * a.Wo;
        ptab[p] = ((a.s * i + (j & 1) * (a.s >> 1) + K) * a.RP + j) * XB | ((a.s * j) & 1);
    }

    struct Pos {
        int tb, n, l, i0, zs;
    };
    // first tile from tb on (steps of nslots) whose source plane exists
    auto settle = [&](Pos &p) {
        const int per = a.Do * a.tiles;
        for (; p.tb < a.ntot; p.tb += a.nslots) {
            p.n = p.tb / per;
            const int r = p.tb - p.n * per;
            p.l = r / a.tiles;
            p.i0 = (r - p.l * a.tiles) * a.TR;
            p.zs = a.sz * p.l + dz - a.kz;
            if (p.zs >= 0 && p.zs < a.D)
                return true;
        }
        return false;
    };
    auto span = [&](const Pos &p, int &lo, int &run) {
        const int r_lo = a.s * p.i0 - K;
        lo = max(0, -r_lo);
        const int hi = min(a.rows, a.H - r_lo);
        run = (hi - lo) * a.W;
        return hi;
    };
    AnyItem<E, MIS> ix[U], id[U];
    auto x_src = [&](const Pos &p, int lo) { // first pixel of the window's rows
        return x + (static_cast<size_t>(p.n) * a.Ci + ci0) * csx + static_cast<size_t>(p.zs) * HWx +
               static_cast<size_t>(a.s * p.i0 - K + lo) * a.W;
    };
    auto dy_src = [&](const Pos &p) {
        return dy + (static_cast<size_t>(p.n) * a.Co + co0) * csy +
               static_cast<size_t>(p.l) * HWy + static_cast<size_t>(p.i0) * a.Wo;
    };
    auto load_x = [&](const Pos &p) {
        int lo, run;
        span(p, lo, run);
#pragma unroll
        for (int u = 0; u < U; ++u) {
            const int i = threadIdx.x + u * kWThreads;
            ix[u].load(x_src(p, lo), csx, (i % XG) * PX, a.Ci - ci0, min((i / XG) * PX, run - PX));
        }
    };
    auto load_dy = [&](const Pos &p) {
        const int M = min(a.TR, a.Ho - p.i0) * a.Wo;
#pragma unroll
        for (int u = 0; u < U; ++u) {
            const int i = threadIdx.x + u * kWThreads;
            id[u].load(dy_src(p), csy, (i % DG) * PX, a.Co - co0, min((i / DG) * PX, M - PX));
        }
    };
    auto commit_x = [&](const Pos &p) {
        int lo, run;
        const int hi = span(p, lo, run);
#pragma unroll
        for (int u = 0; u < U; ++u) {
            const int i = threadIdx.x + u * kWThreads;
            const int f = min((i / XG) * PX, run - PX);
            ix[u].align(x_src(p, lo), csx, (i % XG) * PX, a.Ci - ci0, f);
            if (a.Ci - ci0 < 32 * A)
                ix[u].drop((i % XG) * PX, a.Ci - ci0);
            if ((i / XG) * PX < run)
                ix[u].template commit<XB>(win, wg, lo, f, i % XG);
        }
        zero_border<XB, XG, kWThreads>(win, wg, lo, hi);
    };
    auto commit_dy = [&](const Pos &p) {
        const int M = min(a.TR, a.Ho - p.i0) * a.Wo;
#pragma unroll
        for (int u = 0; u < U; ++u) {
            const int i = threadIdx.x + u * kWThreads;
            const int f = min((i / DG) * PX, M - PX);
            id[u].align(dy_src(p), csy, (i % DG) * PX, a.Co - co0, f);
            if (a.Co - co0 < 32 * NCO)
                id[u].drop((i % DG) * PX, a.Co - co0);
            if ((i / DG) * PX < M)
                id[u].template commit_flat<DB>(dyl, f, i % DG);
        }
        // the slots past the last pixel, up to a whole step
        const int Mp = (M + 15) & ~15;
        for (int i = threadIdx.x; i < (Mp - M) * DG; i += kWThreads)
            *reinterpret_cast<uint4 *>(dyl + (M + i / DG) * DB + 16 * (i % DG)) =
                make_uint4(0, 0, 0, 0);
    };

    floatx16 acc[NCO][TPW];
#pragma unroll
    for (int c = 0; c < NCO; ++c)
#pragma unroll
        for (int t = 0; t < TPW; ++t)
            acc[c][t] = floatx16{};
    // float32: sums of up to run_steps steps, not yet in acc
    constexpr int RC = F32 ? NCO : 1, RT = F32 ? TPW : 1;
    floatx16 run[RC][RT];
    int nrun = 0;
#pragma unroll
    for (int c = 0; c < RC; ++c)
#pragma unroll
        for (int t = 0; t < RT; ++t)
            run[c][t] = floatx16{};
    auto end_run = [&]() {
        if constexpr (F32)
#pragma unroll
            for (int c = 0; c < NCO; ++c)
#pragma unroll
                for (int t = 0; t < TPW; ++t) {
                    acc[c][t] += run[c][t];
                    run[c][t] = floatx16{};
                }
    };

    unsigned char *xb = win + ai * CB;
    const int prow = a.RP * XB;

    // this wave's taps: offsets (wave-uniform), parity of their columns.  The
    // bias is tap T; the taps past it compute sums that are not read.
    int toff[TPW];
    bool todd[TPW];
#pragma unroll
    for (int t = 0; t < TPW; ++t) {
        toff[t] = 0;
        todd[t] = false;
#pragma unroll
        for (int g = 0; g < G; ++g)
            if (g * TPW + t < T && grp == g) {
                toff[t] = a.toff[g * TPW + t];
                todd[t] = (tab.dq[g * TPW + t] & 1) != 0;
            }
    }
    const bool has_bias = grp == T / TPW;

    // one step: 16 pixels of the tile from p0 on; TAIL: only `left` of them exist
    auto step = [&](auto tail, int p0, int left) {
        constexpr bool TAIL = decltype(tail)::value;
        if constexpr (F32) {
            float av[NCO][8];
            int b0[8], b1[8]; // window bytes of the centre, and where the tap's column is odd
#pragma unroll
            for (int h = 0; h < 8; ++h) {
                const int p = p0 + 2 * h + (lane >> 5);
                const int e = ptab[p];
                b0[h] = (e & ~1) + 4 * (lane & 31);
                b1[h] = b0[h] + ((e & 1) ? prow : 0);
#pragma unroll
                for (int c = 0; c < NCO; ++c)
                    av[c][h] = *reinterpret_cast<const float *>(dyl + p * DB + c * CB +
                                                                4 * (lane & 31));
            }
            // a tap's operands are read during the products of the tap before
            // (left alone, each product waits for its own read), whose sums
            // are added in turn between this tap's products
            float bv[2][8];
            auto read = [&](int t) {
#pragma unroll
                for (int h = 0; h < 8; ++h) {
                    float v = *reinterpret_cast<const float *>(xb + (todd[t] ? b1[h] : b0[h]) +
                                                               toff[t]);
                    if (t == T % TPW && has_bias)
                        v = 1.f;
                    if (TAIL)
                        v = 2 * h + (lane >> 5) < left ? v : 0.f;
                    bv[t & 1][h] = v;
                }
            };
            floatx16 s[2][NCO];
            read(0);
#pragma unroll
            for (int t = 0; t < TPW; ++t) {
                if (t + 1 < TPW)
                    read(t + 1);
#pragma unroll
                for (int c = 0; c < NCO; ++c)
                    s[t & 1][c] = floatx16{};
#pragma unroll
                for (int h = 0; h < 8; ++h) {
                    __builtin_amdgcn_sched_barrier(0);
#pragma unroll
                    for (int c = 0; c < NCO; ++c) {
                        s[t & 1][c] = __builtin_amdgcn_mfma_f32_32x32x2f32(
                            av[c][h], bv[t & 1][h], s[t & 1][c], 0, 0, 0);
                        if (t > 0)
#pragma unroll
                            for (int r = 2 * h; r < 2 * h + 2; ++r)
                                run[c][t - 1][r] += s[(t - 1) & 1][c][r];
                    }
                }
            }
#pragma unroll
            for (int c = 0; c < NCO; ++c)
                run[c][TPW - 1] += s[(TPW - 1) & 1][c];
            if (++nrun == a.run_steps) {
                nrun = 0;
                end_run();
            }
        } else {
            // pixels 8 (lane / 32) + (lane % 16) / 4 and 4 further on;
            // channels 16 ((lane / 16) % 2) + 4 (lane % 4) ..
            const int pl = 8 * (lane >> 5) + ((lane & 15) >> 2);
            const int cl = 32 * ((lane >> 4) & 1) + 8 * (lane & 3);
            const int e0 = ptab[p0 + pl], e1 = ptab[p0 + pl + 4];
            unsigned char *x00 = xb + (e0 & ~1) + cl, *x10 = xb + (e1 & ~1) + cl;
            unsigned char *x01 = x00 + ((e0 & 1) ? prow : 0);
            unsigned char *x11 = x10 + ((e1 & 1) ? prow : 0);
            bf16x8 av[NCO];
#pragma unroll
            for (int c = 0; c < NCO; ++c) {
                unsigned char *d = dyl + (p0 + pl) * DB + c * CB + cl;
                av[c] = tr_read(d, d + 4 * DB);
            }
            // halves of the operand's dwords that lie past the tile's end
            const int lv = left - 8 * (lane >> 5);
#pragma unroll
            for (int t = 0; t < TPW; ++t) {
                uint4 u = __builtin_bit_cast(uint4, tr_read((todd[t] ? x01 : x00) + toff[t],
                                                            (todd[t] ? x11 : x10) + toff[t]));
                if (t == T % TPW && has_bias)
                    u = make_uint4(0x3f803f80u, 0x3f803f80u, 0x3f803f80u, 0x3f803f80u);
                if (TAIL) {
                    u.x &= lv >= 2 ? 0xffffffffu : lv == 1 ? 0xffffu : 0u;
                    u.y &= lv >= 4 ? 0xffffffffu : lv == 3 ? 0xffffu : 0u;
                    u.z &= lv >= 6 ? 0xffffffffu : lv == 5 ? 0xffffu : 0u;
                    u.w &= lv >= 8 ? 0xffffffffu : lv == 7 ? 0xffffu : 0u;
                }
                const bf16x8 bv = __builtin_bit_cast(bf16x8, u);
#pragma unroll
                for (int c = 0; c < NCO; ++c)
                    acc[c][t] =
                        __builtin_amdgcn_mfma_f32_32x32x16_bf16(av[c], bv, acc[c][t], 0, 0, 0);
            }
        }
    };

    Pos cur{slot, 0, 0, 0, 0};
    bool more = settle(cur);
    if (PF && more) {
        load_x(cur);
        load_dy(cur);
    }
    while (more) {
        Pos nxt = cur;
        nxt.tb += a.nslots;
        more = settle(nxt);
        if (!PF)
            load_x(cur);
        __syncthreads(); // the previous tile's readers are done (and the table is written)
        commit_x(cur);
        if (!PF)
            load_dy(cur);
        commit_dy(cur);
        __syncthreads();
        if (PF && more) {
            load_x(nxt);
            load_dy(nxt);
        }
        const int M = min(a.TR, a.Ho - cur.i0) * a.Wo;
        const int nst = M >> 4;
        for (int q = ks; q < nst; q += KS)
            step(std::false_type{}, q * 16, 16);
        if ((M & 15) != 0 && nst % KS == ks)
            step(std::true_type{}, nst * 16, M & 15);
        cur = nxt;
    }

    end_run();
    // add the pixel splits, then one slot of partial sums:
    // part[type][slot][wave role][tap][co tile][r][lane]
    constexpr int WE = NCO * TPW * 16 * 64; // floats per wave
    float *red = reinterpret_cast<float *>(smem);
    const int role = wave % (G * A);
#pragma unroll
    for (int k = 1; k < KS; ++k) {
        __syncthreads();
        if (ks == k) {
#pragma unroll
            for (int c = 0; c < NCO; ++c)
#pragma unroll
                for (int t = 0; t < TPW; ++t)
#pragma unroll
                    for (int r = 0; r < 16; ++r)
                        red[role * WE + ((t * NCO + c) * 16 + r) * 64 + lane] = acc[c][t][r];
        }
        __syncthreads();
        if (ks == 0) {
#pragma unroll
            for (int c = 0; c < NCO; ++c)
#pragma unroll
                for (int t = 0; t < TPW; ++t)
#pragma unroll
                    for (int r = 0; r < 16; ++r)
                        acc[c][t][r] += red[role * WE + ((t * NCO + c) * 16 + r) * 64 + lane];
        }
    }
    if (ks == 0) {
        float *o = part + ((static_cast<size_t>(type) * a.nslots + slot) * (G * A) + role) * WE;
#pragma unroll
        for (int c = 0; c < NCO; ++c)
#pragma unroll
            for (int t = 0; t < TPW; ++t)
#pragma unroll
                for (int r = 0; r < 16; ++r)
                    o[((t * NCO + c) * 16 + r) * 64 + lane] = acc[c][t][r];
    }
}

// dw and db from the slots, in a fixed order and in 64 bits (the loads bound
// it): a block owns 64 consecutive partial elements (one wave's width) and its
// waves every kRedWaves-th slot, eight loads in flight each; the waves' sums
// are added through LDS.  One
// thread per element over all slots was bound by its chain of loads (256
// slots of 64 KB: 18.7 us).
struct RedArgs {
    int Ci, Co, Z, T, nci, nco, nslots, NCO, A, TPW, G, kz;
    int per; // floats per slot
};
constexpr int kRedWaves = 8;

__global__ __launch_bounds__(64 * kRedWaves) void reduce_any_k(const float *__restrict__ part,
                                                               float *__restrict__ dw,
                                                               float *__restrict__ db, RedArgs a)
{
    __shared__ double sums[kRedWaves][64];
    const int type = blockIdx.y;
    const int lane = threadIdx.x & 63;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    // what this block's elements are: [wave role][tap][co tile][r][lane]
    const int r = blockIdx.x & 15;
    int q = blockIdx.x >> 4;
    const int c = q % a.NCO;
    q /= a.NCO;
    const int t = q % a.TPW;
    q /= a.TPW;
    const int tap = (q % a.G) * a.TPW + t, ai = q / a.G;
    const int cob = type % a.nco, cib = (type / a.nco) % a.nci, dz = type / (a.nco * a.nci);
    const bool bias = tap == a.T;
    const int co0 = (cob * a.NCO + c) * 32 + 8 * (r >> 2) + (r & 3);
    const int ci0 = (cib * a.A + ai) * 32;
    if (tap > a.T || co0 >= a.Co || ci0 >= a.Ci ||
        (bias && (db == nullptr || ci0 != 0 || dz != a.kz)))
        return; // the same for the whole block
    const float *p = part + static_cast<size_t>(type) * a.nslots * a.per + blockIdx.x * 64 + lane;
    double s[8] = {};
    int i = wave;
    for (; i + 7 * kRedWaves < a.nslots; i += 8 * kRedWaves)
#pragma unroll
        for (int u = 0; u < 8; ++u)
            s[u] += p[static_cast<size_t>(i + u * kRedWaves) * a.per];
    for (; i < a.nslots; i += kRedWaves)
        s[0] += p[static_cast<size_t>(i) * a.per];
    sums[wave][lane] = ((s[0] + s[1]) + (s[2] + s[3])) + ((s[4] + s[5]) + (s[6] + s[7]));
    __syncthreads();
    if (wave != 0)
        return;
    double sum = 0.0;
#pragma unroll
    for (int k = 0; k < kRedWaves; ++k)
        sum += sums[k][lane];
    const float v = static_cast<float>(sum);
    const int co = co0 + 4 * (lane >> 5), ci = ci0 + (lane & 31);
    if (co >= a.Co || ci >= a.Ci || (bias && ci != 0))
        return;
    if (bias)
        db[co] = v;
    else
        dw[(static_cast<size_t>(co) * a.Ci + ci) * a.Z * a.T + dz * a.T + tap] = v;
}

// ------------------------------------------------------------------- host

constexpr size_t kAnyLds = 160 * 1024;

// Clocks of a compute unit for `slots` blocks of every type at the tile of
// `pl`: rounds of tiles (products of two waves a SIMD, and staging), and the
// partial sums of all slots, written and read again at about 3 TB/s.
double tile_cost(const WAnyPlan &pl, Dtype d, long ntot, int slots, int items, size_t slot,
                 int cus)
{
    const WAnyArgs &a = pl.a;
    const int KS = 8 / (pl.G * pl.A);
    const int steps = (a.npix / 16 + KS - 1) / KS;
    const double mf = steps * 2.0 * pl.TPW * pl.NCO * (d == F32 ? 8 * 64 : 32);
    const double waves = std::max(1.0, pl.types * slots / static_cast<double>(cus));
    const double rounds = static_cast<double>((ntot + slots - 1) / slots);
    return waves * rounds * (mf + 4000 + items * 4.0) + slot * slots * 0.0008;
}

// The tile (rows of it) and the number of slots for A input-channel tiles
// and U items per thread, the cheapest that fits.
bool plan_tile(const ConvShape &sh, Dtype d, int A, int U, int cus, WAnyPlan &best)
{
    const int es = d == F32 ? 4 : 2, PX = 16 / es;
    const int K = sh.k;
    WAnyPlan pl{};
    WAnyArgs &a = pl.a;
    a.N = sh.N;
    a.Ci = sh.Ci;
    a.Co = sh.Co;
    a.D = sh.D;
    a.H = sh.H;
    a.W = sh.W;
    a.Do = sh.Do;
    a.Ho = sh.Ho;
    a.Wo = sh.Wo;
    a.s = sh.s;
    a.sz = sh.sz;
    a.kz = sh.kz;
    a.Z = sh.Z;
    pl.NCO = (d != F32 || K == 1) && sh.Co > 32 ? 2 : 1;
    pl.TPW = role_tpw(d == F32, K, pl.NCO);
    pl.G = role_g(d == F32, K, pl.NCO);
    pl.A = A;
    pl.U = U;
    a.nco = (sh.Co + 32 * pl.NCO - 1) / (32 * pl.NCO);
    a.nci = (sh.Ci + 32 * A - 1) / (32 * A);
    pl.types = a.Z * a.nci * a.nco;
    const int XB = A * 32 * es, DB = pl.NCO * 32 * es;
    if (static_cast<long>(sh.D) * sh.H * sh.W * XB >= kAnyMaxSpan ||
        static_cast<long>(sh.Do) * sh.Ho * sh.Wo * DB >= kAnyMaxSpan)
        return false;
    const int we = pl.NCO * pl.TPW * 16 * 64;
    const int KS = 8 / (pl.G * A);
    // one block per compute unit in all; every slot costs a write and a read
    // of its partial sums.  No more slots than the scratch array of
    // hexconv_bwd_noalloc holds (at k > 1 256 slots would take 80 MB of its
    // 64), and no shape of which it holds not even one, so that this call
    // takes every shape that the other kernels' workspaces allow.
    const size_t slot = static_cast<size_t>(pl.types) * pl.G * A * we * 4;
    if (slot > HEX_NOALLOC_SCRATCH_BYTES)
        return false;
    const int most = std::max(1, std::min(cus / pl.types,
                                          static_cast<int>(HEX_NOALLOC_SCRATCH_BYTES / slot)));
    const int cols = sh.W + 2 * K;
    a.WCs = (cols + a.s - 1) / a.s;
    // slots of 64 bytes: rows of a multiple of 4 keep the 256-byte phase of
    // consecutive columns when odd columns read one row further down
    a.WCs = (a.WCs + 3) & ~3;
    a.RP = a.s * a.WCs;
    bool found = false;
    for (int TR = std::min(sh.Ho, std::max(1, 512 / sh.Wo)); TR >= 1; --TR) {
        const int tiles = (sh.Ho + TR - 1) / TR;
        if (found && tiles == a.tiles)
            continue; // the same rows per tile
        a.TR = (sh.Ho + tiles - 1) / tiles;
        a.tiles = tiles;
        a.rows = a.s * (a.TR - 1) + (sh.Wo > 1 ? a.s / 2 : 0) + 2 * K + 1;
        const int M = a.TR * sh.Wo;
        a.npix = (M + 15) & ~15;
        const int ix = (XB / 16) * ((std::min(a.rows, sh.H) * sh.W + PX - 1) / PX);
        const int id = (DB / 16) * ((M + PX - 1) / PX);
        const size_t dyb = static_cast<size_t>(a.npix) * DB;
        const size_t xb = static_cast<size_t>(a.rows) * a.RP * XB;
        pl.lds = dyb + xb + static_cast<size_t>(a.npix) * 4;
        if (pl.lds > kAnyLds || ix > U * kWThreads || id > U * kWThreads)
            continue;
        const long ntot = static_cast<long>(sh.N) * sh.Do * tiles;
        if (ntot > (1L << 30))
            break;
        const int slots = static_cast<int>(std::min<long>(ntot, most));
        const double cost = tile_cost(pl, d, ntot, slots, ix + id, slot, cus);
        if (found && cost >= best.cost)
            continue;
        found = true;
        a.x_off = static_cast<int>(dyb);
        a.tab_off = static_cast<int>(dyb + xb);
        a.ntot = static_cast<int>(ntot);
        a.nslots = slots;
        pl.ws = slot * slots;
        pl.cost = cost;
        best = pl;
        // the pixel splits are added through LDS
        if (KS > 1)
            best.lds = std::max(best.lds, static_cast<size_t>(pl.G) * A * we * 4);
    }
    if (!found)
        return false;
    WAnyArgs &b = best.a;
    const int split = 8 / (best.G * best.A);
    const double steps = std::ceil(static_cast<double>(b.ntot) / b.nslots) *
                         ((b.npix / 16 + split - 1) / split);
    b.run_steps = std::max(kRunSteps, static_cast<int>(std::lround(std::sqrt(steps))));
    int t = 0;
    for (int dq = -K; dq <= K; ++dq)
        for (int i = 0; i < col_len(K, dq); ++i, ++t) {
            const int c = K + dq;
            b.toff[t] = ((col_ds_lo(K, dq) + i + floor_half(dq)) * b.RP + (c % b.s) * b.WCs +
                         c / b.s) * XB;
        }
    return true;
}

bool plan_wgrad(const ConvShape &sh, Dtype d, WAnyPlan &pl)
{
    if (sh.k < 1 || sh.k > 3 || sh.Wo < (d == F32 ? 4 : 8) || sh.Ho < 1)
        return false;
    // bfloat16: two input-channel tiles share the dy tile (at k = 3 the taps
    // take every wave), and one item per thread where that holds a tile
    const int A = (d != F32 && sh.Ci > 32 && sh.k < 3) ? 2 : 1;
    const int cus = device_cus();
    bool ok = false;
    for (int aa = A; aa >= 1 && !ok; --aa)
        for (int u = d == F32 ? 2 : 1; u <= 2 && !ok; ++u)
            ok = plan_tile(sh, d, aa, u, cus, pl);
    return ok;
}

template <typename E, int K, int NCO, int A>
hipError_t launch_u(const WAnyPlan &pl, const void *x, const void *dy, float *part, hipStream_t st)
{
    const dim3 grid(pl.types * pl.a.nslots), block(kWThreads);
    const E *xe = static_cast<const E *>(x), *de = static_cast<const E *>(dy);
    // the next tile's items fit beside the sums except at 160 registers of
    // sums (k > 1: bfloat16 with two tiles of output channels, float32) and at
    // 128 registers of items
    constexpr bool sums = K == 1 || (sizeof(E) == 2 && NCO == 1);
#define HEX_WA(UV, PFV, MISV)                                                                \
    HEX_LAUNCH((wgrad_any_k<E, K, NCO, A, UV, PFV, MISV>), grid, block, pl.lds, st, xe, de,  \
               part, pl.a)
    if constexpr (sizeof(E) == 4) {
        HEX_WA(2, sums, false);
    } else {
        const bool mis = ((pl.a.W | pl.a.Wo) & 1) != 0; // some runs start at an odd element
        if (pl.U == 1) {
            if (mis)
                HEX_WA(1, NCO == 1, true);
            else
                HEX_WA(1, sums, false);
        } else if (mis) {
            HEX_WA(2, false, true);
        } else {
            HEX_WA(2, false, false);
        }
    }
#undef HEX_WA
    return hipGetLastError();
}

template <typename E, int K>
hipError_t launch_k(const WAnyPlan &pl, const void *x, const void *dy, float *part, hipStream_t st)
{
    if constexpr (sizeof(E) == 4) {
        if constexpr (K == 1)
            if (pl.NCO == 2)
                return launch_u<E, K, 2, 1>(pl, x, dy, part, st);
        return launch_u<E, K, 1, 1>(pl, x, dy, part, st);
    } else {
        if constexpr (K < 3)
            if (pl.A == 2)
                return pl.NCO == 2 ? launch_u<E, K, 2, 2>(pl, x, dy, part, st)
                                   : launch_u<E, K, 1, 2>(pl, x, dy, part, st);
        return pl.NCO == 2 ? launch_u<E, K, 2, 1>(pl, x, dy, part, st)
                           : launch_u<E, K, 1, 1>(pl, x, dy, part, st);
    }
}

template <typename E>
hipError_t launch_e(const WAnyPlan &pl, int k, const void *x, const void *dy, float *part,
                    hipStream_t st)
{
    switch (k) {
    case 1:
        return launch_k<E, 1>(pl, x, dy, part, st);
    case 2:
        return launch_k<E, 2>(pl, x, dy, part, st);
    default:
        return launch_k<E, 3>(pl, x, dy, part, st);
    }
}

} // namespace

bool wgrad_any_plan(const ConvShape &sh, Dtype d, WAnyPlan &pl)
{
    // Few input channels leave most of a 32-channel tile empty: in float32,
    // whose products take 16 times as long, another kernel is then the faster
    // one (64 images of 41 x 43, us here against generic: k = 1 4 -> 16
    // channels 47 / 65, 3 -> 16 46 / 58, 2 -> 16 45 / 38; 8 volumes of 12
    // planes, 3 -> 16 104 / 189, 2 -> 8 slower).
    if (d == F32 && (sh.Ci * sh.T < 20 || (sh.Z > 1 && sh.Ci < 3)))
        return false;
    if (!plan_wgrad(sh, d, pl))
        return false;
    pl.us = d == F32 ? 8.2 + 1.20 * pl.cost / 2400 : 10.5 + 1.14 * pl.cost / 2400;
    return true;
}

hipError_t wgrad_any(const void *x, const void *dy, float *dw, float *db, void *ws,
                     const ConvShape &sh, Dtype d, const WAnyPlan &pl, hipStream_t st)
{
    float *part = static_cast<float *>(ws);
    hipError_t e = d == F32 ? launch_e<float>(pl, sh.k, x, dy, part, st)
                            : launch_e<bf16raw>(pl, sh.k, x, dy, part, st);
    if (e != hipSuccess)
        return e;
    const WAnyArgs &a = pl.a;
    const int per = pl.G * pl.A * pl.NCO * pl.TPW * 16 * 64;
    const RedArgs r{a.Ci, a.Co, a.Z, sh.T, a.nci, a.nco, a.nslots, pl.NCO, pl.A,
                    pl.TPW, pl.G, a.kz, per};
    HEX_LAUNCH(reduce_any_k, dim3(per / 64, pl.types), dim3(64 * kRedWaves), 0, st, part, dw, db, r);
    return hipGetLastError();
}

} // namespace hexk
