// chanlast.h -- channel-last windows in LDS for matrix-core kernels over
// planes of any size (k_conv_any.hip, k_wgrad_any.hip).
//
// A window holds rows of one plane of NCHW (or NCDHW) data with the channels
// of a slot contiguous, so a matrix-core operand is one 16-byte LDS read at
// the slot of a pixel plus a tap's offset, for any row length, stride and
// column parity.  Whole rows are contiguous in memory per channel, so the
// rows that exist are read as one flat run: an item is PX channels times PX
// consecutive pixels (PX = 8 for bfloat16, 4 for float32), PX 16-byte loads
// of elements that need not be aligned (a row of odd length starts anywhere;
// global memory takes 16-byte accesses at any element), transposed in
// registers and written as PX 16-byte LDS stores, one per pixel's slot.  The
// last item of a run is moved back to end with it and writes some slots a
// second time with the same values, so no load leaves the run.
#pragma once

#include "hexdev.h"

namespace hexk {

template <typename E> struct AnyE;
template <> struct AnyE<float> {
    static constexpr int PX = 4;
};
template <> struct AnyE<bf16raw> {
    static constexpr int PX = 8;
};

// Bytes that the channels of one staged block may span, so that an item's
// offset from the block's first element fits 32 bits.
constexpr long kAnyMaxSpan = 1L << 31;

// Columns of a window: column c (0 <= c < s * WCs) of a row lives at slot
// column (c % s) * WCs + c / s, so that consecutive outputs of a stride-s
// convolution read consecutive slots; a row holds RP = s * WCs slots.
struct WinGeom {
    int rows;  // window rows
    int RP;    // slots per row
    int WCs;   // slots per residue class
    int s;     // columns are split by residue mod s
    int coff;  // window column of plane column 0
    int W;     // plane columns
    __device__ __forceinline__ int slot(int row, int col) const
    {
        if (s == 1)
            return row * RP + col;
        const int q = col / s;
        return row * RP + (col - q * s) * WCs + q;
    }
};

// One item: channels [c, c + PX) of the flat pixels [f, f + PX) of a run.
// MIS: bfloat16 runs that may start at an odd element.  Loads at addresses
// that are no multiple of 4 take about twice as long (64 x 48 -> 48 channels,
// 128 x 127 against 128 x 126: 147 against 95 us), so those read the aligned
// words around the item, one word more, and align() shifts them.
template <typename E, bool MIS> struct AnyItem {
    static constexpr int PX = AnyE<E>::PX;
    uint4 v[PX];
    uint32_t ex[MIS ? PX : 1];

    // src: the run's first pixel of channel 0 (the same for the whole block;
    // a lane's offset from it fits 32 bits, kAnyMaxSpan).  Channels >= nc
    // read channel nc - 1 and are zeroed by drop(): the loads carry no
    // condition, else each becomes a branch of its own.
    __device__ __forceinline__ void load(const E *src, uint32_t cstride, int c, int nc, int f)
    {
        if constexpr (MIS) {
            const uintptr_t s = reinterpret_cast<uintptr_t>(src);
            const char *base = reinterpret_cast<const char *>(s & ~static_cast<uintptr_t>(3));
            const uint32_t s2 = s & 2;
#pragma unroll
            for (int e = 0; e < PX; ++e) {
                const uint32_t off = (min(c + e, nc - 1) * cstride + f) * 2 + s2;
                const char *p = base + (off & ~3u);
                __builtin_memcpy(&v[e], __builtin_assume_aligned(p, 4), 16);
                // the word with the last element (the last loaded one where
                // the item starts on a word: nothing past the item is read)
                const char *q = base + ((off & ~3u) + ((off & 2) ? 16 : 12));
                ex[e] = *reinterpret_cast<const uint32_t *>(q);
            }
        } else {
#pragma unroll
            for (int e = 0; e < PX; ++e) {
                const uint32_t off = (min(c + e, nc - 1) * cstride + f) * sizeof(E);
                __builtin_memcpy(&v[e], reinterpret_cast<const char *>(src) + off, 16);
            }
        }
    }

    // MIS: the words of an item that starts at an odd element, shifted; the
    // arguments of the load
    __device__ __forceinline__ void align(const E *src, uint32_t cstride, int c, int nc, int f)
    {
        if constexpr (MIS) {
            const uint32_t s2 = reinterpret_cast<uintptr_t>(src) & 2;
#pragma unroll
            for (int e = 0; e < PX; ++e) {
                const uint32_t off = (min(c + e, nc - 1) * cstride + f) * 2 + s2;
                const uint32_t sh = (off & 2) * 8; // 0 or 16
                v[e].x = __builtin_amdgcn_alignbit(v[e].y, v[e].x, sh);
                v[e].y = __builtin_amdgcn_alignbit(v[e].z, v[e].y, sh);
                v[e].z = __builtin_amdgcn_alignbit(v[e].w, v[e].z, sh);
                v[e].w = __builtin_amdgcn_alignbit(ex[e], v[e].w, sh);
            }
        }
    }

    // channels c + e >= nc become zero
    __device__ __forceinline__ void drop(int c, int nc)
    {
#pragma unroll
        for (int e = 0; e < PX; ++e) {
            const uint32_t m = c + e < nc ? 0xffffffffu : 0u;
            v[e].x &= m;
            v[e].y &= m;
            v[e].z &= m;
            v[e].w &= m;
        }
    }

    // the PX channels of pixel px as one 16-byte vector
    __device__ __forceinline__ uint4 pixel(int px) const
    {
        if constexpr (PX == 4) {
            const uint32_t a[4] = {comp(v[0], px), comp(v[1], px), comp(v[2], px), comp(v[3], px)};
            return make_uint4(a[0], a[1], a[2], a[3]);
        } else {
            uint32_t q[4];
#pragma unroll
            for (int j = 0; j < 4; ++j) {
                const uint32_t a = comp(v[2 * j], px >> 1), b = comp(v[2 * j + 1], px >> 1);
                // low or high halves of (a, b)
                q[j] = (px & 1) ? __builtin_amdgcn_perm(b, a, 0x07060302u)
                                : __builtin_amdgcn_perm(b, a, 0x05040100u);
            }
            return make_uint4(q[0], q[1], q[2], q[3]);
        }
    }

    __device__ static __forceinline__ uint32_t comp(const uint4 &u, int i)
    {
        return i == 0 ? u.x : i == 1 ? u.y : i == 2 ? u.z : u.w;
    }

    // Window slots of the flat pixels f .. f + PX - 1 of a run that starts
    // at window row row0, plane column 0; g: 16-byte vector within the slot.
    template <int SB>
    __device__ __forceinline__ void commit(unsigned char *__restrict__ win, const WinGeom &wg,
                                           int row0, int f, int g) const
    {
        int row = f / wg.W;
        int col = f - row * wg.W;
        row += row0;
        if (wg.s == 1) {
            int slot = row * wg.RP + col + wg.coff;
#pragma unroll
            for (int px = 0; px < PX; ++px) {
                *reinterpret_cast<uint4 *>(win + slot * SB + 16 * g) = pixel(px);
                ++slot;
                if (++col == wg.W) {
                    col = 0;
                    slot += wg.RP - wg.W;
                }
            }
        } else {
            int cq = (col + wg.coff) / wg.s;
            int cr = col + wg.coff - cq * wg.s;
            int base = row * wg.RP;
            const int q0 = wg.coff / wg.s, r0 = wg.coff - q0 * wg.s; // column 0
#pragma unroll
            for (int px = 0; px < PX; ++px) {
                *reinterpret_cast<uint4 *>(win + (base + cr * wg.WCs + cq) * SB + 16 * g) =
                    pixel(px);
                if (++cr == wg.s) {
                    cr = 0;
                    ++cq;
                }
                if (++col == wg.W) {
                    col = 0;
                    cr = r0;
                    cq = q0;
                    base += wg.RP;
                }
            }
        }
    }

    // Slots f .. f + PX - 1 of a plain list of pixels.
    template <int SB>
    __device__ __forceinline__ void commit_flat(unsigned char *__restrict__ lst, int f, int g) const
    {
#pragma unroll
        for (int px = 0; px < PX; ++px)
            *reinterpret_cast<uint4 *>(lst + (f + px) * SB + 16 * g) = pixel(px);
    }
};

// Zero the slots of a window that hold no element of the plane: the columns
// left of 0 and right of W - 1 in every row, and the rows before `lo` and
// from `hi` on.  NG 16-byte vectors per slot.
template <int SB, int NG, int NTHR>
__device__ __forceinline__ void zero_border(unsigned char *__restrict__ win, const WinGeom &wg,
                                            int lo, int hi)
{
    const int side = wg.RP - wg.W;
    const int n1 = wg.rows * side * NG;
    for (int i = threadIdx.x; i < n1; i += NTHR) {
        const int g = i % NG, r = i / NG;
        const int row = r / side;
        int col = r - row * side;
        col = col < wg.coff ? col : col + wg.W;
        *reinterpret_cast<uint4 *>(win + wg.slot(row, col) * SB + 16 * g) = make_uint4(0, 0, 0, 0);
    }
    const int nbad = lo + wg.rows - hi;
    const int n2 = nbad * wg.W * NG;
    for (int i = threadIdx.x; i < n2; i += NTHR) {
        const int g = i % NG, r = i / NG;
        int row = r / wg.W;
        const int col = r - row * wg.W + wg.coff;
        row = row < lo ? row : row - lo + hi;
        *reinterpret_cast<uint4 *>(win + wg.slot(row, col) * SB + 16 * g) = make_uint4(0, 0, 0, 0);
    }
}

} // namespace hexk
