// Workgroup-level exact arithmetic on little-endian 32-bit-limb numbers.
//
// One workgroup of T threads (T/64 wavefronts) owns one multi-precision
// instance.  Operands live in LDS (or are read straight from global memory
// through a view).
//
// Here: the views operands are read through, and the vector-ALU product, whose
// two passes (copy, mul) are called by all T threads with the same arguments,
// begin with a workgroup barrier so that they see every earlier write, and leave
// their results unsynchronised.
// The primitives header (mp_prims_hip.hpp) must be included first.
#pragma once

#include <stdint.h>

namespace mp {

constexpr int kRCol = 4;                 // product columns per lane
constexpr int kStrip = kLanes * kRCol;   // product columns per wave pass
constexpr int kPad = kStrip + 8;         // zero guard on both sides of a staged window operand


// control block at the start of the instance's LDS (32-bit words)
constexpr int kCtlOver = 0;      // 16 per-wave carries that run through a wave's columns
constexpr int kCtlStrip = 16;    // strip carries: one word per strip, or two (vector ALU: up to 64 strips)
constexpr int kCtlPrec = 16;     // before them, precisions: four words per wave
constexpr int kCtlBcast = 144;   // 16 broadcast scalars
constexpr int kCtlWords = 160;

#define MP_HD __host__ __device__ __forceinline__

MP_HD constexpr int r4(int x) { return (x + 3) & ~3; }
MP_HD constexpr int hmax(int a, int b) { return a > b ? a : b; }
MP_HD constexpr int hmin(int a, int b) { return a < b ? a : b; }

MP_DEV int imin(int a, int b) { return a < b ? a : b; }
MP_DEV int imax(int a, int b) { return a > b ? a : b; }

// ------------------------------------------------------------------ views

// limb k of a number stored at p[0..len) placed at offset `off`: p[k - off]
// inside the stored range, zero elsewhere.  off > 0 multiplies by B^off,
// off < 0 takes the whole shift by -off limbs (floor).
struct Span {
    const uint32_t *p;
    int off;
    int len;
    MP_DEV uint32_t operator()(int k) const
    {
        unsigned i = (unsigned)(k - off);
        return i < (unsigned)len ? p[i] : 0u;
    }
};

// B^e
struct PowB {
    int e;
    MP_DEV uint32_t operator()(int k) const { return k == e ? 1u : 0u; }
};

// dst[k] = src(k) for k in [0, n), zero for k in [n, clear)
template <int T, class FS>
MP_DEV void copy(uint32_t *dst, int n, int clear, const FS &src)
{
    sync();
    const int e = imax(n, clear);
    int k = (int)threadIdx.x;
    for (; k + 3 * T < e; k += 4 * T) {
        const uint32_t y0 = k < n ? src(k) : 0u, y1 = k + T < n ? src(k + T) : 0u;
        const uint32_t y2 = k + 2 * T < n ? src(k + 2 * T) : 0u, y3 = k + 3 * T < n ? src(k + 3 * T) : 0u;
        dst[k] = y0;
        dst[k + T] = y1;
        dst[k + 2 * T] = y2;
        dst[k + 3 * T] = y3;
    }
    for (; k < e; k += T) dst[k] = k < n ? src(k) : 0u;
}

// ------------------------------------------------------------- multiply

// Turns the 96-bit column sums lo/hi of strip s (first column K0; lane l
// holds columns K0 + 4l .. K0 + 4l + 3) into limbs: lane-local carry, the
// neighbour's carry by shuffle, then a carry-lookahead over the wave from
// ballots.  The limbs go to p, the carry leaving the strip to the strip slot s.
MP_DEV void strip_resolve(uint32_t *ctl, int s, int K0, const uint64_t (&lo)[4], const uint32_t (&hi)[4],
                          uint32_t *p, int ncols)
{
    const int l = lane();
    const int k0 = K0 + l * kRCol;
    // lane-local carry: z = column sums as limbs, c = carry into column k0+4
    uint32_t z[4];
    uint64_t c = 0;
#pragma unroll
    for (int r = 0; r < 4; r++) {
        const uint64_t t = lo[r] + c;
        const uint32_t kap = t < c ? 1u : 0u;
        z[r] = (uint32_t)t;
        c = ((uint64_t)(hi[r] + kap) << 32) | (t >> 32);
    }
    // add the carry of the lane below (< 2^46), leaving a 1-bit carry g
    const uint64_t cp = ((uint64_t)shfl_up1((uint32_t)(c >> 32)) << 32) | shfl_up1((uint32_t)c);
    uint64_t acc = (uint64_t)z[0] + (uint32_t)cp;
    z[0] = (uint32_t)acc;
    acc = (acc >> 32) + (cp >> 32) + z[1];
    z[1] = (uint32_t)acc;
    acc = (acc >> 32) + z[2];
    z[2] = (uint32_t)acc;
    acc = (acc >> 32) + z[3];
    z[3] = (uint32_t)acc;
    const bool g = (acc >> 32) != 0;
    const bool pr = (z[0] & z[1] & z[2] & z[3]) == 0xFFFFFFFFu;
    const uint64_t G = ballot(g), P = ballot(pr), X = G | P;
    const uint64_t sum = X + G;
    uint32_t ci = (uint32_t)(((sum ^ X ^ G) >> l) & 1u);
#pragma unroll
    for (int r = 0; r < 4; r++) {
        z[r] += ci;
        ci &= (z[r] == 0u) ? 1u : 0u;
    }
    if (k0 + 3 < ncols) {
        store4(p + k0, z[0], z[1], z[2], z[3]);
    } else {
#pragma unroll
        for (int r = 0; r < 4; r++)
            if (k0 + r < ncols) p[k0 + r] = z[r];
    }
    if (l == kLanes - 1) {
        const uint64_t e = c + (sum < X ? 1u : 0u);
        ctl[kCtlStrip + 2 * s] = (uint32_t)e;
        ctl[kCtlStrip + 2 * s + 1] = (uint32_t)(e >> 32);
    }
}


// p[0, na + nb) = a * b but for the carries between strips (in the strip slots;
// mul_valu_instance adds them).  `a` (na limbs, readable up to 3 limbs past its end)
// is the row operand, read with wave-uniform addresses; `bw` points at limb 0
// of the window operand (nb limbs) staged in LDS with kPad zero limbs on both
// sides, 16-byte aligned.  The shorter operand should be the rows: the waste of
// a strip is then only the triangles at the ramps.
//
// Column strips of kStrip columns are dealt to the waves; lane l of the wave
// owns kRCol consecutive columns and keeps their 96-bit sums in registers
// while it walks the rows in blocks of 4 (the load-balanced classical
// schedule of Sec. 3.3 becomes a row walk per strip: one window load and 16
// limb products per lane per block).  The strip's sums are turned into limbs
// in-wave (lane-local carry, neighbour carry by shuffle, lookahead by
// ballot).
template <int T>
MP_DEV void mul(uint32_t *ctl, uint32_t *p, const uint32_t *a, int na, const uint32_t *bw, int nb)
{
    constexpr int W = T / kLanes;
    sync();
    const int ncols = na + nb, nstrips = (ncols + kStrip - 1) / kStrip;
    const int w = wave_index(), l = lane();
    for (int s = w; s < nstrips; s += W) {
        const int K0 = s * kStrip, k0 = K0 + l * kRCol;
        const int ilo = imax(0, K0 - nb + 1) & ~3;
        const int ihi = imin(na, imin(K0 + kStrip, ncols));
        uint64_t lo[4] = {0, 0, 0, 0};
        uint32_t hi[4] = {0, 0, 0, 0};
        if (ilo < ihi) {
            // column k0+r, row i+t takes window limb k0 + r - i - t; per block
            // of rows i..i+3 the lane needs window limbs k0-i-3 .. k0-i+3
            const uint32_t *wp = bw + (k0 - ilo);
            const uint32_t *ap = a + ilo;
            int nblk = (ihi - ilo) >> 2;
            for (; nblk >= 2; nblk -= 2) {
                const Limb4 w0 = load4(wp), w1 = load4(wp - 4), w2 = load4(wp - 8);
                const uint32_t a0 = ap[0], a1 = ap[1], a2 = ap[2], a3 = ap[3];
                const uint32_t a4 = ap[4], a5 = ap[5], a6 = ap[6], a7 = ap[7];
                mac4(lo, hi, a0, w0.x, w0.y, w0.z, w0.w);
                mac4(lo, hi, a1, w1.w, w0.x, w0.y, w0.z);
                mac4(lo, hi, a2, w1.z, w1.w, w0.x, w0.y);
                mac4(lo, hi, a3, w1.y, w1.z, w1.w, w0.x);
                mac4(lo, hi, a4, w1.x, w1.y, w1.z, w1.w);
                mac4(lo, hi, a5, w2.w, w1.x, w1.y, w1.z);
                mac4(lo, hi, a6, w2.z, w2.w, w1.x, w1.y);
                mac4(lo, hi, a7, w2.y, w2.z, w2.w, w1.x);
                keep(w2.x);   // keeps the third window load one aligned 16-byte read
                wp -= 8;
                ap += 8;
            }
            const int rem = (ihi - ilo) - ((ihi - ilo) & ~7);   // rows left: 0..7
            if (rem > 0) {
                // last rows: those at or past ihi (<= na) read as zero
                const int i = ihi - rem;
                const Limb4 w0 = load4(wp), w1 = load4(wp - 4), w2 = load4(wp - 8);
                const uint32_t a0 = ap[0];
                const uint32_t a1 = i + 1 < ihi ? ap[1] : 0u, a2 = i + 2 < ihi ? ap[2] : 0u;
                const uint32_t a3 = i + 3 < ihi ? ap[3] : 0u, a4 = i + 4 < ihi ? ap[4] : 0u;
                const uint32_t a5 = i + 5 < ihi ? ap[5] : 0u, a6 = i + 6 < ihi ? ap[6] : 0u;
                mac4(lo, hi, a0, w0.x, w0.y, w0.z, w0.w);
                mac4(lo, hi, a1, w1.w, w0.x, w0.y, w0.z);
                mac4(lo, hi, a2, w1.z, w1.w, w0.x, w0.y);
                mac4(lo, hi, a3, w1.y, w1.z, w1.w, w0.x);
                if (rem > 4) {
                    mac4(lo, hi, a4, w1.x, w1.y, w1.z, w1.w);
                    mac4(lo, hi, a5, w2.w, w1.x, w1.y, w1.z);
                    mac4(lo, hi, a6, w2.z, w2.w, w1.x, w1.y);
                }
            }
        }
        strip_resolve(ctl, s, K0, lo, hi, p, ncols);
    }
}

}  // namespace mp
