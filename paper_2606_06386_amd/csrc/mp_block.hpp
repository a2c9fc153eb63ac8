// Block division: one workgroup divides u by v in blocks of quotient limbs.
//
// First W ~ B^(k+dp+2) / v is computed for a precision of dp <= 255 limbs (and
// two guard limbs) by Newton steps on one wave.  Then the quotient's d = h - k
// limbs are found in nb blocks from the top, block i holding the limbs
// [o_i, o_(i-1)):
//     q_i = floor(R_top W / B^(dp+3)),   R_top = floor(R / B^(o_i+k-1))
//     R  <- R - v q_i B^(o_i)
// with a signed remainder R that starts as u.  All products run on the int8
// matrix cores over balanced radix-256 digits; the digits of v and of W are
// made once per instance, those of R_top and of -q_i once per block, and R is
// added to the accumulators of the second product, so the subtraction costs
// no pass of its own.  After the last block r = R up to a few multiples of v.
//
// Against one full-precision inverse followed by u * shinv and v * q (Alg. 1
// and 3 as printed) this needs no Newton step beyond 257 limbs and fewer limb
// products (a 2048 by 1024-limb division: 1.08e6 instead of 1.78e6), and every
// operand converted to digits is at most one block long.
//
// Error bounds.  With W = B^(k+dp+2)/v - E and |E| <= 3 (see newton),
// |R| < 2.1 v B^(o_(i-1)) gives R_top W / B^(dp+3) = R / (v B^(o_i)) + e with
// |e| < 2^-20; the floor and the columns of R_top W below cA add at most one
// unit each, so q_i is within (-2, 1] of the real ratio: after the block
// -1.1 v B^(o_i) < R < 2.1 v B^(o_i).  R is therefore exact as a signed
// (k + 2)-limb number above o_i, q_i as a signed (limbs + 1)-limb number
// whose top limb is its sign, and at most two corrections each way remain.
#pragma once

#include "launch.hpp"
#include "mp_strip.hpp"

namespace mp {

enum : int32_t { kInstOk = 0, kInstDivZero = 1, kInstQWidth = 2, kInstInternal = 3 };

// The quotient's d limbs: nb blocks of bi limbs, the first (top) of
// d - (nb - 1) bi; dp limbs of precision of W serve the longest of them.  bi
// is a multiple of 4, so that every block starts at a 16-byte boundary of R;
// dp + 1 is a multiple of 8, so that the quotient product starts two columns
// below the quotient's limbs.
struct BlockSplit {
    int nb, bi, dp;
};

// Longest block: R_top (3 limbs more), the quotient's columns (3 more) and
// every Newton product then fit the 256 limbs of one strip, which one wave
// holds in registers, four limbs per lane, from the accumulators to the digits
// of the next product.
constexpr int kBlockMax = 252;

MP_HD constexpr int block_precision(int b) { return ((b + 8) & ~7) - 1; }

MP_HD BlockSplit block_split(int d, int bmax)
{
    if (d <= bmax) return BlockSplit{1, 0, block_precision(d)};
    const int nb = 1 + (d - 1) / bmax, even = r4((d + nb - 1) / nb), bi = even < bmax ? even : bmax;
    const int b0 = d - (nb - 1) * bi;
    return BlockSplit{nb, bi, block_precision(b0 > bi ? b0 : bi)};
}

// longest block for a limit on the iterates of the Newton steps (the small_limit knob)
MP_HD int block_limit(int limit) { return hmax(16, hmin(kBlockMax, (2 * limit - 16) & ~3)); }

// ---------------------------------------------------------------- LDS layout
//
// ctl | pad | V planes 0 .. 3 | T planes 0, 1 | W reversed | -q reversed | W | R
// (pads of zero half-blocks before the first plane and after each; T: R_top, and
// the residuals of the Newton steps).  R holds the dividend's h limbs and above
// them the quotient: limb j of q goes to R[k + 2 + j], which the remainder has
// left by the time the block is done.
struct BodyPlan {
    int nV, lyV, offV;        // limbs of the divisor's planes, distance of the planes, first word
    int offT;                 // T's two planes of 32 blocks
    int offX, offQ, offW, offR;   // W's reversed digits, -q's, W's limbs, R
    int capR;
    int total;
};

constexpr int kPad4 = kPadWords / 2;             // zero words a strip reads on each side of one of four planes
constexpr int kPlaneT = 4 * kStripBlks;          // words of T's planes
constexpr int kLyT = kPlaneT + kPadWords;        // distance of T's planes

// distance of V's planes of n words: a pad between them, and 16 modulo 32
MP_HD constexpr int plane_distance(int n) { return ((n + kPad4 + 15) & ~31) + 16; }

// behind the plan, Mode::kShared: partial sums of the quotient products, by the waves [1, kShares)
constexpr int kShares = 4, kPartWords = (kShares - 1) * 1024;

// a dividend of at most nu and a divisor of at most nv limbs (each one more
// inside, for divisors of one limb, which are shifted up by one)
MP_HD constexpr BodyPlan plan_body(int nu, int nv)
{
    BodyPlan p{};
    const int ny = (nv < nu ? nv : nu) + 2;            // digit limbs of the divisor
    const int dm = block_precision(hmin(kBlockMax, nu + 1));
    p.nV = (ny + 15) & ~15;
    p.offV = kCtlWords + kPad4;
    p.lyV = plane_distance(p.nV >> 2);
    p.offT = p.offV + 4 * p.lyV + kPadWords - kPad4;
    p.offX = r4(p.offT + 2 * kLyT + kXLow);
    p.offQ = r4(p.offX + dm + 4 + kXPad + kXLow);
    p.offW = p.offQ + 3 + dm + 1 + kXPad;
    p.offR = r4(p.offW + dm + 4);
    p.capR = r4(nu + 8);
    p.total = p.offR + p.capR;
    return p;
}

// the quad of limbs of each lane (see quad_limb) to T's planes, zeros from limb n on
MP_DEV void store_T(int l, uint32_t *td, const uint32_t (&z)[4], int n)
{
    const int g = quad_limb(l);
    store4(td + (l >> 5) * kLyT + 4 * (l & 31), g < n ? z[0] : 0u, g + 1 < n ? z[1] : 0u, g + 2 < n ? z[2] : 0u,
           g + 3 < n ? z[3] : 0u);
}

// R's quad of limbs at k0, its columns in [0, ncols)
MP_DEV Limb4 quad_in(const uint32_t *R, int ncols, int k0)
{
    return k0 >= 0 && k0 < ncols ? load4(R + k0) : Limb4{0u, 0u, 0u, 0u};
}

MP_DEV void quad_out(uint32_t *R, int ncols, int k0, const uint32_t (&z)[4])
{
    if (k0 < 0) return;
    if (k0 + 3 < ncols) {
        store4(R + k0, z[0], z[1], z[2], z[3]);
    } else {
#pragma unroll
        for (int j = 0; j < 4; j++)
            if (k0 + j < ncols) R[k0 + j] = z[j];
    }
}

// R[c] += column c of x * y for c in [0, ncols), mod B^ncols, but for the
// strips' carries: the carry of strip s goes to the control slots of s, and
// strip_carries adds it.  x has at most kBlockMax + 1 limbs, y at least ncols
// digit limbs, and the strips end at ncols (rounded up to 8 limbs), so that
// every strip but the lowest needs every diagonal of x: a wave takes two of
// these at a time (strip_sums2).  FAST, few strips: one each, which takes less
// time as long as there are waves and LDS reads do not bind (4096 by 1024 limbs,
// four strips on eight waves: 55 us, in pairs 61; four on four waves of up to
// four instances, 700 divisions of 2048 by 1024: 42 us, in pairs 39).  The
// lowest, partial strip comes last.  Shared quotient products: the first wave,
// which stores the quotient's limbs before, takes the last share.  R is 16-byte
// aligned.
template <int T, Mode M, class FX, class FY>
MP_DEV void strips(uint32_t *ctl, const FX &xs, const FY &ys, uint32_t *R, int ncols, int base, int nstrips)
{
    constexpr int W = T / kLanes;
    constexpr bool FAST = M != Mode::kPacked;
    const int w = wave_index(), n = nstrips - 1, b = base >> 3;
    const int step = FAST && n <= (T == 256 ? 2 : 4) ? 1 : 2, units = (n + step - 1) / step;
    for (int u = M == Mode::kShared ? (w ? w : W) - 1 : w; u <= units; u += W) {   // (unit `units`: the lowest strip)
        const int i = u < units ? 1 + u * step : 0, l = lane_at(u);
        const ShortDigits x = xs(l);
        const Planes4 y = ys(l);
        if (step == 2 && u < units && i < n) {
            MfmaAcc accE, accO;
            strip_sums2<FAST>(x, y, b + i * kStripBlks, accE, accO);
            const int k0 = base + i * kStrip + 16 * (l & 31) + 4 * (l >> 5);
            uint32_t zE[4], zO[4];
            const int e = strip_limbs2(l, accE, accO, [&](int odd) { return quad_in(R, ncols, k0 + 8 * odd); }, zE, zO);
            quad_out(R, ncols, k0, zE);
            quad_out(R, ncols, k0 + 8, zO);
            if (l < 2) ctl[kCtlStrip + i + l] = l ? (uint32_t)e : 0u;
        } else {
            const MfmaAcc acc = strip_sums<FAST>(x, y, b + i * kStripBlks);
            const int k0 = base + i * kStrip + quad_limb(l);
            uint32_t z[4];
            const int e = strip_limbs<true>(l, acc, quad_in(R, ncols, k0), z);
            quad_out(R, ncols, k0, z);
            if (l == 0) ctl[kCtlStrip + i] = (uint32_t)e;
        }
    }
}

// adds the strips' carries to dst (see strips), by one wave after a barrier:
// lane s adds the signed carry of strip s - 1 to the first two limbs of strip
// s; a carry or borrow out of those (rare) ripples on
MP_DEV void strip_carries(int s, const uint32_t *ctl, uint32_t *dst, int ncols, int base, int nstrips)
{
    const int cb = base + s * kStrip;
    const bool on = s >= 1 && s < nstrips, two = on && cb + 1 < ncols;
    const int e = on ? (int)ctl[kCtlStrip + s - 1] : 0;
    const uint64_t x = ((uint64_t)(two ? dst[cb + 1] : 0u) << 32) | (on ? dst[cb] : 0u), y = x + (uint64_t)(int64_t)e;
    if (on) dst[cb] = (uint32_t)y;
    if (two) dst[cb + 1] = (uint32_t)(y >> 32);
    uint64_t up = ballot(two && e > 0 && y < x), m = up | ballot(two && e < 0 && y > x);
    while (m) {
        const int t = __builtin_ctzll(m), c = base + t * kStrip + 2;
        m &= m - 1;
        if (c < ncols) ripple(s, dst + c, ncols - c, (up >> t) & 1u);
    }
    wave_sync();
}

// ---------------------------------------------------------------- division

// the limbs of a number shifted up by sv limbs
struct Shifted {
    const uint32_t *p;
    int n, sv;
    MP_DEV uint32_t operator()(int k) const
    {
        const unsigned i = (unsigned)(k - sv);
        return i < (unsigned)n ? p[i] : 0u;
    }
};

// limb n - 64 + l of x (zero below its first): most numbers fill their row
MP_DEV uint32_t top_limb(int l, const uint32_t *x, int n) { return n - kLanes + l >= 0 ? x[n - kLanes + l] : 0u; }

// Number of significant limbs of x[0, n) (global memory), the same in all waves:
// by every wave from its top_limb, or else by all of them together, 8 limbs per
// thread and step (one wave by itself took eight steps of 5000 cycles for 8192
// limbs).  slot: two words per wave.
template <int T>
MP_DEV int precision(int l, int w, const uint32_t *x, int n, uint32_t top, uint32_t *slot)
{
    constexpr int W = T / kLanes, R = 8;
    const uint64_t m = ballot(top != 0u);
    if (m) return n - __builtin_clzll(m);
    for (int s = (n - 1) / (R * T); s >= 0; s--) {
        const int r0 = (s * W + w) * R;
        uint32_t v[R];
#pragma unroll
        for (int j = 0; j < R; j++) {
            const int i = (r0 + j) * kLanes + l;
            v[j] = i < n ? x[i] : 0u;
        }
        int found = 0;
#pragma unroll
        for (int j = 0; j < R; j++) {
            const uint64_t mj = ballot(v[j] != 0u);
            if (mj) found = (r0 + j + 1) * kLanes - __builtin_clzll(mj);
        }
        uint32_t *sl = slot + (s & 1) * W;       // (the step before may still be read)
        if (l == 0) sl[w] = (uint32_t)found;
        sync();
        const uint32_t f = l < W ? sl[l] : 0u;
        const uint64_t mf = ballot(f != 0u);
        if (mf) return (int)readlane(f, 63 - __builtin_clzll(mf));
    }
    return 0;
}

// whether x[0, n) is zero, by one wave, 1024 limbs at a time
MP_DEV bool all_zero(int l, const uint32_t *x, int n)
{
    for (int b = n; b > 0; b -= 16 * kLanes) {
        uint32_t any = 0;
#pragma unroll
        for (int j = 0; j < 16; j++) {
            const int i = b - (j + 1) * kLanes + l;
            any |= i >= 0 ? x[i] : 0u;
        }
        if (ballot(any != 0u)) return false;
    }
    return true;
}

// x >= y for numbers of n limbs, by one wave, 64 limbs at a time from the top
template <class FX, class FY>
MP_DEV bool not_less(int l, int n, const FX &x, const FY &y)
{
    for (int c = n - 1; c >= 0; c -= kLanes) {
        const int j = c - (kLanes - 1) + l;
        const uint32_t a = j >= 0 ? x(j) : 0u, b = j >= 0 ? y(j) : 0u;
        const uint64_t ne = ballot(a != b), gt = ballot(a > b);
        if (ne) return (gt >> (63 - __builtin_clzll(ne))) & 1u;
    }
    return true;
}

constexpr int kStartLimbs = 46;   // longest iterate of newton_start

// limbs a Newton step to f limbs starts from: the first step's are exact to one
// unit, so it needs one limb less (see newton)
MP_HD int newton_from(int f) { return (f + (f <= 2 * kStartLimbs - 2 ? 3 : 4)) >> 1; }

// limbs of the iterate the Newton steps to F limbs start from
MP_HD int start_limbs(int F)
{
    while (F > kStartLimbs) F = newton_from(F);
    return F;
}

// lane j >= 1: bits [24 (j - 1), 24 j) below the leading bit of v, which is lz
// bits below the top of limb k (lane 0: 0)
template <class FV>
MP_DEV uint32_t start_digits(int l, const FV &v, int k, int lz)
{
    const int p = 32 * (k + 1) - lz - 24 * l, i = p >> 5;
    const uint32_t lo = i >= 0 ? v(i) : 0u, hi = i >= -1 ? v(i + 1) : 0u;
    return l ? alignbit(hi, lo, (uint32_t)p & 31u) & 0xFFFFFFu : 0u;
}

// w[0, f] = floor(B^(k+f) / v) or one less, 4 <= f <= kStartLimbs, by one wave
// from the start_digits V of v: a division of 2^(e-48) by v' = v / 2^(32(k+1)-lz)
// in signed digits of 48 bits.  Lane j holds weight 2^(-24j): the remainder r in
// signed 25-bit parts a, and v' shifted down to the next digit's place (the
// upper and the lower half of the digit: vA, vB).  A step takes the digit from
// the leading lanes of r (as an integer modulo 2^64, which drops the lanes
// above: they cancel) times 1 / v' in double precision, to within 2^-2 of r/v':
// |r| stays below 0.8 v' 2^(-48 t).  It costs about 270 cycles, nearly all of
// it one dependent chain through scalar and vector units; a Newton step on the matrix core
// costs 4700 to 5600 however short its operands (its LDS round trips and carry
// passes), so 25 steps here (37 limbs) beat the five Newton steps from the 112
// bits of one reciprocal.  (46 limbs are what 63 lanes of 24 bits leave exact to
// one unit.)  scratch: 64 words.
MP_DEV void newton_start(int l, uint32_t V, int lz, int f, uint32_t *scratch, uint32_t *w)
{
    constexpr double kRound = 0x1.8p52;          // (adding it leaves the integer in the low mantissa bits)
    const int e = 39 + ((lz + 1) & 7);           // (the result ends at a byte)
    const int n = (32 * (f - 1) + lz - e + 8 + 47) / 48 + 1, x = 48 * (n - 1) + e - 32 * (f - 1) - lz;
    const double d = (double)(int)readlane(V, 1) * 0x1p-24 + (double)(int)readlane(V, 2) * 0x1p-48 +
                     (double)(int)readlane(V, 3) * 0x1p-72;
    double r = __builtin_amdgcn_rcp(d);
    r = __builtin_fma(r, __builtin_fma(-d, r, 1.0), r);
    r = __builtin_fma(r, __builtin_fma(-d, r, 1.0), r);
    constexpr int kHalf = 1 << 23;
    int vA = -(int)shfl_up1(V), vB = (int)shfl_up1((uint32_t)vA);
    int a = (l == 1 ? 1 << (e - 24) : 0) + kHalf, digit = 0;   // (a: the part plus kHalf)
    for (int t = 0; t < n; t++) {
        const int a0 = (int)readlane((uint32_t)a, 2 * t), a1 = (int)readlane((uint32_t)a, 2 * t + 1),
                  a2 = (int)readlane((uint32_t)a, 2 * t + 2), a3 = (int)readlane((uint32_t)a, 2 * t + 3) - kHalf;
        // (as a double: the bits of kRound, less the three kHalf)
        const int64_t S = (int64_t)((uint64_t)(int64_t)a0 << 48) + ((int64_t)a1 * (1 << 24) + a2);
        const int64_t bits = 0x4338000000000000ll - (int64_t)((uint64_t)kHalf * ((1ull << 48) + (1ull << 24) + 1)) + S;
        const double rem = __builtin_fma((double)a3, 0x1p-24, __builtin_bit_cast(double, bits) - kRound);
        const uint64_t b = __builtin_bit_cast(uint64_t, __builtin_fma(rem, r, kRound + kHalf));
        // the digit's halves, the lower one in [-2^23, 2^23)
        const int ql = (int)((uint32_t)b & 0xFFFFFFu) - kHalf;
        const int qh = (int)(alignbit((uint32_t)(b >> 32), (uint32_t)b, 24) << 5) >> 5;
        const int64_t P = (int64_t)qh * vA + (a + (int64_t)ql * vB);
        a = (int)((uint32_t)P & 0xFFFFFFu) + (int)shfl_down1(alignbit((uint32_t)((uint64_t)P >> 32), (uint32_t)P, 24));
        digit = l == 2 * t + 1 ? qh : l == 2 * t + 2 ? ql : digit;
        vA = (int)shfl_up1((uint32_t)vB);
        vB = (int)shfl_up1((uint32_t)vA);
    }
    // the borrows of the digits (lane 1 the highest), their bytes, and the limbs
    const uint64_t G = __builtin_bitreverse64(ballot(digit < 0)), X = G | __builtin_bitreverse64(ballot(digit == 0));
    const uint32_t z = (uint32_t)digit - (inverse_ballot(__builtin_bitreverse64((X + G) ^ X ^ G)) ? 1u : 0u);
    scratch[l] = 0u;
    wave_sync();
    if (l >= 1 && l <= 2 * n) {
        uint8_t *at = reinterpret_cast<uint8_t *>(scratch) + 3 * (2 * n - l);
        at[0] = (uint8_t)z;
        at[1] = (uint8_t)(z >> 8);
        at[2] = (uint8_t)(z >> 16);
    }
    wave_sync();
    if (l <= f) {
        const int o = (x >> 3) + 4 * l;
        w[l] = alignbyte(scratch[(o >> 2) + 1], scratch[o >> 2], (uint32_t)o & 3u);
    }
    wave_sync();
}

// W ~ B^(k+F) / v, F = dp + 2, by one wave: w[0, F] its limbs, xw the reversed
// digits of its F + 2 digit limbs (all words from xw - kXLow to their upper pad
// are zero before).  vd: the planes (distance lv) of v's digits, td: T's planes
// (their pads zero).  w holds newton_start's start_limbs(F) limbs below its top.
//
// The iterate for f limbs is w ~ B^(k+f)/v, the top of the final one: w[F - f,
// F].  A step to f' <= 2f - 3 limbs takes the middle columns of v w as the
// residual e = (v w - B^(k+f)) / B^c and adds -w e: both products fill one
// 256-column strip, and both results go from the accumulators to the digits of
// the next product in registers.  With |E| the error of w in units of its last
// limb, the new one is at most E^2 / B (quadratic term; E^2 in the first step,
// to 2f - 2 limbs, where newton_start's |E| is 1) + 1 (floor) + 0.1:
// limbs of v below s are left out (but for those the strip reads anyway), s <=
// k - 1 - f', which moves e by less than B^f, and columns of e below c = sh - f
// - 2, of either sign and below 2^26 B^c.  So |E| <= 3 at the end.
//
// The correction ends in the old iterate's last limb, which the second product
// takes as an addend.  As long as that limb neither overflows (it moves by a
// few units) nor passes another balancing carry up than before, the digits
// above it stay as they are and only the new limbs' are written; otherwise all
// digits are made again from the limbs.
template <bool FAST>
MP_DEV void newton(int k, int dp, const uint32_t *vd, int lv, uint32_t *td, uint32_t *w,
                   uint32_t *xw)
{
    const int F = dp + 2, l = lane_at(k), g = quad_limb(l);
    const Limb4 none{0u, 0u, 0u, 0u};
    int f = start_limbs(F);
    bool again = true;                           // the digits are to be made from the limbs
    for (;;) {
        wave_sync();
        if (again) balance_rows(l, 0, (f + 65) >> 6, f + 1, 0u, Span{w + F - f, 0, f + 1}, StoreRev{xw, f + 2});
        if (f == F) break;
        const uint32_t last = uniform(w[F - f]);
        int fn = F;                              // the next step of the schedule that ends at F
        while (newton_from(fn) > f) fn = newton_from(fn);
        const int s = imax(0, k - 1 - fn) & ~15;
        const int sh = k - s + 2 * f - fn;       // w e / B^sh is the correction
        const int c0 = imax(0, sh - f - 2) & ~7, nx = k + 2 - s - c0;
        wave_sync();
        // -e: the two's complement of the columns [c0, c0 + nx) of v w (B^(k+f-s) lies above them), as digits
        uint32_t z[4];
        strip_limbs<false>(l, strip_sums<FAST>(short_digits(l, xw, f + 2), planes4(l, vd + (s >> 2), lv, k + 2 - s), c0 >> 3), none, z);
#pragma unroll
        for (int j = 0; j < 4; j++) z[j] = g + j < nx ? ~z[j] : 0u;
        quad_balance(z, 1u);
        store_T(l, td, z, nx);
        wave_sync();
        // the new limbs: columns [shc, shc + m) of w (-e), and the old last limb at column shc + m
        const int shc = sh - c0, cB = (shc - 2) & ~7, m = fn - f, i0 = cB + g - shc, at = shc + m - cB;
        Limb4 add{i0 == m ? last : 0u, i0 + 1 == m ? last : 0u, i0 + 2 == m ? last : 0u, i0 + 3 == m ? last : 0u};
        strip_limbs<true>(l, strip_sums<FAST>(short_digits(l, xw, f + 2), planes(l, td, kLyT, nx), cB >> 3), add, z);
        const int over = (int)quad_get(z, at + 1);
        const uint32_t nl = quad_get(z, at);                 // the old last limb, moved
#pragma unroll
        for (int j = 0; j < 4; j++) {
            const bool in = (unsigned)(i0 + j) <= (unsigned)m;
            if (in) w[F - fn + i0 + j] = z[j];
            z[j] = in ? z[j] : 0u;
        }
        const bool odd = quad_balance(z, 0u);                // (a limb that passes its carry on: look at all)
        again = odd || over != 0 || (nl > kBalTop) != (last > kBalTop);
        if (again) {
            add_small(l, w + F - f + 1, f, over);
        } else {
#pragma unroll
            for (int j = 0; j < 4; j++)
                if ((unsigned)(i0 + j) <= (unsigned)m) xw[fn + 1 - i0 - j] = bswap(z[j]);
        }
        f = fn;
    }
}

// the digits of R_top, nt limbs at src, to T's planes td
MP_DEV void top_digits(int l, const uint32_t *src, int nt, uint32_t *td)
{
    const int g = quad_limb(l);
    uint32_t z[4];
#pragma unroll
    for (int j = 0; j < 4; j++) z[j] = g + j < nt ? src[g + j] : 0u;
    quad_balance(z, 0u);
    store_T(l, td, z, nt);
}

// word of the 16-byte aligned place of -q's digits where those of a block of b limbs start: a lane's quad ends there on an aligned word
MP_DEV int quotient_at(int b) { return (1 - b) & 3; }

// the reversed digits of -q_i to xq + quotient_at(b); q: limbs of R_top W /
// B^(dp+1), limb 2 + j is limb j of q_i, 2 + b its sign
MP_DEV void quotient_digits(int l, const uint32_t (&q)[4], int b, uint32_t *xq)
{
    const int g = quad_limb(l) - 2, at = quotient_at(b);
    uint32_t z[4];
#pragma unroll
    for (int j = 0; j < 4; j++) z[j] = g + j < 0 ? 0xFFFFFFFFu : ~q[j];   // (the two columns below pass the +1 on)
    quad_balance(z, 1u);
    if (g <= b) {                                 // (digits below limb 0 are zero)
        store4(xq + at + b - g - 3, g + 3 <= b ? bswap(z[3]) : 0u, g + 2 <= b ? bswap(z[2]) : 0u,
               g + 1 <= b ? bswap(z[1]) : 0u, bswap(z[0]));
    }
    if (l < kXPad - 2) xq[at + b + 3 + l] = 0u;
}

// the b limbs of q_i (see quotient_digits) to the quotient's limbs Q
MP_DEV void quotient_limbs(int l, uint32_t *Q, const uint32_t (&q)[4], int b)
{
    const int g = quad_limb(l) - 2;
#pragma unroll
    for (int j = 0; j < 4; j++)
        if ((unsigned)(g + j) < (unsigned)b) Q[g + j] = q[j];
}

// its sign to the n limbs above them (or, for the first block, one more limb)
MP_DEV void quotient_sign(int l, uint32_t *Q, int sign, int n)
{
    if (n == 0) {
        if (l == 0) Q[0] = (uint32_t)sign;
    } else {
        add_small(l, Q, n + 1, sign);
    }
}

// limbs of a dividend: an array, or B^e
MP_DEV uint32_t top_limb(int l, const Span &u, int n) { return top_limb(l, u.p, n); }
MP_DEV uint32_t top_limb(int, const PowB &, int) { return 0u; }
template <int T>
MP_DEV int precision(int l, int w, const Span &u, int n, uint32_t top, uint32_t *slot)
{
    return precision<T>(l, w, u.p, n, top, slot);
}
template <int T>
MP_DEV int precision(int, int, const PowB &u, int, uint32_t, uint32_t *)
{
    return u.e + 1;
}

// Whether a comparison shows the quotient to be 0 or 1: u has h limbs, d - 1 more
// than v, whose top limb k is vk (v is not B^k).
MP_DEV bool quotient_below_two(int l, const Span &u, int h, int d, uint32_t vk, const uint32_t *v, int)
{
    return d == 1 && (vk >> 31 || !not_less(l, h, u, Span{v, 0, h}));   // (vk >= 2^31: u < B^h <= 2v)
}

// (B^e of v's length is less than v, of one limb more than 2v if v > B^e / 2)
MP_DEV bool quotient_below_two(int l, const PowB &, int, int d, uint32_t vk, const uint32_t *v, int k)
{
    return d == 1 || (d == 2 && (vk > 0x80000000u || (vk == 0x80000000u && !all_zero(l, v, k))));
}

// The n <= 3 limbs of U by the limb v: the quotient's limbs to a, the remainder
// returned.  The digits are chosen in double precision, a relative 2^-40 low (at
// most 2^-8 of a unit), so they are exact or one too small.
template <class FU>
MP_DEV uint32_t short_division(const FU &U, int n, uint32_t v, uint32_t (&a)[3])
{
    const double d = (double)v;
    double r = __builtin_amdgcn_rcp(d);
    r = __builtin_fma(r, __builtin_fma(-d, r, 1.0), r);
    r = __builtin_fma(r, __builtin_fma(-d, r, 1.0), r);
    r -= r * 0x1p-40;
    uint32_t rem = 0;
#pragma unroll 1
    for (int i = n - 1; i >= 0; i--) {
        const uint64_t x = (uint64_t)rem << 32 | U(i);
        const uint32_t q = (uint32_t)((double)x * r);
        const uint64_t m = x - (uint64_t)q * v;
        a[2] = a[1];
        a[1] = a[0];
        a[0] = q + (m >= v ? 1u : 0u);
        rem = (uint32_t)(m >= v ? m - v : m);
    }
    return rem;
}

// Divisions that need no inverse, by all waves: of up to three limbs by one (k =
// 0), and those of quotient_below_two.  A call, made once nothing else is
// live: inlined, its registers pass the 64 of the packed kernels (one spilled,
// random divisor lengths 1 to 2% slower).
template <int T, class FU>
__device__ __attribute__((noinline)) void divide_without_inverse(FU U, int h, int k, uint32_t vk, const uint32_t *v,
                                                                 uint32_t *q, int nq, uint32_t *r, int nr,
                                                                 int32_t *status)
{
    constexpr int W = T / kLanes;
    const int l = lane(), w = wave_index(), t = w * kLanes + l;
    bool ok = true;
    if (k == 0) {
        uint32_t a[3] = {0u, 0u, 0u};
        const uint32_t rem = short_division(U, h, vk, a);
        ok = (nq > 2 || a[2] == 0u) && (nq > 1 || a[1] == 0u);
        for (int i = t; i < nq; i += T) q[i] = !ok ? 0u : i == 0 ? a[0] : i == 1 ? a[1] : i == 2 ? a[2] : 0u;
        for (int i = t; i < nr; i += T) r[i] = ok && i == 0 ? rem : 0u;
    } else {
        const bool one = not_less(l, h, U, Span{v, 0, k + 1});
        for (int i = t; i < nq; i += T) q[i] = one && i == 0 ? 1u : 0u;
        if (nr) {                                     // r = u - q v, both of k + 1 limbs
            const int rows = (k + 64) >> 6, per = (rows + W - 1) / W, r0 = w * per, r1 = imin(rows, r0 + per);
            if (r0 < r1) addsub_rows(l, r0, r1, k + 1, true, U, Span{v, 0, one ? k + 1 : 0}, r);
            for (int i = k + 1 + t; i < nr; i += T) r[i] = 0u;
        }
    }
    if (status && t == 0) *status = ok ? kInstOk : kInstQWidth;
}

// (q, r) with u = q v + r, 0 <= r < v: q has nq limbs, r (unless null) nv.
// U(i) is limb i of the dividend, which has at most nu limbs; bmax: longest
// block.
template <int T, Mode M, class FU>
MP_DEV void divide_instance(uint32_t *lds, const FU &U, int nu, const uint32_t *v, int nv, uint32_t *q, int nq,
                            uint32_t *r, int32_t *status, int bmax)
{
    constexpr int W = T / kLanes;
    constexpr bool FAST = M != Mode::kPacked, SHARED = M == Mode::kShared;
    uint32_t *ctl = lds;
    const BodyPlan pl = plan_body(nu, nv);
    uint32_t *Vd = lds + pl.offV, *Td = lds + pl.offT, *XW = lds + pl.offX, *XQ = lds + pl.offQ;
    uint32_t *R = lds + pl.offR, *part = lds + r4(pl.total);
    const int w = wave_index(), l0 = lane_at(nu), t = w * kLanes + l0, nr = r ? nv : 0;
    MP_RSTAMP(14);
    MP_STAMP(0);
    // precisions, and the cases that need no division
    const uint32_t tu = top_limb(l0, U, nu), tv = top_limb(l0, v, nv);
    int h = precision<T>(l0, w, U, nu, tu, ctl + kCtlPrec), k = precision<T>(l0, w, v, nv, tv, ctl + kCtlPrec + 2 * W) - 1;
    if (k < 0 || h <= k) {                            // v = 0, or u < v: (0, u)
        for (int i = t; i < nq; i += T) q[i] = 0u;
        for (int i = t; i < nr; i += T) r[i] = k >= 0 && i < h ? U(i) : 0u;
        if (status && t == 0) *status = k < 0 ? kInstDivZero : kInstOk;
        return;
    }
    const int d = h - k;
    const uint32_t vk = k >= nv - kLanes ? readlane(tv, k - nv + kLanes) : uniform(v[k]);
    if (vk == 1u && all_zero(l0, v, k)) {   // v = B^k: q = u >> k, r the limbs below
        const bool ok = d <= nq;                         // (limb h - 1 is not zero)
        for (int i = t; i < nq; i += T) q[i] = ok && i < d ? U(i + k) : 0u;
        for (int i = t; i < nr; i += T) r[i] = ok && i < k ? U(i) : 0u;
        if (status && t == 0) *status = ok ? kInstOk : kInstQWidth;
        return;
    }
    if (d - 1 > nq) {                                 // q >= B^(d-2): it needs more than nq limbs
        for (int i = t; i < nq; i += T) q[i] = 0u;
        for (int i = t; i < nr; i += T) r[i] = 0u;
        if (status && t == 0) *status = kInstQWidth;
        return;
    }
    // Without the inverse they take (us; with it): 4096 of 64 by 64 limbs and a
    // quotient of 0 or 1 6.8 (19.8), of 1 by 1 limb 5.7 (18.7), 4096 inverses of B^7
    // by 8 limbs 5.4 (17.9), any one of these 4.4 (6.6).
    if (__builtin_expect(d <= 3, 0) && (k == 0 || quotient_below_two(l0, U, h, d, vk, v, k))) {
        divide_without_inverse<T>(U, h, k, vk, v, q, nq, r, nr, status);
        return;
    }
    const int sv = k == 0 ? 1 : 0;                    // a one-limb divisor: u B / (v B)
    h += sv;
    k += sv;
    const Shifted Vv{v, nv, sv};
    const BlockSplit bs = block_split(d, bmax);
    const int dp = bs.dp, nb = bs.nb, bi = bs.bi;
    MP_STAMP(1);
    // The first wave: the start of the inverse; the others: the divisor's digits
    // and the zero pads.  What the first wave does by itself, here and in the
    // blocks, goes before other instances' work on its SIMD, since three waves
    // wait for it: 4096 divisions of 2048 by 1024 limbs take 124 -> 119 us, 1024
    // inverses 41 -> 39.
    if (w == 0) {
        wave_priority<3>();
        const int l = lane_at(k), lz = __builtin_clz(vk);
        const int f = start_limbs(dp + 2);
        newton_start(l, start_digits(l, Vv, k, lz), lz, f, Td, lds + pl.offW + dp + 2 - f);
    } else {
        const int t1 = t - kLanes;
        const int nw = pl.nV >> 2;                    // words of V's planes
        for (int i = t1; i < pl.lyV - nw; i += T - kLanes) {
            if (i < kPad4) lds[pl.offV - kPad4 + i] = 0u;
#pragma unroll
            for (int p = 0; p < 4; p++) Vd[p * pl.lyV + nw + i] = 0u;
        }
        for (int i = t1; i < kPadWords; i += T - kLanes) Td[i - kPadWords] = Td[i + kPlaneT] = Td[i + kLyT + kPlaneT] = 0u;
        for (int i = pl.offX - kXLow + t1; i < pl.offW; i += T - kLanes) lds[i] = 0u;
        const int rows = (pl.nV + 63) >> 6, per = (rows + W - 2) / (W - 1);
        const int r0 = (w - 1) * per, r1 = imin(rows, r0 + per);
        if (r0 < r1) balance_rows(l0, r0, r1, k + 1, 0u, Vv, StorePlane4{Vd, pl.nV, pl.lyV});
    }
    sync();
    MP_STAMP(9);
    // W by the first wave, while the others read the dividend (zeros above it)
    if (w == 0) {
        newton<FAST>(k, dp, Vd, pl.lyV, Td, lds + pl.offW, XW);
    } else {
        constexpr int S = T - kLanes;
        for (int i0 = t - kLanes; i0 < pl.capR; i0 += 8 * S) {
            uint32_t a[8];
#pragma unroll
            for (int j = 0; j < 8; j++) {
                const int i = i0 + j * S - sv;
                a[j] = i >= 0 && i < nu ? U(i) : 0u;
            }
#pragma unroll
            for (int j = 0; j < 8; j++)
                if (i0 + j * S < pl.capR) R[i0 + j * S] = a[j];
        }
    }
    sync();
    MP_STAMP(2);
    bool good = true;
    const int n2 = k + 2, bs2 = (n2 + kStrip - 1) / kStrip, base2 = ((n2 + 7) & ~7) - bs2 * kStrip;
    const Limb4 none{0u, 0u, 0u, 0u};
    // the lanes' addresses of the products' operands, where registers allow
    const int lf = lane_at(nb);
    const ShortDigits xw0 = short_digits(lf, XW, dp + 4), xq0 = short_digits(lf, XQ, 0);
    const Planes4 yv0 = planes4(lf, Vd, pl.lyV, n2);
    Planes yt0 = planes(lf, Td, kLyT, 0);
    int o = d;
    for (int i = 0; i < nb; i++) {
        const int op = o;
        o = (nb - 1 - i) * bi;
        const int b = op - o, nt = b + 3;             // limbs of this block, of R_top
        const int l = lane_at(i);
        uint32_t q[4];                                // (the first wave's) q_i
        const int cq = (dp + 1) >> 3;                 // block of the product's first column
        // R_top is read before the strips' carries are added, which the last wave
        // does during the product, if those lie below R_top (the top strip starts
        // three limbs below it): but for a ripple of one unit into R_top's
        // lowest limb, which the quotient's error bound has room for.  The limbs
        // from k + 2 + o on are R_top's by then, and the quotient's next.
        const bool late = bs2 == 1 || b + ((n2 + 7) & ~7) <= k + 253;
        if (w == 0) {
            if (i && !late) strip_carries(l, ctl, R + op, n2, base2, bs2);
            top_digits(l, R + o + k - 1, nt, Td);
            MP_STAMP(16 + 3 * (i % 5));   // (trace build: the phases of the last five blocks)
        }
        sync();
        const bool carries = w == W - 1 && i && late;
        if constexpr (SHARED) {
            MfmaAcc acc;
            if (w < kShares) {
                yt0.ny = nt;
                acc = strip_sums<FAST>(xw0, yt0, cq, w, kShares);
                if (w) acc_store(l, acc, part + (w - 1) * 1024);
            }
            sync();
            if (w == 0) {
#pragma unroll
                for (int j = 0; j < kShares - 1; j++) acc_add(l, acc, part + j * 1024);
                strip_limbs<false>(l, acc, none, q);
                quotient_digits(l, q, b, XQ);
            } else if (carries) {
                strip_carries(l, ctl, R + op, n2 - b, base2, bs2);
            }
        } else if (carries) {
            strip_carries(l, ctl, R + op, n2 - b, base2, bs2);
        } else if (w == 0) {
            if constexpr (FAST) {
                yt0.ny = nt;
                strip_limbs<false>(l, strip_sums<FAST>(xw0, yt0, cq), none, q);
            } else {
                strip_limbs<false>(
                    l, strip_sums<FAST>(short_digits(l, XW, dp + 4), planes(l, Td, kLyT, nt), cq), none, q);
            }
            uint32_t *Q = R + k + 2 + o;
            const int sign = (int)quad_get(q, b + 2);
            quotient_limbs(l, Q, q, b);
            quotient_digits(l, q, b, XQ);
            quotient_sign(l, Q + b, sign, d - op);
        }
        sync();
        MP_STAMP(17 + 3 * (i % 5));
        if (SHARED && w == 0) {
            uint32_t *Q = R + k + 2 + o;
            quotient_limbs(l, Q, q, b);
            quotient_sign(l, Q + b, (int)quad_get(q, b + 2), d - op);
        }
        // R -= v q_i
        if (w == 0) wave_priority<0>();
        strips<T, M>(
            ctl, [&](int lu) {
                return FAST ? short_digits(xq0, quotient_at(b), b + 1)
                            : short_digits(lu, XQ + quotient_at(b), b + 1);
            },
            [&](int lu) { return FAST ? yv0 : planes4(lu, Vd, pl.lyV, n2); }, R + o, n2, base2, bs2);
        if (w == 0) wave_priority<3>();
        sync();
        MP_STAMP(18 + 3 * (i % 5));
    }
    if (w == 0) {
        strip_carries(lane_at(nb), ctl, R, n2, base2, bs2);
        wave_priority<0>();
    }
    sync();
    MP_STAMP(6);
    // corrections: R is a signed (k + 2)-limb number in (-1.1 v, 2.1 v)
    uint32_t *Q = R + k + 2, *Ra = R, *Rb = Vd;       // (the divisor's digits are no longer needed)
    int delta = 0;
    for (int it = 0; good; it++) {
        bool neg = (int32_t)uniform(Ra[k + 1]) < 0, ge = uniform(Ra[k + 1]) != 0u;
        if (!ge) ge = not_less(lane_at(it), k + 1, [&](int j) { return Ra[j]; }, Vv);   // (equal: R = v)
        if (!neg && !ge) break;
        if (it == 4) {
            good = false;
            break;
        }
        const int rows = (n2 + 63) >> 6, per = (rows + W - 1) / W;
        const int r0 = w * per, r1 = imin(rows, r0 + per);
        if (r0 < r1) addsub_rows(lane_at(it), r0, r1, n2, !neg, Span{Ra, 0, n2}, Vv, Rb);
        delta += neg ? -1 : 1;
        sync();
        uint32_t *x = Ra;
        Ra = Rb;
        Rb = x;
    }
    if (good && delta) {
        if (w == 0) add_small(lane_at(delta), Q, d + 1, delta);
        sync();
    }
    MP_STAMP(7);
    int32_t st = good ? kInstOk : kInstInternal;
    if (good && uniform(Q[d]) != 0u) st = kInstInternal;
    if (st == kInstOk && d > nq) {                    // (d <= nq + 1)
        if (uniform(Q[d - 1]) != 0u) st = kInstQWidth;
    }
    const bool ok = st == kInstOk;
    const int te = w * kLanes + lane_at(st);
    for (int i = te; i < nq; i += T) q[i] = ok && i < d ? Q[i] : 0u;
    for (int i = te; i < nr; i += T) r[i] = ok && i <= k - sv ? Ra[i + sv] : 0u;
    if (status && te == 0) *status = st;
    MP_STAMP(8);
    MP_RSTAMP(15);
}

}  // namespace mp
