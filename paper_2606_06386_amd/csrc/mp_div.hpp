// One multi-precision product, shifted inverse or division per workgroup.
//
// The division is the paper's shifted-inverse method:
//   Alg. 1 (Shinv): special cases, 2-limb initial approximation
//                   w = floor(B^3 / (v_{k-1} + v_k B)), then Refine: Newton
//                   steps with shorter iterates (l doubling) and divisor
//                   prefixes (v >> s limbs), 2 guard limbs.
//   Alg. 1 (Step):  w' = shift_m(w) +- shift_{2m-H}(w * x), the negative
//                   branch rounded toward -infinity.
//   Alg. 2 (PowDiff): (sign, |B^h - v w|) from the full product, or from the
//                   low L limbs of v w (the close product).
//   Alg. 3 (Div):   q = shift_{-h}(u * shinv_h(v)), m = v q, then quotient
//                   corrections.
// All numbers are little-endian base B = 2^32 limbs; h, k, l, m, s, g count
// limbs.  Readings taken where the printed algorithms are silent or garbled:
//   * the Refine loop runs 2 + ceil(log2(h-k-1)) times, 2 times when
//     h-k-1 <= 1;
//   * Step's rounding test looks at the h-2m (not 2m-h) low limbs of w*x;
//   * PowDiff's sign is 1 iff B^h - v*w >= 0;
//   * the computed inverse can be floor(B^h/v) - 1 as well as + 1, and the
//     clipped products below move it by at most one more unit either way, so
//     the division corrects q0 by up to four subtractions and five additions
//     of v (q - 4 <= q0 <= q + 3 is what the bound allows; one more step
//     each way is a safety margin that reports INTERNAL instead of a wrong
//     answer), and the stand-alone shinv ends with an exact fix-up.
//
// Two kernels share the work of one instance.  The head (one wave per
// instance, many instances per compute unit) computes the initial
// approximation and the early Refine iterations, whose operands are short;
// it leaves their state in a record at the start of the instance's own output
// row (q for a division, w for a shifted inverse).  The body (one workgroup
// per instance) picks the record up and runs the remaining iterations and
// the quotient and remainder products.  Without a record the body runs every
// step itself.
#pragma once

#include <stdint.h>

#include "launch.hpp"

namespace mp {

enum : int32_t { kInstOk = 0, kInstDivZero = 1, kInstQWidth = 2, kInstInternal = 3 };

#define MP_HD __host__ __device__ __forceinline__

MP_HD constexpr int r4(int x) { return (x + 3) & ~3; }
MP_HD constexpr int hmax(int a, int b) { return a > b ? a : b; }

MP_HD constexpr int hmin(int a, int b) { return a < b ? a : b; }

// LDS layout of a head's wave (32-bit words)
struct Plan {
    int capV, capW, capX, capR, capSB, capP;
    int offV, offW, offX, offR, offSB, offP;   // offR: word 0 of the reversed digits, offSB: limb 0 of the window
    int vbase;                                 // index of the divisor limb stored at offV (limbs below are not held)
    int capY;          // longest operand whose matrix-core digit planes (with their zero pads) fit the window area
    int sbLo, sbHi;    // the window area is SB[-sbLo, sbHi), kept zero where nothing is staged
    int total;
};

// A division's quotient limbs d = h - k are found in blocks (mp_block.hpp):
// nb blocks of bi limbs, the first (top) of d - (nb - 1) bi; dp limbs of
// precision of the inverse serve the longest of them.  bi is a multiple of 4,
// so that every block starts at a 16-byte boundary of the remainder.
struct BlockSplit {
    int nb, bi, dp;
};

// longest block: the last Newton step reaches 2^j + 1 limbs, and 257 limbs is
// the longest iterate whose steps fit one wave's head
constexpr int kBlockMax = 257;
constexpr int kSmallBlock = 16;   // without a head: inverses that fit one limb per lane throughout

MP_HD BlockSplit block_split(int d, int bmax)
{
    if (d <= bmax) return BlockSplit{1, 0, d > 2 ? d : 2};
    const int top = bmax & ~3, nb = 1 + (d - bmax + top - 1) / top;
    const int even = r4((d + nb - 1) / nb), bi = even < top ? even : top, b0 = d - (nb - 1) * bi;
    return BlockSplit{nb, bi, b0 > bi ? b0 : bi};
}

// longest block whose Newton steps all have iterates (l + 3 limbs) shorter than `limit` limbs
MP_HD int block_limit(int limit)
{
    int b = 3;
    while (2 * b - 1 <= kBlockMax && b + 3 < limit) b = 2 * b - 1;
    return b;
}

// LDS layout of one wave's head (the Refine iterations whose iterate has fewer
// than `limit` limbs, so l <= limit - 4): a short control block (a head's
// products have at most kHeadStrips strips and it broadcasts nothing through
// LDS), the divisor limbs [vbase, k] it reads (v' = v >> s has at most 2l + 2
// limbs), the iterate (at most 2l + 2 limbs after the last of these
// iterations), PowDiff's residual (at most 3l + 3 limbs, B^h' minus a
// product), the reversed digits of a matrix-core product's shorter operand
// (the iterate, at most l + 4 limbs), the window operand with its zero
// guards, and products (w * x: at most 4l + 9 limbs).  Every use is guarded;
// an iteration that would overrun returns false and the body does it instead.
// The window's guards cover both product engines: the one-wave VALU product
// reads strip [K0, K0 + 64) with rows [ilo, ihi) within 65 limbs below the
// window and 63 above it; the matrix-core digit planes of a long operand of
// up to capY = 2 limit + 8 limbs (v' and PowDiff's residual in the
// iterations a head runs) need 4 kYPadBlk zero words below the window and
// reach 8 ((capY + 8) / 8) + 8 kYPadBlk words above its start (a longer
// operand takes the VALU product).  Sized so that 16 heads share a compute
// unit's LDS up to the largest limit.
constexpr int kHeadMinLimit = 16;   // smallest small_limit (lower knob values count as this)
constexpr int kHeadMaxLimit = 140;   // largest small_limit: every head operand then fits kHeadMaxLimbs
constexpr int kHeadPad = kLanes + 8; // zero guard on both sides of a head's VALU window operand
// (the longest one-wave linear operation of a head is bounded by capP, capX or
// capW + l, all below 4 * limit + 8 limbs)
static_assert(4 * kHeadMaxLimit + 8 <= kHeadMaxLimbs, "head operands must fit one wave's addsub");
static_assert(4 * kHeadMaxLimit + 8 <= kHeadStrips * kStrip, "a head's products must fit its strip slots");

MP_HD constexpr Plan plan_head(int limit, int vbase)
{
    Plan p{};
    const int L = limit < kHeadMinLimit ? kHeadMinLimit : limit > kHeadMaxLimit ? kHeadMaxLimit : limit;
    p.vbase = vbase;
    p.capV = r4(2 * L);
    p.capW = r4(2 * L + 8);
    p.capX = r4(3 * L + 8);
    p.capR = r4(L + 4);
    p.capSB = r4(3 * L + 8);
    p.capP = r4(4 * L + 8);
    p.capY = 2 * L + 8;
    p.sbLo = hmax(kHeadPad, 4 * kYPadBlk);
    p.sbHi = hmax(p.capSB + kHeadPad, 8 * ((p.capY + 8) >> 3) + 8 * kYPadBlk);
    p.offV = kHeadCtlWords;
    p.offW = p.offV + p.capV;
    p.offX = p.offW + p.capW;
    p.offR = p.offX + p.capX + kXPad;
    p.offSB = p.offR + p.capR + kXPad + p.sbLo;
    p.offP = p.offSB + p.sbHi;
    p.total = p.offP + p.capP + 4;
    return p;
}

// Record of the head in one of the instance's output rows (the longer of q and
// r; w for a shifted inverse), in 32-bit words:
//   [0] kRecValid, or 0 when there is none
//   [1] h   [2] k   [3] limbs u and v are shifted up by (1 for a one-limb divisor)
//   [4] limbs of W   [5] dp   [6] blocks   [7] limbs of the blocks below the first
//   [kRecHdr, kRecHdr + [4]) the limbs of W, about B^(k + dp + 2) / v
constexpr uint32_t kRecValid = 0x52454332u;
constexpr int kRecHdr = 8;
// longest inverse a record of `row` limbs can hold (dp + 3 limbs and the header)
MP_HD int record_block(int row) { return row - kRecHdr - 3; }
constexpr int kHeadWaves = 4;   // head instances (waves) per workgroup
static_assert(16 * plan_head(kHeadMaxLimit, 0).total * 4 <= 160 * 1024, "16 heads must share a compute unit's LDS");

MP_HD int mul_lds_words(int na, int nb)
{
    const int lo = na < nb ? na : nb, hi = na < nb ? nb : na;
    return kCtlWords + kXPad + r4(lo + 1) + kXPad + 4 + kPad + r4(hi + 1) + kPad + r4(na + nb) + 4;
}

// ------------------------------------------------------------------ helpers

// p[c0, ncols) = columns c0 .. ncols-1 of x*y (c0 = 0: x*y mod B^ncols; see
// mul and mul_mfma for c0 > 0, a multiple of 8); returns the precision of the
// result.  Long enough products run on the matrix cores (long operand's
// digits in sb, short operand's reversed digits in xr, which holds xrcap
// limbs); the rest walk the rows on the VALU with the longer operand staged in
// sb as window.
//
// MF = false builds the vector-ALU path only (for code that never has an
// operand long enough for the matrix cores).
template <int T, bool MF, class FL, class FS>
MP_DEV int product_views(uint32_t *ctl, uint32_t *p, int ncols, const FL &lng, int nl, const uint32_t *lng_lds,
                         const FS &sht, int ns, const uint32_t *sht_lds, uint32_t *sb, int &sbext,
                         uint32_t *xr, int xrcap, int mfma_min, int c0 = 0, bool want_prec = true,
                         bool sht_ready = false)
{
    int r;
    if constexpr (MF) {
        if (ns >= mfma_min && ns + 1 <= xrcap) {
            mfma_operands<T>(ctl, lng, nl, sb, sbext, sht, ns, xr, sht_ready);
            sbext = mfma_ext(nl);
            r = mul_mfma<T>(ctl, p, ncols, sb, nl, xr, ns, c0, want_prec);
            return r;
        }
    }
    copy<T>(sb, nl, sbext, lng);
    sbext = nl;
    if constexpr (T == kLanes) r = mul1<T>(ctl, p, ncols, sht_lds, ns, sb, nl, c0, want_prec);
    else r = mul<T>(ctl, p, ncols, sht_lds, ns, sb, nl, c0, want_prec);
    return r;
}

template <int T, bool MF = true>
MP_DEV int product(uint32_t *ctl, uint32_t *p, int ncols, const uint32_t *x, int nx,
                   const uint32_t *y, int ny, uint32_t *sb, int &sbext, uint32_t *xr, int xrcap, int mfma_min,
                   int c0 = 0, bool want_prec = true, bool sht_ready = false)
{
    const uint32_t *sht = nx >= ny ? y : x, *lng = nx >= ny ? x : y;
    const int ns = nx >= ny ? ny : nx, nl = nx >= ny ? nx : ny;
    return product_views<T, MF>(ctl, p, ncols, Span{lng, 0, nl}, nl, lng, Span{sht, 0, ns}, ns, sht, sb, sbext,
                                xr, xrcap, mfma_min, c0, want_prec, sht_ready);
}

// ------------------------------------------------------- Alg. 1 Refine

// (trace build: sub-steps of two of a head's iterations, i = 3 in slots 5-7
// and i = 6 in slots 8-10: PowDiff's product, its residual, Step's product)
#define MP_HEAD_SUB(i, k)                                       \
    do {                                                        \
        if constexpr (T == kLanes) {                            \
            if ((i) == 3) MP_WSTAMP(5 + (k));                   \
            else if ((i) == 6) MP_WSTAMP(8 + (k));              \
        }                                                       \
    } while (0)

// Iteration i of the Refine loop (Alg. 1): PowDiff, then Step, updating the
// iterate W (nonzero limbs inside [0, we), precision nw) and l.  Run by T
// threads (the workgroup, or one wave in a head); MF as for product_views.
template <int T, bool MF = true>
MP_DEV bool refine_iter(uint32_t *ctl, const Plan &pl, const Knobs &kn, uint32_t *lds, int h, int k, int i, int &l,
                        int &we, int &nw, int &sbext)
{
    uint32_t *V = lds + pl.offV, *W = lds + pl.offW, *X = lds + pl.offX;
    uint32_t *SB = lds + pl.offSB, *P = lds + pl.offP, *XR = lds + pl.offR;
    const int g = 2, d = h - k;
    const int m = imin(d + 1 - l, l);
    const int s = imax(0, k - 2 * l + 1 - g);
    const int H = k + l + m - s + g;
    if (s < pl.vbase) return false;      // (a head holds only the limbs its iterations read)
    const uint32_t *vp = V + (s - pl.vbase);   // divisor prefix shift_{-s}(v)
    const int nvp = k + 1 - s;
    const int hp = H - m, lp = l - g;   // PowDiff(v', w, H - m, l - g)
    const int L = nvp + nw - lp + 1;
    // a product goes to the matrix cores only if its longer operand's digit
    // planes fit the window area
    const int mm_pd = imax(nvp, nw) <= pl.capY ? kn.mfma_min : (1 << 30);
    bool sign;
    int nx;
    if (L >= hp) {                      // full product, compare with B^hp
        const int np0 = nvp + nw;
        if (np0 > pl.capP) return false;
        const int np = product<T, MF>(ctl, P, np0, vp, nvp, W, nw, SB, sbext, XR, pl.capR, mm_pd);
        MP_HEAD_SUB(i, 0);
        if (np <= hp) {                 // P < B^hp: x = B^hp - P
            if (hp > pl.capX) return false;
            sign = true;
            addsub<T>(ctl, hp, true, 0u, Zero{}, Span{P, 0, np}, Store{X, 0, hp});
        } else {                        // x = P - B^hp
            if (np > pl.capX) return false;
            sign = false;
            addsub<T>(ctl, np, true, 0u, Span{P, 0, np}, PowB{hp}, Store{X, 0, np});
        }
        nx = read_prec<T>(ctl);
    } else {                            // close product: P = v'w mod B^L
        if (L > pl.capP || L > pl.capX) return false;
        const int np = product<T, MF>(ctl, P, L, vp, nvp, W, nw, SB, sbext, XR, pl.capR, mm_pd);
        MP_HEAD_SUB(i, 0);
        if (np == 0) {                  // v'w = B^hp exactly
            sign = true;
            nx = 0;
        } else if (np < L) {            // top limb 0: v'w = B^hp + P
            sign = false;
            nx = np;
            copy<T>(X, np, 0, Span{P, 0, np});
        } else {                        // v'w = B^hp - (B^L - P)
            sign = true;
            addsub<T>(ctl, L, true, 0u, Zero{}, Span{P, 0, L}, Store{X, 0, L});
            nx = read_prec<T>(ctl);
        }
    }
    // Step: res = shift_m(w) +- shift_{2m-H}(w x); then w = shift_{-post}(res).
    // When nw + nx <= sh, w x < B^sh: the shifted product is 0 and, in the
    // negative branch, its nonzero low part borrows one; no product is formed.
    // Otherwise only the columns of w x from cs = sh - 2 (rounded down to a
    // multiple of 8) up are formed: the columns below change the shifted
    // product by less than one unit of the iterate's last guard limb, and the
    // sticky bit of the negative branch is taken from the formed columns below
    // sh.  The matrix-core digits can make the dropped part negative (less
    // than 2^17 cs B^cs in size), so the formed sum T may exceed w x: one more
    // column holds T < 2 B^(nw+nx), and w x >= B^(nw+nx-2) >= B^(sh-1) keeps
    // T > 0.
    MP_HEAD_SUB(i, 1);
    const int sh = H - 2 * m;
    const int post = i < 2 ? m : 1;
    int nt = 0, cs = 0;
    uint32_t below = 0;   // borrow of a product that lies wholly below sh
    if (nx && nw + nx <= sh) {
        below = sign ? 0u : 1u;
    } else if (nx) {
        nt = nw + nx;
        cs = imax(sh - 2, 0) & ~7;
        if (cs) nt += 1;
        if (nt - cs > pl.capP) return false;
        // w is the shorter operand of both products on the matrix cores: its
        // digits from PowDiff's product are still in XR
        const bool w_ready = MF && nvp >= nw && nw < nx && nw >= mm_pd && nw + 1 <= pl.capR;
        const int mm_st = imax(nw, nx) <= pl.capY ? kn.mfma_min : (1 << 30);
        // column c of the product goes to P[c - cs]
        product<T, MF>(ctl, P - cs, nt, W, nw, X, nx, SB, sbext, XR, pl.capR, mm_st, cs, false, w_ready);
    }
    MP_HEAD_SUB(i, 2);
    // the sticky borrow of the negative branch (any nonzero formed column
    // below sh) is found by the Step's own addsub before its carry scan
    const int stop = !sign && nt > cs ? imin(sh, nt) - cs : 0;
    const int nres = imax(nw + m, nt - sh) + 1;
    if (nres - post > pl.capW) return false;
    const uint32_t co = addsub<T>(ctl, nres, !sign, below, Span{W, m, nw}, Span{P, cs - sh, imax(nt - cs, 0)},
                                  Store{W, post, pl.capW}, StickyAny<T>{P, stop});
    if (!sign && co) return false;
    we = nres - post;
    nw = read_prec<T>(ctl, post);
    if (i >= 2) l = l + m - 1;
    return true;
}

// ------------------------------------------------ one-wave tiny iterations
//
// A Refine iteration whose operands, products and result all fit 64 limbs,
// run by one wave with limb j of every intermediate in lane j: the same
// arithmetic as refine_iter (the same products, the same clipping of the Step
// product at cs, the same sticky borrow), with every carry resolved by the
// ballot lookahead in registers instead of a pass through LDS.  Only the
// divisor prefix and the iterate are read from LDS and only the new iterate is
// written back.

// the carry (or borrow) into each lane of a one-limb-per-lane addition
// (subtraction) whose lanes generate g and propagate p, with carry-in cin;
// cout gets the carry out of lane 63
MP_DEV uint32_t lane_carry_in(bool g, bool p, uint32_t cin, uint32_t &cout)
{
    const uint64_t G = ballot(g), P = ballot(p), X = G | P;
    const uint64_t s0 = X + G;
    cout = (s0 < X ? 1u : 0u) | ((~P == 0 ? 1u : 0u) & cin);
    const uint64_t cm = (X + G + (uint64_t)cin) ^ X ^ G;
    return (uint32_t)(cm >> lane()) & 1u;
}

// a - b - bin in lanes [0, n) (zero above); bout: the borrow out of lane n - 1
MP_DEV uint32_t lane_sub(uint32_t a, uint32_t b, int n, uint32_t bin, uint32_t &bout)
{
    const bool in = lane() < n;
    const uint32_t d = in ? a - b : 0u;
    const uint32_t bi = lane_carry_in(in && a < b, !in || d == 0u, bin, bout);
    return in ? d - bi : 0u;
}

// a + b + cin in lanes [0, n) (zero above); cout: the carry out of lane n - 1
MP_DEV uint32_t lane_add(uint32_t a, uint32_t b, int n, uint32_t cin, uint32_t &cout)
{
    const bool in = lane() < n;
    const uint64_t s = (uint64_t)a + b;
    const uint32_t z = in ? (uint32_t)s : 0u;
    const uint32_t ci = lane_carry_in(in && (s >> 32) != 0, !in || z == 0xFFFFFFFFu, cin, cout);
    return in ? z + ci : 0u;
}

// 1 + the highest lane holding a nonzero limb (0 when none)
MP_DEV int lane_prec(uint32_t z)
{
    const uint64_t m = ballot(z != 0u);
    return m ? 64 - __builtin_clzll(m) : 0;
}

// column K0 + lane of a * b with the carries between columns K0 .. K0 + 63
// and none from below K0: rows a_i (i < na) from rowf(i) (wave-uniform i),
// window limbs b_j (j < nb) from LDS, read per lane with a range mask
template <class FR>
MP_DEV uint32_t lane_mul(const FR &rowf, int na, const uint32_t *b, int nb, int K0)
{
    const int l = lane(), k = K0 + l;
    const int ilo = imax(0, K0 - nb + 1), ihi = imin(na, K0 + kLanes);
    uint64_t lo[4] = {0, 0, 0, 0};
    uint32_t hi[4] = {0, 0, 0, 0};
    for (int i = ilo; i < ihi; i += 4) {
        uint32_t a[4], w[4];
#pragma unroll
        for (int j = 0; j < 4; j++) {
            a[j] = i + j < ihi ? rowf(i + j) : 0u;
            const int c = k - i - j;
            w[j] = (unsigned)c < (unsigned)nb ? b[c] : 0u;
        }
        mac4x(lo, hi, a[0], w[0], a[1], w[1], a[2], w[2], a[3], w[3]);
    }
    uint64_t sl = lo[0];
    uint32_t sh = hi[0];
#pragma unroll
    for (int r = 1; r < 4; r++) {
        const uint64_t t = sl + lo[r];
        sh += hi[r] + (t < sl ? 1u : 0u);
        sl = t;
    }
    // S = s0 + s1 B + s2 B^2 per column: t = s0 + s1 of the lane below + s2 of the lane two below
    const uint32_t s1m = shfl_up1((uint32_t)(sl >> 32)), s2m = shfl_up2(sh);
    const uint64_t t = (uint64_t)(uint32_t)sl + s1m + s2m;
    const uint32_t cm = shfl_up1((uint32_t)(t >> 32));
    const uint64_t y = (uint64_t)(uint32_t)t + cm;
    uint32_t top_carry;   // leaves column K0 + 63: above every column a caller keeps
    const uint32_t z = (uint32_t)y;
    return z + lane_carry_in((y >> 32) != 0, z == 0xFFFFFFFFu, 0u, top_carry);
}

struct LdsRows {
    const uint32_t *p;
    MP_DEV uint32_t operator()(int i) const { return p[i]; }
};
struct LaneRows {
    uint32_t x;
    MP_DEV uint32_t operator()(int i) const { return readlane(x, i); }
};

// whether Refine iteration i (with l, nw, we) fits one limb per lane throughout
MP_DEV bool iter_fits_wave(const Plan &pl, int h, int k, int l, int nw, int we)
{
    const int g = 2, d = h - k;
    const int m = imin(d + 1 - l, l);
    const int s = imax(0, k - 2 * l + 1 - g);
    const int H = k + l + m - s + g;
    const int nvp = k + 1 - s;
    const int hp = H - m, lp = l - g;
    const int L = nvp + nw - lp + 1;
    const int ncA = L >= hp ? nvp + nw : L;
    const int nxmax = imax(ncA, hp);
    const int sh = H - 2 * m;
    const int cs = imax(sh - 2, 0) & ~7;
    return s >= pl.vbase && ncA <= kLanes && hp <= kLanes && nw + nxmax + 1 - cs <= kLanes &&
           imax(nw + m, nw + nxmax + 1 - sh) + 1 <= kLanes && we <= kLanes;
}

// Refine iteration i (as refine_iter) by one wave in registers, for an
// iteration that iter_fits_wave accepts
MP_DEV bool refine_iter_wave(const Plan &pl, uint32_t *lds, int h, int k, int i, int &l, int &we, int &nw)
{
    uint32_t *V = lds + pl.offV, *W = lds + pl.offW;
    const int g = 2, d = h - k;
    const int m = imin(d + 1 - l, l);
    const int s = imax(0, k - 2 * l + 1 - g);
    const int H = k + l + m - s + g;
    const int nvp = k + 1 - s;
    const int hp = H - m, lp = l - g;
    const int L = nvp + nw - lp + 1;
    const bool full = L >= hp;
    const int ncA = full ? nvp + nw : L;          // columns PowDiff forms
    const int sh = H - 2 * m;
    const int cs = imax(sh - 2, 0) & ~7;
    const int post = i < 2 ? m : 1;
    const uint32_t *vp = V + (s - pl.vbase);
    wave_sync();
    const int ln = lane();
    // PowDiff: P = v' w (all columns, or mod B^L), then x = |v' w - B^hp|
    uint32_t P = lane_mul(LdsRows{W}, nw, vp, nvp, 0);
    if (ln >= ncA) P = 0u;
    const int np = lane_prec(P);
    bool sign;
    uint32_t x, bo;
    if (full) {
        if (np <= hp) {                 // x = B^hp - P
            sign = true;
            x = lane_sub(0u, P, hp, 0u, bo);
        } else {                        // x = P - B^hp
            sign = false;
            x = lane_sub(P, ln == hp ? 1u : 0u, np, 0u, bo);
        }
    } else if (np == 0) {               // v'w = B^hp exactly
        sign = true;
        x = 0u;
    } else if (np < L) {                // v'w = B^hp + P
        sign = false;
        x = P;
    } else {                            // v'w = B^hp - (B^L - P)
        sign = true;
        x = lane_sub(0u, P, L, 0u, bo);
    }
    const int nx = lane_prec(x);
    // Step: res = shift_m(w) +- shift_{2m-H}(w x), formed from column cs up
    int nt = 0, cse = 0;
    uint32_t below = 0, Ps = 0u;
    if (nx && nw + nx <= sh) {
        below = sign ? 0u : 1u;
    } else if (nx) {
        nt = nw + nx;
        cse = cs;
        if (cse) nt += 1;
        Ps = lane_mul(LaneRows{x}, nx, W, nw, cse);
        if (ln >= nt - cse) Ps = 0u;
    }
    const int stop = !sign && nt > cse ? imin(sh, nt) - cse : 0;
    const bool sticky = ballot(ln < stop && Ps != 0u) != 0;
    const int nres = imax(nw + m, nt - sh) + 1;
    if (nres - post > pl.capW) return false;
    const uint32_t wk = (unsigned)(ln - m) < (unsigned)nw ? W[ln - m] : 0u;
    const int src = ln + sh - cse;   // column ln + sh of w x, at lane src of Ps
    const uint32_t yk = shfl(Ps, src < kLanes ? src : 0);
    const uint32_t y = (src < kLanes && src < nt - cse) ? yk : 0u;
    const uint32_t cin = sticky ? 1u : below;
    uint32_t co;
    const uint32_t res = sign ? lane_add(wk, y, nres, cin, co) : lane_sub(wk, y, nres, cin, co);
    if (!sign && co) return false;
    wave_sync();
    if (ln >= post && ln < nres) W[ln - post] = res;
    we = nres - post;
    nw = imax(lane_prec(res) - post, 0);
    if (i >= 2) l = l + m - 1;
    return true;
}

MP_HD int refine_iters(int d)   // Alg. 1's iteration count for h - k = d >= 1
{
    int r = 0;
    while (d - 1 > 1 && (1 << r) < d - 1) r++;
    return 2 + r;
}

// l at the start of Refine iteration i (d = h - k)
MP_HD int refine_l(int d, int i)
{
    int l = 2;
    for (int j = 2; j < i; j++) l = l + (d + 1 - l < l ? d + 1 - l : l) - 1;
    return l;
}

// floor(B^3 / V) for B <= V < B^2, by one wave (every lane gets the result):
// the quotient is B^2 when V = B and below B^2 otherwise.  Its bits are found
// six at a time from the top: in each round lane j tests whether the bits
// known so far followed by j (and zeros below) times V is at most B^3; the
// lanes that pass are 0 .. J (the product grows with j), so J is the next six
// bits.  Ten rounds of six bits and one of four: exact integer arithmetic, no
// division.
MP_DEV void inv96_wave(uint64_t V, uint64_t &q, uint32_t &q64)
{
    q = 0;
    q64 = 0;
    if (V == (1ull << 32)) {
        q64 = 1;
        return;
    }
    const unsigned __int128 B3 = ((unsigned __int128)1) << 96;
    const uint64_t j = (uint64_t)lane();
    for (int sh = 58; sh >= 0; sh -= 6) {
        const uint64_t c = q | (j << (sh < 4 ? 0 : sh));
        const bool ok = (sh >= 4 || j < 16) && (unsigned __int128)c * V <= B3;
        const uint64_t m = ballot(ok);
        q |= (uint64_t)(63 - __builtin_clzll(m)) << (sh < 4 ? 0 : sh);
        if (sh < 4) break;
        if (sh == 4) sh = 6;   // the last round takes bits 3 .. 0
    }
}

// Alg. 1's initial approximation w = shift_g(floor(B^3 / V)), V = v_{k-1} + v_k B
// (in registers), by one wave: w0 <= B^2 has 3 limbs (65 bits when V = B)
MP_DEV void head_init(uint64_t Vt, uint32_t *W, int &we, int &nw)
{
    uint64_t w0;
    uint32_t w64;
    inv96_wave(Vt, w0, w64);
    if (lane() == 0) {
        W[0] = 0u;
        W[1] = 0u;
        W[2] = (uint32_t)w0;
        W[3] = (uint32_t)(w0 >> 32);
        W[4] = w64;
    }
    nw = (int)uniform(w64 ? 5u : (w0 >> 32) ? 4u : 3u);
    we = 5;
}

// ------------------------------------------------------------------- head

// number of significant limbs of x[0, n) (global memory), by one wave from the top
MP_DEV int wave_prec(const uint32_t *x, int n)
{
    for (int top = n; top > 0; top -= kLanes) {
        const int i = top - kLanes + lane();
        const uint64_t m = ballot(i >= 0 && x[i] != 0u);
        if (m) return top - kLanes + 64 - __builtin_clzll(m);
    }
    return 0;
}

// index of the lowest nonzero limb of x[0, n) (n when there is none), by one wave
MP_DEV int wave_low(const uint32_t *x, int n)
{
    for (int base = 0; base < n; base += kLanes) {
        const int i = base + lane();
        const uint64_t m = ballot(i < n && x[i] != 0u);
        if (m) return base + __builtin_ctzll(m);
    }
    return n;
}

// The head of one instance with h, k = prec(v) - 1 and vlow (index of v's
// lowest nonzero limb), by one wave in its own LDS area (plan_head words):
// splits the quotient's limbs into blocks and computes the inverse W they
// need (Alg. 1's initial approximation and Refine for h' = k + dp), recorded
// in rec[0, nrec).  rec[0] = 0 when there is nothing to divide (u < v, v a
// power of B), the quotient cannot fit nq limbs, or the record the row.  With
// have_top, vtop holds v_{k-1} + v_k B (read by the caller), else they are
// read here.  A divisor of one limb is divided as v B into u B.
MP_DEV void head_refine(uint32_t *lds, int h, int k, int vlow, const uint32_t *v, uint64_t vtop, bool have_top,
                        uint32_t *rec, int nrec, int nq, const Knobs &kn)
{
    constexpr int T = kLanes;
    uint32_t *ctl = lds;
    const int g = 2, sv = k == 0 ? 1 : 0;
    bool go = k >= 0 && h > k && h - k - 1 <= nq;
    uint64_t Vt = vtop;
    if (go && !have_top) Vt = sv ? (uint64_t)v[0] << 32 : ((uint64_t)v[k] << 32) | v[k - 1];
    if (go) go = !(vlow == k && (uint32_t)(Vt >> 32) == 1u);
    const int bmax = hmin(block_limit(kn.small_limit), record_block(nrec));
    if (!go || bmax < kSmallBlock) {
        if (lane() == 0) rec[0] = 0u;
        return;
    }
    h += sv;
    k += sv;
    const BlockSplit bs = block_split(h - k, bmax);
    const int hh = k + bs.dp, ns = refine_iters(bs.dp);
    const int vbase = imax(0, k - 2 * refine_l(bs.dp, ns - 1) + 1 - g);
    const Plan pl = plan_head(kn.small_limit, vbase);
    uint32_t *V = lds + pl.offV, *W = lds + pl.offW, *SB = lds + pl.offSB;
    // the divisor limbs [vbase, k] (at most 2 l + 2 <= capV <= 5 T): every read
    // in flight at once; the LDS areas are zeroed and the initial approximation
    // (from the top limbs in registers) computed while they arrive, then they
    // are stored
    int we = 0, nw = 0, sbext = 0, l = 2;
    {
        static_assert(r4(2 * kHeadMaxLimit) <= 5 * T, "a head stages its divisor limbs in one round");
        const int nvs = k + 1 - vbase, first = vbase - sv;
        uint32_t a[5];
#pragma unroll
        for (int j = 0; j < 5; j++) {
            const int i = lane() + j * T;
            a[j] = i < nvs && first + i >= 0 ? v[first + i] : 0u;
        }
        for (int i = lane(); i < pl.capW; i += T) W[i] = 0u;
        for (int i = lane() - pl.sbLo; i < pl.sbHi; i += T) SB[i] = 0u;
        wave_sync();
        head_init(Vt, W, we, nw);
#pragma unroll
        for (int j = 0; j < 5; j++)
            if (lane() + j * T < nvs) V[lane() + j * T] = a[j];
    }
    MP_WSTAMP(2);   // (trace build: staging and the initial approximation)
    MP_WSTAMP(3);
    bool ok = k + 1 - vbase <= pl.capV;
    int i = 0;
    // the first iterations in registers, one limb per lane; the rest through LDS
    for (; i < ns && ok && iter_fits_wave(pl, hh, k, l, nw, we); i++) {
        ok = refine_iter_wave(pl, lds, hh, k, i, l, we, nw);
        MP_WSTAMP(16 + (i & 15));
    }
    for (; i < ns && ok; i++) {
        ok = refine_iter<T>(ctl, pl, kn, lds, hh, k, i, l, we, nw, sbext);
        MP_WSTAMP(16 + (i & 15));
    }
    ok = ok && nw <= bs.dp + 3;
    wave_sync();
    for (int i = lane(); ok && i < nw; i += T) rec[kRecHdr + i] = W[i];
    if (lane() == 0) {
        rec[1] = (uint32_t)h;
        rec[2] = (uint32_t)k;
        rec[3] = (uint32_t)sv;
        rec[4] = (uint32_t)nw;
        rec[5] = (uint32_t)bs.dp;
        rec[6] = (uint32_t)bs.nb;
        rec[7] = (uint32_t)bs.bi;
        rec[0] = ok ? kRecValid : 0u;
    }
    MP_WSTAMP(4);
    MP_WRSTAMP(15);   // (trace build: real time at the end and the start of a head)
}

// prec(x[0, n)) when x[0, n) is nonzero below its top 64 limbs or in them:
// the ballot of the top chunk m (read by the caller) decides it, else the
// scan goes on downwards
MP_DEV int wave_prec_from(const uint32_t *x, int n, uint64_t m)
{
    if (m) return n - kLanes + 64 - __builtin_clzll(m);
    return n > kLanes ? wave_prec(x, n - kLanes) : 0;
}

// k = prec(v) - 1 and the index of v's lowest nonzero limb, by one wave
// from the ballots of v's top 64 limbs (mv) and bottom 64 limbs (mb), read
// by the caller; a chunk of 64 zero limbs sends the scan on
MP_DEV void wave_vshape(const uint32_t *v, int nv, uint64_t mv, uint64_t mb, int &k, int &vlow)
{
    k = wave_prec_from(v, nv, mv) - 1;
    vlow = mb ? __builtin_ctzll(mb) : wave_low(v, k + 1);
}

// v_{k-1} + v_k B from the registers of v's top 64 limbs (lane j holds limb
// nv - 64 + j), when both limbs lie in that chunk
MP_DEV bool wave_vtop(uint32_t vt, int nv, int k, uint64_t &V)
{
    const int j = k - (nv - kLanes);   // lane of v_k
    if (k < 1 || j < 1 || j >= kLanes) return false;
    V = ((uint64_t)readlane(vt, j) << 32) | readlane(vt, j - 1);
    return true;
}

// the head of a division: the top 64 limbs of u and of v and the bottom 64 of
// v are read together, which settles both precisions and v's lowest nonzero
// limb in one round trip unless a number has 64 zero limbs at that end
MP_DEV void head_divrem(uint32_t *lds, const uint32_t *u, int nu, const uint32_t *v, int nv, uint32_t *rec, int nrec,
                        int nq, const Knobs &kn)
{
    MP_WSTAMP(0);
    MP_WRSTAMP(14);
    const int iu = nu - kLanes + lane(), iv = nv - kLanes + lane(), il = lane();
    const uint32_t ut = iu >= 0 ? u[iu] : 0u, vt = iv >= 0 ? v[iv] : 0u, vb = il < nv ? v[il] : 0u;
    const uint64_t mu = ballot(ut != 0u), mv = ballot(vt != 0u), mb = ballot(vb != 0u);
    const int h = wave_prec_from(u, nu, mu);
    int k, vlow;
    wave_vshape(v, nv, mv, mb, k, vlow);
    uint64_t vtop = 0;
    const bool top = wave_vtop(vt, nv, k, vtop);
    MP_WSTAMP(1);
    head_refine(lds, h, k, vlow, v, vtop, top, rec, nrec, nq, kn);
}

// the head of a shifted inverse floor(B^h / v): the division of B^h
MP_DEV void head_shinv(uint32_t *lds, int h, const uint32_t *v, int nv, uint32_t *rec, int nrec, const Knobs &kn)
{
    const int iv = nv - kLanes + lane(), il = lane();
    const uint32_t vt = iv >= 0 ? v[iv] : 0u, vb = il < nv ? v[il] : 0u;
    int k, vlow;
    wave_vshape(v, nv, ballot(vt != 0u), ballot(vb != 0u), k, vlow);
    uint64_t vtop = 0;
    const bool top = wave_vtop(vt, nv, k, vtop);
    head_refine(lds, h + 1, k, vlow, v, vtop, top, rec, nrec, nrec, kn);
}

// ------------------------------------------------------------ instances

// c = a * b  (c has na + nb limbs)
template <int T>
MP_DEV void mul_instance(uint32_t *lds, const uint32_t *a, int na, const uint32_t *b, int nb, uint32_t *c,
                         const Knobs &kn)
{
    uint32_t *ctl = lds;
    const int nlo = na < nb ? na : nb, nhi = na < nb ? nb : na;
    const uint32_t *sht = na < nb ? a : b, *lng = na < nb ? b : a;
    uint32_t *A = lds + kCtlWords + kXPad;          // short operand (rows, or reversed digits)
    uint32_t *SBbase = A + r4(nlo + 1) + kXPad + 4;
    uint32_t *SB = SBbase + kPad;                   // long operand (window, or digits)
    uint32_t *P = SB + r4(nhi + 1) + kPad;
    int np;
    MP_RSTAMP(6);
    MP_STAMP(0);
    if (nlo >= kn.mfma_min) {
        copy<T>(SBbase, 0, 2 * kPad + r4(nhi + 1), Zero{});
        MP_STAMP(1);
        mfma_operands<T>(ctl, Span{lng, 0, nhi}, nhi, SB, 0, Span{sht, 0, nlo}, nlo, A);
        MP_STAMP(2);
        np = mul_mfma<T>(ctl, P, na + nb, SB, nhi, A, nlo, 0, false);
        MP_STAMP(3);
    } else {
        copy<T>(A, nlo, r4(nlo) + 4, Span{sht, 0, nlo});
        copy<T>(SBbase, kPad + nhi, 2 * kPad + r4(nhi), Span{lng, kPad, nhi});
        np = mul<T>(ctl, P, na + nb, A, nlo, SB, nhi, 0, false);
    }
    (void)np;
    bar<T>();
    MP_STAMP(4);
    for (int i = tid<T>(); i < na + nb; i += T) c[i] = P[i];
    MP_STAMP(5);
    MP_RSTAMP(7);
}

}  // namespace mp
