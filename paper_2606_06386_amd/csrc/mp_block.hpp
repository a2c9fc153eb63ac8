// Block division: one workgroup divides u by v in blocks of quotient limbs.
//
// The head leaves an approximation W of B^(k+dp+2) / v (dp at most 257 limbs
// of precision, two guard limbs).  The quotient's d = h - k limbs are found in
// nb blocks from the top, block i holding the limbs [o_i, o_(i-1)):
//     q_i = floor(R_top W / B^(dp+3)),   R_top = floor(R / B^(o_i+k-1))
//     R  <- R - v q_i B^(o_i)
// with a signed remainder R that starts as u.  Both products run on the int8
// matrix cores over balanced radix-256 digits; the digits of v and of W are
// made once per instance, those of R_top and of -q_i once per block, and R is
// added to the accumulators of the second product, so the subtraction costs
// no pass of its own.  After the last block r = R up to a few multiples of v.
//
// Against one full-precision inverse followed by u * shinv and v * q this
// needs no Newton iteration beyond 257 limbs and about half the limb products
// (a 2048 by 1024-limb division: 1.2e6 instead of 1.8e6), and every operand
// converted to digits is at most one block long.
//
// Error bounds (W = B^(k+dp+2)/v - E with |E| a few units; measured at most 2
// over structured divisors, and clipping adds at most one per iteration):
// |R| < 2.1 v B^(o_(i-1)) gives R_top W / B^(dp+3) = R / (v B^(o_i)) + e with
// |e| < 2^-20; the floor and the columns of R_top W below cA add at most one
// unit each, so q_i is within (-2, 1] of the real ratio: after the block
// -1.1 v B^(o_i) < R < 2.1 v B^(o_i).  R is therefore exact as a signed
// (k + 2)-limb number above o_i, q_i as a signed (limbs + 1)-limb number
// whose top limb is its sign, and at most two corrections each way remain.
#pragma once

#include "mp_div.hpp"

namespace mp {

// ---------------------------------------------------------------- LDS layout
//
// ctl | pad | V plane 0 | pad | V plane 1 | pad | R_top plane 0 | pad |
// R_top plane 1 | pad | W reversed | -q reversed | P | R
// (pads of kYPadBlk zero blocks shared by their neighbours).  R holds the
// dividend's h limbs and above them the quotient: limb j of q goes to
// R[k + 2 + j], which the remainder has left by the time the block is done.
struct BodyPlan {
    int nbV, lyV, offV;       // 8-limb blocks of the divisor's digits, distance of the planes, first word
    int nbT, lyT, offT;       // the same for R_top
    int offW, offQ, offP, offR;
    int capR;
    int total;
};

constexpr int kPadWords = 4 * kYPadBlk;

// a dividend of at most nu and a divisor of at most nv limbs (each one more
// inside, for divisors of one limb, which are shifted up by one)
MP_HD constexpr BodyPlan plan_body(int nu, int nv)
{
    BodyPlan p{};
    const int ny = (nv < nu ? nv : nu) + 2;            // digit limbs of the divisor
    const int dm = hmin(kBlockMax, hmax(nu + 1, 40));  // longest block and inverse
    p.nbV = (ny + 7) >> 3;
    p.nbT = (dm + 3 + 7) >> 3;
    p.offV = kCtlWords + kPadWords;
    p.lyV = 4 * p.nbV + kPadWords;
    p.offT = p.offV + 2 * p.lyV;
    p.lyT = 4 * p.nbT + kPadWords;
    p.offW = p.offT + 2 * p.lyT + kXPad;
    p.offQ = r4(p.offW + dm + 4 + kXPad);
    p.offP = r4(p.offQ + dm + 1 + kXPad);
    p.offR = p.offP + r4(dm + 16);
    p.capR = r4(nu + 8);
    p.total = p.offR + p.capR;
    return p;
}

// ------------------------------------------------------------- row passes
//
// Linear passes over limbs in rows of 64, limb 64 r + l in lane l of the wave
// that owns row r.  Carries inside a row come from one addition of ballot
// masks on the scalar unit; rows of one wave chain through the scalar carry;
// the carry into a wave's first row is found by looking back from it for a
// limb that does not propagate (the row below, but for runs of 64 propagating
// limbs), so waves need no exchange.  A row costs about ten vector
// instructions for 64 limbs; a pass that gives each thread a chunk of limbs
// costs about twelve per limb and thread.

// carries into the lanes of one row: bit l of the result; cin becomes the carry out
MP_DEV uint64_t row_carries(uint64_t G, uint64_t P, uint32_t &cin)
{
    const uint64_t X = G | P;
    const unsigned __int128 s = (unsigned __int128)X + G + cin;
    cin = (uint32_t)(s >> 64);
    return (uint64_t)s ^ X ^ G;
}

// the carry out of a row of generate and propagate masks that does not wholly propagate
MP_DEV uint32_t row_carry_out(uint64_t G, uint64_t P)
{
    return (uint32_t)(G >> (63 - __builtin_clzll(~P))) & 1u;
}

constexpr uint32_t kBal = 0x80808080u;

// out(k, digit limb) for the limbs k of rows [r0, r1): the balanced radix-256
// digits of the n-limb number x with carry-in cin0 at limb 0.  Limb n gets the
// top carry digit (0 or 1), limbs above it zero.
template <class FX, class FO>
MP_DEV void balance_rows(int r0, int r1, int n, uint32_t cin0, const FX &x, const FO &out)
{
    uint32_t c = cin0;
    for (int r = r0 - 1; r >= 0; r--) {          // (rows below r0 lie inside [0, n))
        const uint32_t s = x(64 * r + lane()) + kBal;
        const uint64_t G = ballot(s < kBal), P = ballot(s == 0xFFFFFFFFu);
        if (~P) {
            c = row_carry_out(G, P);
            break;
        }
    }
    for (int r = r0; r < r1; r += 4) {
        uint32_t xv[4];
#pragma unroll
        for (int j = 0; j < 4; j++) {
            const int k = 64 * (r + j) + lane();
            xv[j] = r + j < r1 && k < n ? x(k) : 0u;
        }
#pragma unroll
        for (int j = 0; j < 4; j++) {
            if (r + j < r1) {
                const int k = 64 * (r + j) + lane();
                const uint32_t a = k < n ? kBal : 0u, s = xv[j] + a;
                const uint64_t cm = row_carries(ballot(s < a), ballot(s == 0xFFFFFFFFu), c);
                out(k, (s + (inverse_ballot(cm) ? 1u : 0u)) ^ a);
            }
        }
    }
}

// digit limb k into the planes at p (plane distance ly), k < n
struct StorePlane {
    uint32_t *p;
    int n, ly;
    MP_DEV void operator()(int k, uint32_t z) const
    {
        if (k < n) p[plane_word(k, ly)] = z;
    }
};

// digit limb k byte-reversed: dst[n - 1 - k], k < n
struct StoreRev {
    uint32_t *p;
    int n;
    MP_DEV void operator()(int k, uint32_t z) const
    {
        if (k < n) p[n - 1 - k] = bswap(z);
    }
};

// dst = x + y or x - y over limbs [0, n) (mod B^n), rows [r0, r1) by this wave; dst is neither operand
template <class FX, class FY>
MP_DEV void addsub_rows(int r0, int r1, int n, bool sub, const FX &x, const FY &y, uint32_t *dst)
{
    uint32_t c = 0;
    for (int r = r0 - 1; r >= 0; r--) {
        const int k = 64 * r + lane();
        const uint32_t a = x(k), b = y(k), z = sub ? a - b : a + b;
        const uint64_t G = ballot(sub ? a < b : z < a), P = ballot(z == (sub ? 0u : 0xFFFFFFFFu));
        if (~P) {
            c = row_carry_out(G, P);
            break;
        }
    }
    for (int r = r0; r < r1; r++) {
        const int k = 64 * r + lane();
        const uint32_t a = k < n ? x(k) : 0u, b = k < n ? y(k) : 0u, z = sub ? a - b : a + b;
        const uint64_t cm = row_carries(ballot(sub ? a < b : z < a), ballot(z == (sub ? 0u : 0xFFFFFFFFu)), c);
        const uint32_t ci = inverse_ballot(cm) ? 1u : 0u;
        if (k < n) dst[k] = sub ? z - ci : z + ci;
    }
}

// p[0, n) += 1 (up) or -= 1, by one wave: stops at the first limb that does not pass the carry on
MP_DEV void ripple(uint32_t *p, int n, bool up)
{
    const uint32_t pass = up ? 0xFFFFFFFFu : 0u;
    for (int b = 0; b < n; b += kLanes) {
        const int k = b + lane();
        wave_sync();
        const uint32_t x = k < n ? p[k] : pass;
        const uint64_t m = ballot(x != pass);
        if (k < n && (m == 0 || lane() <= __builtin_ctzll(m))) p[k] = up ? x + 1u : x - 1u;
        wave_sync();
        if (m) return;
    }
}

// p[0, n) += s for a small signed s, by one wave
MP_DEV void add_small(uint32_t *p, int n, int s)
{
    if (s == 0 || n <= 0) return;
    wave_sync();
    const uint32_t x = uniform(p[0]), z = x + (uint32_t)s;
    wave_sync();
    if (lane() == 0) p[0] = z;
    wave_sync();
    if (s > 0 ? z < x : z > x) ripple(p + 1, n - 1, s > 0);
}

// ---------------------------------------------------------------- products
//
// One strip (256 limb columns) of a product is one 32x32 matrix-core tile
// accumulated over the diagonals d:  D[t][n] += sum_r X_d[t][r] Y_d[r][n] with
//   X_d[t][r] = e_(32d + t - r)           (Toeplitz slice of the short operand)
//   Y_d[r][n] = d_(32 (S0 + n - d) + r)   (32 blocks of 32 digits of the long one)
// so D[t][n] is the sum of byte column 32 (S0 + n) + t.  The lane that feeds
// row p of X supplies t = 16 ((p >> 2) & 1) + 4 (p >> 3) + (p & 3): the
// accumulator's row order then leaves lane (n, h) with the 16 byte columns of
// the four consecutive limb columns 8n + 4h .. 8n + 4h + 3, and no exchange
// between lanes is needed to form limbs.

struct Operands {
    const uint32_t *x;   // this lane's word of the reversed short digits at diagonal 0
    uint32_t sft;        // and its byte shift
    int dmax;            // last diagonal that touches the short digits
    const uint32_t *y;   // this lane's word of the long digits' planes for block 0
    int nyblk;           // blocks of the long digits
};

// xr: nx reversed digit limbs; yb: planes (distance ly) of ny digit limbs
MP_DEV Operands operands(const uint32_t *xr, int nx, const uint32_t *yb, int ly, int ny)
{
    const int l = lane(), p = l & 31, h = l >> 5;
    const int ox = 4 * nx - 1 - (16 * ((p >> 2) & 1) + 4 * (p >> 3) + (p & 3)) + 16 * h;
    return Operands{xr + (ox >> 2), (uint32_t)ox & 3u, (4 * nx + 30) >> 5, yb + h * ly + 4 * p, (ny + 7) >> 3};
}

// the accumulator of the strip whose first block is S0
MP_DEV MfmaAcc strip_sums(const Operands &o, int S0)
{
    MfmaAcc acc = mfma_zero();
    int d = uniform(imax(0, S0 - o.nyblk + 1));
    const int dhi = uniform(imin(o.dmax, S0 + 31));
    const uint32_t *x = o.x - 8 * d, *y = o.y + 4 * (S0 - d);
    for (; d + 3 <= dhi; d += 4) {
        const XRaw r0 = xraw(x), r1 = xraw(x - 8), r2 = xraw(x - 16), r3 = xraw(x - 24);
        const Limb4 y0 = load4(y), y1 = load4(y - 4), y2 = load4(y - 8), y3 = load4(y - 12);
        acc = mfma_x(acc, xfrag(r0, o.sft), y0);
        acc = mfma_x(acc, xfrag(r1, o.sft), y1);
        acc = mfma_x(acc, xfrag(r2, o.sft), y2);
        acc = mfma_x(acc, xfrag(r3, o.sft), y3);
        sched_loads_first();
        x -= 32;
        y -= 16;
    }
    for (; d <= dhi; d++) {
        acc = mfma_x(acc, xfrag(xraw(x), o.sft), load4(y));
        x -= 8;
        y -= 4;
    }
    return acc;
}

// sum of a[j] 256^j, j = 0..3, plus c (exact, signed)
MP_DEV int64_t byte_sum(const MfmaAcc &a, int j, int64_t c)
{
    int b1 = 256, b2 = 65536, b3 = 16777216;
    asm("" : "+s"(b1), "+s"(b2), "+s"(b3));   // (keeps the products multiply-adds instead of 64-bit shifts)
    c += mfma_get(a, j);
    c += (int64_t)mfma_get(a, j + 1) * b1;
    c += (int64_t)mfma_get(a, j + 2) * b2;
    c += (int64_t)mfma_get(a, j + 3) * b3;
    return c;
}

// The limbs of a strip from its byte sums plus four addend limbs per lane:
// z gets the limbs of columns 8n + 4h .. + 3 with every carry inside the strip
// resolved.  A lane's four columns pass a signed carry on; it is biased by
// 2^31 (subtracted again in the next lane's lowest column, or, below the first
// column of the number, put in as `below` = 2^31) so that it is never
// negative.  Returns the strip's carry into its next column, biased the same
// way (0 <= carry < 2^33): the next strip's own bias takes the 2^31 off again.
MP_DEV uint64_t strip_limbs(const MfmaAcc &a, const Limb4 &add, uint32_t below, uint32_t (&z)[4])
{
    int64_t t = byte_sum(a, 0, (int64_t)add.x - ((int64_t)1 << 31));
    z[0] = (uint32_t)t;
    t = byte_sum(a, 4, (t >> 32) + (int64_t)add.y);
    z[1] = (uint32_t)t;
    t = byte_sum(a, 8, (t >> 32) + (int64_t)add.z);
    z[2] = (uint32_t)t;
    t = byte_sum(a, 12, (t >> 32) + (int64_t)add.w);
    z[3] = (uint32_t)t;
    const uint32_t c = (uint32_t)(t >> 32) + 0x80000000u;
    // the lane below (n, 1) is (n, 0); below (n, 0) it is (n - 1, 1)
    uint32_t lo, hi;
    half_swap(c, lo, hi);                 // lo: lane l gets c of lane l & 31; hi: of lane (l & 31) + 32
    const uint32_t up = shfl_up1(hi);
    const uint32_t prev = lane() >= 32 ? lo : (lane() == 0 ? below : up);
    uint32_t co;
    z[0] = __builtin_addc(z[0], prev, 0u, &co);
    z[1] = __builtin_addc(z[1], 0u, co, &co);
    z[2] = __builtin_addc(z[2], 0u, co, &co);
    z[3] = __builtin_addc(z[3], 0u, co, &co);
    const uint64_t G = ballot(co != 0u);
    uint64_t e = readlane(c, kLanes - 1);
    if (G) {
        // lookahead over the 32 lane pairs (n, 0), (n, 1)
        const uint64_t P = ballot((z[0] & z[1] & z[2] & z[3]) == 0xFFFFFFFFu);
        const uint32_t Gl = (uint32_t)G, Gh = (uint32_t)(G >> 32), Pl = (uint32_t)P, Ph = (uint32_t)(P >> 32);
        const uint32_t Gp = Gh | (Ph & Gl), X = Gp | (Ph & Pl);
        const uint64_t s = (uint64_t)X + Gp;
        const uint32_t cl = (uint32_t)s ^ X ^ Gp, ch = Gl | (Pl & cl);
        e += s >> 32;
        const uint32_t ci = inverse_ballot((uint64_t)ch << 32 | cl) ? 1u : 0u;
        z[0] = __builtin_addc(z[0], ci, 0u, &co);
        z[1] = __builtin_addc(z[1], 0u, co, &co);
        z[2] = __builtin_addc(z[2], 0u, co, &co);
        z[3] += co;
    }
    return e;
}

// dst[c] = limb of column c of x * y (+ R, when ADD: dst's own limbs) for c in
// [c0, ncols), mod B^(ncols - c0) above c0, but for the strips' carries: the
// carry of strip s goes to the control slots of s, and strip_carries adds it.
// Strips are dealt to the workgroup's waves round robin; dst is 16-byte
// aligned, c0 a multiple of 8 (0 with ADD).
template <int T, bool ADD>
MP_DEV void strips(uint32_t *ctl, const Operands &o, uint32_t *dst, int c0, int ncols, int base, int nstrips)
{
    const int l = lane(), k = 8 * (l & 31) + 4 * (l >> 5);
    for (int s = wave_index(); s < nstrips; s += T / kLanes) {
        const int k0 = base + s * kStrip + k;
        Limb4 add{0u, 0u, 0u, 0u};
        if (ADD && k0 >= 0 && k0 < ncols) add = load4(dst + k0);
        const MfmaAcc acc = strip_sums(o, (base >> 3) + s * (kStrip / 8));
        uint32_t z[4];
        const uint64_t e = strip_limbs(acc, add, s == 0 ? 0x80000000u : 0u, z);
        if (k0 >= c0) {
            if (k0 + 3 < ncols) {
                store4(dst + k0, z[0], z[1], z[2], z[3]);
            } else {
#pragma unroll
                for (int j = 0; j < 4; j++)
                    if (k0 + j < ncols) dst[k0 + j] = z[j];
            }
        }
        if (l == 0) {
            ctl[kCtlStrip + 2 * s] = (uint32_t)e;
            ctl[kCtlStrip + 2 * s + 1] = (uint32_t)(e >> 32);
        }
    }
}

// adds the strips' carries to dst (see strips), by one wave after a barrier:
// lane s adds the carry of strip s - 1 to the first two limbs of strip s; a
// carry out of those (rare) ripples on
MP_DEV void strip_carries(const uint32_t *ctl, uint32_t *dst, int ncols, int base, int nstrips)
{
    const int s = lane(), cb = base + s * kStrip;
    const bool on = s >= 1 && s < nstrips, two = on && cb + 1 < ncols;
    uint32_t co = 0;
    if (on) {
        const uint32_t z0 = __builtin_addc(dst[cb], ctl[kCtlStrip + 2 * s - 2], 0u, &co);
        const uint32_t z1 = __builtin_addc(two ? dst[cb + 1] : 0u, ctl[kCtlStrip + 2 * s - 1], co, &co);
        dst[cb] = z0;
        if (two) dst[cb + 1] = z1;
    }
    uint64_t m = ballot(two && co != 0u);
    while (m) {
        const int c = base + __builtin_ctzll(m) * kStrip + 2;
        m &= m - 1;
        if (c < ncols) ripple(dst + c, ncols - c, true);
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

// W for an instance without a head record, by one wave: the top limbs of v
// (at pv) and the first Refine iterations in registers, for at most
// kSmallBlock limbs of precision.  V and Wl are scratch for the divisor
// prefix and the iterate (2 kSmallBlock + 8 words each).  Returns prec(W),
// 0 if an iteration does not fit (never for dp <= kSmallBlock).
MP_DEV int small_inverse(uint32_t *lds, int offV, int offW, int k, int dp, const Shifted &v)
{
    const int iters = refine_iters(dp), hh = k + dp;
    Plan pl{};
    pl.vbase = imax(0, k - 2 * refine_l(dp, iters - 1) - 1);
    pl.capV = pl.capW = 2 * kSmallBlock + 8;
    pl.offV = offV;
    pl.offW = offW;
    for (int i = lane(); i < k + 1 - pl.vbase; i += kLanes) lds[offV + i] = v(pl.vbase + i);
    for (int i = lane(); i < pl.capW; i += kLanes) lds[offW + i] = 0u;
    wave_sync();
    int we = 0, nw = 0, l = 2;
    head_init((uint64_t)uniform(v(k)) << 32 | uniform(v(k - 1)), lds + offW, we, nw);
    for (int i = 0; i < iters; i++)
        if (!iter_fits_wave(pl, hh, k, l, nw, we) || !refine_iter_wave(pl, lds, hh, k, i, l, we, nw)) return 0;
    wave_sync();
    return nw;
}

// (q, r) with u = q v + r, 0 <= r < v: q has nq limbs, r (unless null) nv.
// U(i) is limb i of the dividend, which has at most nu limbs.  rec: the head's
// record, or nullptr when no head ran.
template <int T, class FU>
MP_DEV void divide_instance(uint32_t *lds, const FU &U, int nu, const uint32_t *v, int nv, uint32_t *q, int nq,
                            uint32_t *r, int32_t *status, const uint32_t *rec)
{
    constexpr int W = T / kLanes;
    uint32_t *ctl = lds;
    const BodyPlan pl = plan_body(nu, nv);
    uint32_t *Vd = lds + pl.offV, *Td = lds + pl.offT, *XW = lds + pl.offW, *XQ = lds + pl.offQ;
    uint32_t *P = lds + pl.offP, *R = lds + pl.offR;
    const int w = wave_index(), t = tid<T>(), nr = r ? nv : 0;
    int h = 0, k = 0, sv = 0, nw = 0, dp = 0, nb = 0, bi = 0;
    const bool valid = rec && uniform(rec[0]) == kRecValid;
    MP_RSTAMP(14);
    MP_STAMP(0);
    bar<T>();
    if (valid) {
        h = (int)uniform(rec[1]);
        k = (int)uniform(rec[2]);
        sv = (int)uniform(rec[3]);
        nw = (int)uniform(rec[4]);
        dp = (int)uniform(rec[5]);
        nb = (int)uniform(rec[6]);
        bi = (int)uniform(rec[7]);
    } else {
        // precisions, and the cases that need no division
        int32_t st = kInstOk;
        h = prec<T>(ctl, nu, U);
        k = prec<T>(ctl, nv, Span{v, 0, nv}) - 1;
        if (k < 0 || h <= k) {                        // v = 0, or u < v: (0, u)
            for (int i = t; i < nq; i += T) q[i] = 0u;
            for (int i = t; i < nr; i += T) r[i] = k >= 0 && i < h ? U(i) : 0u;
            if (status && t == 0) *status = k < 0 ? kInstDivZero : kInstOk;
            return;
        }
        const uint32_t vk = uniform(v[k]);
        const bool pow = vk == 1u && prec<T>(ctl, k, Span{v, 0, nv}) == 0;
        const int d0 = h - k;
        if (d0 - 1 > nq) {                            // q >= B^(d-2): it needs more than nq limbs
            st = kInstQWidth;
        } else if (pow) {                             // v = B^k: q = u >> k, r the limbs below
            if (d0 > nq && uniform(U(h - 1)) != 0u) {
                st = kInstQWidth;
            } else {
                for (int i = t; i < nq; i += T) q[i] = i < d0 ? U(i + k) : 0u;
                for (int i = t; i < nr; i += T) r[i] = i < k ? U(i) : 0u;
                if (status && t == 0) *status = st;
                return;
            }
        }
        if (st != kInstOk) {
            for (int i = t; i < nq; i += T) q[i] = 0u;
            for (int i = t; i < nr; i += T) r[i] = 0u;
            if (status && t == 0) *status = st;
            return;
        }
        if (k == 0) {                                 // one limb: u B / (v B)
            sv = 1;
            k = 1;
            h += 1;
        }
        const BlockSplit bs = block_split(h - k, kSmallBlock);
        dp = bs.dp;
        nb = bs.nb;
        bi = bs.bi;
        if (w == 0) {
            const int nw0 = small_inverse(lds, pl.offP, pl.offQ, k, dp, Shifted{v, nv, sv});
            if (lane() == 0) ctl[kCtlBcast] = (uint32_t)nw0;
        }
        bar<T>();
        nw = (int)uniform(ctl[kCtlBcast]);
    }
    MP_STAMP(1);
    const int d = h - k;
    // the dividend's limbs and zeros above them; the divisor's digits; W's; zero pads
    {
        for (int i0 = t; i0 < pl.capR; i0 += 8 * T) {
            uint32_t a[8];
#pragma unroll
            for (int j = 0; j < 8; j++) {
                const int i = i0 + j * T - sv;
                a[j] = i >= 0 && i < nu ? U(i) : 0u;
            }
#pragma unroll
            for (int j = 0; j < 8; j++)
                if (i0 + j * T < pl.capR) R[i0 + j * T] = a[j];
        }
        for (int i = t; i < 5 * kPadWords; i += T) {   // the planes' pads
            const int b = i / kPadWords, j = i - b * kPadWords;
            const int at = b < 3 ? pl.offV + b * pl.lyV : pl.offT + (b - 2) * pl.lyT;
            lds[at - kPadWords + j] = 0u;
        }
        const int rows = (8 * pl.nbV + 63) >> 6, per = (rows + W - 1) / W;
        const int r0 = w * per, r1 = imin(rows, r0 + per);
        if (r0 < r1)
            balance_rows(r0, r1, k + 1, 0u, Shifted{v, nv, sv}, StorePlane{Vd, 8 * pl.nbV, pl.lyV});
        if (w == W - 1) {
            // W's reversed digits (one digit limb more than its limbs)
            const uint32_t *ws = valid ? rec + kRecHdr : lds + pl.offQ;
            balance_rows(0, (nw + 64) >> 6, nw, 0u, Span{ws, 0, nw}, StoreRev{XW, nw + 1});
            if (lane() < kXPad) XW[lane() - kXPad] = 0u;
            else if (lane() < 2 * kXPad) XW[nw + 1 + lane() - kXPad] = 0u;
        }
    }
    bar<T>();
    if (w == 0 && lane() < kXPad) XQ[lane() - kXPad] = 0u;   // (after W's digits: an own W was in XQ)
    MP_STAMP(2);
    bool good = nw > 0 && nw <= dp + 3;
    const int n2 = k + 2, bs2 = (n2 + kStrip - 1) / kStrip, base2 = ((n2 + 7) & ~7) - bs2 * kStrip;
    int o = d;
    for (int i = 0; i < nb && good; i++) {
        const int op = o;
        o = (nb - 1 - i) * bi;
        const int b = op - o, nt = b + 3;             // limbs of this block, of R_top
        // R complete, R_top's digits
        if (w == 0) {
            if (i) strip_carries(ctl, R + op, n2, base2, bs2);
            const uint32_t *src = R + o + k - 1;
            balance_rows(0, (8 * pl.nbT + 63) >> 6, nt, 0u, Span{src, 0, nt}, StorePlane{Td, imin(nt, 8 * pl.nbT), pl.lyT});
            for (int j = nt + lane(); j < 8 * pl.nbT; j += kLanes) Td[plane_word(j, pl.lyT)] = 0u;
        }
        bar<T>();
        MP_STAMP(16 + 4 * (i & 3));   // (trace build: the phases of the last four blocks)
        // q_i = R_top W / B^(dp+3): columns from cA up
        const int shA = dp + 3, cA = (shA - 2) & ~7, nA = shA + b + 1, sA = (nA - cA + kStrip - 1) / kStrip;
        strips<T, false>(ctl, operands(XW, nw + 1, Td, pl.lyT, nt), P - cA, cA, nA, cA, sA);
        bar<T>();
        MP_STAMP(17 + 4 * (i & 3));
        // its limbs to the quotient, the reversed digits of -q_i
        if (w == 0) {
            strip_carries(ctl, P - cA, nA, cA, sA);
            const uint32_t *src = P + (shA - cA);
            const int nd = b + 1;
            uint32_t *Q = R + k + 2 + o;
            balance_rows(0, (nd + 63) >> 6, nd, 1u, [&](int j) { return ~src[j]; }, StoreRev{XQ, nd});
            if (lane() < kXPad) XQ[nd + lane()] = 0u;
            for (int j = lane(); j < b; j += kLanes) Q[j] = src[j];
            const int s = (int)uniform(src[b]);       // q_i's sign limb
            wave_sync();
            if (i == 0) {
                if (lane() == 0) Q[b] = (uint32_t)s;
            } else {
                add_small(Q + b, d + 1 - op, s);
            }
        }
        bar<T>();
        MP_STAMP(18 + 4 * (i & 3));
        // R -= v q_i
        strips<T, true>(ctl, operands(XQ, b + 1, Vd, pl.lyV, k + 2), R + o, 0, n2, base2, bs2);
        bar<T>();
        MP_STAMP(19 + 4 * (i & 3));
    }
    if (w == 0 && good) strip_carries(ctl, R, n2, base2, bs2);
    bar<T>();
    MP_STAMP(6);
    // corrections: R is a signed (k + 2)-limb number in (-1.1 v, 2.1 v)
    uint32_t *Q = R + k + 2, *Ra = R, *Rb = Vd;       // (the divisor's digits are no longer needed)
    const Shifted Vv{v, nv, sv};
    int delta = 0;
    for (int it = 0; good; it++) {
        bool neg = (int32_t)uniform(Ra[k + 1]) < 0, ge = uniform(Ra[k + 1]) != 0u;
        if (!ge) {                                    // compare with v from the top, 64 limbs at a time
            ge = true;                                // (equal: R = v)
            for (int c = k; c >= 0; c -= kLanes) {
                const int j = c - (kLanes - 1) + lane();
                const uint32_t a = j >= 0 ? Ra[j] : 0u, x = j >= 0 ? Vv(j) : 0u;
                const uint64_t ne = ballot(a != x), gt = ballot(a > x);
                if (ne) {
                    ge = (gt >> (63 - __builtin_clzll(ne))) & 1u;
                    break;
                }
            }
        }
        if (!neg && !ge) break;
        if (it == 4) {
            good = false;
            break;
        }
        const int rows = (n2 + 63) >> 6, per = (rows + W - 1) / W;
        const int r0 = w * per, r1 = imin(rows, r0 + per);
        if (r0 < r1) addsub_rows(r0, r1, n2, !neg, Span{Ra, 0, n2}, Vv, Rb);
        delta += neg ? -1 : 1;
        bar<T>();
        uint32_t *x = Ra;
        Ra = Rb;
        Rb = x;
    }
    if (good && delta) {
        if (w == 0) add_small(Q, d + 1, delta);
        bar<T>();
    }
    MP_STAMP(7);
    int32_t st = good ? kInstOk : kInstInternal;
    if (good && uniform(Q[d]) != 0u) st = kInstInternal;
    if (st == kInstOk && d > nq) {                    // (d <= nq + 1)
        if (uniform(Q[d - 1]) != 0u) st = kInstQWidth;
    }
    const bool ok = st == kInstOk;
    for (int i = t; i < nq; i += T) q[i] = ok && i < d ? Q[i] : 0u;
    for (int i = t; i < nr; i += T) r[i] = ok && i <= k - sv ? Ra[i + sv] : 0u;
    if (status && t == 0) *status = st;
    MP_STAMP(8);
    MP_RSTAMP(15);
}

}  // namespace mp
