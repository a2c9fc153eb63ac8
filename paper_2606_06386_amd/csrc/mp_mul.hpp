// Products, one per workgroup: c = a * b (the method's Mult, Sec. 3.3).
//
// On the int8 matrix cores (mul_instance) each wave owns G adjacent strips of
// 256 columns and all their diagonals.  With d = r + 32 m, strip i of the group
// at diagonal d reads the long operand's blocks from S0 + 32 (i - m) - r on: for
// a fixed r they depend on q = i - m only.  So for each r the wave walks q
// downwards with one fragment of the long operand per step and a window of G
// Toeplitz fragments m = i - q of the short one, of which one is new: two
// fragments read for G products.  LDS reads bound a product otherwise (18 LDS
// cycles per fragment pair against 8 matrix-core cycles of a compute unit's
// four): G = 4 reads 4.5 cycles' worth per product, pairs of strips with one
// shared fragment 13.  4096 products of 2048 x 2048 limbs: 301 -> 264 us (the
// matrix cores busy 67% of the time, at the 1.7 GHz the chip holds under them),
// 256 of 8192 x 8192: 254 -> 210 us, 2000 of 1531 x 333: 34 -> 25 us.
//
// The limbs go from the accumulators to global memory in registers; a strip's
// carry goes to the next strip of the group in registers and to the next
// group through LDS.
//
// Short operands (below mfma_min limbs) take the vector ALU (mul_valu_instance).
#pragma once

#include <stdint.h>

#include "launch.hpp"
#include "mp_strip.hpp"

namespace mp {

struct MulPlan {
    int nbY, lyY, offY, offX, total;   // long digits: blocks, distance of the planes, first word; reversed short digits
};

MP_HD constexpr MulPlan plan_mul(int na, int nb)
{
    MulPlan p{};
    const int lo = hmin(na, nb), hi = hmax(na, nb);
    p.nbY = (hi + 1 + 7) >> 3;
    p.offY = kCtlWords + kPadWords;
    p.lyY = 4 * p.nbY + kPadWords;
    p.offX = p.offY + 2 * p.lyY + kXPad;
    p.total = r4(p.offX + lo + 1 + kXPad);
    return p;
}

MP_HD int mul_valu_lds_words(int na, int nb)
{
    const int lo = na < nb ? na : nb, hi = na < nb ? nb : na;
    return kCtlWords + r4(lo + 1) + 4 + kPad + r4(hi + 1) + kPad + r4(na + nb) + 4;
}

struct Operands {
    uint32_t x, sft;     // the short digits (see ShortDigits)
    int dmax;
    uint32_t y;          // LDS byte address of this lane's word of the long digits' planes for block 0
    int nyblk;           // blocks of the long digits
};

// xr: nx reversed digit limbs; yb: planes (distance ly) of ny digit limbs
MP_DEV Operands operands(int l, const uint32_t *xr, int nx, const uint32_t *yb, int ly, int ny)
{
    const ShortDigits s = short_digits(l, xr, nx);
    return Operands{s.x, s.sft, s.dmax, lds_address(yb) + 4 * ((l >> 5) * ly + 4 * (l & 31)), (ny + 7) >> 3};
}

// acc += the diagonals [d, dhi] of the strip whose first block is S0
MP_DEV void diagonal_sums(const Operands &o, int S0, int d, int dhi, MfmaAcc &acc)
{
    constexpr int D = 4;   // diagonals whose operands are in flight
    uint32_t x = opaque(o.x - 32 * (d + D - 1)), y = opaque(o.y + 16 * (S0 - d - (D - 1)));
    int n = uniform(dhi - d + 1);
    for (; n >= D; n -= D) {
        XRaw r[D];
        Limb4 v[D];
#pragma unroll
        for (int j = 0; j < D; j++) {
            r[j] = xraw_at(x, 8 * (D - 1 - j));
            v[j] = lds_quad(y, D - 1 - j);
        }
#pragma unroll
        for (int j = 0; j < D; j++) acc = mfma_x(acc, xfrag(r[j], o.sft), v[j]);
        sched_loads_first();
        x -= 32 * D;
        y -= 16 * D;
    }
    for (; n > 0; n--) {
        acc = mfma_x(acc, xfrag(xraw_at(x, 8 * (D - 1)), o.sft), lds_quad(y, D - 1));
        x -= 32;
        y -= 16;
    }
}

// The sums of G adjacent strips, the first starting at block S0, for a short
// operand of fewer than 32 G diagonals: those that every strip needs share
// each Toeplitz fragment, the rest strip by strip.
template <int G>
MP_DEV void group_sums_short(const Operands &o, int S0, MfmaAcc (&acc)[G])
{
#pragma unroll
    for (int i = 0; i < G; i++) acc[i] = mfma_zero();
    const int lo = imax(0, S0 + 32 * (G - 1) - o.nyblk + 1), hi = imin(o.dmax, S0 + 31);
    if constexpr (G == 1) {
        diagonal_sums(o, S0, lo, hi, acc[0]);
        return;
    }
    uint32_t x = opaque(o.x - 32 * lo), y = opaque(o.y + 16 * (S0 - lo));
    for (int n = uniform(hi - lo); n >= 0; n--) {
        const XRaw r = xraw_at(x, 0);
        Limb4 v[G];
#pragma unroll
        for (int i = 0; i < G; i++) v[i] = lds_quad(y, 32 * i);
        const XFrag f = xfrag(r, o.sft);
#pragma unroll
        for (int i = 0; i < G; i++) acc[i] = mfma_x(acc[i], f, v[i]);
        sched_loads_first();
        x -= 32;
        y -= 16;
    }
#pragma unroll
    for (int i = 0; i < G; i++) {
        const int S = S0 + 32 * i, li = imax(0, S - o.nyblk + 1), hi_i = imin(o.dmax, S + 31);
        if (lo > hi) {
            diagonal_sums(o, S, li, hi_i, acc[i]);
        } else {
            diagonal_sums(o, S, li, lo - 1, acc[i]);
            diagonal_sums(o, S, hi + 1, hi_i, acc[i]);
        }
    }
}

// Scheduling of G steps: all their LDS reads first, then per step the aligns of
// its new fragment and its products
template <int G>
MP_DEV void sched_chunk()
{
    __builtin_amdgcn_sched_group_barrier(0x100, 8 * G, 0);   // DS reads
#pragma unroll
    for (int u = 0; u < G; u++) {
        __builtin_amdgcn_sched_group_barrier(0x002, 4, 0);   // VALU
        __builtin_amdgcn_sched_group_barrier(0x008, G, 0);   // MFMA
    }
}

// The same for a short operand of at least 32 G diagonals, with a window of G
// Toeplitz fragments (see the top of this file).  For each r the steps q are:
// head (q > 0): strips i >= q, the fragments m = i - q < G - 1; main: all
// strips, one new fragment per step; tail (m beyond the last fragment M for
// the upper strips): strips i <= q + M, no new fragment.
template <int G>
MP_DEV void group_sums(const Operands &o, int S0, MfmaAcc (&acc)[G])
{
#pragma unroll
    for (int i = 0; i < G; i++) acc[i] = mfma_zero();
    for (int r = 0; r < 32; r++) {
        const int M = (o.dmax - r) >> 5;                              // m = 0 .. M, M >= G - 1
        const int qt = imin(G - 1, (o.nyblk - 1 - S0 + r) >> 5);      // steps qt .. qb hold nonzero blocks
        const int qb = imax(-M, -((S0 + 31 - r) >> 5));
        int q = imin(qt, 0);
        if (q < qb) continue;
        uint32_t x = opaque(o.x - 32 * r + 1024 * q), y = opaque(o.y + 16 * (S0 - r + 32 * q));   // of X_(-q), Y_q
        XFrag w[G];                                                   // w[i] = X_(i-q)
#pragma unroll
        for (int i = 0; i + 1 < G; i++)
            if (i - q <= M) w[i] = xfrag(xraw_at(x - 1024 * i, 0), o.sft);
#pragma unroll
        for (int h = G - 1; h >= 1; h--)
            if (h <= qt) {
                const Limb4 v = lds_quad(y + 512 * h, 0);
#pragma unroll
                for (int i = h; i < G; i++) acc[i] = mfma_x(acc[i], w[i - h], v);
            }
        int n = q - imax(qb, G - 1 - M) + 1;                          // main steps
        q -= imax(n, 0);
        for (; n >= G; n -= G) {
            XRaw raw[G];
            Limb4 v[G];
#pragma unroll
            for (int u = 0; u < G; u++) {
                raw[u] = xraw_at(x - 1024 * (G - 1 + u), 0);
                v[u] = lds_quad(y - 512 * u, 0);
            }
#pragma unroll
            for (int u = 0; u < G; u++) {
                w[(u + G - 1) % G] = xfrag(raw[u], o.sft);
#pragma unroll
                for (int i = 0; i < G; i++) acc[i] = mfma_x(acc[i], w[(u + i) % G], v[u]);
            }
            sched_chunk<G>();
            x -= 1024 * G;
            y -= 512 * G;
        }
        for (; n > 0; n--) {
            w[G - 1] = xfrag(xraw_at(x - 1024 * (G - 1), 0), o.sft);
            const Limb4 v = lds_quad(y, 0);
#pragma unroll
            for (int i = 0; i < G; i++) acc[i] = mfma_x(acc[i], w[i], v);
#pragma unroll
            for (int i = 0; i + 1 < G; i++) w[i] = w[i + 1];
            x -= 1024;
            y -= 512;
        }
        for (; q >= qb; q--) {
            const Limb4 v = lds_quad(y, 0);
#pragma unroll
            for (int i = 0; i + 1 < G; i++)
                if (i <= q + M) acc[i] = mfma_x(acc[i], w[i], v);
#pragma unroll
            for (int i = 0; i + 2 < G; i++) w[i] = w[i + 1];
            y -= 512;
        }
    }
}

// z += e at limb 0 of the 256-limb number; returns the signed carry out
MP_DEV int quad_add_signed(int l, uint32_t (&z)[4], int e)
{
    const bool first = l == 0;
    const uint32_t x[4] = {z[0], z[1], z[2], z[3]};
    const int el = first ? e : 0;
    if (add64_carry(z[0], z[1], el) == ballot(el < 0)) return 0;
    const uint32_t s = (uint32_t)(e >> 31), b[4] = {first ? (uint32_t)e : s, s, s, s};
#pragma unroll
    for (int j = 0; j < 4; j++) z[j] = x[j];
    return (int)quad_add(z, b, 0u) + (e >> 31);
}

// c = a * b  (c has na + nb limbs) by W = T / 64 waves: wave w owns the groups
// w and (K = 2) w + W of G strips each; na + nb <= 256 G K W limbs
template <int T, int G, int K>
MP_DEV void mul_instance(uint32_t *lds, const uint32_t *a, int na, const uint32_t *b, int nb, uint32_t *c)
{
    constexpr int W = T / kLanes;
    uint32_t *ctl = lds;
    const MulPlan pl = plan_mul(na, nb);
    const int nx = na < nb ? na : nb, ny = na < nb ? nb : na, nc = na + nb;
    const uint32_t *x = na < nb ? a : b, *y = na < nb ? b : a;
    uint32_t *Y = lds + pl.offY, *X = lds + pl.offX;
    const int w = wave_index(), l = lane_at(nc), t = w * kLanes + l;
    MP_RSTAMP(6);
    MP_STAMP(0);
    for (int i = t; i < 3 * kPadWords; i += T) {
        const int p = i / kPadWords;
        Y[p * pl.lyY - kPadWords + i - p * kPadWords] = 0u;
    }
    if (w == 0 && l < 2 * kXPad) X[l < kXPad ? l - kXPad : nx + 1 + l - kXPad] = 0u;
    {
        // rows of both operands, dealt to the waves in contiguous runs
        const int ry = (8 * pl.nbY + 63) >> 6, rx = (nx + 64) >> 6, per = (ry + rx + W - 1) / W;
        const int r0 = w * per, r1 = r0 + per;
        if (r0 < ry) balance_rows(l, r0, imin(ry, r1), ny, 0u, Span{y, 0, ny}, StorePlane{Y, 8 * pl.nbY, pl.lyY});
        if (r1 > ry && r0 < ry + rx)
            balance_rows(l, imax(0, r0 - ry), imin(rx, r1 - ry), nx, 0u, Span{x, 0, nx}, StoreRev{X, nx + 1});
    }
    sync();
    MP_STAMP(1);
    const int ns = (nc + kStrip - 1) / kStrip;
    uint32_t z[K][G][4];
#pragma unroll
    for (int k = 0; k < K; k++) {
        // With one group per wave the middle ones have the most diagonals:
        // neighbouring workgroups of a compute unit (256 apart) deal them to
        // different SIMDs.  Groups w and w + W together have as many for every w.
        const int g = K == 1 && G > 1 ? (w + (int)(blockIdx.x >> 8)) % W : w + W * k, s0 = g * G;
        int e = 0;
        if (s0 < ns) {
            const int lk = lane_at(k);
            MfmaAcc acc[G];
            const Operands o = operands(lk, X, nx + 1, Y, pl.lyY, ny + 1);
            if (G > 1 && o.dmax + 1 >= 32 * G) group_sums<G>(o, s0 * (kStrip / 8), acc);
            else group_sums_short<G>(o, s0 * (kStrip / 8), acc);
            MP_STAMP(2 + k);
#pragma unroll
            for (int i = 0; i < G; i++) {
                const int ei = strip_limbs<false>(lk, acc[i], Limb4{0u, 0u, 0u, 0u}, z[k][i]);
                e = ei + (i ? quad_add_signed(lk, z[k][i], e) : 0);
            }
        }
        if (l == 0) ctl[kCtlStrip + g] = (uint32_t)e;
    }
    sync();
    MP_STAMP(4);
    const bool quads = ((nc | (int)((uintptr_t)c >> 2)) & 3) == 0;
#pragma unroll
    for (int k = 0; k < K; k++) {
        const int g = K == 1 && G > 1 ? (w + (int)(blockIdx.x >> 8)) % W : w + W * k, s0 = g * G;
        // the carry of the group below; one that runs through the whole group
        // (long runs of zeros or ones) is added once everything is stored
        int over = 0;
        if (s0 < ns) {
            over = g ? (int)uniform(ctl[kCtlStrip + g - 1]) : 0;
#pragma unroll
            for (int i = 0; i < G; i++)
                if (over) over = quad_add_signed(l, z[k][i], over);
#pragma unroll
            for (int i = 0; i < G; i++) {
                const int k0 = (s0 + i) * kStrip + quad_limb(l);
                if (quads) {
                    if (k0 < nc) store4(c + k0, z[k][i][0], z[k][i][1], z[k][i][2], z[k][i][3]);
                } else {
#pragma unroll
                    for (int j = 0; j < 4; j++)
                        if (k0 + j < nc) c[k0 + j] = z[k][i][j];
                }
            }
        }
        if (l == 0) ctl[kCtlOver + g] = (uint32_t)over;
    }
    sync();
    if (w == 0) {
        const int v = l < K * W ? (int)ctl[kCtlOver + l] : 0;
        for (uint64_t m = ballot(v != 0); m; m &= m - 1) {
            const int i = __builtin_ctzll(m), at = (i + 1) * G * kStrip;
            if (at < nc) ripple(l, c + at, nc - at, (int)readlane((uint32_t)v, i) > 0);
        }
    }
    MP_STAMP(5);
    MP_RSTAMP(7);
}

// c = a * b on the vector ALU
template <int T>
MP_DEV void mul_valu_instance(uint32_t *lds, const uint32_t *a, int na, const uint32_t *b, int nb, uint32_t *c)
{
    uint32_t *ctl = lds;
    const int nlo = na < nb ? na : nb, nhi = na < nb ? nb : na;
    const uint32_t *sht = na < nb ? a : b, *lng = na < nb ? b : a;
    uint32_t *A = lds + kCtlWords;                  // short operand (rows)
    uint32_t *SB = A + r4(nlo + 1) + 4 + kPad;      // long operand (window)
    uint32_t *P = SB + r4(nhi + 1) + kPad;
    copy<T>(A, nlo, r4(nlo) + 4, Span{sht, 0, nlo});
    copy<T>(SB - kPad, kPad + nhi, 2 * kPad + r4(nhi), Span{lng, kPad, nhi});
    mul<T>(ctl, P, A, nlo, SB, nhi);
    sync();
    if (wave_index() == 0) {
        // lane s adds the 64-bit carry of strip s - 1 to the first two limbs of strip s (a carry out of those ripples on)
        const int nc = na + nb, ns = (nc + kStrip - 1) / kStrip, s = lane(), at = s * kStrip;
        const bool on = s >= 1 && s < ns, two = on && at + 1 < nc;
        const uint64_t x = ((uint64_t)(two ? P[at + 1] : 0u) << 32) | (on ? P[at] : 0u);
        const uint32_t *e = ctl + kCtlStrip + 2 * (on ? s - 1 : 0);
        const uint64_t y = x + (on ? ((uint64_t)e[1] << 32) | e[0] : 0u);
        if (on) P[at] = (uint32_t)y;
        if (two) P[at + 1] = (uint32_t)(y >> 32);
        for (uint64_t m = ballot(two && y < x); m; m &= m - 1) {
            const int k = __builtin_ctzll(m) * kStrip + 2;
            if (k < nc) ripple(lane(), P + k, nc - k, true);
        }
    }
    sync();
    for (int i = (int)threadIdx.x; i < na + nb; i += T) c[i] = P[i];
}

}  // namespace mp
