// Carry passes and products shared by the division (mp_block.hpp) and the
// product (mp_mul.hpp): balanced radix-256 digits, exact int8 matrix-core
// products of them, and the way back to limbs.
//
// A number is rewritten in radix 256 with balanced digits in [-128, 127]:
// adding 0x80 to every byte and carrying makes the digit bytes
// (x + 0x8080...80) XOR 0x8080...80 limb by limb, and the carry out of the top
// limb is one more digit (0 or 1).  The byte-column sums of a product of such
// digits are exact int32 values (below 2^29 for 8192-limb operands).
#pragma once

#include <stdint.h>

namespace mp {

constexpr int kPadBlk = 32, kPadWords = 4 * kPadBlk;   // zero blocks a strip may read on each side of a digit plane
constexpr int kXPad = 16;            // zero words it reads on each side of the reversed short operand
constexpr int kXLow = kXPad + 8;     // and below it where diagonals are taken in pairs

constexpr int kStripBlks = kStrip / 8;

// The long operand's digits lie in two planes of 16-byte half-blocks (plane h
// holds bytes 16h .. 16h + 15 of every 32-byte block), so that the lanes of
// either half-wave read 32 consecutive 16-byte chunks of one plane; the short
// operand's lie byte-reversed, so that a Toeplitz row is 16 consecutive bytes.
// word of the planes holding limb k: block k / 8, plane (k / 4) % 2, word k % 4
MP_DEV int plane_word(int k, int ly) { return ((k >> 1) & ~3) + (k & 3) + ((k >> 2) & 1) * ly; }

// A divisor's lie in four, 2r + h holding the half-blocks h of the even (r = 0)
// or odd blocks, so that every second of 64 blocks is read in consecutive chunks
// (see strip_sums2).  Planes 16 words apart modulo 32 keep the even and odd
// lanes of a read of 32 consecutive blocks on different banks (if the first is
// an odd one, all but three in sixteen).
MP_DEV int plane4_word(int k, int ly)
{
    return (((k >> 3) & 1) * 2 + ((k >> 2) & 1)) * ly + ((k >> 4) << 2) + (k & 3);
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

constexpr uint32_t kBal = 0x80808080u, kBalTop = 0x7F7F7F7Fu;   // (limbs above kBalTop carry)
constexpr int kRowBatch = 5;   // rows read at once (an iterate's 257 + 2 limbs)

// out(k, digit limb) for the limbs k of rows [r0, r1): the balanced radix-256
// digits of the n-limb number x with carry-in cin0 at limb 0.  Limb n gets the
// top carry digit (0 or 1), limbs above it zero.
template <class FX, class FO>
MP_DEV void balance_rows(int ln, int r0, int r1, int n, uint32_t cin0, const FX &x, const FO &out)
{
    uint32_t c = cin0;
    for (int r = r0 - 1; r >= 0; r--) {          // (rows below r0 lie inside [0, n))
        const uint32_t s = x(64 * r + ln) + kBal;
        const uint64_t G = ballot(s < kBal), P = ballot(s == 0xFFFFFFFFu);
        if (~P) {
            c = row_carry_out(G, P);
            break;
        }
    }
    for (int r = r0; r < r1; r += kRowBatch) {
        uint32_t xv[kRowBatch];
#pragma unroll
        for (int j = 0; j < kRowBatch; j++) {
            const int k = 64 * (r + j) + ln;
            xv[j] = r + j < r1 && k < n ? x(k) : 0u;
        }
#pragma unroll
        for (int j = 0; j < kRowBatch; j++) {
            if (r + j < r1) {
                const int k = 64 * (r + j) + ln;
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

struct StorePlane4 {
    uint32_t *p;
    int n, ly;
    MP_DEV void operator()(int k, uint32_t z) const
    {
        if (k < n) p[plane4_word(k, ly)] = z;
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
MP_DEV void addsub_rows(int ln, int r0, int r1, int n, bool sub, const FX &x, const FY &y, uint32_t *dst)
{
    uint32_t c = 0;
    for (int r = r0 - 1; r >= 0; r--) {
        const int k = 64 * r + ln;
        const uint32_t a = x(k), b = y(k), z = sub ? a - b : a + b;
        const uint64_t G = ballot(sub ? a < b : z < a), P = ballot(z == (sub ? 0u : 0xFFFFFFFFu));
        if (~P) {
            c = row_carry_out(G, P);
            break;
        }
    }
    for (int r = r0; r < r1; r++) {
        const int k = 64 * r + ln;
        const uint32_t a = k < n ? x(k) : 0u, b = k < n ? y(k) : 0u, z = sub ? a - b : a + b;
        const uint64_t cm = row_carries(ballot(sub ? a < b : z < a), ballot(z == (sub ? 0u : 0xFFFFFFFFu)), c);
        const uint32_t ci = inverse_ballot(cm) ? 1u : 0u;
        if (k < n) dst[k] = sub ? z - ci : z + ci;
    }
}

// p[0, n) += 1 (up) or -= 1, by one wave: stops at the first limb that does not pass the carry on
MP_DEV void ripple(int l, uint32_t *p, int n, bool up)
{
    const uint32_t pass = up ? 0xFFFFFFFFu : 0u;
    for (int b = 0; b < n; b += kLanes) {
        const int k = b + l;
        wave_sync();
        const uint32_t x = k < n ? p[k] : pass;
        const uint64_t m = ballot(x != pass);
        if (k < n && (m == 0 || l <= __builtin_ctzll(m))) p[k] = up ? x + 1u : x - 1u;
        wave_sync();
        if (m) return;
    }
}

// p[0, n) += s for a small signed s, by one wave
MP_DEV void add_small(int l, uint32_t *p, int n, int s)
{
    if (s == 0 || n <= 0) return;
    wave_sync();
    const uint32_t x = uniform(p[0]), z = x + (uint32_t)s;
    wave_sync();
    if (l == 0) p[0] = z;
    wave_sync();
    if (s > 0 ? z < x : z > x) ripple(l, p + 1, n - 1, s > 0);
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

// X_d of this lane: 16 bytes of the reversed short digits from word xp on,
// shifted by sft bytes (five words read, four byte aligns)
struct XRaw {
    uint32_t w0, w1, w2, w3, w4;
};
struct XFrag {
    uint32_t a, b, c, d;
};

MP_DEV XFrag xfrag(const XRaw &r, uint32_t sft)
{
    return XFrag{alignbyte(r.w1, r.w0, sft), alignbyte(r.w2, r.w1, sft), alignbyte(r.w3, r.w2, sft),
                 alignbyte(r.w4, r.w3, sft)};
}

// Scheduling of one diagonal step: its LDS reads first (all in flight
// together), then the vector ALU work (byte aligns, addresses), then the
// matrix-core products; without this the scheduler of a kernel near its
// register limit interleaves them and pays one LDS round trip per product.
MP_DEV void sched_loads_first()
{
    __builtin_amdgcn_sched_group_barrier(0x100, 32, 0);   // DS reads
    __builtin_amdgcn_sched_group_barrier(0x002, 32, 0);   // VALU
    __builtin_amdgcn_sched_group_barrier(0x008, 4, 0);    // MFMA
}

MP_DEV MfmaAcc mfma_x(MfmaAcc acc, const XFrag &x, const Limb4 &y)
{
    return mfma_i8(acc, x.a, x.b, x.c, x.d, y.x, y.y, y.z, y.w);
}

struct ShortDigits {
    uint32_t x;          // LDS byte address of this lane's word of the reversed short digits at diagonal 0
    uint32_t sft;        // and its byte shift
    int dmax;            // last diagonal that touches them
};

// xr: nx reversed digit limbs
MP_DEV ShortDigits short_digits(int l, const uint32_t *xr, int nx)
{
    const int p = l & 31, h = l >> 5;
    const int ox = 16 * h - 1 - (16 * ((p >> 2) & 1) + 4 * (p >> 3) + (p & 3));   // (from the end of the digits)
    return ShortDigits{lds_address(xr + nx) + 4 * (ox >> 2), (uint32_t)ox & 3u, (4 * nx + 30) >> 5};
}

// those of nx limbs from word `at` on, from those of none at word 0
MP_DEV ShortDigits short_digits(const ShortDigits &none, int at, int nx)
{
    return ShortDigits{none.x + 4 * (at + nx), none.sft, (4 * nx + 30) >> 5};
}

MP_DEV XRaw xraw_at(uint32_t a, int w)
{
    return XRaw{lds_word(a, w), lds_word(a, w + 1), lds_word(a, w + 2), lds_word(a, w + 3), lds_word(a, w + 4)};
}

// ny digit limbs in two planes at p: LDS byte address of this lane's half of the
// 32 blocks from B on
struct Planes {
    static constexpr int kStep = 32;   // (two blocks)
    uint32_t y;
    int ny;
    MP_DEV uint32_t at(int B) const { return y + 16 * B; }
};

MP_DEV Planes planes(int l, const uint32_t *p, int ly, int ny)
{
    return Planes{lds_address(p) + 4 * (l >> 5) * ly + 16 * (l & 31), ny};
}

// the same in four planes, and of the 32 blocks B, B + 2, ..
struct Planes4 {
    static constexpr int kStep = 16;
    uint32_t even, odd;   // from block 0 and from block 1 on
    uint32_t alt;         // the blocks 0, 2, ..
    int ly, ny;
    MP_DEV uint32_t at(int B) const
    {
        const uint32_t e = even, o = odd;
        return (B & 1 ? o : e) + 16 * (B >> 1);
    }
    MP_DEV uint32_t alternate(int B) const { return alt + 8 * (B & 1) * ly + 16 * (B >> 1); }
};

MP_DEV Planes4 planes4(int l, const uint32_t *p, int ly, int ny)
{
    const uint32_t a = lds_address(p) + 4 * (l >> 5) * ly;
    const int n = l & 31, r = 8 * ly;
    return Planes4{a + 16 * (n >> 1) + (n & 1 ? r : 0), a + 16 * ((n + 1) >> 1) + (n & 1 ? 0 : r), a + 16 * n, ly, ny};
}

// the operands of two diagonals, the second at the addresses x and y1
struct Diagonals {
    XRaw r0, r1;
    Limb4 v0, v1;
    MP_DEV void load(uint32_t x, uint32_t y0, uint32_t y1)
    {
        r0 = xraw_at(x, 8);
        v0 = lds_quad(y0, 0);
        r1 = xraw_at(x, 0);
        v1 = lds_quad(y1, 0);
    }
    MP_DEV void add(MfmaAcc &acc, uint32_t sft) const
    {
        acc = mfma_x(acc, xfrag(r0, sft), v0);
        acc = mfma_x(acc, xfrag(r1, sft), v1);
    }
};

// The accumulator of the strip whose first block is S0, or the share `part` of
// `parts` of its diagonals (the first share the smallest).  Steps of two
// diagonals; the last may pass the end: it reads zeros there (of the short
// digits, or blocks below the long ones').  FAST, for kernels with registers to
// spare and few waves per SIMD to hide LDS reads behind: the next step's
// operands in flight.
template <bool FAST, class Y>
MP_DEV MfmaAcc strip_sums(const ShortDigits &o, const Y &q, int S0, int part = 0, int parts = 1)
{
    MfmaAcc acc = mfma_zero();
    const int dlo = imax(0, S0 - ((q.ny + 7) >> 3) + 1), dhi = imin(o.dmax, S0 + 31);
    int n = uniform(dhi - dlo + 2) >> 1;         // steps
    if (n <= 0) return acc;
    const int first = n * part / parts, d0 = dlo + 2 * first;
    n = n * (part + 1) / parts - first;
    // (address of a step's second diagonal: the first lies at a positive offset)
    uint32_t x = opaque(o.x - 32 * (d0 + 1)), y0 = opaque(q.at(S0 - d0)), y1 = opaque(q.at(S0 - d0 - 1));
    constexpr int S = Y::kStep;
    if constexpr (FAST) {
        Diagonals a, b;
        a.load(x, y0, y1);
        for (; n >= 2; n -= 2) {                 // (the reads past the last step are not used)
            b.load(x - 64, y0 - S, y1 - S);
            a.add(acc, o.sft);
            sched_loads_first();
            x -= 128;
            y0 -= 2 * S;
            y1 -= 2 * S;
            a.load(x, y0, y1);
            b.add(acc, o.sft);
            sched_loads_first();
        }
        if (n) a.add(acc, o.sft);
    } else {
        for (; n > 0; n--) {
            Diagonals a;
            a.load(x, y0, y1);
            a.add(acc, o.sft);
            sched_loads_first();
            x -= 64;
            y0 -= S;
            y1 -= S;
        }
    }
    return acc;
}

// Two adjacent strips at once, of every second block each: accE holds the sums of
// the blocks P0, P0 + 2, .., accO those between.  Both must need all diagonals
// [0, dmax] (P0 >= dmax - 31).  What the even blocks multiply by diagonal m the
// odd ones multiply by m + 1, so a step reads one fragment of each operand for
// two products (18 LDS cycles; two fragments of the long operand, for strips one
// behind the other, 26: LDS reads bind a compute unit full of instances).
template <bool FAST>
MP_DEV void strip_sums2(const ShortDigits &o, const Planes4 &q, int P0, MfmaAcc &accE, MfmaAcc &accO)
{
    accE = mfma_zero();
    accO = mfma_zero();
    const int dmax = uniform(o.dmax), odd = dmax & 1;
    XFrag w = xfrag(xraw_at(o.x, 0), o.sft);     // X_m
    accO = mfma_x(accO, w, lds_quad(q.alternate(P0 + 1), 0));
    const auto step = [&](const XRaw &r, const Limb4 &v) {
        accE = mfma_x(accE, w, v);
        w = xfrag(r, o.sft);
        accO = mfma_x(accO, w, v);
    };
    if (odd) step(xraw_at(o.x - 32, 0), lds_quad(q.alternate(P0), 0));
    // (m, m + 1) per step
    uint32_t x = opaque(o.x - 32 * (odd + 2)), y0 = opaque(q.alternate(P0 - odd)),
             y1 = opaque(q.alternate(P0 - odd - 1));
    int n = dmax >> 1;
    if constexpr (FAST) {
        Diagonals a, b;
        a.load(x, y0, y1);
        for (; n >= 2; n -= 2) {                 // (the reads past the last step are not used)
            b.load(x - 64, y0 - 16, y1 - 16);
            step(a.r0, a.v0);
            step(a.r1, a.v1);
            sched_loads_first();
            x -= 128;
            y0 -= 32;
            y1 -= 32;
            a.load(x, y0, y1);
            step(b.r0, b.v0);
            step(b.r1, b.v1);
            sched_loads_first();
        }
        if (n) {
            step(a.r0, a.v0);
            step(a.r1, a.v1);
            a.v0 = lds_quad(y0 - 16, 0);
        }
        accE = mfma_x(accE, w, a.v0);            // (m = dmax)
    } else {
        for (; n > 0; n--) {
            const XRaw r0 = xraw_at(x, 8);
            const Limb4 v0 = lds_quad(y0, 0);
            step(r0, v0);
            sched_loads_first();
            const XRaw r1 = xraw_at(x, 0);
            const Limb4 v1 = lds_quad(y1, 0);
            step(r1, v1);
            sched_loads_first();
            x -= 64;
            y0 -= 16;
            y1 -= 16;
        }
        accE = mfma_x(accE, w, lds_quad(y0, 0));
    }
}

// an accumulator through LDS, 1024 words from p, and its sum with another
MP_DEV void acc_store(int l, const MfmaAcc &a, uint32_t *p)
{
#pragma unroll
    for (int j = 0; j < 4; j++)
        store4(p + 256 * j + 4 * l, (uint32_t)a[4 * j], (uint32_t)a[4 * j + 1], (uint32_t)a[4 * j + 2],
               (uint32_t)a[4 * j + 3]);
}

MP_DEV void acc_add(int l, MfmaAcc &a, const uint32_t *p)
{
#pragma unroll
    for (int j = 0; j < 4; j++) {
        const Limb4 v = load4(p + 256 * j + 4 * l);
        a[4 * j] += (int)v.x;
        a[4 * j + 1] += (int)v.y;
        a[4 * j + 2] += (int)v.z;
        a[4 * j + 3] += (int)v.w;
    }
}

// A number of up to 256 limbs in one wave's registers: lane (n, h) = n + 32 h
// holds the limbs 8n + 4h .. 8n + 4h + 3, which is also the half-block h of
// block n in the planes.
MP_DEV int quad_limb(int l) { return 8 * (l & 31) + 4 * (l >> 5); }

// limb i (the same in every lane) of such a number
MP_DEV uint32_t quad_get(const uint32_t (&z)[4], int i)
{
    const int j = i & 3;
    const uint32_t x = j == 0 ? z[0] : j == 1 ? z[1] : j == 2 ? z[2] : z[3];
    return readlane(x, ((i >> 3) & 31) + ((i & 4) << 3));
}

// the lanes next above those of mask m (in limb order), the lowest lane getting cin
MP_DEV uint64_t quad_up(uint64_t m, uint32_t cin)
{
    const uint32_t lo = (uint32_t)m, hi = (uint32_t)(m >> 32);
    return (uint64_t)lo << 32 | (hi << 1 | cin);
}

// z += b + cin, b[j] in limb j of each lane's four; returns the carry out of
// the 256 limbs.  The general case: a lookahead over the 32 lane pairs (n, 0),
// (n, 1).
MP_DEV uint32_t quad_add(uint32_t (&z)[4], const uint32_t (&b)[4], uint32_t cin)
{
    uint32_t co = 0;
#pragma unroll
    for (int j = 0; j < 4; j++) z[j] = __builtin_addc(z[j], b[j], co, &co);
    const uint64_t G = ballot(co != 0u), P = ballot((z[0] & z[1] & z[2] & z[3]) == 0xFFFFFFFFu);
    const uint32_t Gl = (uint32_t)G, Gh = (uint32_t)(G >> 32), Pl = (uint32_t)P, Ph = (uint32_t)(P >> 32);
    const uint32_t Gp = Gh | (Ph & Gl), X = Gp | (Ph & Pl);
    const uint64_t s = (uint64_t)X + Gp + cin;
    const uint32_t cl = (uint32_t)s ^ X ^ Gp, ch = Gl | (Pl & cl);
    z[0] = __builtin_addc(z[0], 0u, inverse_ballot((uint64_t)ch << 32 | cl) ? 1u : 0u, &co);
    z[1] = __builtin_addc(z[1], 0u, co, &co);
    z[2] = __builtin_addc(z[2], 0u, co, &co);
    z[3] += co;
    return (uint32_t)(s >> 32);
}

// The balanced digits of the number in z, with carry-in cin.  A limb above
// kBalTop carries, whatever comes in; a limb equal to it passes an incoming
// carry on, which shows as a sum of 0: then (one limb in 2^32) the carries are
// resolved in full.  Returns whether that was so.
MP_DEV bool quad_balance(uint32_t (&z)[4], uint32_t cin)
{
    const uint32_t x[4] = {z[0], z[1], z[2], z[3]};
    const uint64_t up = quad_up(add_above(z, kBal, kBalTop), cin);
    z[0] = add_mask(z[0], kBal, up);
    const uint32_t a = z[0] < z[1] ? z[0] : z[1], b = z[2] < z[3] ? z[2] : z[3];
    const bool odd = ballot((a < b ? a : b) == 0u) != 0;
    if (odd) {
        const uint32_t bal[4] = {kBal, kBal, kBal, kBal};
#pragma unroll
        for (int j = 0; j < 4; j++) z[j] = x[j];
        quad_add(z, bal, cin);
    }
#pragma unroll
    for (int j = 0; j < 4; j++) z[j] ^= kBal;
    return odd;
}

// The four limbs of a lane's columns from its accumulator plus (ADD) four
// addend limbs, and their signed carry into the next lane.
template <bool ADD>
MP_DEV uint32_t quad_sums(const MfmaAcc &a, const Limb4 &add, uint32_t (&z)[4])
{
    // every term one 64-bit multiply-add (the carry's weight hidden apart from
    // w0, or the compiler adds before it multiplies, in 64 bits)
    int w0 = 1, w1 = 256, w2 = 65536, w3 = 16777216, wc = 1;
    asm("" : "+s"(w0), "+s"(w1), "+s"(w2), "+s"(w3), "+s"(wc));
    const uint32_t ad[4] = {add.x, add.y, add.z, add.w};
    int64_t s[4];
#pragma unroll
    for (int j = 0; j < 4; j++) {
        s[j] = (int64_t)mfma_get(a, 4 * j) * w0;
        s[j] += (int64_t)mfma_get(a, 4 * j + 1) * w1;
        s[j] += (int64_t)mfma_get(a, 4 * j + 2) * w2;
        s[j] += (int64_t)mfma_get(a, 4 * j + 3) * w3;
        if constexpr (ADD) s[j] = (int64_t)((uint64_t)ad[j] * (uint32_t)w0 + (uint64_t)s[j]);
    }
#pragma unroll
    for (int j = 1; j < 4; j++) s[j] += (int64_t)(int32_t)(s[j - 1] >> 32) * wc;
#pragma unroll
    for (int j = 0; j < 4; j++) z[j] = (uint32_t)s[j];
    return (uint32_t)(s[3] >> 32);
}

// The limbs of a strip from its accumulator plus (ADD) four addend limbs per
// lane: z gets the limbs of columns 8n + 4h .. + 3 with the carries inside the
// strip resolved; returns the strip's signed carry into its next column.
// Every lane's four columns are chained exactly and pass a signed carry to the
// next lane, where it is absorbed by the two lowest limbs; only if it is not
// (about one lane in 2^40, or runs of zero or all-ones limbs) the carries are
// resolved in full, biased by 2^31 to be non-negative.
template <bool ADD>
MP_DEV int strip_limbs(int l, const MfmaAcc &a, const Limb4 &add, uint32_t (&z)[4])
{
    const uint32_t c = quad_sums<ADD>(a, add, z);
    const uint32_t z0 = z[0], z1 = z[1];
    // the lane below (n, 1) is (n, 0); below (n, 0) it is (n - 1, 1)
    uint32_t lo, hi;
    half_swap(c, lo, hi);                 // lo: lane l gets c of lane l & 31; hi: of lane (l & 31) + 32
    const uint32_t up = shfl_up1(hi);     // (0 in lane 0)
    const int prev = (int)(l >= 32 ? lo : up);
    const uint64_t odd = add64_carry(z[0], z[1], prev) ^ ballot(prev < 0);
    int e = (int)readlane(c, kLanes - 1);
    if (odd) {
        // z + sum (c + 2^31) - sum 2^31, each sum over the lanes above the lowest
        const bool first = l == 0;
        const uint32_t b[4] = {first ? 0u : (uint32_t)prev + 0x80000000u, 0u, 0u, 0u};
        const uint32_t m[4] = {first ? 0xFFFFFFFFu : 0x7FFFFFFFu, 0xFFFFFFFFu, 0xFFFFFFFFu, 0xFFFFFFFFu};
        z[0] = z0;
        z[1] = z1;
        e += (int)quad_add(z, b, 0u);
        e += (int)quad_add(z, m, 1u) - 1;
    }
    return e;
}

// z += b + cin for a number of 512 limbs, zE the lanes' quads of its even
// blocks and zO those of its odd ones (in limb order: E of (n, 0), E of (n, 1), O
// of (n, 0), O of (n, 1)); returns the carry out
MP_DEV uint32_t quad2_add(uint32_t (&zE)[4], uint32_t (&zO)[4], const uint32_t (&bE)[4], const uint32_t (&bO)[4],
                          uint32_t cin)
{
    uint32_t cE = 0, cO = 0;
#pragma unroll
    for (int j = 0; j < 4; j++) {
        zE[j] = __builtin_addc(zE[j], bE[j], cE, &cE);
        zO[j] = __builtin_addc(zO[j], bO[j], cO, &cO);
    }
    const uint64_t GE = ballot(cE != 0u), GO = ballot(cO != 0u);
    const uint64_t PE = ballot((zE[0] & zE[1] & zE[2] & zE[3]) == 0xFFFFFFFFu),
                   PO = ballot((zO[0] & zO[1] & zO[2] & zO[3]) == 0xFFFFFFFFu);
    const uint32_t g0 = (uint32_t)GE, g1 = (uint32_t)(GE >> 32), g2 = (uint32_t)GO, g3 = (uint32_t)(GO >> 32);
    const uint32_t p0 = (uint32_t)PE, p1 = (uint32_t)(PE >> 32), p2 = (uint32_t)PO, p3 = (uint32_t)(PO >> 32);
    const uint32_t G = g3 | (p3 & (g2 | (p2 & (g1 | (p1 & g0))))), X = G | (p0 & p1 & p2 & p3);
    const uint64_t s = (uint64_t)X + G + cin;
    const uint32_t c0 = (uint32_t)s ^ X ^ G, c1 = g0 | (p0 & c0), c2 = g1 | (p1 & c1), c3 = g2 | (p2 & c2);
    cE = inverse_ballot((uint64_t)c1 << 32 | c0) ? 1u : 0u;
    cO = inverse_ballot((uint64_t)c3 << 32 | c2) ? 1u : 0u;
#pragma unroll
    for (int j = 0; j < 4; j++) {
        zE[j] = __builtin_addc(zE[j], 0u, cE, &cE);
        zO[j] = __builtin_addc(zO[j], 0u, cO, &cO);
    }
    return (uint32_t)(s >> 32);
}

// the same as strip_limbs<true> for the 512 limbs of strip_sums2 (add(0): the
// addend quad of the even blocks, add(1): of the odd ones)
template <class FA>
MP_DEV int strip_limbs2(int l, const MfmaAcc &aE, const MfmaAcc &aO, const FA &add, uint32_t (&zE)[4],
                        uint32_t (&zO)[4])
{
    const uint32_t cE = quad_sums<true>(aE, add(0), zE);
    wave_sync();                          // (one addend at a time: registers)
    const uint32_t cO = quad_sums<true>(aO, add(1), zO);
    const uint32_t xE[2] = {zE[0], zE[1]}, xO[2] = {zO[0], zO[1]};
    uint32_t loE, hiE, loO, hiO;
    half_swap(cE, loE, hiE);
    half_swap(cO, loO, hiO);
    const uint32_t up = shfl_up1(hiO);    // (0 in lane 0)
    const int pE = (int)(l >= 32 ? loE : up), pO = (int)(l >= 32 ? loO : hiE);
    const uint64_t odd = (add64_carry(zE[0], zE[1], pE) ^ ballot(pE < 0)) | (add64_carry(zO[0], zO[1], pO) ^ ballot(pO < 0));
    int e = (int)readlane(cO, kLanes - 1);
    if (odd) {
        const bool first = l == 0;
        const uint32_t bE[4] = {first ? 0u : (uint32_t)pE + 0x80000000u, 0u, 0u, 0u};
        const uint32_t bO[4] = {(uint32_t)pO + 0x80000000u, 0u, 0u, 0u};
        const uint32_t mE[4] = {first ? 0xFFFFFFFFu : 0x7FFFFFFFu, 0xFFFFFFFFu, 0xFFFFFFFFu, 0xFFFFFFFFu};
        const uint32_t mO[4] = {0x7FFFFFFFu, 0xFFFFFFFFu, 0xFFFFFFFFu, 0xFFFFFFFFu};
#pragma unroll
        for (int j = 0; j < 2; j++) {
            zE[j] = xE[j];
            zO[j] = xO[j];
        }
        e += (int)quad2_add(zE, zO, bE, bO, 0u);
        e += (int)quad2_add(zE, zO, mE, mO, 1u) - 1;
    }
    return e;
}

}  // namespace mp
