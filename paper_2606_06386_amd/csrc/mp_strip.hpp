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

constexpr int kYPadBlk = 31;   // zero blocks a strip reads on each side of a digit plane
constexpr int kXPad = 16;      // zero words it reads on each side of the reversed short operand

#ifndef MP_DIAGS
#define MP_DIAGS 2
#endif
constexpr int kDiags = MP_DIAGS;   // diagonals per step of a product

constexpr int kPadBlk = kYPadBlk + kDiags - 1, kPadWords = 4 * kPadBlk;
constexpr int kXLow = kXPad + 8 * (kDiags - 1);   // zero words below the reversed digits

constexpr int kStripBlks = kStrip / 8;

// The long operand's digits lie in two planes of 16-byte half-blocks (plane h
// holds bytes 16h .. 16h + 15 of every 32-byte block), so that the lanes of
// either half-wave read 32 consecutive 16-byte chunks of one plane; the short
// operand's lie byte-reversed, so that a Toeplitz row is 16 consecutive bytes.
// word of the planes holding limb k: block k / 8, plane (k / 4) % 2, word k % 4
MP_DEV int plane_word(int k, int ly) { return ((k >> 1) & ~3) + (k & 3) + ((k >> 2) & 1) * ly; }

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
constexpr int kRowBatch = 5;   // rows read at once (a block's 257 + 3 limbs)

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

struct Operands {
    uint32_t x;          // LDS byte address of this lane's word of the reversed short digits at diagonal 0
    uint32_t sft;        // and its byte shift
    int dmax;            // last diagonal that touches the short digits
    uint32_t y;          // LDS byte address of this lane's word of the long digits' planes for block 0
    int nyblk;           // blocks of the long digits
};

// xr: nx reversed digit limbs; yb: planes (distance ly) of ny digit limbs
MP_DEV Operands operands(int l, const uint32_t *xr, int nx, const uint32_t *yb, int ly, int ny)
{
    const int p = l & 31, h = l >> 5;
    const int ox = 16 * h - 1 - (16 * ((p >> 2) & 1) + 4 * (p >> 3) + (p & 3));   // (from the end of the digits)
    return Operands{lds_address(xr + nx) + 4 * (ox >> 2), (uint32_t)ox & 3u, (4 * nx + 30) >> 5,
                    lds_address(yb) + 4 * (h * ly + 4 * p), (ny + 7) >> 3};
}

MP_DEV XRaw xraw_at(uint32_t a, int w)
{
    return XRaw{lds_word(a, w), lds_word(a, w + 1), lds_word(a, w + 2), lds_word(a, w + 3), lds_word(a, w + 4)};
}

// the operands of N diagonals, the last at the addresses x and y
template <int N>
struct Diagonals {
    XRaw r[N];
    Limb4 y[N];
    MP_DEV void load(uint32_t xa, uint32_t ya)
    {
#pragma unroll
        for (int j = 0; j < N; j++) {
            r[j] = xraw_at(xa, 8 * (N - 1 - j));
            y[j] = lds_quad(ya, N - 1 - j);
        }
    }
    MP_DEV void add(MfmaAcc &acc, uint32_t sft) const
    {
#pragma unroll
        for (int j = 0; j < N; j++) acc = mfma_x(acc, xfrag(r[j], sft), y[j]);
    }
};

// The accumulator of the strip whose first block is S0, or the share `part` of
// `parts` of its diagonals (the first share the smallest).  Steps of kDiags
// diagonals; the last may pass the end: it reads zeros there (of the short
// digits, or blocks below the long ones').  FAST, for kernels with registers to
// spare and few waves per SIMD to hide LDS reads behind: the next step's
// operands in flight.
template <bool FAST>
MP_DEV MfmaAcc strip_sums(const Operands &o, int S0, int part = 0, int parts = 1)
{
    constexpr int D = kDiags;
    MfmaAcc acc = mfma_zero();
    const int dlo = imax(0, S0 - o.nyblk + 1), dhi = imin(o.dmax, S0 + 31);
    int n = uniform(dhi - dlo + D) / D;          // steps
    if (n <= 0) return acc;
    const int first = n * part / parts, d0 = dlo + D * first;
    n = n * (part + 1) / parts - first;
    // (addresses of a step's last diagonal: the others lie at positive offsets)
    uint32_t x = opaque(o.x - 32 * (d0 + D - 1)), y = opaque(o.y + 16 * (S0 - d0 - (D - 1)));
    if constexpr (FAST) {
        Diagonals<D> a, b;
        a.load(x, y);
        for (; n >= 2; n -= 2) {                 // (the reads past the last step are not used)
            b.load(x - 32 * D, y - 16 * D);
            a.add(acc, o.sft);
            sched_loads_first();
            x -= 64 * D;
            y -= 32 * D;
            a.load(x, y);
            b.add(acc, o.sft);
            sched_loads_first();
        }
        if (n) a.add(acc, o.sft);
    } else {
        for (; n > 0; n--) {
            Diagonals<D> a;
            a.load(x, y);
            a.add(acc, o.sft);
            sched_loads_first();
            x -= 32 * D;
            y -= 16 * D;
        }
    }
    return acc;
}

// The same for two adjacent strips at once over the diagonals [0, dmax], which
// both must need in full (SA >= dmax - 31): each X fragment serves both, and one
// address steps over two diagonals.
MP_DEV void strip_sums2(const Operands &o, int SA, MfmaAcc &accA, MfmaAcc &accB)
{
    accA = mfma_zero();
    accB = mfma_zero();
    uint32_t x = o.x, y = o.y + 16 * SA;
    const auto one = [&](int j) {                // diagonal j below the addresses
        const XRaw r = xraw_at(x, -8 * j);
        const Limb4 va = lds_quad(y, -j), vb = lds_quad(y, kStripBlks - j);
        const XFrag f = xfrag(r, o.sft);
        accA = mfma_x(accA, f, va);
        accB = mfma_x(accB, f, vb);
        sched_loads_first();
    };
    const int n = uniform(o.dmax) + 1;
    if (n & 1) {
        one(0);
        x -= 32;
        y -= 16;
    }
    x = opaque(x - 32);                          // (offsets from an address are not negative)
    y = opaque(y - 16);
    for (int i = n >> 1; i > 0; i--) {
        one(-1);
        one(0);
        x -= 64;
        y -= 32;
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
    const uint32_t c = (uint32_t)(s[3] >> 32);
    // the lane below (n, 1) is (n, 0); below (n, 0) it is (n - 1, 1)
    uint32_t lo, hi;
    half_swap(c, lo, hi);                 // lo: lane l gets c of lane l & 31; hi: of lane (l & 31) + 32
    const uint32_t up = shfl_up1(hi);     // (0 in lane 0)
    const int prev = (int)(l >= 32 ? lo : up);
    const uint64_t neg = ballot(prev < 0);
    const uint64_t odd = add64_carry(z[0], z[1], prev) ^ neg;
    int e = (int)readlane(c, kLanes - 1);
    if (odd) {
        // z + sum (c + 2^31) - sum 2^31, each sum over the lanes above the lowest
        const bool first = l == 0;
        const uint32_t b[4] = {first ? 0u : (uint32_t)prev + 0x80000000u, 0u, 0u, 0u};
        const uint32_t m[4] = {first ? 0xFFFFFFFFu : 0x7FFFFFFFu, 0xFFFFFFFFu, 0xFFFFFFFFu, 0xFFFFFFFFu};
#pragma unroll
        for (int j = 0; j < 4; j++) z[j] = (uint32_t)s[j];
        e += (int)quad_add(z, b, 0u);
        e += (int)quad_add(z, m, 1u) - 1;
    }
    return e;
}

}  // namespace mp
