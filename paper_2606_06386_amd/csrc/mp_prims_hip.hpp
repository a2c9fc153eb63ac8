// Workgroup and wavefront primitives for gfx950 (CDNA4, wave64).
//
// The multi-precision code in the other headers is written against
// exactly this small set of operations: thread index, workgroup barrier,
// wave ballot / shuffles, a wave-uniform broadcast, and the 4x4 block of
// 32x32->64-bit multiply-accumulates that dominates every product.
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

#define MP_DEV __device__ __forceinline__

// Phase tracing (a diagnostic build option, off by default): with
// MP_PHASE_TRACE defined, MP_STAMP(id) records the shader clock of
// workgroup thread 0 in slot id (< 32) of the workgroup's row of
// mp_trace_buf (one per translation unit, for up to 8192 workgroups).
#ifdef MP_PHASE_TRACE
static __device__ uint64_t mp_trace_buf[8192 * 32];
#define MP_STAMP(id)                                                                                          \
    do {                                                                                                      \
        if (threadIdx.x == 0 && blockIdx.x < 8192) mp_trace_buf[(size_t)blockIdx.x * 32 + (id)] = __builtin_readcyclecounter(); \
    } while (0)
// MP_RSTAMP(id): the constant-rate (100 MHz) real-time counter instead, which
// gives the shader clock rate of the run against the cycle stamps
#define MP_RSTAMP(id)                                                                                         \
    do {                                                                                                      \
        if (threadIdx.x == 0 && blockIdx.x < 8192) mp_trace_buf[(size_t)blockIdx.x * 32 + (id)] = __builtin_amdgcn_s_memrealtime(); \
    } while (0)
#else
#define MP_STAMP(id) \
    do {             \
    } while (0)
#define MP_RSTAMP(id) \
    do {              \
    } while (0)
#endif

namespace mp {

constexpr int kLanes = 64;  // CDNA wavefront width

MP_DEV int lane() { return (int)(threadIdx.x & (kLanes - 1)); }
// the lane, computed anew where the scalar `at` changes: what follows from it is
// not kept in registers across a loop in which `at` does
MP_DEV int lane_at(int at)
{
    int l;
    asm("v_mbcnt_lo_u32_b32 %0, -1, 0\n\tv_mbcnt_hi_u32_b32 %0, -1, %0" : "=v"(l) : "s"(at));
    return l;
}
MP_DEV void sync() { __syncthreads(); }
// orders this wave's LDS accesses before and after it (a wave runs in
// lockstep and the LDS serves one wave's requests in order; only the
// compiler must not move accesses across)
MP_DEV void wave_sync() { asm volatile("" ::: "memory"); }
MP_DEV uint64_t ballot(bool p) { return __ballot(p); }

// this wave's claim on its SIMD's issue slots, 0 (all waves at first) to 3
template <int P>
MP_DEV void wave_priority()
{
    __builtin_amdgcn_s_setprio(P);
}

// index of the wave in its workgroup
MP_DEV int wave_index() { return (int)__builtin_amdgcn_readfirstlane(threadIdx.x / kLanes); }

// DPP controls (GFX9 data-parallel primitives: a VALU source operand read
// from another lane of the same wave, no LDS round trip)
constexpr int kDppWaveShl1 = 0x130;      // lane i reads lane i + 1
constexpr int kDppWaveShr1 = 0x138;      // lane i reads lane i - 1

// x of the lane the DPP control selects; lanes without a source receive 0
template <int CTRL>
MP_DEV uint32_t dpp(uint32_t x)
{
    return (uint32_t)__builtin_amdgcn_update_dpp(0, (int)x, CTRL, 0xF, 0xF, true);
}

// value held by lane-1 (lane 0 receives 0)
MP_DEV uint32_t shfl_up1(uint32_t x) { return dpp<kDppWaveShr1>(x); }

// value held by lane+1 (lane 63 receives 0)
MP_DEV uint32_t shfl_down1(uint32_t x) { return dpp<kDppWaveShl1>(x); }

// value of x in lane l (l wave-uniform)
MP_DEV uint32_t readlane(uint32_t x, int l) { return __builtin_amdgcn_readlane(x, l); }

// bit l of a wave-uniform mask, in lane l
MP_DEV bool inverse_ballot(uint64_t m) { return __builtin_amdgcn_inverse_ballot_w64(m); }

// lo: the lower 32 lanes' x in both halves of the wave, hi: the upper 32 lanes' x
MP_DEV void half_swap(uint32_t x, uint32_t &lo, uint32_t &hi)
{
    const auto r = __builtin_amdgcn_permlane32_swap(x, x, false, false);
    lo = r[0];
    hi = r[1];
}

// a value every lane of the wave already agrees on, moved to a scalar register
MP_DEV uint32_t uniform(uint32_t x) { return __builtin_amdgcn_readfirstlane(x); }
MP_DEV int uniform(int x) { return (int)__builtin_amdgcn_readfirstlane((uint32_t)x); }

// acc[r] += a * b[r] for r = 0..3, each acc a 96-bit column sum held as a
// 64-bit low part and a 32-bit high part.  v_mad_u64_u32 forms a*b + lo with
// the carry out in an SGPR pair; v_addc folds the carry into hi.  On gfx950 a
// VALU carry write needs two wait states before a VALU reads it; the three
// independent multiplies placed between each write and its read provide them.
MP_DEV void mac4(uint64_t (&lo)[4], uint32_t (&hi)[4], uint32_t a,
                 uint32_t b0, uint32_t b1, uint32_t b2, uint32_t b3)
{
    uint64_t c0, c1, c2, c3;
    asm volatile(
        "v_mad_u64_u32 %0, %8, %12, %13, %0\n\t"
        "v_mad_u64_u32 %1, %9, %12, %14, %1\n\t"
        "v_mad_u64_u32 %2, %10, %12, %15, %2\n\t"
        "v_mad_u64_u32 %3, %11, %12, %16, %3\n\t"
        "v_addc_co_u32_e64 %4, %8, 0, %4, %8\n\t"
        "v_addc_co_u32_e64 %5, %9, 0, %5, %9\n\t"
        "v_addc_co_u32_e64 %6, %10, 0, %6, %10\n\t"
        "v_addc_co_u32_e64 %7, %11, 0, %7, %11"
        : "+v"(lo[0]), "+v"(lo[1]), "+v"(lo[2]), "+v"(lo[3]),
          "+v"(hi[0]), "+v"(hi[1]), "+v"(hi[2]), "+v"(hi[3]),
          "=&s"(c0), "=&s"(c1), "=&s"(c2), "=&s"(c3)
        : "v"(a), "v"(b0), "v"(b1), "v"(b2), "v"(b3));
}

// (hi:lo) += c (sign-extended) in every lane; returns the lanes whose addition
// carried out of the 64 bits (of the unsigned value: for negative c, those that
// did not borrow).  A VALU carry needs two wait states before a VALU reads it.
MP_DEV uint64_t add64_carry(uint32_t &lo, uint32_t &hi, int c)
{
    uint64_t m;
    asm("v_add_co_u32_e64 %0, %2, %0, %3\n\t"
        "s_nop 1\n\t"
        "v_addc_co_u32_e64 %1, %2, %1, %4, %2"
        : "+&v"(lo), "+&v"(hi), "=&s"(m)
        : "v"(c), "v"(c >> 31));
    return m;
}

// z[j] = z[j] + a + carry from z[j-1] > t for j = 1..3 (a limb above t passes a
// carry up); returns the lanes whose z[3] does.  z[0] is left to the caller.
MP_DEV uint64_t add_above(uint32_t (&z)[4], uint32_t a, uint32_t t)
{
    uint64_t g0, g1, g2, g3, co;
    asm("v_cmp_lt_u32_e64 %3, %9, %8\n\t"
        "v_cmp_lt_u32_e64 %4, %9, %0\n\t"
        "v_cmp_lt_u32_e64 %5, %9, %1\n\t"
        "v_cmp_lt_u32_e64 %6, %9, %2\n\t"
        "v_addc_co_u32_e64 %0, %7, %0, %10, %3\n\t"
        "v_addc_co_u32_e64 %1, %7, %1, %10, %4\n\t"
        "v_addc_co_u32_e64 %2, %7, %2, %10, %5"
        : "+&v"(z[1]), "+&v"(z[2]), "+&v"(z[3]), "=&s"(g0), "=&s"(g1), "=&s"(g2), "=&s"(g3), "=&s"(co)
        : "v"(z[0]), "v"(t), "v"(a));
    return g3;
}

// x + a + (bit of m for the lane), m from the scalar unit
MP_DEV uint32_t add_mask(uint32_t x, uint32_t a, uint64_t m)
{
    uint32_t r;
    uint64_t co;
    asm("v_addc_co_u32_e64 %0, %1, %2, %3, %4" : "=v"(r), "=&s"(co) : "v"(x), "v"(a), "s"(m));
    return r;
}

// bytes [sel, sel + 4) of the 8-byte value hi:lo (sel in 0..3)
MP_DEV uint32_t alignbyte(uint32_t hi, uint32_t lo, uint32_t sel) { return __builtin_amdgcn_alignbyte(hi, lo, sel); }

// bits [n, n + 32) of the 8-byte value hi:lo (n in 0..31)
MP_DEV uint32_t alignbit(uint32_t hi, uint32_t lo, uint32_t n) { return __builtin_amdgcn_alignbit(hi, lo, n); }

MP_DEV uint32_t bswap(uint32_t x) { return __builtin_bswap32(x); }

// ---------------------------------------------------------- int8 matrix core
// v_mfma_i32_32x32x32_i8: D[32x32] += X[32x32] * Y[32x32], int8 inputs, int32
// sums.  Lane l supplies X row l%32 and Y column l%32, each as 16 bytes
// (k = 16*(l/32) + byte index, the same k order for X and Y), and receives
// D[8*(v/4) + 4*(l/32) + v%4][l%32] in accumulator element v.
typedef int MfmaFrag __attribute__((ext_vector_type(4)));
typedef int MfmaAcc __attribute__((ext_vector_type(16)));

MP_DEV MfmaAcc mfma_zero() { return MfmaAcc{}; }
MP_DEV MfmaAcc mfma_i8(MfmaAcc acc, uint32_t x0, uint32_t x1, uint32_t x2, uint32_t x3,
                       uint32_t y0, uint32_t y1, uint32_t y2, uint32_t y3)
{
    const MfmaFrag x = {(int)x0, (int)x1, (int)x2, (int)x3}, y = {(int)y0, (int)y1, (int)y2, (int)y3};
    return __builtin_amdgcn_mfma_i32_32x32x32_i8(x, y, acc, 0, 0, 0);
}
MP_DEV int mfma_get(const MfmaAcc &acc, int v) { return acc[v]; }

// marks a value as used without emitting any instruction
MP_DEV void keep(uint32_t x) { asm volatile("" : : "v"(x)); }

// 16-byte vector load and store of four limbs; p must be 16-byte aligned
struct Limb4 {
    uint32_t x, y, z, w;
};

MP_DEV Limb4 load4(const uint32_t *p)
{
    const uint4 v = *reinterpret_cast<const uint4 *>(__builtin_assume_aligned(p, 16));
    return Limb4{v.x, v.y, v.z, v.w};
}

MP_DEV void store4(uint32_t *p, uint32_t a, uint32_t b, uint32_t c, uint32_t d)
{
    *reinterpret_cast<uint4 *>(__builtin_assume_aligned(p, 16)) = make_uint4(a, b, c, d);
}

// LDS by byte address: the products' loops step plain 32-bit addresses and
// reach a step's operands by constant offsets
typedef __attribute__((address_space(3))) const uint32_t LdsWord;
typedef uint32_t Vec4 __attribute__((ext_vector_type(4)));
typedef __attribute__((address_space(3))) const Vec4 LdsQuad;

MP_DEV uint32_t lds_address(const uint32_t *p) { return (uint32_t)(uintptr_t)(LdsWord *)p; }
MP_DEV uint32_t lds_word(uint32_t a, int w) { return ((LdsWord *)(uintptr_t)a)[w]; }
MP_DEV Limb4 lds_quad(uint32_t a, int q)
{
    const Vec4 v = ((LdsQuad *)(uintptr_t)a)[q];
    return Limb4{v.x, v.y, v.z, v.w};
}
// the same value, whose origin the compiler does not see
MP_DEV uint32_t opaque(uint32_t x)
{
    asm("" : "+v"(x));
    return x;
}

}  // namespace mp
