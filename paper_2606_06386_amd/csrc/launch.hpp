// Host-side launchers of the division kernels (defined in kernels.hip, one
// translation unit per kernel family and workgroup size so that they compile
// in parallel).
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

#include "../../include/mpdiv.h"

namespace mp {

// sets a kernel's dynamic-LDS limit to at least `bytes` on the current device
// (cached: no runtime call once the limit is high enough)
bool lds_attr(const void *kernel, size_t bytes);

constexpr int kMaxLimbs = 8192;   // widest operand (2^18 bits)

// limbs of the four pools of a ragged batch
struct PoolLimbs {
    int64_t u, v, q, r;
};

// widths in range and every operand inside its pool (no overflow: widths are
// small, offsets not negative)
__device__ __forceinline__ bool desc_ok(const mp_desc_t &d, const PoolLimbs &p)
{
    return d.nu >= 1 && d.nu <= kMaxLimbs && d.nv >= 1 && d.nv <= kMaxLimbs && d.nq >= 1 && d.u_off >= 0 &&
           d.v_off >= 0 && d.q_off >= 0 && d.r_off >= 0 && d.u_off <= p.u - d.nu && d.v_off <= p.v - d.nv &&
           d.q_off <= p.q - d.nq && d.r_off <= p.r - d.nv;
}

// Products on the matrix cores, a wave taking one strip of 256 columns, two
// adjacent ones, four, or twice four; or on the vector ALU
enum class MulKind { kStrip, kPair, kQuad, kQuads, kValu };

template <int T>
hipError_t launch_mul(int grid, hipStream_t st, const uint32_t *a, int na, const uint32_t *b, int nb, uint32_t *c,
                      MulKind kind);

// Division kernels, by the room the batch leaves them: eight waves per SIMD; or
// built for four, with products that keep more reads in flight; the latter with
// four waves sharing a block's quotient product
enum class Mode { kPacked, kFast, kShared };

// bmax: longest block of quotient limbs
template <int T, Mode M>
hipError_t launch_shinv(int grid, size_t lds, hipStream_t st, const uint32_t *v, int nv, int h, uint32_t *w, int nw,
                        int32_t *status, int bmax);

template <int T, Mode M>
hipError_t launch_divrem(int grid, size_t lds, hipStream_t st, const uint32_t *u, int nu, const uint32_t *v, int nv,
                         uint32_t *q, int nq, uint32_t *r, int32_t *status, int bmax);

template <int T>
hipError_t launch_ragged(int grid, size_t lds, hipStream_t st, const uint32_t *up, const uint32_t *vp,
                         const mp_desc_t *desc, uint32_t *qp, uint32_t *rp, int32_t *status, int32_t *ws, int cls,
                         int count, int cus, int bmax);

// one workgroup per instance, descriptors checked by the workgroup (no workspace)
template <int T, Mode M>
hipError_t launch_ragged_direct(int count, size_t lds, hipStream_t st, const uint32_t *up, const uint32_t *vp,
                                const mp_desc_t *desc, uint32_t *qp, uint32_t *rp, int32_t *status,
                                const PoolLimbs &pools, int bmax);

}  // namespace mp
