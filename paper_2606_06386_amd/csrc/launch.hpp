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

// Products on the matrix cores, a wave taking one strip of 256 columns, two
// adjacent ones, four, or twice four; or on the vector ALU
enum class MulKind { kStrip, kPair, kQuad, kQuads, kValu };

template <int T>
hipError_t launch_mul(int grid, hipStream_t st, const uint32_t *a, int na, const uint32_t *b, int nb, uint32_t *c,
                      MulKind kind);

// Division kernels; bmax: longest block of quotient limbs.  FAST: built for four
// waves per SIMD instead of eight, with products that keep more reads in flight.
template <int T, bool FAST>
hipError_t launch_shinv(int grid, size_t lds, hipStream_t st, const uint32_t *v, int nv, int h, uint32_t *w, int nw,
                        int32_t *status, int bmax);

template <int T, bool FAST>
hipError_t launch_divrem(int grid, size_t lds, hipStream_t st, const uint32_t *u, int nu, const uint32_t *v, int nv,
                         uint32_t *q, int nq, uint32_t *r, int32_t *status, int bmax);

template <int T, bool FAST>
hipError_t launch_ragged(int grid, size_t lds, hipStream_t st, const uint32_t *up, const uint32_t *vp,
                         const mp_desc_t *desc, uint32_t *qp, uint32_t *rp, int32_t *status, int32_t *ws, int cls,
                         int count, int bmax);

}  // namespace mp
