// Division kernels and their launchers.
//
// One workgroup per instance (or, for the persistent ragged kernels, per
// instance taken from a work queue).  The workgroup size follows the operand
// width so that every linear pass handles at most 16 limbs per thread:
//   width <= 2048 limbs -> 256 threads, <= 4096 -> 512, <= 8192 -> 1024.
// All operands and intermediates of an instance live in dynamic LDS laid out
// by plan_body (20 KB at 2^16 bits, 74 KB at most at 2^18).
//
// The build compiles this file once per kernel family and workgroup size
// (MP_KFAMILY: 0 product, 1 shifted inverse, 2 division, 3 ragged division;
// MP_KT: threads), each object holding one explicit instantiation
// of a launcher, so the translation units compile in parallel.
#include "mp_prims_hip.hpp"
#include "mp_core.hpp"
#include "mp_strip.hpp"
#include "mp_mul.hpp"
#include "mp_block.hpp"

namespace mp {

// Registers of the division kernels.  An instance spends much of its time in
// phases that one of its waves runs (Newton steps, a block's digits and
// quotient product), so further resident instances fill the other waves' issue
// slots: eight waves per SIMD (64 vector and 96 scalar registers), which the LDS
// of a 2^16-bit instance, 20 KB, also allows.  4096 divisions of 2048 by 1024
// limbs take 122 us, at seven waves 133; 2048 of random divisor lengths 72 and
// 99 us.
#define MP_OCCUPANCY __attribute__((amdgpu_waves_per_eu(M == Mode::kPacked ? 8 : 4, 8)))
#define MP_SHARED_OCCUPANCY __attribute__((amdgpu_waves_per_eu(8, 8)))
// products: four waves per SIMD (four accumulators and a window of four fragments per wave)
#define MP_MUL_OCCUPANCY __attribute__((amdgpu_waves_per_eu(4, 8)))

// Workspace of a ragged batch (int32): [0, 4) instances per class, [4, 8)
// queue heads, then one list of instance indices per class, each `count` long.
constexpr int kClasses = 4;
constexpr int kWsHeader = 16;

MP_DEV int64_t uniform64(int64_t x)
{
    const uint32_t lo = uniform((uint32_t)x), hi = uniform((uint32_t)((uint64_t)x >> 32));
    return (int64_t)(((uint64_t)hi << 32) | lo);
}

template <int T, int G, int K>
__global__ __launch_bounds__(T) MP_MUL_OCCUPANCY void k_mul(const uint32_t *a, int na, const uint32_t *b, int nb,
                                                            uint32_t *c)
{
    extern __shared__ __align__(16) uint32_t lds[];
    const size_t j = blockIdx.x;
    mul_instance<T, G, K>(lds, a + j * na, na, b + j * nb, nb, c + j * (size_t)(na + nb));
}

template <int T>
__global__ __launch_bounds__(T) void k_mul_valu(const uint32_t *a, int na, const uint32_t *b, int nb, uint32_t *c)
{
    extern __shared__ __align__(16) uint32_t lds[];
    const size_t j = blockIdx.x;
    mul_valu_instance<T>(lds, a + j * na, na, b + j * nb, nb, c + j * (size_t)(na + nb));
}

template <int T, Mode M>
__global__ __launch_bounds__(T) MP_OCCUPANCY void k_shinv(const uint32_t *v, int nv, int h, uint32_t *w, int nw,
                                                          int32_t *status, int bmax)
{
    extern __shared__ __align__(16) uint32_t lds[];
    const size_t j = blockIdx.x;
    uint32_t *wj = w + j * nw;
    divide_instance<T, M>(lds, PowB{h}, h + 1, v + j * nv, nv, wj, nw, nullptr, status ? status + j : nullptr,
                       bmax);
}

template <int T, Mode M>
__global__ __launch_bounds__(T) MP_OCCUPANCY void k_divrem(const uint32_t *u, int nu, const uint32_t *v, int nv,
                                                           uint32_t *q, int nq, uint32_t *r, int32_t *status,
                                                           int bmax)
{
    extern __shared__ __align__(16) uint32_t lds[];
    const size_t j = blockIdx.x;
    uint32_t *qj = q + j * nq, *rj = r + j * nv;
    divide_instance<T, M>(lds, Span{u + j * nu, 0, nu}, nu, v + j * nv, nv, qj, nq, rj, status ? status + j : nullptr,
                       bmax);
}

// instance j of a ragged batch
template <int T, Mode M>
MP_DEV void ragged_instance(uint32_t *lds, const uint32_t *up, const uint32_t *vp, const mp_desc_t *desc, uint32_t *qp,
                            uint32_t *rp, int32_t *status, int j, int bmax)
{
    // every value below is the same on all lanes: keep it in scalar registers
    const mp_desc_t &d = desc[j];
    const int64_t uo = uniform64(d.u_off), vo = uniform64(d.v_off), qo = uniform64(d.q_off), ro = uniform64(d.r_off);
    const int nu = uniform(d.nu), nv = uniform(d.nv), nq = uniform(d.nq);
    divide_instance<T, M>(lds, Span{up + uo, 0, nu}, nu, vp + vo, nv, qp + qo, nq, rp + ro, status + j, bmax);
}

// one workgroup per instance of a small ragged batch, whatever its width
template <int T, Mode M>
__global__ __launch_bounds__(T) MP_OCCUPANCY void k_ragged_direct(const uint32_t *up, const uint32_t *vp,
                                                                  const mp_desc_t *desc, uint32_t *qp, uint32_t *rp,
                                                                  int32_t *status, PoolLimbs pools, int bmax)
{
    extern __shared__ __align__(16) uint32_t lds[];
    const int j = blockIdx.x;
    if (!desc_ok(desc[j], pools)) {
        if (threadIdx.x == 0) status[j] = MP_INST_BADDESC;
        return;
    }
    ragged_instance<T, M>(lds, up, vp, desc, qp, rp, status, j, bmax);
}

// Persistent workgroups of one class: take the next instance of the class's
// queue until it is empty.  Of 1024 threads, only some of the workgroups launched
// stay, at most two per compute unit, which hold all its waves: one per unit if the instances would not give half
// the units a second one, since two slow each other down (300 of a batch of 1200:
// 184 us for the batch, in pairs 191); and three on two units beside a class of
// the next width, whose workgroups then find LDS on every other unit (4096 of
// mixed widths 417 -> 413 us, of widths spread evenly in their logarithm 419 ->
// 394).
template <int T>
__global__ __launch_bounds__(T) MP_SHARED_OCCUPANCY void k_ragged(const uint32_t *up, const uint32_t *vp,
                                                                  const mp_desc_t *desc, uint32_t *qp, uint32_t *rp,
                                                                  int32_t *status, int32_t *ws, int cls, int count,
                                                                  int cus, int bmax)
{
    extern __shared__ __align__(16) uint32_t lds[];
    const int n = ws[cls];
    if (T == 1024) {
        const int some = cus + (cus >> 1);
        const bool beside = cls == kClasses - 1 && ws[cls - 1] >= cus;
        if ((int)blockIdx.x >= (n <= some ? cus : beside ? some : 2 * cus)) return;
    }
    for (;;) {
        __syncthreads();
        if (threadIdx.x == 0) lds[kCtlBcast + 2] = (uint32_t)atomicAdd(&ws[kClasses + cls], 1);
        __syncthreads();
        const int idx = uniform((int)lds[kCtlBcast + 2]);
        if (idx >= n) break;
        ragged_instance<T, Mode::kPacked>(lds, up, vp, desc, qp, rp, status, uniform(ws[kWsHeader + (size_t)cls * count + idx]),
                                  bmax);
    }
}

template <int T>
hipError_t launch_mul(int grid, hipStream_t st, const uint32_t *a, int na, const uint32_t *b, int nb, uint32_t *c,
                      MulKind kind)
{
    auto *fn = kind == MulKind::kStrip   ? k_mul<T, 1, 1>
               : kind == MulKind::kPair  ? k_mul<T, 2, 1>
               : kind == MulKind::kQuad  ? k_mul<T, 4, 1>
               : kind == MulKind::kQuads ? k_mul<T, 4, 2>
                                         : k_mul_valu<T>;
    const size_t lds = (size_t)4 * (kind == MulKind::kValu ? mul_valu_lds_words(na, nb) : plan_mul(na, nb).total);
    if (!lds_attr(reinterpret_cast<const void *>(fn), lds)) return hipErrorInvalidValue;
    hipLaunchKernelGGL(fn, dim3(grid), dim3(T), lds, st, a, na, b, nb, c);
    return hipGetLastError();
}

template <int T, Mode M>
hipError_t launch_shinv(int grid, size_t lds, hipStream_t st, const uint32_t *v, int nv, int h, uint32_t *w, int nw,
                        int32_t *status, int bmax)
{
    if (!lds_attr(reinterpret_cast<const void *>(&k_shinv<T, M>), lds)) return hipErrorInvalidValue;
    hipLaunchKernelGGL((k_shinv<T, M>), dim3(grid), dim3(T), lds, st, v, nv, h, w, nw, status, bmax);
    return hipGetLastError();
}

template <int T, Mode M>
hipError_t launch_divrem(int grid, size_t lds, hipStream_t st, const uint32_t *u, int nu, const uint32_t *v, int nv,
                         uint32_t *q, int nq, uint32_t *r, int32_t *status, int bmax)
{
    if (!lds_attr(reinterpret_cast<const void *>(&k_divrem<T, M>), lds)) return hipErrorInvalidValue;
    hipLaunchKernelGGL((k_divrem<T, M>), dim3(grid), dim3(T), lds, st, u, nu, v, nv, q, nq, r, status, bmax);
    return hipGetLastError();
}

template <int T>
hipError_t launch_ragged(int grid, size_t lds, hipStream_t st, const uint32_t *up, const uint32_t *vp,
                         const mp_desc_t *desc, uint32_t *qp, uint32_t *rp, int32_t *status, int32_t *ws, int cls,
                         int count, int cus, int bmax)
{
    if (!lds_attr(reinterpret_cast<const void *>(&k_ragged<T>), lds)) return hipErrorInvalidValue;
    hipLaunchKernelGGL(k_ragged<T>, dim3(grid), dim3(T), lds, st, up, vp, desc, qp, rp, status, ws, cls, count, cus,
                       bmax);
    return hipGetLastError();
}

template <int T, Mode M>
hipError_t launch_ragged_direct(int count, size_t lds, hipStream_t st, const uint32_t *up, const uint32_t *vp,
                                const mp_desc_t *desc, uint32_t *qp, uint32_t *rp, int32_t *status,
                                const PoolLimbs &pools, int bmax)
{
    if (!lds_attr(reinterpret_cast<const void *>(&k_ragged_direct<T, M>), lds)) return hipErrorInvalidValue;
    hipLaunchKernelGGL((k_ragged_direct<T, M>), dim3(count), dim3(T), lds, st, up, vp, desc, qp, rp, status, pools,
                       bmax);
    return hipGetLastError();
}

#if defined(MP_KFAMILY) && defined(MP_KT)
// (Mode::kFast serves workgroups of 256 and 512 threads only, see division_shape)
#if MP_KFAMILY == 0
template hipError_t launch_mul<MP_KT>(int, hipStream_t, const uint32_t *, int, const uint32_t *, int, uint32_t *,
                                      MulKind);
#elif MP_KFAMILY == 1
#define MP_SHINV(M)                                                                                                 \
    template hipError_t launch_shinv<MP_KT, M>(int, size_t, hipStream_t, const uint32_t *, int, int, uint32_t *,    \
                                               int, int32_t *, int);
MP_SHINV(Mode::kPacked)
MP_SHINV(Mode::kShared)
#if MP_KT <= 512
MP_SHINV(Mode::kFast)
#endif
#elif MP_KFAMILY == 2
#define MP_DIVREM(M)                                                                                                \
    template hipError_t launch_divrem<MP_KT, M>(int, size_t, hipStream_t, const uint32_t *, int, const uint32_t *,  \
                                                int, uint32_t *, int, uint32_t *, int32_t *, int);
MP_DIVREM(Mode::kPacked)
MP_DIVREM(Mode::kShared)
#if MP_KT <= 512
MP_DIVREM(Mode::kFast)
#endif
#elif MP_KFAMILY == 3
template hipError_t launch_ragged<MP_KT>(int, size_t, hipStream_t, const uint32_t *, const uint32_t *,
                                         const mp_desc_t *, uint32_t *, uint32_t *, int32_t *, int32_t *, int, int,
                                         int, int);
#if MP_KT == 1024
#define MP_DIRECT(M)                                                                                                \
    template hipError_t launch_ragged_direct<1024, M>(int, size_t, hipStream_t, const uint32_t *, const uint32_t *, \
                                                      const mp_desc_t *, uint32_t *, uint32_t *, int32_t *,         \
                                                      const PoolLimbs &, int);
MP_DIRECT(Mode::kPacked)
MP_DIRECT(Mode::kShared)
#endif
#endif
#endif

}  // namespace mp

#if defined(MP_PHASE_TRACE) && MP_KFAMILY == 0 && MP_KT == 128
// copies the stamps of the first `blocks` product workgroups (32 per workgroup) to host memory
extern "C" int mp_trace_read_mul(uint64_t *dst, int blocks)
{
    return (int)hipMemcpyFromSymbol(dst, HIP_SYMBOL(mp_trace_buf), (size_t)blocks * 32 * sizeof(uint64_t), 0,
                                    hipMemcpyDeviceToHost);
}
#endif

#if defined(MP_PHASE_TRACE) && MP_KFAMILY == 2
#define MP_TRACE_NAME2(t) mp_trace_read_divrem_##t
#define MP_TRACE_NAME(t) MP_TRACE_NAME2(t)
// copies the stamps of the first `blocks` workgroups (32 per workgroup) to host memory
extern "C" int MP_TRACE_NAME(MP_KT)(uint64_t *dst, int blocks)
{
    return (int)hipMemcpyFromSymbol(dst, HIP_SYMBOL(mp_trace_buf), (size_t)blocks * 32 * sizeof(uint64_t), 0,
                                    hipMemcpyDeviceToHost);
}
#endif
