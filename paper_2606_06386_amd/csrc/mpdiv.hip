// C ABI of libmpdiv (see include/mpdiv.h): argument checks, launch
// configuration and the ragged-batch preparation kernel.  The division
// kernels themselves are in kernels.hip.
#include "mp_prims_hip.hpp"
#include "mp_core.hpp"
#include "mp_strip.hpp"
#include "mp_mul.hpp"
#include "mp_block.hpp"
#include "launch.hpp"

#include "../../include/mpdiv.h"

#include <atomic>
#include <mutex>
#include <string.h>

namespace {

constexpr int kLdsWords = 160 * 1024 / 4;   // gfx950: 160 KB of LDS per workgroup

// run-time knobs (mp_set_knob)
std::atomic<int32_t> g_mfma_min{64}, g_small_limit{MP_SMALL_LIMIT_AUTO};

constexpr int kAutoLimit = 136, kMaxLimit = 140;

// longest block of a launch's divisions
int block_max()
{
    const int sl = g_small_limit.load();
    return mp::block_limit(sl == MP_SMALL_LIMIT_AUTO ? kAutoLimit : sl);
}

// LDS of a division kernel
size_t body_bytes(int nu, int nv, mp::Mode mode = mp::Mode::kPacked)
{
    const int n = mp::plan_body(nu, nv).total;
    return (size_t)4 * (mode == mp::Mode::kShared ? mp::r4(n) + mp::kPartWords : n);
}

// ------------------------------------------------------------ ragged batches
//
// Workspace (int32): [0, 4) instances per class, [4, 8) queue heads, then one
// list of instance indices per class, each `count` long.
constexpr int kClasses = 4;
constexpr int kClassWidth[kClasses] = {1024, 2048, 4096, 8192};
constexpr int kWsHeader = 16;
static_assert(mp::plan_body(kClassWidth[kClasses - 1], kClassWidth[kClasses - 1]).total <= kLdsWords,
              "an instance of the widest class fits the LDS of a workgroup");

__device__ __forceinline__ int width_class(int nu)
{
    return nu <= 1024 ? 0 : nu <= 2048 ? 1 : nu <= 4096 ? 2 : 3;
}

// Queue order within a class: by falling cost, in kBins steps, so that no long
// instance starts when the others are nearly done.  An instance of nb blocks
// (and Newton steps worth four) costs a fixed time per block and one that grows
// with the divisor.
constexpr int kBins = 16;

__device__ __forceinline__ int cost_of(int nu, int nv) { return ((nu > nv ? nu - nv : 0) / 136 + 5) * (4096 + nv); }

__device__ __forceinline__ int cost_bin(int c, int nu, int nv)
{
    const int most = cost_of(kClassWidth[c], kClassWidth[c] / 2);
    const int bin = (int)((int64_t)cost_of(nu, nv) * kBins / most);
    return bin < kBins ? kBins - 1 - bin : 0;
}

// one workgroup: validate descriptors and bucket instance indices by class and cost
__global__ __launch_bounds__(1024) void k_ragged_prep(const mp_desc_t *desc, int count, mp::PoolLimbs pools,
                                                      int32_t *status, int32_t *ws)
{
    __shared__ int cnt[kClasses][kBins];
    if (threadIdx.x < kClasses * kBins) cnt[0][threadIdx.x] = 0;
    __syncthreads();
    for (int j = threadIdx.x; j < count; j += blockDim.x) {
        const mp_desc_t d = desc[j];
        if (!mp::desc_ok(d, pools)) {
            status[j] = MP_INST_BADDESC;
            continue;
        }
        const int c = width_class(d.nu);
        atomicAdd(&cnt[c][cost_bin(c, d.nu, d.nv)], 1);
    }
    __syncthreads();
    if (threadIdx.x < kClasses) {          // counts to first slots
        int sum = 0;
        for (int i = 0; i < kBins; i++) {
            const int n = cnt[threadIdx.x][i];
            cnt[threadIdx.x][i] = sum;
            sum += n;
        }
        ws[threadIdx.x] = sum;
        ws[kClasses + threadIdx.x] = 0;
    }
    __syncthreads();
    for (int j = threadIdx.x; j < count; j += blockDim.x) {
        const mp_desc_t d = desc[j];
        if (!mp::desc_ok(d, pools)) continue;
        const int c = width_class(d.nu);
        ws[kWsHeader + (size_t)c * count + atomicAdd(&cnt[c][cost_bin(c, d.nu, d.nv)], 1)] = j;
    }
}

struct RaggedConfig {
    int threads[kClasses] = {256, 256, 512, 1024};
    int wgs_per_cu[kClasses] = {4, 4, 2, 2};
};
RaggedConfig g_ragged;
std::mutex g_ragged_mu;

int threads_for(int width)
{
    return width <= 2048 ? 256 : width <= 4096 ? 512 : 1024;
}

// How a batch of products splits its strips of 256 columns over waves.  Few
// products leave compute units idle: the more waves share one the better, down
// to one strip each.  Many are bound by LDS reads (18 cycles per matrix-core
// product where one strip reads its own fragments, 9 for a pair of strips, 4.5
// for four), and then by uneven waves: four strips at either end of a product
// have a third of the work of four in the middle, which two groups per wave
// (w and w + W) even out, at the price of fewer waves.  us for lo x hi limbs,
// batch: strip / pair / four / two fours per wave
//   1024 x 1024:  256: 10 / 16 / 23 / 42;   1024: 27 / 29 / 28 / 44;   4096: 98 / 95 / 85 / 110
//   2048 x 2048:  128: 18 / 23 / 34 / 52;    512: 43 / 40 / 46 / 67;   4096: 327 / 284 / 276 / 264
//   4096 x 4096:  128: 59 / 46 / 58 / 74;    512: 154 / 131 / 117 / 128; 1024: 304 / 259 / 229 / 233
//   8192 x 8192:  128: 218 / - / 143 / 167;  256: 294 / - / 210 / 227
//   8192 x 2000:  256: 78 / - / 62 / 66;    1024: 298 / - / 242 / 221
//   2048 x 300:   256: 10 / - / 11 / 14;    4096: 65 / - / 60 / 63
// (A short operand below 1016 limbs leaves four strips no window of fragments:
// they share single ones, evenly.)  The batches' limits are in strips: 24, 32 and
// 64 for each of the 256 compute units.
struct MulShape {
    int threads;
    mp::MulKind kind;
};

MulShape mul_shape(int lo, int nc, int64_t batch)
{
    const int ns = (nc + mp::kStrip - 1) / mp::kStrip;
    const int64_t strips = batch * ns;
    if (ns <= 6 || (ns <= 16 && strips <= 6144)) return {ns <= 4 ? 256 : ns <= 8 ? 512 : 1024, mp::MulKind::kStrip};
    if (ns > 8 && ns <= 32 && lo >= 1016 && strips <= (ns <= 16 ? 16384 : 8192))
        return {ns <= 16 ? 512 : 1024, mp::MulKind::kPair};
    if (lo >= 1016 && ((ns > 8 && ns <= 16) || (ns > 32 && strips > 16384)))
        return {ns <= 16 ? 128 : 512, mp::MulKind::kQuads};
    return {ns <= 8 ? 128 : ns <= 16 ? 256 : ns <= 32 ? 512 : 1024, mp::MulKind::kQuad};
}

// the current device is gfx950 (checked once per device)
bool device_ok()
{
    static int checked[64];   // 0 unknown, 1 ok, 2 not usable
    int dev = 0;
    if (hipGetDevice(&dev) != hipSuccess || dev < 0 || dev >= 64) return false;
    if (checked[dev] == 0) {
        hipDeviceProp_t prop;
        bool ok = hipGetDeviceProperties(&prop, dev) == hipSuccess &&
                  strncmp(prop.gcnArchName, "gfx950", 6) == 0;
        checked[dev] = ok ? 1 : 2;
    }
    return checked[dev] == 1;
}

}  // namespace

// raise a kernel's dynamic LDS limit to at least `bytes` on the current
// device; the attribute is set only when it grows, so repeated launches (and
// launches under stream capture) make no further runtime call
bool mp::lds_attr(const void *fn, size_t bytes)
{
    struct Entry {
        const void *fn;
        int dev;
        size_t bytes;
    };
    static Entry seen[256];
    static int nseen;
    static std::mutex mu;
    int dev = 0;
    if (hipGetDevice(&dev) != hipSuccess) return false;
    std::lock_guard<std::mutex> lock(mu);
    Entry *e = nullptr;
    for (int i = 0; i < nseen; i++)
        if (seen[i].fn == fn && seen[i].dev == dev) e = &seen[i];
    if (e && e->bytes >= bytes) return true;
    if (hipFuncSetAttribute(fn, hipFuncAttributeMaxDynamicSharedMemorySize, (int)bytes) != hipSuccess) return false;
    if (!e && nseen < 256) e = &seen[nseen++];
    if (e) *e = Entry{fn, dev, bytes};
    return true;
}

namespace {

mp_status_t status_of(hipError_t e) { return e == hipSuccess ? MP_OK : MP_ERR_LAUNCH; }

mp_status_t launch_mul_threads(int T, int grid, hipStream_t st, const uint32_t *a, int na, const uint32_t *b, int nb,
                               uint32_t *c, mp::MulKind kind)
{
    switch (T) {
    case 128: return status_of(mp::launch_mul<128>(grid, st, a, na, b, nb, c, kind));
    case 256: return status_of(mp::launch_mul<256>(grid, st, a, na, b, nb, c, kind));
    case 512: return status_of(mp::launch_mul<512>(grid, st, a, na, b, nb, c, kind));
    default: return status_of(mp::launch_mul<1024>(grid, st, a, na, b, nb, c, kind));
    }
}

// compute units of the current device (queried once per device)
int device_cus()
{
    static int cus[64];
    int dev = 0;
    if (hipGetDevice(&dev) != hipSuccess || dev < 0 || dev >= 64) return 0;
    if (cus[dev] == 0) {
        hipDeviceProp_t prop;
        if (hipGetDeviceProperties(&prop, dev) != hipSuccess) return 0;
        cus[dev] = prop.multiProcessorCount;
    }
    return cus[dev];
}

// The division kernel of a batch of `batch` workgroups of T threads.  Those
// built for four waves per SIMD finish sooner as long as the device holds the
// batch at that; and up to three instances per compute unit are faster if four
// waves share each quotient product (us, one wave and four: 1 of 1024 by 512
// limbs 21.7 and 20.5, 768 24.7 and 24.5, 1024 25.6 and 26.1; when it was made,
// 512 of 4096 by 2048 73.5 and 70.2, 256 of 8192 by 4096 135 and 124), which is
// every such batch of more than 256 threads per instance.
mp::Mode division_mode(int T, int64_t batch)
{
    const int cus = device_cus();
    return batch * (T / 64) > (int64_t)16 * cus ? mp::Mode::kPacked
           : batch <= (int64_t)3 * cus          ? mp::Mode::kShared
                                                : mp::Mode::kFast;
}

struct DivShape {
    int threads;
    mp::Mode mode;
};

// In large batches of wide operands LDS allows few instances per compute unit:
// half the waves with twice the registers each do better if they still take
// the remainder update's strips in one round (pairs, and the lowest), that is if
// the divisor is short enough (us, whole and half: 600 divisions of 4096 by 1638
// limbs 77.6 and 72.9, 2000 of 2500 by 1500 89.0 and 86.0, by 1875 72.9 and 73.6,
// 2000 of 4096 by 3072 131 and 137; 1000 of 8192 by 1228 340 and 301, by 4915 308
// and 311).
DivShape division_shape(int nu, int nv, int64_t batch)
{
    const int T = threads_for(nu);
    const mp::Mode mode = division_mode(T, batch);
    if (mode == mp::Mode::kPacked && T >= 512 && nv + 2 <= (T / 64 - 1) * mp::kStrip) return {T / 2, mp::Mode::kFast};
    return {T, mode};
}

// The work queue of mp_divrem_ragged_static: a library-owned array of one
// ragged workspace for MP_STATIC_MAX_COUNT instances (1 MiB), one copy per
// GPU, kept until the process ends.  Host code never uses the array's name as
// an address: static_scratch() returns this device's copy's address, fetched
// once per device with that device current.
static __device__ __align__(256) int32_t scratch[kWsHeader + kClasses * MP_STATIC_MAX_COUNT];

int32_t *static_scratch()
{
    static void *ptr[64];
    static std::mutex mu;
    int dev = 0;
    if (hipGetDevice(&dev) != hipSuccess || dev < 0 || dev >= 64) return nullptr;
    std::lock_guard<std::mutex> lock(mu);
    if (!ptr[dev]) {
        void *p = nullptr;
        if (hipGetSymbolAddress(&p, HIP_SYMBOL(scratch)) != hipSuccess || !p) return nullptr;
        ptr[dev] = p;
    }
    return (int32_t *)ptr[dev];
}

// A ragged batch of at most two instances per compute unit: one launch of one
// 1024-thread workgroup per instance with the LDS of the widest division
// (two per unit), which checks its own descriptor.  No instance waits for
// another, so neither the preparation kernel nor the classes' streams gain
// anything: 5 instances take 53 us (prepared 105), 256 122 (187), 512 142
// (178); 700 would run in rounds of 512, 10% slower than by classes.  False: the
// batch is larger.
bool ragged_direct(const uint32_t *u_pool, const uint32_t *v_pool, const mp_desc_t *desc, uint32_t *q_pool,
                   uint32_t *r_pool, const mp::PoolLimbs &pools, int32_t *inst_status, int32_t count, hipStream_t st,
                   mp_status_t *result)
{
    const int cus = device_cus();
    if (count > 2 * cus) return false;
    const mp::Mode mode = division_mode(1024, count);
    const auto launch = mode == mp::Mode::kPacked ? mp::launch_ragged_direct<1024, mp::Mode::kPacked>
                                                  : mp::launch_ragged_direct<1024, mp::Mode::kShared>;
    *result = status_of(launch(count, body_bytes(mp::kMaxLimbs, mp::kMaxLimbs, mode), st, u_pool, v_pool, desc, q_pool,
                               r_pool, inst_status, pools, block_max()));
    return true;
}

// Streams and events of the concurrent class kernels.  The widest class, most
// of a batch's time, runs on the caller's stream: with a stream for each class
// a fifth one shares a hardware queue (of four), and the whole batch waits
// for whatever is queued there (4096 mixed instances took 530 us where a stream
// for each class took 600 to 750 from one process to the next).
constexpr int kForked = kClasses - 1;
struct Forks {
    hipStream_t fs[kForked];
    hipEvent_t ev_fork, ev_join[kForked];
};

// The launches of a larger ragged batch: descriptor check and bucketing, then
// one persistent kernel per width class, the widest on st, the others each on
// its own fork stream joined back into st (all on st, one after another, when
// fk is null).  The preparation kernel sets every counter of the workspace, so
// it needs no clearing.  Called with g_ragged_mu held.
mp_status_t ragged_launch(const uint32_t *u_pool, const uint32_t *v_pool, const mp_desc_t *desc, uint32_t *q_pool,
                          uint32_t *r_pool, const mp::PoolLimbs &pools, int32_t *inst_status, int32_t count,
                          int32_t *ws, hipStream_t st, const Forks *fk)
{
    const int cus = device_cus();
    if (cus <= 0) return MP_ERR_DEVICE;
    const int bmax = block_max();
    hipLaunchKernelGGL(k_ragged_prep, dim3(1), dim3(1024), 0, st, desc, count, pools, inst_status, ws);
    if (hipGetLastError() != hipSuccess) return MP_ERR_LAUNCH;
    if (fk && hipEventRecord(fk->ev_fork, st) != hipSuccess) return MP_ERR_LAUNCH;
    mp_status_t result = MP_OK;
    int forks = kForked;                              // the fork streams [forks, kForked) hold work
    for (int c = kClasses - 1; c >= 0 && result == MP_OK; c--) {
        const bool forked = fk && c < kForked;
        hipStream_t fs = forked ? fk->fs[c] : st;
        if (forked && hipStreamWaitEvent(fs, fk->ev_fork, 0) != hipSuccess) {
            result = MP_ERR_LAUNCH;
            break;
        }
        if (forked) forks = c;
        const int T = g_ragged.threads[c];
        const size_t bytes = body_bytes(kClassWidth[c], kClassWidth[c]);   // the class's widest instance
        const int fit = (int)(((size_t)kLdsWords * 4) / bytes);
        const int wpc = g_ragged.wgs_per_cu[c] < fit ? g_ragged.wgs_per_cu[c] : fit;
        const auto launch = T == 256   ? mp::launch_ragged<256>
                            : T == 512 ? mp::launch_ragged<512>
                                       : mp::launch_ragged<1024>;
        result = status_of(launch(cus * wpc, bytes, fs, u_pool, v_pool, desc, q_pool, r_pool, inst_status, ws, c,
                                  count, cus, bmax));
        if (forked && hipEventRecord(fk->ev_join[c], fs) != hipSuccess) result = MP_ERR_LAUNCH;
    }
    // (also after a failure: what runs on a fork stream must not outlive the caller's order)
    for (int c = forks; c < kForked; c++)
        if (hipStreamWaitEvent(st, fk->ev_join[c], 0) != hipSuccess) result = MP_ERR_LAUNCH;
    return result;
}

}  // namespace

extern "C" {

const char *mp_status_str(mp_status_t s)
{
    switch (s) {
    case MP_OK: return "MP_OK";
    case MP_ERR_ARG: return "MP_ERR_ARG: invalid argument";
    case MP_ERR_SIZE: return "MP_ERR_SIZE: operand wider than mp_max_limbs()";
    case MP_ERR_LAUNCH: return "MP_ERR_LAUNCH: kernel launch failed";
    case MP_ERR_DEVICE: return "MP_ERR_DEVICE: no usable gfx950 device";
    case MP_ERR_COUNT: return "MP_ERR_COUNT: count exceeds MP_STATIC_MAX_COUNT (the static work queue's size)";
    }
    return "unknown mp_status_t";
}

int32_t mp_max_limbs(void) { return mp::kMaxLimbs; }

mp_status_t mp_set_knob(int32_t knob, int32_t value)
{
    switch (knob) {
    case MP_KNOB_MFMA_MIN:
        if (value < 1) return MP_ERR_ARG;
        g_mfma_min.store(value);
        return MP_OK;
    case MP_KNOB_SMALL_LIMIT:
        if (value != MP_SMALL_LIMIT_AUTO && (value < 0 || value > kMaxLimit)) return MP_ERR_ARG;
        g_small_limit.store(value);
        return MP_OK;
    }
    return MP_ERR_ARG;
}

int32_t mp_get_knob(int32_t knob)
{
    switch (knob) {
    case MP_KNOB_MFMA_MIN: return g_mfma_min.load();
    case MP_KNOB_SMALL_LIMIT: return g_small_limit.load();
    }
    return -1;
}

int64_t mp_lds_bytes(int32_t op, int32_t n1, int32_t n2)
{
    if (n1 <= 0 || n2 <= 0 || n1 > mp::kMaxLimbs || n2 > mp::kMaxLimbs) return -1;
    switch (op) {
    case MP_OP_MUL: return (int64_t)4 * (mp::hmin(n1, n2) < g_mfma_min.load() ? mp::mul_valu_lds_words(n1, n2)
                                                                        : mp::plan_mul(n1, n2).total);
    case MP_OP_DIVREM: return (int64_t)body_bytes(n1, n2);
    case MP_OP_SHINV: return (int64_t)body_bytes(n2 + 1, n1);
    }
    return -1;
}

mp_status_t mp_mul_batch(const uint32_t *a, int32_t na, const uint32_t *b, int32_t nb,
                         uint32_t *c, int32_t batch, void *stream)
{
    if (!a || !b || !c || na <= 0 || nb <= 0 || batch < 0) return MP_ERR_ARG;
    if (na > mp::kMaxLimbs || nb > mp::kMaxLimbs) return MP_ERR_SIZE;
    if (batch == 0) return MP_OK;
    if (!device_ok()) return MP_ERR_DEVICE;
    hipStream_t st = (hipStream_t)stream;
    const int lo = na < nb ? na : nb;
    if (lo < g_mfma_min.load())
        return launch_mul_threads(threads_for((na + nb + 1) / 2), batch, st, a, na, b, nb, c, mp::MulKind::kValu);
    const MulShape m = mul_shape(lo, na + nb, batch);
    return launch_mul_threads(m.threads, batch, st, a, na, b, nb, c, m.kind);
}

mp_status_t mp_shinv_batch(const uint32_t *v, int32_t nv, int32_t h, uint32_t *w, int32_t nw,
                           int32_t *inst_status, int32_t batch, void *stream)
{
    if (!v || !w || nv <= 0 || nw <= 0 || h < 0 || batch < 0) return MP_ERR_ARG;
    if (nv > mp::kMaxLimbs || h > mp::kMaxLimbs) return MP_ERR_SIZE;
    if (batch == 0) return MP_OK;
    if (!device_ok()) return MP_ERR_DEVICE;
    const DivShape shape = division_shape(h > 0 ? h : 1, nv, batch);
    const size_t bytes = body_bytes(h + 1, nv, shape.mode);
    if (bytes > (size_t)kLdsWords * 4) return MP_ERR_SIZE;
    hipStream_t st = (hipStream_t)stream;
    const int bmax = block_max();
    using mp::Mode;
    const auto launch =
        shape.mode == Mode::kFast     ? (shape.threads == 256 ? mp::launch_shinv<256, Mode::kFast>
                                                              : mp::launch_shinv<512, Mode::kFast>)
        : shape.mode == Mode::kShared ? (shape.threads == 256   ? mp::launch_shinv<256, Mode::kShared>
                                         : shape.threads == 512 ? mp::launch_shinv<512, Mode::kShared>
                                                                : mp::launch_shinv<1024, Mode::kShared>)
                                      : (shape.threads == 256   ? mp::launch_shinv<256, Mode::kPacked>
                                         : shape.threads == 512 ? mp::launch_shinv<512, Mode::kPacked>
                                                                : mp::launch_shinv<1024, Mode::kPacked>);
    return status_of(launch(batch, bytes, st, v, nv, h, w, nw, inst_status, bmax));
}

mp_status_t mp_divrem_batch(const uint32_t *u, int32_t nu, const uint32_t *v, int32_t nv,
                            uint32_t *q, int32_t nq, uint32_t *r, int32_t *inst_status,
                            int32_t batch, void *stream)
{
    if (!u || !v || !q || !r || nu <= 0 || nv <= 0 || nq <= 0 || batch < 0) return MP_ERR_ARG;
    if (nu > mp::kMaxLimbs || nv > mp::kMaxLimbs) return MP_ERR_SIZE;
    if (batch == 0) return MP_OK;
    if (!device_ok()) return MP_ERR_DEVICE;
    const DivShape shape = division_shape(nu, nv, batch);
    const size_t bytes = body_bytes(nu, nv, shape.mode);
    if (bytes > (size_t)kLdsWords * 4) return MP_ERR_SIZE;
    hipStream_t st = (hipStream_t)stream;
    const int bmax = block_max();
    using mp::Mode;
    const auto launch =
        shape.mode == Mode::kFast     ? (shape.threads == 256 ? mp::launch_divrem<256, Mode::kFast>
                                                              : mp::launch_divrem<512, Mode::kFast>)
        : shape.mode == Mode::kShared ? (shape.threads == 256   ? mp::launch_divrem<256, Mode::kShared>
                                         : shape.threads == 512 ? mp::launch_divrem<512, Mode::kShared>
                                                                : mp::launch_divrem<1024, Mode::kShared>)
                                      : (shape.threads == 256   ? mp::launch_divrem<256, Mode::kPacked>
                                         : shape.threads == 512 ? mp::launch_divrem<512, Mode::kPacked>
                                                                : mp::launch_divrem<1024, Mode::kPacked>);
    return status_of(launch(batch, bytes, st, u, nu, v, nv, q, nq, r, inst_status, bmax));
}

int64_t mp_ragged_workspace_bytes(int32_t count)
{
    return count < 0 ? 0 : (int64_t)4 * (kWsHeader + (int64_t)kClasses * count);
}

mp_status_t mp_ragged_config(int32_t cls, int32_t threads, int32_t wgs_per_cu)
{
    if (cls < 0 || cls >= kClasses || wgs_per_cu < 1 || wgs_per_cu > 8) return MP_ERR_ARG;
    if (threads != 256 && threads != 512 && threads != 1024) return MP_ERR_ARG;
    if (threads * 8 < kClassWidth[cls]) return MP_ERR_ARG;
    std::lock_guard<std::mutex> lock(g_ragged_mu);
    g_ragged.threads[cls] = threads;
    g_ragged.wgs_per_cu[cls] = wgs_per_cu;
    return MP_OK;
}

mp_status_t mp_divrem_ragged(const uint32_t *u_pool, int64_t u_limbs, const uint32_t *v_pool, int64_t v_limbs,
                             const mp_desc_t *desc, uint32_t *q_pool, int64_t q_limbs, uint32_t *r_pool,
                             int64_t r_limbs, int32_t *inst_status, int32_t count, void *workspace,
                             void *stream)
{
    if (!u_pool || !v_pool || !desc || !q_pool || !r_pool || !inst_status || !workspace || count < 0)
        return MP_ERR_ARG;
    if (u_limbs < 0 || v_limbs < 0 || q_limbs < 0 || r_limbs < 0) return MP_ERR_ARG;
    if (count == 0) return MP_OK;
    if (!device_ok()) return MP_ERR_DEVICE;
    hipStream_t st = (hipStream_t)stream;
    const mp::PoolLimbs pools{u_limbs, v_limbs, q_limbs, r_limbs};
    mp_status_t direct;
    if (ragged_direct(u_pool, v_pool, desc, q_pool, r_pool, pools, inst_status, count, st, &direct)) return direct;
    std::lock_guard<std::mutex> lock(g_ragged_mu);
    int dev = 0;
    if (hipGetDevice(&dev) != hipSuccess || dev < 0 || dev >= 64) return MP_ERR_DEVICE;
    // fork streams and events (default priority), one set per caller stream
    // (up to kForkSets per device, made on first use), so batches launched on
    // different streams run their class kernels side by side; further caller
    // streams share the last set (correct, only serialised)
    constexpr int kForkSets = 8;
    static Forks forks[64][kForkSets];
    static hipStream_t owner[64][kForkSets];
    static int nsets[64];
    int f = 0;
    while (f < nsets[dev] && owner[dev][f] != st) f++;
    if (f == nsets[dev]) {
        // no set for this stream yet: none is made while the stream is being
        // captured into a graph (the kernels then run in order on it)
        hipStreamCaptureStatus cap = hipStreamCaptureStatusNone;
        if (hipStreamIsCapturing(st, &cap) != hipSuccess) return MP_ERR_LAUNCH;
        if (cap != hipStreamCaptureStatusNone)
            return ragged_launch(u_pool, v_pool, desc, q_pool, r_pool, pools, inst_status, count,
                                 (int32_t *)workspace, st, nullptr);
        if (f == kForkSets) {
            f = kForkSets - 1;
        } else {
            Forks &fk = forks[dev][f];
            for (int c = 0; c < kForked; c++) {
                if (hipStreamCreateWithFlags(&fk.fs[c], hipStreamNonBlocking) != hipSuccess ||
                    hipEventCreateWithFlags(&fk.ev_join[c], hipEventDisableTiming) != hipSuccess)
                    return MP_ERR_LAUNCH;
            }
            if (hipEventCreateWithFlags(&fk.ev_fork, hipEventDisableTiming) != hipSuccess) return MP_ERR_LAUNCH;
            owner[dev][f] = st;
            nsets[dev] = f + 1;
        }
    }
    return ragged_launch(u_pool, v_pool, desc, q_pool, r_pool, pools, inst_status, count, (int32_t *)workspace, st,
                         &forks[dev][f]);
}

mp_status_t mp_divrem_ragged_static(const uint32_t *u_pool, int64_t u_limbs, const uint32_t *v_pool,
                                    int64_t v_limbs, const mp_desc_t *desc, uint32_t *q_pool, int64_t q_limbs,
                                    uint32_t *r_pool, int64_t r_limbs, int32_t *inst_status, int32_t count,
                                    void *stream)
{
    if (!u_pool || !v_pool || !desc || !q_pool || !r_pool || !inst_status || count < 0) return MP_ERR_ARG;
    if (u_limbs < 0 || v_limbs < 0 || q_limbs < 0 || r_limbs < 0) return MP_ERR_ARG;
    if (count > MP_STATIC_MAX_COUNT) return MP_ERR_COUNT;
    if (count == 0) return MP_OK;
    if (!device_ok()) return MP_ERR_DEVICE;
    const mp::PoolLimbs pools{u_limbs, v_limbs, q_limbs, r_limbs};
    mp_status_t direct;
    if (ragged_direct(u_pool, v_pool, desc, q_pool, r_pool, pools, inst_status, count, (hipStream_t)stream, &direct))
        return direct;
    std::lock_guard<std::mutex> lock(g_ragged_mu);
    int32_t *ws = static_scratch();
    if (!ws) return MP_ERR_DEVICE;
    return ragged_launch(u_pool, v_pool, desc, q_pool, r_pool, pools, inst_status, count, ws, (hipStream_t)stream,
                         nullptr);
}

}  // extern "C"
