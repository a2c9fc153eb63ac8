/* The HIP runtime calls libmpdiv's host code makes, as a record: each prints one
 * line, and the FAKE_HIP_FAIL-th launch (or attribute call, event record, stream
 * wait: any of those printed with a '#') fails.  Loaded before the library, with its
 * symbols visible to it, so that the order of launches, events and waits can be
 * read without a GPU. */
#include <hip/hip_runtime_api.h>
#include <cstdio>
#include <cstdlib>
#include <cstring>
#include <map>
#include <string>

static std::map<const void *, std::string> names;
static hipError_t last = hipSuccess;
static long streams = 0x100, events = 0x1000;

static hipError_t call(const char *what, const void *a, const void *b)
{
    static const int fail = getenv("FAKE_HIP_FAIL") ? atoi(getenv("FAKE_HIP_FAIL")) : 0;
    static int n = 0;
    const hipError_t e = ++n == fail ? hipErrorOutOfMemory : hipSuccess;
    printf("#%s %p %p %s\n", what, a, b, e == hipSuccess ? "ok" : "failed");
    last = e;
    return e;
}

extern "C" {
void **__hipRegisterFatBinary(const void *) { static void *h; return &h; }
void __hipUnregisterFatBinary(void **) {}
void __hipRegisterFunction(void **, const void *f, char *, const char *name, unsigned, void *, void *, void *, void *, int *) { names[f] = name; }
void __hipRegisterVar(void **, void *, char *, char *, int, size_t, int, int) {}

static hipStream_t pushed;
hipError_t __hipPushCallConfiguration(dim3, dim3, size_t, hipStream_t s) { pushed = s; return hipSuccess; }
hipError_t __hipPopCallConfiguration(dim3 *g, dim3 *b, size_t *m, hipStream_t *s)
{
    *g = *b = dim3(1);
    *m = 0;
    *s = pushed;
    return hipSuccess;
}
hipError_t hipLaunchKernel(const void *f, dim3, dim3, void **, size_t, hipStream_t s)
{
    printf("%s\n", names[f].c_str());
    return call("launch", s, nullptr);
}
hipError_t hipGetLastError() { const hipError_t e = last; last = hipSuccess; return e; }
hipError_t hipFuncSetAttribute(const void *, hipFuncAttribute, int) { return call("attribute", nullptr, nullptr); }
hipError_t hipGetDevice(int *d) { *d = 0; return hipSuccess; }
hipError_t hipGetDevicePropertiesR0600(hipDeviceProp_tR0600 *p, int)
{
    memset(p, 0, sizeof *p);
    strcpy(p->gcnArchName, "gfx950:sramecc+:xnack-");
    p->multiProcessorCount = 256;
    return hipSuccess;
}
hipError_t hipGetSymbolAddress(void **p, const void *) { *p = (void *)0x2000; return hipSuccess; }
hipError_t hipStreamCreateWithFlags(hipStream_t *s, unsigned) { *s = (hipStream_t)++streams; return hipSuccess; }
hipError_t hipEventCreateWithFlags(hipEvent_t *e, unsigned) { *e = (hipEvent_t)++events; return hipSuccess; }
hipError_t hipStreamIsCapturing(hipStream_t, hipStreamCaptureStatus *c)
{
    *c = getenv("FAKE_HIP_CAPTURE") ? hipStreamCaptureStatusActive : hipStreamCaptureStatusNone;
    return hipSuccess;
}
hipError_t hipEventRecord(hipEvent_t e, hipStream_t s) { return call("record", s, e); }
hipError_t hipStreamWaitEvent(hipStream_t s, hipEvent_t e, unsigned) { return call("wait", s, e); }
}
