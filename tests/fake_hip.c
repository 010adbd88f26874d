/* A stand-in for the HIP runtime, preloaded by test_host_calls.py: two devices of 256 compute units,
 * device memory that is host memory, streams that finish at once, and kernels that do nothing.  It keeps
 * a log of what the host code asked for: one line per allocation, device selection and launch, each
 * with the device that was current. */
#define _GNU_SOURCE
#include <hip/hip_runtime_api.h>
#include <stdarg.h>
#include <stdio.h>
#include <stdlib.h>
#include <string.h>

static int cur = 0;
static char* text = NULL;
static size_t len = 0, cap = 0;

static void say(const char* fmt, ...)
{
    char line[512];
    va_list ap;
    va_start(ap, fmt);
    int n = vsnprintf(line, sizeof line, fmt, ap);
    va_end(ap);
    if (n >= (int)sizeof line) n = (int)sizeof line - 1;
    if (len + (size_t)n + 1 > cap) {
        cap = 2 * cap + 4096 + (size_t)n;
        text = realloc(text, cap);
    }
    memcpy(text + len, line, (size_t)n + 1);
    len += (size_t)n;
}

const char* fake_log(void) { return text ? text : ""; }
void fake_clear(void)
{
    len = 0;
    if (text) text[0] = 0;
}
void fake_current(int d) { cur = d; }  /* what another part of the program left current */

hipError_t hipGetDeviceCount(int* n) { *n = 2; return hipSuccess; }
hipError_t hipSetDevice(int d) { cur = d; say("device %d\n", d); return hipSuccess; }
hipError_t hipGetDevicePropertiesR0600(hipDeviceProp_tR0600* p, int d)
{
    (void)d;
    memset(p, 0, sizeof *p);
    p->multiProcessorCount = 256;
    strcpy(p->gcnArchName, "gfx950");
    return hipSuccess;
}
hipError_t hipDeviceGetAttribute(int* v, hipDeviceAttribute_t a, int d) { (void)a; (void)d; *v = 100000; return hipSuccess; }
hipError_t hipDeviceSynchronize(void) { return hipSuccess; }
const char* hipGetErrorString(hipError_t e) { (void)e; return "error"; }
hipError_t hipGetLastError(void) { return hipSuccess; }

hipError_t hipMalloc(void** p, size_t n) { say("malloc %d %zu\n", cur, n); *p = malloc(n ? n : 1); return hipSuccess; }
hipError_t hipMallocAsync(void** p, size_t n, hipStream_t s)
{
    (void)s;
    say("async %d %zu\n", cur, n);
    *p = malloc(n ? n : 1);
    return hipSuccess;
}
hipError_t hipFree(void* p) { free(p); return hipSuccess; }
hipError_t hipFreeAsync(void* p, hipStream_t s) { (void)s; free(p); return hipSuccess; }
hipError_t hipHostMalloc(void** p, size_t n, unsigned f) { (void)f; say("pinned %d %zu\n", cur, n); *p = calloc(1, n ? n : 1); return hipSuccess; }
hipError_t hipHostFree(void* p) { free(p); return hipSuccess; }
hipError_t hipMemcpy(void* d, const void* s, size_t n, hipMemcpyKind k) { (void)k; memcpy(d, s, n); return hipSuccess; }
hipError_t hipMemcpyAsync(void* d, const void* s, size_t n, hipMemcpyKind k, hipStream_t st)
{
    (void)k;
    (void)st;
    memcpy(d, s, n);
    return hipSuccess;
}
hipError_t hipMemset(void* d, int v, size_t n) { memset(d, v, n); return hipSuccess; }
hipError_t hipGetSymbolAddress(void** p, const void* sym)
{
    (void)sym;
    static void* block = NULL;
    if (!block) block = malloc(16u << 20);
    *p = block;
    return hipSuccess;
}

hipError_t hipEventCreate(hipEvent_t* e) { *e = (hipEvent_t)malloc(1); return hipSuccess; }
hipError_t hipEventCreateWithFlags(hipEvent_t* e, unsigned f) { (void)f; return hipEventCreate(e); }
hipError_t hipEventDestroy(hipEvent_t e) { free(e); return hipSuccess; }
hipError_t hipEventRecord(hipEvent_t e, hipStream_t s) { (void)e; (void)s; return hipSuccess; }
hipError_t hipEventQuery(hipEvent_t e) { (void)e; return hipSuccess; }
hipError_t hipEventSynchronize(hipEvent_t e) { (void)e; return hipSuccess; }
hipError_t hipEventElapsedTime(float* ms, hipEvent_t a, hipEvent_t b) { (void)a; (void)b; *ms = 1.0f; return hipSuccess; }
hipError_t hipStreamCreateWithFlags(hipStream_t* s, unsigned f) { (void)f; *s = (hipStream_t)malloc(1); return hipSuccess; }
hipError_t hipStreamDestroy(hipStream_t s) { free(s); return hipSuccess; }
hipError_t hipStreamSynchronize(hipStream_t s) { (void)s; return hipSuccess; }
hipError_t hipStreamWaitEvent(hipStream_t s, hipEvent_t e, unsigned f) { (void)s; (void)e; (void)f; return hipSuccess; }
hipError_t hipStreamIsCapturing(hipStream_t s, hipStreamCaptureStatus* c)
{
    (void)s;
    *c = hipStreamCaptureStatusNone;
    return hipSuccess;
}
hipError_t hipOccupancyMaxActiveBlocksPerMultiprocessor(int* n, const void* f, int t, size_t l)
{
    (void)f; (void)t; (void)l;
    *n = 2;
    return hipSuccess;
}

/* kernels by the names that the library registers */
#define MAX_KERNELS 256
static struct { const void* host; const char* name; } kernels[MAX_KERNELS];
static int n_kernels = 0;
void** __hipRegisterFatBinary(const void* d) { (void)d; static void* h; return &h; }
void __hipUnregisterFatBinary(void** m) { (void)m; }
void __hipRegisterFunction(void** m, const void* host, char* dev, const char* name, unsigned t, void* a, void* b,
                           void* c, void* d, int* w)
{
    (void)m; (void)dev; (void)t; (void)a; (void)b; (void)c; (void)d; (void)w;
    if (n_kernels < MAX_KERNELS) {
        kernels[n_kernels].host = host;
        kernels[n_kernels++].name = name;
    }
}
void __hipRegisterVar(void** m, void* v, char* h, char* d, int e, size_t s, int c, int g)
{
    (void)m; (void)v; (void)h; (void)d; (void)e; (void)s; (void)c; (void)g;
}

static dim3 cfg_grid, cfg_block;
static size_t cfg_lds;
static hipStream_t cfg_stream;
hipError_t __hipPushCallConfiguration(dim3 g, dim3 b, size_t l, hipStream_t s)
{
    cfg_grid = g; cfg_block = b; cfg_lds = l; cfg_stream = s;
    return hipSuccess;
}
hipError_t __hipPopCallConfiguration(dim3* g, dim3* b, size_t* l, hipStream_t* s)
{
    *g = cfg_grid; *b = cfg_block; *l = cfg_lds; *s = cfg_stream;
    return hipSuccess;
}
hipError_t hipLaunchKernel(const void* f, dim3 g, dim3 b, void** args, size_t lds, hipStream_t s)
{
    (void)args; (void)s;
    const char* name = "?";
    for (int i = 0; i < n_kernels; ++i)
        if (kernels[i].host == f) name = kernels[i].name;
    say("launch %d %u %u %zu %s\n", cur, g.x, b.x, lds, name);
    return hipSuccess;
}
