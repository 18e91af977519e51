/* A HIP runtime without a GPU, for tests of the library's host code: device memory is host
 * memory, streams and events are nothing, and a kernel launch is recorded and not run.  Loaded
 * with RTLD_GLOBAL before the library, it takes the place of the runtime.  A test can make the
 * launches of one kernel, or the allocations of pinned memory, fail, and reads back what was
 * launched (a kernel's name and the words of its first arguments). */
#define __HIP_PLATFORM_AMD__ 1
#include <hip/hip_runtime_api.h>
#include <stdlib.h>
#include <string.h>

#define MAX_FN 512
#define MAX_LAUNCH 4096
#define ARG_WORDS 8

static struct { const void *fn; char name[256]; } fns[MAX_FN];
static int n_fns;
struct launch { char name[256]; unsigned grid, block; };
static struct launch launches[MAX_LAUNCH];
static unsigned long long arg0[MAX_LAUNCH][ARG_WORDS];
static int n_launches, n_syncs;
static hipError_t last_error = hipSuccess;
static char fail_name[256];
static int fail_pinned;

int fake_launches(void) { return n_launches; }
const char *fake_launch_name(int i) { return launches[i].name; }
unsigned fake_launch_grid(int i) { return launches[i].grid; }
const unsigned long long *fake_launch_arg0(int i) { return arg0[i]; }
int fake_syncs(void) { return n_syncs; }
void fake_reset(void) { n_launches = n_syncs = 0; }
void fake_fail_kernel(const char *part) { strncpy(fail_name, part, sizeof fail_name - 1); }
void fake_fail_pinned(int on) { fail_pinned = on; }

static hipError_t fail(hipError_t e) { return last_error = e; }

void **__hipRegisterFatBinary(const void *data) { (void)data; return calloc(1, sizeof(void *)); }
void __hipUnregisterFatBinary(void **h) { free(h); }
void __hipRegisterFunction(void **h, const void *fn, char *dev, const char *name, unsigned limit, void *tid, void *bid,
                           void *bdim, void *gdim, int *wsize)
{
    (void)h, (void)dev, (void)limit, (void)tid, (void)bid, (void)bdim, (void)gdim, (void)wsize;
    if (n_fns < MAX_FN) {
        fns[n_fns].fn = fn;
        strncpy(fns[n_fns].name, name, sizeof fns[0].name - 1);
        n_fns++;
    }
}
void __hipRegisterVar(void **h, void *var, char *host, char *dev, int ext, size_t size, int constant, int global)
{
    (void)h, (void)var, (void)host, (void)dev, (void)ext, (void)size, (void)constant, (void)global;
}
static dim3 cfg_grid, cfg_block;
static size_t cfg_shared;
static hipStream_t cfg_stream;
hipError_t __hipPushCallConfiguration(dim3 grid, dim3 block, size_t shared, hipStream_t s)
{
    cfg_grid = grid, cfg_block = block, cfg_shared = shared, cfg_stream = s;
    return hipSuccess;
}
hipError_t __hipPopCallConfiguration(dim3 *grid, dim3 *block, size_t *shared, hipStream_t *s)
{
    *grid = cfg_grid, *block = cfg_block, *shared = cfg_shared, *s = cfg_stream;
    return hipSuccess;
}
hipError_t hipLaunchKernel(const void *fn, dim3 grid, dim3 block, void **args, size_t shared, hipStream_t s)
{
    (void)shared, (void)s;
    const char *name = "?";
    for (int i = 0; i < n_fns; i++)
        if (fns[i].fn == fn)
            name = fns[i].name;
    if (fail_name[0] && strstr(name, fail_name))
        return fail(hipErrorLaunchFailure);
    if (n_launches < MAX_LAUNCH) {
        strncpy(launches[n_launches].name, name, sizeof launches[0].name - 1);
        launches[n_launches].grid = grid.x;
        launches[n_launches].block = block.x;
        /* (the caller's argument block: at least the first argument, read as far as the next) */
        memset(arg0[n_launches], 0, sizeof arg0[0]);
        memcpy(arg0[n_launches], args[0], sizeof arg0[0]);
        n_launches++;
    }
    return hipSuccess;
}

hipError_t hipGetLastError(void) { hipError_t e = last_error; last_error = hipSuccess; return e; }
const char *hipGetErrorString(hipError_t e) { (void)e; return "injected"; }
hipError_t hipGetDeviceCount(int *n) { *n = 1; return hipSuccess; }
hipError_t hipSetDevice(int d) { (void)d; return hipSuccess; }
hipError_t hipGetDevice(int *d) { *d = 0; return hipSuccess; }
hipError_t hipGetDeviceProperties(hipDeviceProp_t *p, int d)
{
    (void)d;
    memset(p, 0, sizeof *p);
    p->multiProcessorCount = 256;
    return hipSuccess;
}
hipError_t hipDeviceGetAttribute(int *v, hipDeviceAttribute_t a, int d) { (void)a, (void)d; *v = 256; return hipSuccess; }
hipError_t hipOccupancyMaxActiveBlocksPerMultiprocessor(int *n, const void *f, int b, size_t s)
{
    (void)f, (void)b, (void)s;
    *n = 2;
    return hipSuccess;
}
hipError_t hipMalloc(void **p, size_t n) { *p = calloc(1, n ? n : 1); return *p ? hipSuccess : fail(hipErrorOutOfMemory); }
hipError_t hipFree(void *p) { free(p); return hipSuccess; }
hipError_t hipHostMalloc(void **p, size_t n, unsigned flags)
{
    (void)flags;
    if (fail_pinned)
        return fail(hipErrorOutOfMemory);
    return hipMalloc(p, n);
}
hipError_t hipHostFree(void *p) { free(p); return hipSuccess; }
hipError_t hipGetSymbolAddress(void **p, const void *sym) { (void)sym; return hipMalloc(p, 8u << 20); }
hipError_t hipMemcpy(void *d, const void *s, size_t n, hipMemcpyKind k) { (void)k; memmove(d, s, n); return hipSuccess; }
hipError_t hipMemcpyAsync(void *d, const void *s, size_t n, hipMemcpyKind k, hipStream_t st)
{
    (void)st;
    return hipMemcpy(d, s, n, k);
}
hipError_t hipStreamCreateWithFlags(hipStream_t *s, unsigned f) { (void)f; return hipMalloc((void **)s, 8); }
hipError_t hipStreamDestroy(hipStream_t s) { return hipFree((void *)s); }
hipError_t hipStreamSynchronize(hipStream_t s) { (void)s; n_syncs++; return hipSuccess; }
hipError_t hipStreamWaitEvent(hipStream_t s, hipEvent_t e, unsigned f) { (void)s, (void)e, (void)f; return hipSuccess; }
hipError_t hipStreamBeginCapture(hipStream_t s, hipStreamCaptureMode m) { (void)s, (void)m; return hipErrorNotSupported; }
hipError_t hipStreamEndCapture(hipStream_t s, hipGraph_t *g) { (void)s; *g = 0; return hipErrorNotSupported; }
hipError_t hipGraphInstantiate(hipGraphExec_t *e, hipGraph_t g, hipGraphNode_t *n, char *b, size_t z)
{
    (void)e, (void)g, (void)n, (void)b, (void)z;
    return hipErrorNotSupported;
}
hipError_t hipGraphLaunch(hipGraphExec_t e, hipStream_t s) { (void)e, (void)s; return hipErrorNotSupported; }
hipError_t hipGraphDestroy(hipGraph_t g) { (void)g; return hipSuccess; }
hipError_t hipGraphExecDestroy(hipGraphExec_t e) { (void)e; return hipSuccess; }
hipError_t hipEventCreate(hipEvent_t *e) { return hipMalloc((void **)e, 8); }
hipError_t hipEventCreateWithFlags(hipEvent_t *e, unsigned f) { (void)f; return hipMalloc((void **)e, 8); }
hipError_t hipEventDestroy(hipEvent_t e) { return hipFree((void *)e); }
hipError_t hipEventRecord(hipEvent_t e, hipStream_t s) { (void)e, (void)s; return hipSuccess; }
hipError_t hipEventQuery(hipEvent_t e) { (void)e; return hipSuccess; }
hipError_t hipEventSynchronize(hipEvent_t e) { (void)e; return hipSuccess; }
hipError_t hipEventElapsedTime(float *ms, hipEvent_t a, hipEvent_t b) { (void)a, (void)b; *ms = 1.0f; return hipSuccess; }
