/* The HIP entry points libpatconv.so calls, without a device: memory is host memory, kernels are noted and not run. Loaded into the
 * global symbol scope ahead of the library, so that a test on the CPU sees which kernel a call takes and what it is launched with. */
#define __HIP_PLATFORM_AMD__
#include <hip/hip_runtime_api.h>
#include <stdlib.h>
#include <string.h>

static struct { const void *fn; char name[256]; } fns[1024];
static int n_fns;
static dim3 cfg_grid, cfg_block;
static size_t cfg_lds;
static hipStream_t cfg_stream;

/* what a test sets and reads */
int stub_capturing, stub_malloc_fails, stub_count;     /* stub_count: the kept kernels of a pack, read back from the device */
int stub_arg, stub_arg_bytes;          /* the argument of a launch that is copied to stub_args */
char stub_args[8192], stub_name[256];  /* of the last launch whose kernel's name holds stub_watch */
char stub_watch[64];
long long stub_grid, stub_lds;

/* operator new of what is loaded after this file: from the time stub_new_left is set to n > 0, the n-th call fails */
int stub_new_left;
extern void _ZSt17__throw_bad_allocv(void);
void *_Znwm(size_t n)
{
    void *p = stub_new_left > 0 && --stub_new_left == 0 ? NULL : malloc(n ? n : 1);
    if (!p) _ZSt17__throw_bad_allocv();
    return p;
}

void **__hipRegisterFatBinary(const void *d) { static void *h; (void)d; return &h; }
void __hipUnregisterFatBinary(void **h) { (void)h; }
void __hipRegisterVar(void **h, void *v, char *hn, const char *dn, int e, size_t s, int c, int g) { (void)h; (void)v; (void)hn; (void)dn; (void)e; (void)s; (void)c; (void)g; }
void __hipRegisterFunction(void **h, const void *fn, char *dev, const char *name, unsigned tl, void *a, void *b, void *c, void *d, int *e)
{
    (void)h; (void)dev; (void)tl; (void)a; (void)b; (void)c; (void)d; (void)e;
    if (n_fns == 1024) abort();
    fns[n_fns].fn = fn;
    strncpy(fns[n_fns++].name, name, 255);
}
hipError_t __hipPushCallConfiguration(dim3 grid, dim3 block, size_t lds, hipStream_t s)
{
    cfg_grid = grid; cfg_block = block; cfg_lds = lds; cfg_stream = s;
    return hipSuccess;
}
hipError_t __hipPopCallConfiguration(dim3 *grid, dim3 *block, size_t *lds, hipStream_t *s)
{
    *grid = cfg_grid; *block = cfg_block; *lds = cfg_lds; *s = cfg_stream;
    return hipSuccess;
}
hipError_t hipLaunchKernel(const void *fn, dim3 grid, dim3 block, void **args, size_t lds, hipStream_t s)
{
    (void)block; (void)s;
    for (int i = 0; i < n_fns; ++i)
        if (fns[i].fn == fn && strstr(fns[i].name, stub_watch)) {
            strcpy(stub_name, fns[i].name);
            stub_grid = (long long)grid.x * grid.y * grid.z;
            stub_lds = (long long)lds;
            if (stub_arg_bytes) memcpy(stub_args, args[stub_arg], (size_t)stub_arg_bytes);
        }
    return hipSuccess;
}
hipError_t hipGetDeviceCount(int *n) { *n = 1; return hipSuccess; }
hipError_t hipSetDevice(int d) { (void)d; return hipSuccess; }
hipError_t hipGetDeviceProperties(hipDeviceProp_t *p, int d)
{
    (void)d;
    memset(p, 0, sizeof(*p));
    p->multiProcessorCount = 256;
    return hipSuccess;
}
hipError_t hipGetSymbolAddress(void **p, const void *s) { static char fixed[64]; (void)s; *p = fixed; return hipSuccess; }
hipError_t hipFuncSetAttribute(const void *f, hipFuncAttribute a, int v) { (void)f; (void)a; (void)v; return hipSuccess; }
hipError_t hipMalloc(void **p, size_t n)
{
    if (stub_malloc_fails) return hipErrorOutOfMemory;
    *p = calloc(1, n);
    return *p ? hipSuccess : hipErrorOutOfMemory;
}
hipError_t hipFree(void *p) { free(p); return hipSuccess; }
hipError_t hipMemcpy(void *d, const void *s, size_t n, hipMemcpyKind k) { (void)k; memcpy(d, s, n); return hipSuccess; }
hipError_t hipMemcpyAsync(void *d, const void *s, size_t n, hipMemcpyKind k, hipStream_t st) { (void)d; (void)s; (void)n; (void)k; (void)st; return hipSuccess; }
hipError_t hipMemcpyWithStream(void *d, const void *s, size_t n, hipMemcpyKind k, hipStream_t st) { (void)s; (void)n; (void)k; (void)st; *(int *)d = stub_count; return hipSuccess; }
hipError_t hipStreamIsCapturing(hipStream_t s, hipStreamCaptureStatus *c)
{
    (void)s;
    *c = stub_capturing ? hipStreamCaptureStatusActive : hipStreamCaptureStatusNone;
    return hipSuccess;
}
hipError_t hipStreamSynchronize(hipStream_t s) { (void)s; return hipSuccess; }
hipError_t hipDeviceSynchronize(void) { return hipSuccess; }
hipError_t hipGetLastError(void) { return hipSuccess; }
const char *hipGetErrorString(hipError_t e) { return e == hipErrorOutOfMemory ? "out of memory" : "error"; }
