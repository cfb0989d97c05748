/* A stand-in for the HIP runtime, so that the library's host code runs on a
 * machine without a GPU: launches are recorded (kernel, grid, workgroup),
 * copies to the host happen when something waits for them, and calls can be
 * made to fail. Loaded before the library with its symbols visible to it. */
#include <hip/hip_runtime_api.h>
#include <stdlib.h>
#include <string.h>

typedef struct { const char *name; unsigned dim[6]; } Launch;
typedef struct { void *dst; const void *src; size_t bytes; } Copy;

static struct { const void *host; const char *name; } kernels[512];
static int nkernels;
static Launch launches[4096];
static int nlaunches, fail_launch, fail_record;
static Copy copies[64];
static int ncopies;
static hipError_t last;
static struct { dim3 grid, block; size_t shared; hipStream_t stream; } config;
static struct { char part[96]; float ms; } costs[64];
static int ncosts;
static double clock_ms;

static const char *kernel_name(const void *f)
{
    for (int k = 0; k < nkernels; ++k)
        if (kernels[k].host == f) return kernels[k].name;
    return "?";
}

static hipError_t done(hipError_t e) { if (e != hipSuccess) last = e; return e; }

static void arrive(void)
{
    for (int k = 0; k < ncopies; ++k) memcpy(copies[k].dst, copies[k].src, copies[k].bytes);
    ncopies = 0;
}

/* ---- what the tests call */
void dbl_reset(void) { nlaunches = fail_launch = fail_record = ncopies = ncosts = 0; last = hipSuccess; }
int dbl_launches(void) { return nlaunches; }
const char *dbl_launch(int k, unsigned *dim) { memcpy(dim, launches[k].dim, sizeof(launches[k].dim)); return launches[k].name; }
void dbl_fail_launch(int k) { fail_launch = k; }            /* the k-th launch from now (1: the next) */
void dbl_fail_record(int on) { fail_record = on; }
int dbl_pending(void) { return ncopies; }                   /* copies that nothing has waited for */
/* launches whose kernel's name holds `part` take `ms` (1 ms else) */
void dbl_cost(const char *part, float ms) { strncpy(costs[ncosts].part, part, 95); costs[ncosts++].ms = ms; }

/* ---- the runtime */
void **__hipRegisterFatBinary(const void *data) { static void *module; (void)data; return &module; }
void __hipUnregisterFatBinary(void **m) { (void)m; }
void __hipRegisterFunction(void **m, const void *host, char *dev, const char *name, unsigned t, void *tid, void *bid, void *b, void *g, int *w)
{
    (void)m; (void)dev; (void)t; (void)tid; (void)bid; (void)b; (void)g; (void)w;
    kernels[nkernels].host = host;
    kernels[nkernels++].name = name;
}
void __hipRegisterVar(void **m, void *var, char *host, char *dev, int ext, size_t size, int c, int g)
{
    (void)m; (void)var; (void)host; (void)dev; (void)ext; (void)size; (void)c; (void)g;
}
hipError_t __hipPushCallConfiguration(dim3 grid, dim3 block, size_t shared, hipStream_t stream)
{
    config.grid = grid; config.block = block; config.shared = shared; config.stream = stream;
    return hipSuccess;
}
hipError_t __hipPopCallConfiguration(dim3 *grid, dim3 *block, size_t *shared, hipStream_t *stream)
{
    *grid = config.grid; *block = config.block; *shared = config.shared; *stream = config.stream;
    return hipSuccess;
}
hipError_t hipLaunchKernel(const void *f, dim3 g, dim3 b, void **args, size_t shared, hipStream_t s)
{
    (void)args; (void)shared; (void)s;
    if (fail_launch > 0 && --fail_launch == 0) return done(hipErrorInvalidConfiguration);
    const char *name = kernel_name(f);
    if (nlaunches < 4096) {
        const Launch l = {name, {g.x, g.y, g.z, b.x, b.y, b.z}};
        launches[nlaunches++] = l;
    }
    float ms = 1.0f;
    for (int k = 0; k < ncosts; ++k)
        if (strstr(name, costs[k].part)) ms = costs[k].ms;
    clock_ms += ms;
    return hipSuccess;
}
hipError_t hipGetLastError(void) { const hipError_t e = last; last = hipSuccess; return e; }
const char *hipGetErrorString(hipError_t e) { return e == hipSuccess ? "no error" : "made to fail"; }
hipError_t hipGetDevice(int *d) { *d = 0; return hipSuccess; }
hipError_t hipGetDeviceProperties(hipDeviceProp_t *p, int d) { (void)d; memset(p, 0, sizeof(*p)); strcpy(p->gcnArchName, "gfx950"); return hipSuccess; }
hipError_t hipDeviceGetAttribute(int *v, hipDeviceAttribute_t a, int d) { (void)a; (void)d; *v = 256; return hipSuccess; }
hipError_t hipDeviceSynchronize(void) { arrive(); return hipSuccess; }
hipError_t hipStreamSynchronize(hipStream_t s) { (void)s; arrive(); return hipSuccess; }
hipError_t hipStreamIsCapturing(hipStream_t s, hipStreamCaptureStatus *st) { (void)s; *st = hipStreamCaptureStatusNone; return hipSuccess; }
hipError_t hipMalloc(void **p, size_t n) { *p = aligned_alloc(256, (n + 255) / 256 * 256); return hipSuccess; }
hipError_t hipFree(void *p) { free(p); return hipSuccess; }
hipError_t hipHostMalloc(void **p, size_t n, unsigned f) { (void)f; *p = calloc(1, n); return hipSuccess; }
hipError_t hipHostFree(void *p) { free(p); return hipSuccess; }
hipError_t hipMemcpyAsync(void *dst, const void *src, size_t n, hipMemcpyKind kind, hipStream_t s)
{
    (void)s;
    if (kind == hipMemcpyDeviceToHost) {
        const Copy c = {dst, src, n};
        copies[ncopies++] = c;
    } else {
        memcpy(dst, src, n);
    }
    return hipSuccess;
}
hipError_t hipEventCreate(hipEvent_t *e) { *e = (hipEvent_t)calloc(1, sizeof(double)); return hipSuccess; }
hipError_t hipEventCreateWithFlags(hipEvent_t *e, unsigned f) { (void)f; return hipEventCreate(e); }
hipError_t hipEventDestroy(hipEvent_t e) { free(e); return hipSuccess; }
hipError_t hipEventRecord(hipEvent_t e, hipStream_t s)
{
    (void)s;
    if (fail_record) return done(hipErrorInvalidHandle);
    *(double *)e = clock_ms;
    return hipSuccess;
}
hipError_t hipEventSynchronize(hipEvent_t e) { (void)e; arrive(); return hipSuccess; }
hipError_t hipEventElapsedTime(float *ms, hipEvent_t a, hipEvent_t b) { *ms = (float)(*(double *)b - *(double *)a); return hipSuccess; }
