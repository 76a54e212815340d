/* A HIP runtime without a GPU, for tests of the library's host code: device addresses are made up, kernels are recorded
 * and not run, allocations can be made to fail.  Loaded with RTLD_GLOBAL before libfastsnarf.so, whose calls then end
 * here (tests/host_path.py). */
#include <hip/hip_runtime_api.h>
#include <stdio.h>
#include <stdlib.h>
#include <string.h>

#define MAX_NAMES 256
#define MAX_LAUNCHES 4096
#define MAX_BLOCKS 4096

static struct { const void *host; const char *name; } names[MAX_NAMES];
static int n_names;
static struct { const char *name; unsigned grid[3], block[3]; size_t shared; char solve[64]; } launches[MAX_LAUNCHES];
static int n_launches;
static struct { char *at; size_t bytes; } blocks[MAX_BLOCKS];
static int n_blocks, bad_frees, fail_in = -1, fail_launch_in = -1, memsets, n_cus = 256, occupancy = 3;
static hipError_t last_error = hipSuccess;
static char *next_address = (char *)0x100000000000ull;
static struct { dim3 grid, block; size_t shared; hipStream_t stream; } config;

/* ---- what the tests call ---- */
void stub_fail_allocation(int n) { fail_in = n; }      /* the n-th allocation from now fails (0: the next one; < 0: none) */
void stub_fail_launch(int n) { fail_launch_in = n; }   /* the n-th launch from now fails */
int stub_memsets(void) { return memsets; }             /* calls of hipMemset so far */
int stub_live_blocks(void) { return n_blocks; }
int stub_bad_frees(void) { return bad_frees; }
void stub_clear_launches(void) { n_launches = 0; }
int stub_launches(void) { return n_launches; }
const char *stub_launch(int i, unsigned *shape)        /* shape: grid x, y, z, block x, y, z, bytes of dynamic LDS */
{
    memcpy(shape, launches[i].grid, 12);
    memcpy(shape + 3, launches[i].block, 12);
    shape[6] = (unsigned)launches[i].shared;
    return launches[i].name;
}

const void *stub_solve_params(int i) { return launches[i].solve; }      /* the SolveP (64 bytes) that a solve kernel was given */

/* ---- the runtime ---- */
hipError_t hipMalloc(void **p, size_t n)
{
    *p = NULL;
    if (fail_in >= 0 && fail_in-- == 0) return hipErrorOutOfMemory;
    if (n_blocks == MAX_BLOCKS) abort();
    blocks[n_blocks].at = next_address;
    blocks[n_blocks++].bytes = n;
    *p = next_address;
    next_address += (n + 511) / 256 * 256;
    return hipSuccess;
}
hipError_t hipFree(void *p)
{
    int i;
    if (!p) return hipSuccess;
    for (i = 0; i < n_blocks; ++i)
        if (blocks[i].at == (char *)p) {
            blocks[i] = blocks[--n_blocks];
            return hipSuccess;
        }
    ++bad_frees;
    return hipErrorInvalidValue;
}
hipError_t hipHostMalloc(void **p, size_t n, unsigned flags) { (void)flags; return (*p = calloc(1, n)) ? hipSuccess : hipErrorOutOfMemory; }
hipError_t hipHostFree(void *p) { free(p); return hipSuccess; }
hipError_t hipHostGetDevicePointer(void **d, void *p, unsigned flags) { (void)flags; *d = p; return hipSuccess; }
hipError_t hipMemset(void *p, int v, size_t n) { (void)p; (void)v; (void)n; ++memsets; return hipSuccess; }
hipError_t hipMemcpyAsync(void *d, const void *s, size_t n, hipMemcpyKind k, hipStream_t st) { (void)d; (void)s; (void)n; (void)k; (void)st; return hipSuccess; }
hipError_t hipGetDevice(int *d) { *d = 0; return hipSuccess; }
hipError_t hipGetLastError(void) { hipError_t e = last_error; last_error = hipSuccess; return e; }
const char *hipGetErrorString(hipError_t e) { (void)e; return "stub"; }
hipError_t hipStreamSynchronize(hipStream_t s) { (void)s; return hipSuccess; }
hipError_t hipDeviceSynchronize(void) { return hipSuccess; }
hipError_t hipDeviceGetAttribute(int *v, hipDeviceAttribute_t a, int d) { (void)a; (void)d; *v = n_cus; return hipSuccess; }
hipError_t hipFuncSetAttribute(const void *f, hipFuncAttribute a, int v) { (void)f; (void)a; (void)v; return hipSuccess; }
hipError_t hipOccupancyMaxActiveBlocksPerMultiprocessor(int *n, const void *f, int b, size_t s) { (void)f; (void)b; (void)s; *n = occupancy; return hipSuccess; }
hipError_t hipGetSymbolAddress(void **p, const void *s) { (void)s; *p = (void *)0x200000000000ull; return hipSuccess; }
hipError_t hipPointerGetAttributes(hipPointerAttribute_t *a, const void *p)
{
    (void)p;
    memset(a, 0, sizeof *a);
    a->type = hipMemoryTypeDevice;
    return hipSuccess;
}
hipError_t hipEventCreate(hipEvent_t *e) { *e = NULL; return hipSuccess; }
hipError_t hipEventDestroy(hipEvent_t e) { (void)e; return hipSuccess; }
hipError_t hipEventRecord(hipEvent_t e, hipStream_t s) { (void)e; (void)s; return hipSuccess; }
hipError_t hipEventSynchronize(hipEvent_t e) { (void)e; return hipSuccess; }
hipError_t hipEventElapsedTime(float *ms, hipEvent_t a, hipEvent_t b) { (void)a; (void)b; *ms = 0.0f; return hipSuccess; }

void **__hipRegisterFatBinary(const void *data) { static void *module; (void)data; return &module; }
void __hipUnregisterFatBinary(void **m) { (void)m; }
void __hipRegisterVar(void **m, void *v, char *h, char *n, int e, size_t s, int c, int g)
{
    (void)m; (void)v; (void)h; (void)n; (void)e; (void)s; (void)c; (void)g;
}
void __hipRegisterFunction(void **m, const void *host, char *dev, const char *name, unsigned limit, void *t, void *b, void *bd, void *gd, int *ws)
{
    (void)m; (void)dev; (void)limit; (void)t; (void)b; (void)bd; (void)gd; (void)ws;
    if (n_names == MAX_NAMES) abort();
    names[n_names].host = host;
    names[n_names++].name = name;
}
hipError_t __hipPushCallConfiguration(dim3 grid, dim3 block, size_t shared, hipStream_t stream)
{
    config.grid = grid;
    config.block = block;
    config.shared = shared;
    config.stream = stream;
    return hipSuccess;
}
hipError_t __hipPopCallConfiguration(dim3 *grid, dim3 *block, size_t *shared, hipStream_t *stream)
{
    *grid = config.grid;
    *block = config.block;
    *shared = config.shared;
    *stream = config.stream;
    return hipSuccess;
}
hipError_t hipLaunchKernel(const void *f, dim3 grid, dim3 block, void **args, size_t shared, hipStream_t stream)
{
    int i;
    (void)stream;
    if (fail_launch_in >= 0 && fail_launch_in-- == 0) return last_error = hipErrorLaunchFailure;
    if (n_launches == MAX_LAUNCHES) abort();
    launches[n_launches].name = "?";
    for (i = 0; i < n_names; ++i)
        if (names[i].host == f) launches[n_launches].name = names[i].name;
    memset(launches[n_launches].solve, 0, 64);
    if (strstr(launches[n_launches].name, "k_solve_ws") || strstr(launches[n_launches].name, "k_solveI")) memcpy(launches[n_launches].solve, args[1], 64);
    launches[n_launches].grid[0] = grid.x; launches[n_launches].grid[1] = grid.y; launches[n_launches].grid[2] = grid.z;
    launches[n_launches].block[0] = block.x; launches[n_launches].block[1] = block.y; launches[n_launches].block[2] = block.z;
    launches[n_launches++].shared = shared;
    return hipSuccess;
}
