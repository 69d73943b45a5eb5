/* Stands in for the HIP runtime under libpf.so on a host without a GPU: notes
 * which kernels the library launches, with what shape, and which attributes it
 * sets on which device.  Loaded before the library with RTLD_GLOBAL, so that its
 * definitions are found first; no kernel runs. */
#define __HIP_PLATFORM_AMD__ 1
#include <hip/hip_runtime_api.h>
#include <pthread.h>
#include <stdio.h>
#include <string.h>
#include <unistd.h>

static int device;
static char text[1 << 16];
static size_t used;
static struct { const void *fn; const char *name; } kernels[512];
static int nkernels;
static __thread dim3 cfg_grid, cfg_block;
static __thread size_t cfg_lds;
static __thread hipStream_t cfg_stream;

void rec_set_device(int d) { device = d; }
void rec_clear(void) { used = 0; text[0] = 0; }
const char *rec_text(void) { return text; }

static const char *name_of(const void *fn) {
    for (int k = 0; k < nkernels; ++k)
        if (kernels[k].fn == fn) return kernels[k].name;
    return "?";
}
static pthread_mutex_t lock = PTHREAD_MUTEX_INITIALIZER;
static void note(const char *what, const void *fn, unsigned a, unsigned b, size_t c) {
    pthread_mutex_lock(&lock);
    used += (size_t)snprintf(text + used, sizeof(text) - used, "%s %d %s %u %u %zu\n", what, device, name_of(fn), a, b, c);
    pthread_mutex_unlock(&lock);
}

void **__hipRegisterFatBinary(const void *data) { static void *module; (void)data; return &module; }
void __hipUnregisterFatBinary(void **module) { (void)module; }
void __hipRegisterFunction(void **module, const void *fn, char *dev, const char *name, unsigned limit, void *tid,
                           void *bid, dim3 *block, dim3 *grid, int *wsize) {
    (void)module; (void)dev; (void)limit; (void)tid; (void)bid; (void)block; (void)grid; (void)wsize;
    kernels[nkernels].fn = fn;
    kernels[nkernels++].name = name;
}
void __hipRegisterVar(void **module, void *var, char *host, char *dev, int ext, size_t size, int constant, int global) {
    (void)module; (void)var; (void)host; (void)dev; (void)ext; (void)size; (void)constant; (void)global;
}
hipError_t __hipPushCallConfiguration(dim3 grid, dim3 block, size_t lds, hipStream_t st) {
    cfg_grid = grid; cfg_block = block; cfg_lds = lds; cfg_stream = st;
    return hipSuccess;
}
hipError_t __hipPopCallConfiguration(dim3 *grid, dim3 *block, size_t *lds, hipStream_t *st) {
    *grid = cfg_grid; *block = cfg_block; *lds = cfg_lds; *st = cfg_stream;
    return hipSuccess;
}
hipError_t hipLaunchKernel(const void *fn, dim3 grid, dim3 block, void **args, size_t lds, hipStream_t st) {
    (void)args; (void)st;
    note("launch", fn, grid.x, block.x, lds);
    return hipSuccess;
}
hipError_t hipLaunchCooperativeKernel(const void *fn, dim3 grid, dim3 block, void **args, unsigned lds, hipStream_t st) {
    (void)args; (void)st;
    note("cooperative", fn, grid.x, block.x, lds);
    return hipSuccess;
}
hipError_t hipFuncSetAttribute(const void *fn, hipFuncAttribute attr, int value) {
    note("attribute", fn, (unsigned)attr, 0, (size_t)value);
    return hipSuccess;
}
hipError_t hipFuncGetAttributes(struct hipFuncAttributes *attr, const void *fn) {
    (void)fn;
    usleep(200000);  /* long enough for another thread to come by */
    memset(attr, 0, sizeof(*attr));
    attr->sharedSizeBytes = 60000;
    return hipSuccess;
}
hipError_t hipOccupancyMaxActiveBlocksPerMultiprocessor(int *n, const void *fn, int threads, size_t lds) {
    (void)fn; (void)lds;
    *n = 2048 / threads;
    return hipSuccess;
}
hipError_t hipDeviceGetAttribute(int *value, hipDeviceAttribute_t attr, int dev) {
    *value = attr == hipDeviceAttributeMultiprocessorCount                  ? 256 >> dev
             : attr == hipDeviceAttributeMaxSharedMemoryPerMultiprocessor ? 160 << 10
                                                                          : 100000;
    return hipSuccess;
}
hipError_t hipGetDevice(int *d) { *d = device; return hipSuccess; }
hipError_t hipGetLastError(void) { return hipSuccess; }
hipError_t hipMemcpyAsync(void *dst, const void *src, size_t n, hipMemcpyKind kind, hipStream_t st) {
    (void)dst; (void)src; (void)n; (void)kind; (void)st;
    return hipSuccess;
}
hipError_t hipGetSymbolAddress(void **p, const void *symbol) {
    (void)symbol;
    *p = (void *)(uintptr_t)(0x100000000ull * (unsigned)(device + 1));
    return hipSuccess;
}
