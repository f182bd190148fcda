/* A HIP runtime that runs nothing, for tests of the library's host code on a
 * machine without a GPU: device memory is host memory, launches are written to
 * a log instead of being run, and one of them can be made to fail.  Loaded
 * with RTLD_GLOBAL before libramppi.so, whose calls it then receives. */
#include <stddef.h>
#include <stdint.h>
#include <stdlib.h>
#include <string.h>

typedef struct {
    uint32_t x, y, z;
} dim3_t;
typedef struct {
    char name[96]; /* mangled kernel name */
    uint32_t grid, block;
    uint64_t lds;
} launch_t;

enum { kMaxLaunches = 256, kMaxKernels = 128 };
static launch_t log_[kMaxLaunches];
static int n_log, fail_at = -1, last_error, resident = 4;
static struct {
    const void* host;
    const char* name;
} kernels[kMaxKernels];
static int n_kernels;
static struct {
    dim3_t grid, block;
    size_t lds;
    void* stream;
} config;

/* the tests' side */
void fake_reset(int fail) { n_log = 0, last_error = 0, fail_at = fail; }
void fake_resident(int per_cu) { resident = per_cu; } /* workgroups of 256 threads a unit holds */
int fake_launches(void) { return n_log; }
const launch_t* fake_launch(int i) { return &log_[i]; }

/* the library's side */
void** __hipRegisterFatBinary(const void* data) { return (void**)&config + 0 * (data != NULL); }
void __hipUnregisterFatBinary(void** m) { (void)m; }
void __hipRegisterFunction(void** m, const void* host, char* dev, const char* name, unsigned limit, void* a, void* b,
                           void* c, void* d, int* w) {
    (void)m, (void)dev, (void)limit, (void)a, (void)b, (void)c, (void)d, (void)w;
    if (n_kernels < kMaxKernels) kernels[n_kernels].host = host, kernels[n_kernels++].name = name;
}
static void* symbol;
void __hipRegisterVar(void** m, void* host, char* dev, const char* name, int ext, size_t size, int con, int global) {
    (void)m, (void)host, (void)dev, (void)name, (void)ext, (void)con, (void)global;
    symbol = calloc(size, 1);
}
int hipGetSymbolAddress(void** out, const void* sym) { return (void)sym, *out = symbol, 0; }

int __hipPushCallConfiguration(dim3_t grid, dim3_t block, size_t lds, void* stream) {
    config.grid = grid, config.block = block, config.lds = lds, config.stream = stream;
    return 0;
}
int __hipPopCallConfiguration(dim3_t* grid, dim3_t* block, size_t* lds, void** stream) {
    *grid = config.grid, *block = config.block, *lds = config.lds, *stream = config.stream;
    return 0;
}
int hipLaunchKernel(const void* host, dim3_t grid, dim3_t block, void** args, size_t lds, void* stream) {
    (void)args, (void)stream;
    const int i = n_log < kMaxLaunches ? n_log++ : kMaxLaunches - 1;
    log_[i].name[0] = 0;
    for (int k = 0; k < n_kernels; ++k)
        if (kernels[k].host == host) strncpy(log_[i].name, kernels[k].name, sizeof log_[i].name - 1);
    log_[i].grid = grid.x, log_[i].block = block.x, log_[i].lds = lds;
    if (i == fail_at) return last_error = 1; /* hipErrorInvalidValue */
    return 0;
}
int hipGetLastError(void) {
    const int e = last_error;
    last_error = 0;
    return e;
}
const char* hipGetErrorString(int e) { return e ? "an error" : "no error"; }

int hipGetDeviceCount(int* n) { return *n = 1, 0; }
int hipGetDevice(int* d) { return *d = 0, 0; }
int hipDeviceGetAttribute(int* v, int attr, int dev) { return (void)attr, (void)dev, *v = 256, 0; }
int hipOccupancyMaxActiveBlocksPerMultiprocessor(int* n, const void* f, int block, size_t lds) {
    return (void)f, (void)lds, *n = resident * 256 / block, 0; /* by waves, as HIP answers */
}
int hipHostMalloc(void** p, size_t n, unsigned flags) { return (void)flags, *p = calloc(n, 1), 0; }
int hipHostFree(void* p) { return free(p), 0; }
int hipHostGetDevicePointer(void** d, void* h, unsigned flags) { return (void)flags, *d = h, 0; }
int hipMemcpyAsync(void* d, const void* s, size_t n, int kind, void* stream) {
    return (void)kind, (void)stream, memcpy(d, s, n), 0;
}
int hipMemsetAsync(void* d, int v, size_t n, void* stream) { return (void)stream, memset(d, v, n), 0; }
int hipStreamSynchronize(void* s) { return (void)s, 0; }
int hipStreamQuery(void* s) { return (void)s, 0; }
int hipStreamCreateWithFlags(void** s, unsigned f) { return (void)f, *s = &config, 0; }
int hipStreamDestroy(void* s) { return (void)s, 0; }
int hipEventCreate(void** e) { return *e = &config, 0; }
int hipEventCreateWithFlags(void** e, unsigned f) { return (void)f, *e = &config, 0; }
int hipEventDestroy(void* e) { return (void)e, 0; }
int hipEventRecord(void* e, void* s) { return (void)e, (void)s, 0; }
int hipEventSynchronize(void* e) { return (void)e, 0; }
int hipEventElapsedTime(float* ms, void* a, void* b) { return (void)a, (void)b, *ms = 0.0f, 0; }
int hipStreamBeginCapture(void* s, int mode) { return (void)s, (void)mode, 0; }
int hipStreamEndCapture(void* s, void** g) { return (void)s, *g = &config, 0; }
int hipGraphInstantiate(void** x, void* g, void* n, char* log, size_t size) {
    return (void)g, (void)n, (void)log, (void)size, *x = &config, 0;
}
int hipGraphLaunch(void* x, void* s) { return (void)x, (void)s, 0; }
int hipGraphDestroy(void* g) { return (void)g, 0; }
int hipGraphExecDestroy(void* x) { return (void)x, 0; }
