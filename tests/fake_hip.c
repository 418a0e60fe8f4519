/* The HIP runtime calls of liblbm.so, on the host and without a GPU: device
 * memory is host memory, a launch is recorded and not run.  For tests of the
 * library's host side: which kernels a call launches, what it does when a
 * launch fails, how much device memory it holds.
 *
 * Loaded before the library with its symbols global, these definitions take
 * the place of the runtime's. */
#define _GNU_SOURCE
#include <stddef.h>
#include <stdint.h>
#include <stdlib.h>
#include <string.h>
#include <sys/mman.h>

typedef struct { uint32_t x, y, z; } Dim3;
enum { kOk = 0, kOutOfMemory = 2, kNotSupported = 801 };

/* kernels by their host stub */
static struct { const void *stub; const char *name; } kernels[4096];
static int n_kernels;
void **__hipRegisterFatBinary(const void *data) { static void *h; (void)data; return &h; }
void __hipRegisterFunction(void **m, const void *stub, char *dev, const char *name, int threads,
                           void *tid, void *bid, Dim3 *bd, Dim3 *gd, int *ws) {
    (void)m; (void)dev; (void)threads; (void)tid; (void)bid; (void)bd; (void)gd; (void)ws;
    if (n_kernels < 4096) {
        kernels[n_kernels].stub = stub;
        kernels[n_kernels++].name = strdup(name);
    }
}
void __hipRegisterVar(void) {}
void __hipUnregisterFatBinary(void **m) { (void)m; }
int __hipPopCallConfiguration(void) { return kNotSupported; }

/* launches */
static struct Launch { const char *name; uint32_t grid, block; int ticks; } launches[65536];
static int n_launches, fail_at = -1;
void fake_reset(int fail) { n_launches = 0; fail_at = fail; }
int fake_launches(void) { return n_launches; }
const struct Launch *fake_launch(int i) { return &launches[i]; }
int hipLaunchKernel(const void *f, Dim3 grid, Dim3 block, void **args, size_t lds, void *stream) {
    (void)lds; (void)stream;
    if (n_launches == fail_at) return kOutOfMemory;
    if (n_launches == 65536) return kOutOfMemory;
    struct Launch *l = &launches[n_launches++];
    memset(l, 0, sizeof *l);
    l->name = "?";
    for (int k = 0; k < n_kernels; ++k)
        if (kernels[k].stub == f) l->name = kernels[k].name;
    l->grid = grid.x;
    l->block = block.x;
    if (strstr(l->name, "k_advance")) l->ticks = *(int *)args[3];
    return kOk;
}

/* memory (pages untouched until written) */
static struct { void *p; size_t n; } blocks[4096];
static size_t live;
size_t fake_live_bytes(void) { return live; }
static int get(void **p, size_t n) {
    void *q = mmap(NULL, n, PROT_READ | PROT_WRITE, MAP_PRIVATE | MAP_ANONYMOUS | MAP_NORESERVE,
                   -1, 0);
    if (q == MAP_FAILED) return kOutOfMemory;
    for (int k = 0; k < 4096; ++k)
        if (!blocks[k].p) {
            blocks[k].p = q;
            blocks[k].n = n;
            live += n;
            *p = q;
            return kOk;
        }
    munmap(q, n);
    return kOutOfMemory;
}
static int put(void *p) {
    for (int k = 0; p && k < 4096; ++k)
        if (blocks[k].p == p) {
            munmap(p, blocks[k].n);
            live -= blocks[k].n;
            blocks[k].p = NULL;
        }
    return kOk;
}
int hipMalloc(void **p, size_t n) { return get(p, n); }
int hipFree(void *p) { return put(p); }
int hipHostMalloc(void **p, size_t n, unsigned flags) { (void)flags; *p = calloc(1, n); return *p ? kOk : kOutOfMemory; }
int hipHostFree(void *p) { free(p); return kOk; }
int hipMemcpyAsync(void *d, const void *s, size_t n, int kind, void *stream) {
    (void)kind; (void)stream;
    memcpy(d, s, n);
    return kOk;
}

/* the rest: a device, streams and events that are always done, no graphs */
int hipGetDevice(int *d) { *d = 0; return kOk; }
int hipSetDevice(int d) { (void)d; return kOk; }
int hipGetLastError(void) { return kOk; }
int hipGetSymbolAddress(void **p, const void *s) { (void)p; (void)s; return kNotSupported; }
static int handle;
int hipStreamCreateWithFlags(void **s, unsigned f) { (void)f; *s = &handle; return kOk; }
int hipStreamDestroy(void *s) { (void)s; return kOk; }
int hipStreamSynchronize(void *s) { (void)s; return kOk; }
int hipEventCreateWithFlags(void **e, unsigned f) { (void)f; *e = &handle; return kOk; }
int hipEventDestroy(void *e) { (void)e; return kOk; }
int hipEventRecord(void *e, void *s) { (void)e; (void)s; return kOk; }
int hipEventSynchronize(void *e) { (void)e; return kOk; }
int hipStreamBeginCapture(void *s, int mode) { (void)s; (void)mode; return kNotSupported; }
int hipStreamEndCapture(void *s, void **g) { (void)s; *g = NULL; return kNotSupported; }
int hipGraphDestroy(void *g) { (void)g; return kOk; }
int hipGraphExecDestroy(void *g) { (void)g; return kOk; }
int hipGraphInstantiate(void) { return kNotSupported; }
int hipGraphLaunch(void *g, void *s) { (void)g; (void)s; return kNotSupported; }
int hipGraphGetNodes(void) { return kNotSupported; }
int hipGraphNodeGetType(void) { return kNotSupported; }
int hipGraphKernelNodeGetParams(void) { return kNotSupported; }
int hipGraphExecKernelNodeSetParams(void) { return kNotSupported; }
