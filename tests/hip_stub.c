/* A HIP runtime for tests of the library's host side without a GPU: device
 * memory is host memory, copies are memcpy, kernels do not run.  Launches,
 * waits, attribute settings, allocations and copies to the host are logged in
 * order with their stream (device, bytes); one launch can be made to fail, and
 * the byte that new memory holds can be set. */
#include <stdlib.h>
#include <string.h>

typedef struct { unsigned x, y, z; } dim3;
typedef void *stream_t;
enum { LAUNCH = 1, SYNC = 2, ATTR = 3, ALLOC = 4, READ = 5 };
enum { SUCCESS = 0, FAILED = 719 };

static struct { int op; const void *what, *where; } entries[1 << 20];
static int n_log, device, error, fail_at = -1, n_launch, fill;
static struct { dim3 grid, block; size_t lds; stream_t stream; } call;

static void put(int op, const void *what, const void *where)
{
    if (n_log < (1 << 20)) {
        entries[n_log].op = op;
        entries[n_log].what = what;
        entries[n_log++].where = where;
    }
}

/* control by the tests */
void stub_reset(int fail) { n_log = n_launch = error = 0; fail_at = fail; }
void stub_device(int d) { device = d; }
void stub_fill(int byte) { fill = byte; }
int stub_size(void) { return n_log; }
int stub_op(int i) { return entries[i].op; }
const void *stub_what(int i) { return entries[i].what; }
const void *stub_where(int i) { return entries[i].where; }

int __hipPushCallConfiguration(dim3 g, dim3 b, size_t lds, stream_t s)
{
    call.grid = g;
    call.block = b;
    call.lds = lds;
    call.stream = s;
    return SUCCESS;
}
int __hipPopCallConfiguration(dim3 *g, dim3 *b, size_t *lds, stream_t *s)
{
    *g = call.grid;
    *b = call.block;
    *lds = call.lds;
    *s = call.stream;
    return SUCCESS;
}
int hipLaunchKernel(const void *f, dim3 g, dim3 b, void **args, size_t lds, stream_t s)
{
    (void)g, (void)b, (void)args, (void)lds;
    if (n_launch++ == fail_at) return error = FAILED;
    put(LAUNCH, f, s);
    return SUCCESS;
}
int hipGetLastError(void)
{
    int e = error;
    error = SUCCESS;
    return e;
}
static void *handle;
void **__hipRegisterFatBinary(const void *d) { (void)d; return &handle; }
void __hipUnregisterFatBinary(void **m) { (void)m; }
void __hipRegisterFunction(void **m, const void *f, char *a, const char *b, unsigned c, void *d, void *e, void *g, void *h, int *i)
{
    (void)m, (void)f, (void)a, (void)b, (void)c, (void)d, (void)e, (void)g, (void)h, (void)i;
}
void __hipRegisterVar(void **m, void *v, char *a, char *b, int c, size_t d, int e, int f)
{
    (void)m, (void)v, (void)a, (void)b, (void)c, (void)d, (void)e, (void)f;
}
const char *hipGetErrorString(int e) { return e ? "failed" : "success"; }
int hipGetDevice(int *d) { *d = device; return SUCCESS; }
int hipDeviceGetAttribute(int *v, int what, int d) { (void)what, (void)d; *v = 256; return SUCCESS; }
int hipFuncSetAttribute(const void *f, int what, int v) { (void)what, (void)v; put(ATTR, f, (void *)(size_t)device); return SUCCESS; }
int hipFuncGetAttributes(void *a, const void *f) { (void)a, (void)f; return FAILED; }
int hipOccupancyMaxActiveBlocksPerMultiprocessor(int *n, const void *f, int b, size_t l) { (void)f, (void)b, (void)l; *n = 1; return SUCCESS; }
int hipGetSymbolAddress(void **p, const void *s) { (void)s; *p = 0; return FAILED; }
int hipMalloc(void **p, size_t n) { put(ALLOC, (void *)n, 0); *p = malloc(n); if (*p) memset(*p, fill, n); return *p ? SUCCESS : 2; }
int hipFree(void *p) { free(p); return SUCCESS; }
int hipHostMalloc(void **p, size_t n, unsigned f) { (void)f; return hipMalloc(p, n); }
int hipHostFree(void *p) { free(p); return SUCCESS; }
int hipMemcpy(void *d, const void *s, size_t n, int k) { (void)k; memmove(d, s, n); return SUCCESS; }
int hipMemcpyAsync(void *d, const void *s, size_t n, int k, stream_t st) { if (k == 2) put(READ, (void *)n, st); memmove(d, s, n); return SUCCESS; }
int hipMemset(void *d, int v, size_t n) { memset(d, v, n); return SUCCESS; }
int hipStreamCreateWithFlags(stream_t *s, unsigned f) { (void)f; *s = malloc(1); return SUCCESS; }
int hipStreamDestroy(stream_t s) { free(s); return SUCCESS; }
int hipStreamSynchronize(stream_t s) { put(SYNC, 0, s); return SUCCESS; }
int hipDeviceSynchronize(void) { put(SYNC, 0, (void *)-1); return SUCCESS; }
int hipStreamWaitEvent(stream_t s, void *e, unsigned f) { (void)s, (void)e, (void)f; return SUCCESS; }
int hipStreamBeginCapture(stream_t s, int m) { (void)s, (void)m; return FAILED; }
int hipStreamEndCapture(stream_t s, void **g) { (void)s; *g = 0; return FAILED; }
int hipGraphInstantiate(void **e, void *g, void **n, char *l, size_t z) { (void)e, (void)g, (void)n, (void)l, (void)z; return FAILED; }
int hipGraphLaunch(void *e, stream_t s) { (void)e, (void)s; return FAILED; }
int hipGraphDestroy(void *g) { (void)g; return SUCCESS; }
int hipGraphExecDestroy(void *g) { (void)g; return SUCCESS; }
int hipEventCreate(void **e) { *e = malloc(1); return SUCCESS; }
int hipEventDestroy(void *e) { free(e); return SUCCESS; }
int hipEventRecord(void *e, stream_t s) { (void)e, (void)s; return SUCCESS; }
int hipEventQuery(void *e) { (void)e; return SUCCESS; }
int hipEventSynchronize(void *e) { (void)e; return SUCCESS; }
int hipEventElapsedTime(float *ms, void *a, void *b) { (void)a, (void)b; *ms = 1.0f; return SUCCESS; }
