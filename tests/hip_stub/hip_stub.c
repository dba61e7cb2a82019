/* A HIP runtime for host-side tests: device memory is host memory, copies are made at once, kernels are recorded instead of
 * run, and a chosen call fails.  What is put on a stream, and what the host waits for, is kept in the order of the calls.  Loaded (with global symbols) before libdeer.so in a process without a GPU. */
#include <stdint.h>
#include <stdlib.h>
#include <string.h>

typedef struct { uint32_t x, y, z; } dim3_t;
typedef struct { char name[256]; const void *fn; } fn_t;
enum { ARG_BYTES = 120 };   /* of a GEMM's arguments: up to the K shares and the row count (see host_engine.GemmArgs) */
typedef struct { char name[256]; uint32_t grid[3], block[3]; char arg[ARG_BYTES]; } launch_t;
enum { OP_LAUNCH, OP_COPY, OP_SYNC, OP_RECORD, OP_WAIT, OP_STREAM_CREATE, OP_EVENT_CREATE, OP_KINDS };
typedef struct { int kind; void *stream, *what; } op_t;   /* what: the event, or a pass's residual rows (see hipLaunchKernel) */

static fn_t fns[1024];
static int n_fns;
static launch_t launches[1 << 16];
static int n_launches, n_syncs, n_copies, launches_left = -1, copies_left = -1, syncs_left = -1, last_error;
static op_t ops[1 << 17];
static int n_ops, op_left[OP_KINDS] = {-1, -1, -1, -1, -1, -1, -1};
static dim3_t cfg_grid, cfg_block;
static void *cfg_stream;
static char symbol[1 << 20];

int stub_launches(void) { return n_launches; }
const char *stub_launch(int i, uint32_t *grid) { memcpy(grid, launches[i].grid, 12); return launches[i].name; }
const char *stub_launch_arg(int i) { return launches[i].arg; }
int stub_syncs(void) { return n_syncs; }
int stub_copies(void) { return n_copies; }
void stub_reset(void) {
    n_launches = n_syncs = n_copies = n_ops = 0; launches_left = copies_left = syncs_left = -1; last_error = 0;
    for (int i = 0; i < OP_KINDS; ++i) op_left[i] = -1;
}
int stub_ops(void) { return n_ops; }
int stub_op(int i, void **stream, void **what) { *stream = ops[i].stream; *what = ops[i].what; return ops[i].kind; }
/* the call after the next n of this kind fails; -1: none (launches, copies and waits of the host: stub_fail) */
void stub_fail_op(int kind, int n) { op_left[kind] = n; }
/* the call after the next n of its kind fails; -1: none */
void stub_fail(int launch, int copy, int sync) { launches_left = launch; copies_left = copy; syncs_left = sync; }

static int due(int *left) { return *left >= 0 && (*left)-- == 0; }
static void op(int kind, void *stream, void *what) {
    if (n_ops == 1 << 17) abort();
    ops[n_ops].kind = kind; ops[n_ops].stream = stream; ops[n_ops++].what = what;
}

static int fatbin;
static void *fatbin_handle = &fatbin;
void **__hipRegisterFatBinary(const void *data) { (void)data; return &fatbin_handle; }
void __hipUnregisterFatBinary(void **m) { (void)m; }
void __hipRegisterFunction(void **m, const void *host, char *dev, const char *name, unsigned lim, void *t, void *b, void *bd, void *gd, int *w) {
    (void)m; (void)dev; (void)lim; (void)t; (void)b; (void)bd; (void)gd; (void)w;
    if (n_fns < 1024) { strncpy(fns[n_fns].name, name, 255); fns[n_fns++].fn = host; }
}
void __hipRegisterVar(void **m, void *v, char *h, char *d, int e, size_t s, int c, int g) { (void)m; (void)v; (void)h; (void)d; (void)e; (void)s; (void)c; (void)g; }
int __hipPushCallConfiguration(dim3_t grid, dim3_t block, size_t shmem, void *stream) { (void)shmem; cfg_grid = grid; cfg_block = block; cfg_stream = stream; return 0; }
int __hipPopCallConfiguration(dim3_t *grid, dim3_t *block, size_t *shmem, void **stream) { *grid = cfg_grid; *block = cfg_block; *shmem = 0; *stream = cfg_stream; return 0; }

int hipLaunchKernel(const void *fn, dim3_t grid, dim3_t block, void **args, size_t shmem, void *stream) {
    (void)shmem;
    if (due(&launches_left)) return last_error = 719;
    if (n_launches == 1 << 16) abort();
    launch_t *l = &launches[n_launches++];
    l->name[0] = 0;
    for (int i = 0; i < n_fns; ++i) if (fns[i].fn == fn) strcpy(l->name, fns[i].name);
    memcpy(l->grid, &grid, 12); memcpy(l->block, &block, 12);
    if (strstr(l->name, "8GemmArgs")) memcpy(l->arg, args[0], ARG_BYTES); else memset(l->arg, 0, ARG_BYTES);
    op(OP_LAUNCH, stream, strstr(l->name, "k_pass_begin") ? *(void **)args[3] : 0);   /* its fourth argument: the pass's residual rows */
    return 0;
}
int hipGetLastError(void) { int e = last_error; last_error = 0; return e; }
const char *hipGetErrorString(int e) { return e ? "planned failure" : "no error"; }
int hipSetDevice(int d) { (void)d; return 0; }
int hipGetSymbolAddress(void **p, const void *s) { (void)s; *p = symbol; return 0; }
int hipMemset(void *p, int v, size_t n) { memset(p, v, n); return 0; }
int hipMemsetAsync(void *p, int v, size_t n, void *s) { (void)s; memset(p, v, n); return 0; }
int hipMemcpy(void *d, const void *s, size_t n, int k) { (void)k; memcpy(d, s, n); return 0; }
int hipMemcpyAsync(void *d, const void *s, size_t n, int k, void *st) {
    (void)k;
    ++n_copies;
    if (due(&copies_left)) return 719;
    op(OP_COPY, st, d);
    memcpy(d, s, n);
    return 0;
}
int hipStreamSynchronize(void *s) { op(OP_SYNC, s, 0); ++n_syncs; return due(&syncs_left) ? 719 : 0; }
int hipHostMalloc(void **p, size_t n, unsigned f) { (void)f; *p = calloc(1, n); return *p ? 0 : 2; }
int hipHostFree(void *p) { free(p); return 0; }
int hipHostGetDevicePointer(void **d, void *h, unsigned f) { (void)f; *d = h; return 0; }
int hipEventCreate(void **e) { *e = calloc(1, 8); return 0; }
int hipEventDestroy(void *e) { free(e); return 0; }
int hipEventRecord(void *e, void *s) { if (due(&op_left[OP_RECORD])) return 719; op(OP_RECORD, s, e); return 0; }
int hipEventSynchronize(void *e) { (void)e; return 0; }
int hipEventElapsedTime(float *ms, void *a, void *b) { (void)a; (void)b; *ms = 1.f; return 0; }
int hipStreamCreateWithFlags(void **s, unsigned f) { (void)f; if (due(&op_left[OP_STREAM_CREATE])) return 719; *s = calloc(1, 8); return 0; }
int hipStreamDestroy(void *s) { free(s); return 0; }
int hipStreamWaitEvent(void *s, void *e, unsigned f) { (void)f; if (due(&op_left[OP_WAIT])) return 719; op(OP_WAIT, s, e); return 0; }
int hipEventCreateWithFlags(void **e, unsigned f) { (void)f; if (due(&op_left[OP_EVENT_CREATE])) return 719; *e = calloc(1, 8); return 0; }
