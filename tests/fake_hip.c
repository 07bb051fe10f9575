/* A HIP runtime without a GPU, for tests of libps.so's host code: memory is
 * host memory that no kernel touches, a launch is recorded and refused where
 * the real runtime refuses it, events read a simulated clock, and stream
 * capture can be told to fail.  Loaded before libps.so with global symbols, in
 * a process of its own (tests/fake_hip.py). */
#include <stdint.h>
#include <stdlib.h>
#include <string.h>

typedef struct { uint32_t x, y, z; } D3;
typedef struct { const void* func; uint64_t blocks, threads, stream; int captured; } Launch;

enum { OK = 0, INVALID = 1, OUT_OF_MEMORY = 2, INVALID_CONFIG = 9, MAX_LAUNCHES = 1 << 20 };

static Launch launches[MAX_LAUNCHES];
static long nlaunch, nreplay, ninst, fail_begin, fail_end, fail_inst, fail_launch = -1;
static int capturing;
static uint64_t next_handle = 16;
static double now_ms, limit_threads = 1e30, slow = 1, overhead_ms;
static int last_error;
static D3 cfg_grid, cfg_block;
static size_t cfg_shmem;
static void* cfg_stream;

/* ---- control */
void fake_reset(void) { nlaunch = nreplay = ninst = 0; fail_begin = fail_end = fail_inst = 0; fail_launch = -1; last_error = 0; }
long fake_launches(Launch** out) { *out = launches; return nlaunch; }
long fake_replays(void) { return nreplay; }
long fake_instantiated(void) { return ninst; }
int fake_last_error(void) { return last_error; }
/* that many of the next begin-capture, end-capture and instantiate calls fail */
void fake_fail(long begin, long end, long inst) { fail_begin = begin; fail_end = end; fail_inst = inst; }
/* launch n (counted from the last reset) and all later ones fail; -1: none */
void fake_fail_launch(long n) { fail_launch = n; }
/* a launch takes overhead ms + its threads in ms, times slow_ above limit threads */
void fake_cost(double limit, double slow_, double overhead) { limit_threads = limit; slow = slow_; overhead_ms = overhead; }

static int err(int e) { if (e) last_error = e; return e; }

/* ---- code objects and launches */
void** __hipRegisterFatBinary(const void* d) { static void* h; (void)d; return &h; }
void __hipUnregisterFatBinary(void** h) { (void)h; }
void __hipRegisterFunction(void** m, const void* f, char* d, const char* n, unsigned l, void* a, void* b, void* c, void* e, int* w) {
  (void)m; (void)f; (void)d; (void)n; (void)l; (void)a; (void)b; (void)c; (void)e; (void)w;
}
void __hipRegisterVar(void** m, void* v, char* h, const char* d, int e, size_t s, int c, int g) {
  (void)m; (void)v; (void)h; (void)d; (void)e; (void)s; (void)c; (void)g;
}
int __hipPushCallConfiguration(D3 g, D3 b, size_t s, void* st) { cfg_grid = g; cfg_block = b; cfg_shmem = s; cfg_stream = st; return OK; }
int __hipPopCallConfiguration(D3* g, D3* b, size_t* s, void** st) { *g = cfg_grid; *b = cfg_block; *s = cfg_shmem; *st = cfg_stream; return OK; }
int hipLaunchKernel(const void* f, D3 g, D3 b, void** args, size_t shmem, void* st) {
  (void)args; (void)shmem;
  const uint64_t blocks = (uint64_t)g.x * g.y * g.z, threads = (uint64_t)b.x * b.y * b.z;
  /* a launch has fewer than 2^32 threads in all and at most 1024 a workgroup */
  if (blocks == 0 || threads == 0 || threads > 1024 || blocks * threads >= (1ull << 32)) return err(INVALID_CONFIG);
  if (nlaunch >= MAX_LAUNCHES || (fail_launch >= 0 && nlaunch >= fail_launch)) return err(OUT_OF_MEMORY);
  const int cap = capturing; /* one thread: the capture's stream or one forked from it */
  launches[nlaunch++] = (Launch){f, blocks, threads, (uint64_t)(uintptr_t)st, cap};
  if (!cap) {
    const double t = (double)(blocks * threads);
    now_ms += overhead_ms + t * (t > limit_threads ? slow : 1) * 1e-6;
  }
  return OK;
}
int hipGetLastError(void) { const int e = last_error; last_error = OK; return e; }
const char* hipGetErrorString(int e) { return e == INVALID_CONFIG ? "invalid configuration" : e == OUT_OF_MEMORY ? "out of memory" : "fake"; }

/* ---- device and memory */
int hipGetDevice(int* d) { *d = 0; return OK; }
int hipSetDevice(int d) { (void)d; return OK; }
int hipGetDevicePropertiesR0600(void* p, int d) { (void)p; (void)d; return INVALID; }
int hipRuntimeGetVersion(int* v) { *v = 0; return OK; }
int hipMalloc(void** p, size_t n) { *p = malloc(n ? n : 1); return *p ? OK : err(OUT_OF_MEMORY); }
int hipFree(void* p) { free(p); return OK; }
int hipMemcpy(void* d, const void* s, size_t n, int k) { (void)k; memcpy(d, s, n); return OK; }
int hipMemcpyAsync(void* d, const void* s, size_t n, int k, void* st) { (void)k; (void)st; memcpy(d, s, n); return OK; }
int hipPointerGetAttributes(int* at, const void* p) { (void)p; at[0] = 2; return OK; } /* device memory */
int hipMemGetAddressRange(void** base, size_t* n, void* p) { *base = p; *n = (size_t)1 << 60; return OK; }
int hipGetSymbolAddress(void** p, const void* s) { static char* b; (void)s; if (!b) b = malloc(1 << 25); *p = b; return OK; }

/* ---- streams and events */
int hipStreamCreateWithFlags(void** s, unsigned f) { (void)f; *s = (void*)(uintptr_t)(next_handle += 16); return OK; }
int hipStreamDestroy(void* s) { (void)s; return OK; }
int hipStreamSynchronize(void* s) { (void)s; return OK; }
int hipStreamWaitEvent(void* s, void* e, unsigned f) { (void)s; (void)e; (void)f; return OK; }
int hipStreamIsCapturing(void* s, int* st) { (void)s; *st = 0; return OK; }
int hipEventCreate(double** e) { *e = calloc(1, sizeof(double)); return OK; }
int hipEventCreateWithFlags(double** e, unsigned f) { (void)f; return hipEventCreate(e); }
int hipEventDestroy(double* e) { free(e); return OK; }
int hipEventRecord(double* e, void* s) { (void)s; *e = now_ms; return OK; }
int hipEventSynchronize(double* e) { (void)e; return OK; }
int hipEventElapsedTime(float* ms, double* a, double* b) { *ms = (float)(*b - *a); return OK; }

/* ---- graphs */
int hipStreamBeginCapture(void* s, int m) { (void)s; (void)m; if (fail_begin > 0) { --fail_begin; return err(OUT_OF_MEMORY); } capturing = 1; return OK; }
int hipStreamEndCapture(void* s, void** g) {
  (void)s;
  capturing = 0;
  *g = NULL;
  if (fail_end > 0) { --fail_end; return err(OUT_OF_MEMORY); }
  *g = (void*)(uintptr_t)(next_handle += 16);
  return OK;
}
int hipGraphInstantiate(void** x, void* g, void** n, char* l, size_t s) {
  (void)g; (void)n; (void)l; (void)s;
  if (fail_inst > 0) { --fail_inst; *x = NULL; return err(OUT_OF_MEMORY); }
  ++ninst;
  *x = (void*)(uintptr_t)(next_handle += 16);
  return OK;
}
int hipGraphDestroy(void* g) { (void)g; return OK; }
int hipGraphExecDestroy(void* x) { (void)x; return OK; }
int hipGraphLaunch(void* x, void* s) { (void)x; (void)s; ++nreplay; return OK; }
