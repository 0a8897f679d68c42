/* Stand-in for the HIP runtime functions libdugks.so calls, for checks of its
 * host code without a GPU: device memory is malloc'ed, copies are done at once,
 * and every launch and every graph, event and stream call is reported to a hook.
 * Loaded with RTLD_GLOBAL before the library, its symbols come first. */
#include <stdint.h>
#include <stdlib.h>
#include <string.h>

typedef struct { uint32_t x, y, z; } dim3;
typedef void (*hook_t)(const char *what, void *obj, dim3 grid, dim3 block, void **args);
static hook_t hook;
static struct { const void *fn; const char *name; } kernels[4096];
static int nkernels, capturing;
static dim3 cfg_grid, cfg_block;
static size_t cfg_shared;
static void *cfg_stream;
static uintptr_t handles = 0x1000;

void stub_set_hook(hook_t h) { hook = h; }
static int tell(const char *what, void *obj) {
  dim3 one = {1, 1, 1};
  if (hook) hook(what, obj, one, one, NULL);
  return 0;
}
static void *handle(void) { return (void *)(handles += 16); }

void **__hipRegisterFatBinary(const void *d) { static void *m; (void)d; return &m; }
void __hipUnregisterFatBinary(void **m) { (void)m; }
void __hipRegisterFunction(void **m, const void *fn, char *dev, const char *name, unsigned n,
                           void *a, void *b, void *c, void *d, int *e) {
  if (nkernels < 4096) { kernels[nkernels].fn = fn; kernels[nkernels++].name = name; }
}
void __hipRegisterVar(void **m, void *v, char *h, char *d, int e, size_t s, int c, int g) {}
int __hipPushCallConfiguration(dim3 g, dim3 b, size_t s, void *st) {
  cfg_grid = g; cfg_block = b; cfg_shared = s; cfg_stream = st;
  return 0;
}
int __hipPopCallConfiguration(dim3 *g, dim3 *b, size_t *s, void **st) {
  *g = cfg_grid; *b = cfg_block; *s = cfg_shared; *st = cfg_stream;
  return 0;
}
int hipLaunchKernel(const void *fn, dim3 g, dim3 b, void **args, size_t s, void *st) {
  const char *name = "?";
  for (int i = 0; i < nkernels; i++)
    if (kernels[i].fn == fn) name = kernels[i].name;
  if (hook) hook(name, st, g, b, args);
  return 0;
}
int hipGetDevice(int *d) { *d = 0; return 0; }
int hipDeviceGetAttribute(int *v, int a, int d) { *v = 256; return 0; }   /* compute units */
int hipOccupancyMaxActiveBlocksPerMultiprocessor(int *n, const void *f, int b, size_t s) {
  *n = 12;
  return 0;
}
int hipDeviceSynchronize(void) { return tell("device_sync", NULL); }
int hipGetLastError(void) { return 0; }
int hipGetSymbolAddress(void **p, const void *s) {
  static void *mem;
  if (!mem) mem = calloc(1, 1 << 20);
  *p = mem;
  return 0;
}
int hipMalloc(void **p, size_t n) { *p = calloc(1, n); return *p ? 0 : 2; }
int hipFree(void *p) { tell("free", p); free(p); return 0; }
int hipHostMalloc(void **p, size_t n, unsigned f) { return hipMalloc(p, n); }
int hipHostFree(void *p) { free(p); return 0; }
int hipMemcpyAsync(void *d, const void *s, size_t n, int k, void *st) { memcpy(d, s, n); return 0; }
int hipMemset(void *d, int v, size_t n) { memset(d, v, n); return 0; }
int hipMemsetAsync(void *d, int v, size_t n, void *st) { memset(d, v, n); return 0; }
int hipEventCreateWithFlags(void **e, unsigned f) { *e = handle(); return 0; }
int hipEventCreate(void **e) { return hipEventCreateWithFlags(e, 0); }
int hipEventDestroy(void *e) { return tell("event_destroy", e); }
int hipEventRecord(void *e, void *st) { return tell("event_record", e); }
int stub_event_sync_rc;
int hipEventSynchronize(void *e) { tell("event_sync", e); return stub_event_sync_rc; }
int hipEventQuery(void *e) { tell("event_query", e); return 600; }        /* not ready */
int hipEventElapsedTime(float *ms, void *a, void *b) {
  *ms = 1.0f;
  tell("elapsed", ms);                                                      /* the hook may set it */
  return 0;
}
int hipStreamCreateWithFlags(void **s, unsigned f) { *s = handle(); return 0; }
int hipStreamDestroy(void *s) { return 0; }
int hipStreamSynchronize(void *s) { return tell("stream_sync", s); }
int hipStreamIsCapturing(void *s, int *c) { *c = capturing; return 0; }
int hipStreamBeginCapture(void *s, int m) { return tell("capture", s); }
int hipStreamEndCapture(void *s, void **g) { *g = handle(); return 0; }
int hipGraphInstantiate(void **x, void *g, void *n, char *l, size_t z) {
  *x = handle();
  return tell("instantiate", *x);
}
int hipGraphLaunch(void *x, void *st) { return tell("graph_launch", x); }
int hipGraphExecDestroy(void *x) { return tell("exec_destroy", x); }
int hipGraphDestroy(void *g) { return 0; }
