/* A stand-in for the HIP runtime, for tests of what the library asks of it on
 * a machine without a GPU: every call that the library makes is written to a
 * log, kernels are not run, and memory copies from the device give counters of
 * a valid call.  Loaded before the library with its symbols global, so that the
 * library's references bind here. */
#include <stdarg.h>
#include <stdint.h>
#include <stdio.h>
#include <stdlib.h>
#include <string.h>

typedef struct { uint32_t x, y, z; } dim3;

static char *g_log;
static size_t g_len, g_cap;
static int g_device, g_capturing;
static uint32_t g_word;       /* what a copy of 4 bytes from the device reads */
static int g_attr_result;
static uintptr_t g_next = 0x1000;

static void put(const char *fmt, ...) {
  char line[512];
  va_list ap;
  va_start(ap, fmt);
  int k = vsnprintf(line, sizeof line, fmt, ap);
  va_end(ap);
  if (g_len + k + 2 > g_cap) g_log = realloc(g_log, g_cap = 2 * (g_len + k + 2) + 65536);
  memcpy(g_log + g_len, line, k);
  g_len += k;
  g_log[g_len++] = '\n';
  g_log[g_len] = 0;
}
const char *fake_log(void) { return g_log ? g_log : ""; }
void fake_clear(void) { g_len = 0; if (g_log) g_log[0] = 0; }
void fake_set(int device, uint32_t word, int attr_result) {
  g_device = device;
  g_word = word;
  g_attr_result = attr_result;
}

static struct { const void *f; char name[256]; } g_fn[512];
static int g_fns;
static const char *fname(const void *f) {
  for (int i = 0; i < g_fns; ++i)
    if (g_fn[i].f == f) return g_fn[i].name;
  return "?";
}
void **__hipRegisterFatBinary(const void *data) { static void *m; (void)data; return &m; }
void __hipUnregisterFatBinary(void **m) { (void)m; }
void __hipRegisterFunction(void **m, const void *f, char *df, const char *name, unsigned lim, void *a, void *b,
                           void *c, void *d, int *e) {
  (void)m; (void)df; (void)lim; (void)a; (void)b; (void)c; (void)d; (void)e;
  if (g_fns < 512) {
    g_fn[g_fns].f = f;
    snprintf(g_fn[g_fns++].name, 256, "%s", name);
  }
}
void __hipRegisterVar(void **m, void *v, char *h, char *d, int e, size_t s, int c, int g) {
  (void)m; (void)v; (void)h; (void)d; (void)e; (void)s; (void)c; (void)g;
}

static struct { dim3 g, b; size_t lds; void *st; } g_conf;
int __hipPushCallConfiguration(dim3 g, dim3 b, size_t lds, void *st) {
  g_conf.g = g; g_conf.b = b; g_conf.lds = lds; g_conf.st = st;
  return 0;
}
int __hipPopCallConfiguration(dim3 *g, dim3 *b, size_t *lds, void **st) {
  *g = g_conf.g; *b = g_conf.b; *lds = g_conf.lds; *st = g_conf.st;
  return 0;
}
int hipLaunchKernel(const void *f, dim3 g, dim3 b, void **args, size_t lds, void *st) {
  (void)args;
  put("launch %s %u %u %u %u lds %zu stream %p device %d%s", fname(f), g.x, g.y, g.z, b.x, lds, st, g_device,
      g_capturing ? " captured" : "");
  return 0;
}

int hipEventCreateWithFlags(void **e, unsigned f) { (void)f; *e = (void *)(g_next += 16); return 0; }
int hipEventRecord(void *e, void *st) { put("record %p stream %p", e, st); return 0; }
int hipStreamWaitEvent(void *st, void *e, unsigned f) { (void)f; put("wait %p stream %p", e, st); return 0; }
int hipStreamCreateWithFlags(void **s, unsigned f) { (void)f; *s = (void *)(g_next += 16); return 0; }
int hipStreamQuery(void *st) { (void)st; return 0; }
int hipStreamSynchronize(void *st) { put("sync stream %p", st); return 0; }
int hipStreamBeginCapture(void *st, int mode) { (void)mode; put("capture stream %p", st); g_capturing = 1; return 0; }
int hipStreamEndCapture(void *st, void **g) {
  put("captured stream %p", st);
  g_capturing = 0;
  *g = (void *)(g_next += 16);
  return 0;
}
int hipGraphInstantiate(void **x, void *g, void **n, char *l, size_t s) {
  (void)g; (void)n; (void)l; (void)s;
  *x = (void *)(g_next += 16);
  return 0;
}
int hipGraphLaunch(void *x, void *st) { put("graph %p stream %p", x, st); return 0; }
int hipGraphDestroy(void *g) { (void)g; return 0; }
int hipGraphExecDestroy(void *x) { (void)x; return 0; }
int hipFuncSetAttribute(const void *f, int attr, int value) {
  put("attribute %s %d %d device %d", fname(f), attr, value, g_device);
  return g_attr_result;
}
int hipGetDevice(int *d) { *d = g_device; return 0; }
int hipGetLastError(void) { return 0; }
const char *hipGetErrorString(int e) { (void)e; return "error"; }
int hipGetSymbolAddress(void **p, const void *s) { (void)s; *p = (void *)0x100000; return 0; }
int hipHostMalloc(void **p, size_t n, unsigned f) { (void)f; *p = calloc(1, n); return *p ? 0 : 2; }

static int copy(void *dst, size_t n) {
  memset(dst, 0, n);
  if (n == 14 * 8) ((int64_t *)dst)[12] = -1; /* herschel_counters: no invalid row */
  if (n == 4) *(uint32_t *)dst = g_word;
  put("copy %zu", n);
  return 0;
}
int hipMemcpy(void *d, const void *s, size_t n, int k) { (void)s; (void)k; return copy(d, n); }
int hipMemcpyAsync(void *d, const void *s, size_t n, int k, void *st) { (void)s; (void)k; (void)st; return copy(d, n); }
