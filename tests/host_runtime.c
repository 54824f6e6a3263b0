/* A stand-in for the GPU runtime, for tests of the library's host code on the
 * CPU: allocations are host memory that is never reused, kernels do not run,
 * and every call goes to a log.  A host-to-device copy whose bytes hold an
 * address inside a freed allocation, a copy to memory that is not live, and a
 * free of anything but a live allocation are faults, counted. */
#include <stddef.h>
#include <stdint.h>
#include <stdio.h>
#include <stdlib.h>
#include <string.h>

typedef struct { uint32_t x, y, z; } dim3_;
typedef struct { char *p; size_t n; int live; } range_;
typedef struct { const void *f; char name[256]; } fn_;

static range_ *ranges;
static int n_ranges, cap_ranges, n_fns, n_faults, capturing;
static fn_ fns[4096];
static size_t limit = SIZE_MAX; /* an allocation above this fails */
static char *text;
static size_t text_len, text_cap;

static void say(const char *op, const void *p, size_t n, const void *stream, const char *name) {
  char line[512];
  int k = snprintf(line, sizeof(line), "%s %p %zu %p %s\n", op, p, n, stream, name);
  if (text_len + k + 1 > text_cap) text = realloc(text, text_cap = 2 * (text_len + k + 1));
  memcpy(text + text_len, line, k + 1);
  text_len += k;
}
const char *host_log(void) { return text ? text : ""; }
void host_clear(void) { text_len = 0; if (text) text[0] = 0; }
int host_faults(void) { return n_faults; }
int host_live(void) { int n = 0; for (int i = 0; i < n_ranges; ++i) n += ranges[i].live; return n; }
void host_limit(size_t n) { limit = n; }
void host_capture(int on) { capturing = on; }

static int find(const char *p) {
  for (int i = 0; i < n_ranges; ++i)
    if (p >= ranges[i].p && p < ranges[i].p + ranges[i].n) return i;
  return -1;
}
static void fault(const char *what, const void *p) { ++n_faults; say("FAULT", p, 0, 0, what); }

static int take(void **p, size_t n) {
  if (n > limit) { *p = 0; return 2; }
  if (n_ranges == cap_ranges) ranges = realloc(ranges, (cap_ranges = 2 * cap_ranges + 64) * sizeof(*ranges));
  ranges[n_ranges].p = *p = aligned_alloc(256, (n + 511) & ~(size_t)255);
  ranges[n_ranges].n = n ? n : 1;
  ranges[n_ranges++].live = 1;
  return 0;
}
static int give(void *p) {
  if (!p) return 0;
  int i = find(p);
  if (i < 0 || !ranges[i].live || ranges[i].p != p) { fault("free", p); return 1; }
  ranges[i].live = 0;
  return 0;
}
static int last_error;
static int note(int rc) { if (rc) last_error = rc; return rc; }

int hipMalloc(void **p, size_t n) { int rc = note(take(p, n)); say("malloc", *p, n, 0, ""); return rc; }
int hipFree(void *p) { say("free", p, 0, 0, ""); return note(give(p)); }
int hipMallocAsync(void **p, size_t n, void *st) {
  int rc = note(take(p, n));
  say("malloc_async", *p, n, st, "");
  return rc;
}
int hipFreeAsync(void *p, void *st) { say("free_async", p, 0, st, ""); return note(give(p)); }
static int copy(void *to, const void *from, size_t n, int kind) {
  if (kind == 1) { /* host to device */
    int i = find(to);
    if (i < 0 || !ranges[i].live || (char *)to + n > ranges[i].p + ranges[i].n) { fault("copy", to); return 0; }
    for (size_t b = 0; b + 8 <= n; b += 8) {
      char *w;
      memcpy(&w, (const char *)from + b, 8);
      i = find(w);
      if (i >= 0 && !ranges[i].live) fault("dangling", w);
    }
    memcpy(to, from, n);
  }
  return 0;
}
int hipMemcpy(void *to, const void *from, size_t n, int kind) { say("copy", to, n, 0, ""); return copy(to, from, n, kind); }
int hipMemcpyAsync(void *to, const void *from, size_t n, int kind, void *st) {
  say("copy_async", to, n, st, "");
  return copy(to, from, n, kind);
}
int hipGetDevice(int *d) { *d = 0; return 0; }
int hipDeviceGetAttribute(int *v, int attr, int dev) {
  (void)dev;
  *v = attr == 63 ? 256 : 160 << 10; /* else the LDS of a block */
  return 0;
}
int hipGetLastError(void) { int rc = last_error; last_error = 0; return rc; }
int hipGetSymbolAddress(void **p, const void *symbol) {
  static char *array; /* the one device array, 96 MiB */
  (void)symbol;
  if (!array) take((void **)&array, 96u << 20);
  *p = array;
  return 0;
}
int hipDeviceSynchronize(void) { say("device_sync", 0, 0, 0, ""); return 0; }
int hipStreamSynchronize(void *st) { say("stream_sync", 0, 0, st, ""); return 0; }
int hipStreamIsCapturing(void *st, int *status) { (void)st; *status = capturing; return 0; }
int hipStreamWaitEvent(void *st, void *e, unsigned flags) { (void)flags; say("wait", e, 0, st, ""); return 0; }
int hipEventCreate(void **e) { *e = malloc(8); say("event", *e, 0, 0, ""); return 0; }
int hipEventCreateWithFlags(void **e, unsigned flags) { (void)flags; return hipEventCreate(e); }
int hipEventDestroy(void *e) { say("event_gone", e, 0, 0, ""); free(e); return 0; }
int hipEventRecord(void *e, void *st) { say("record", e, 0, st, ""); return 0; }
int hipEventSynchronize(void *e) { say("event_sync", e, 0, 0, ""); return 0; }
int hipEventElapsedTime(float *ms, void *a, void *b) { (void)a; (void)b; *ms = 0; return 0; }

void **__hipRegisterFatBinary(const void *b) { static void *h; (void)b; return &h; }
void __hipUnregisterFatBinary(void **h) { (void)h; }
void __hipRegisterVar(void **h, void *v, char *hv, char *name, int ext, size_t n, int c, int g) {
  (void)h; (void)v; (void)hv; (void)name; (void)ext; (void)n; (void)c; (void)g;
}
void __hipRegisterFunction(void **h, const void *f, char *df, const char *name, unsigned limit_, void *a, void *b,
                           void *c, void *d, int *w) {
  (void)h; (void)df; (void)limit_; (void)a; (void)b; (void)c; (void)d; (void)w;
  if (n_fns == 4096) return;
  fns[n_fns].f = f;
  snprintf(fns[n_fns++].name, 256, "%s", name);
}
static dim3_ c_grid, c_block;
static size_t c_lds;
static void *c_stream;
int __hipPushCallConfiguration(dim3_ g, dim3_ b, size_t lds, void *st) {
  c_grid = g; c_block = b; c_lds = lds; c_stream = st;
  return 0;
}
int __hipPopCallConfiguration(dim3_ *g, dim3_ *b, size_t *lds, void **st) {
  *g = c_grid; *b = c_block; *lds = c_lds; *st = c_stream;
  return 0;
}
int hipLaunchKernel(const void *f, dim3_ g, dim3_ b, void **args, size_t lds, void *st) {
  const char *name = "?";
  (void)args; (void)lds;
  for (int i = 0; i < n_fns; ++i)
    if (fns[i].f == f) name = fns[i].name;
  if (!g.x || !g.y || !g.z || g.y > 65535 || g.z > 65535 || !b.x || b.x > 1024) { fault("launch", 0); return note(9); }
  say("launch", 0, g.x, st, name);
  return 0;
}
