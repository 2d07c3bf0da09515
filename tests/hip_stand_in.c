/* Stand-in for the HIP runtime, for tests of the library's host code without a GPU: device memory is host memory, kernels do not
 * run, and what the host asks for is written down.  A replayed round reports a token and a match index to the pinned memory as its
 * last kernel would.  Loaded with RTLD_GLOBAL before libppd.so, whose calls then come here.  One thread, one context at a time. */
#include <stdint.h>
#include <stdio.h>
#include <stdlib.h>
#include <string.h>

typedef int err_t;
typedef struct { uint32_t x, y, z; } dim3_t;
enum { MAX_NAMES = 4096, MAX_NODES = 4096, SEQ = 10 };      /* SEQ: word of the pinned memory that counts finished rounds (2 + PPD_MAX_K) */
typedef struct { int n; const char *node[MAX_NODES]; int under_way; } graph_t;

static struct { const void *host; const char *name; } names[MAX_NAMES];
static int n_names, capturing;
static graph_t *cap, *last_launch;
static int32_t *pinned;
static struct { dim3_t g, b; size_t lds; void *st; } conf;

/* what the tests read and set */
char si_log[1 << 22];                    /* a line each: K kernel, G graph launch with its nodes behind it, S synchronisation, C capture */
static size_t log_at;
int si_destroyed_under_way;              /* executable graphs destroyed before the stream was waited for behind their last launch */
int si_destroyed;
int32_t si_token = 1, si_match = -1;     /* what the next rounds report */
void si_clear(void) { log_at = 0; si_log[0] = 0; }

static void line(const char *kind, const char *what) {
  const size_t n = strlen(kind) + strlen(what) + 3;
  if (log_at + n >= sizeof si_log) abort();
  log_at += (size_t)sprintf(si_log + log_at, "%s %s\n", kind, what);
}
static const char *name_of(const void *f) {
  for (int i = 0; i < n_names; ++i) if (names[i].host == f) return names[i].name;
  abort();
}

void **__hipRegisterFatBinary(const void *d) { static void *p; (void)d; return &p; }
void __hipUnregisterFatBinary(void **m) { (void)m; }
void __hipRegisterFunction(void **m, const void *host, char *dn, const char *dev, unsigned t, void *a, void *b, void *c, void *d, int *w) {
  (void)m; (void)dn; (void)t; (void)a; (void)b; (void)c; (void)d; (void)w;
  if (n_names == MAX_NAMES) abort();
  names[n_names].host = host; names[n_names++].name = dev;
}
void __hipRegisterVar(void **m, void *v, char *a, const char *b, int c, size_t d, int e, int f) { (void)m; (void)v; (void)a; (void)b; (void)c; (void)d; (void)e; (void)f; }
err_t __hipPushCallConfiguration(dim3_t g, dim3_t b, size_t lds, void *st) { conf.g = g; conf.b = b; conf.lds = lds; conf.st = st; return 0; }
err_t __hipPopCallConfiguration(dim3_t *g, dim3_t *b, size_t *lds, void **st) { *g = conf.g; *b = conf.b; *lds = conf.lds; *st = conf.st; return 0; }

err_t hipLaunchKernel(const void *f, dim3_t g, dim3_t b, void **args, size_t lds, void *st) {
  (void)args; (void)st;
  if (!g.x || !g.y || !g.z || !b.x || lds > 160 * 1024) abort();
  if (!capturing) { line("K", name_of(f)); return 0; }
  if (cap->n == MAX_NODES) abort();
  cap->node[cap->n++] = name_of(f);
  return 0;
}
err_t hipStreamBeginCapture(void *s, int mode) { (void)s; (void)mode; capturing = 1; cap = calloc(1, sizeof *cap); line("C", ""); return 0; }
err_t hipStreamEndCapture(void *s, void **g) { (void)s; capturing = 0; *g = cap; cap = NULL; return 0; }
err_t hipGraphInstantiate(void **e, void *g, void *a, char *b, size_t c) { (void)a; (void)b; (void)c; *e = malloc(sizeof(graph_t)); memcpy(*e, g, sizeof(graph_t)); return 0; }
err_t hipGraphDestroy(void *g) { free(g); return 0; }
err_t hipGraphLaunch(void *e, void *s) {
  graph_t *g = e;
  (void)s;
  line("G", "");
  for (int i = 0; i < g->n; ++i) line("K", g->node[i]);
  if (last_launch) last_launch->under_way = 0;             /* (has ended before this round reports) */
  g->under_way = 1; last_launch = g;
  pinned[0] = si_token; pinned[1] = si_match; pinned[SEQ] += 1;
  return 0;
}
err_t hipGraphExecDestroy(void *e) {
  graph_t *g = e;
  si_destroyed += 1;
  si_destroyed_under_way += g->under_way;
  if (last_launch == g) last_launch = NULL;
  free(g);
  return 0;
}
err_t hipStreamSynchronize(void *s) { if (s && last_launch) last_launch->under_way = 0; line("S", ""); return 0; }

err_t hipMalloc(void **p, size_t n) { *p = calloc(1, n ? n : 1); return *p ? 0 : 2; }
err_t hipFree(void *p) { free(p); return 0; }
err_t hipHostMalloc(void **p, size_t n, unsigned f) { (void)f; *p = pinned = calloc(1, n); return 0; }
err_t hipHostFree(void *p) { free(p); return 0; }
err_t hipHostGetDevicePointer(void **d, void *h, unsigned f) { (void)f; *d = h; return 0; }
err_t hipMemcpyAsync(void *d, const void *s, size_t n, int k, void *st) { (void)k; (void)st; memcpy(d, s, n); return 0; }
err_t hipMemcpyWithStream(void *d, const void *s, size_t n, int k, void *st) { (void)k; (void)st; memcpy(d, s, n); return 0; }
err_t hipMemsetAsync(void *d, int v, size_t n, void *st) { (void)st; if (capturing) abort(); memset(d, v, n); return 0; }
err_t hipMemsetD32Async(void *d, int v, size_t n, void *st) { (void)st; if (capturing) abort(); for (size_t i = 0; i < n; ++i) ((int *)d)[i] = v; return 0; }
err_t hipStreamCreateWithFlags(void **s, unsigned f) { (void)f; *s = malloc(8); return 0; }
err_t hipStreamDestroy(void *s) { free(s); return 0; }
err_t hipStreamWaitEvent(void *s, void *e, unsigned f) { (void)s; (void)e; (void)f; return 0; }
err_t hipEventCreateWithFlags(void **e, unsigned f) { (void)f; *e = malloc(8); return 0; }
err_t hipEventCreate(void **e) { *e = malloc(8); return 0; }
err_t hipEventDestroy(void *e) { free(e); return 0; }
err_t hipEventRecord(void *e, void *s) { (void)e; (void)s; return 0; }
err_t hipEventSynchronize(void *e) { (void)e; return 0; }
err_t hipEventElapsedTime(float *f, void *a, void *b) { (void)a; (void)b; *f = 1.f; return 0; }
err_t hipGetLastError(void) { return 0; }
err_t hipFuncSetAttribute(const void *f, int a, int v) { (void)f; (void)a; (void)v; return 0; }
err_t hipGetDevice(int *d) { *d = 0; return 0; }
err_t hipDeviceGetAttribute(int *v, int a, int d) { (void)a; (void)d; *v = 256; return 0; }
err_t hipGetSymbolAddress(void **p, const void *s) { (void)p; (void)s; return 1; }
