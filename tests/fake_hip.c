/* A stand-in for the HIP runtime on a machine without a GPU, for tests of the
 * library's host code: "device" memory is host memory filled with 0xff, kernels
 * are named in a log instead of run, and allocations and copies fail on demand.
 * Of the kernels it imitates the clearing of a handle's control words and,
 * when asked, the orbit form's refusal. */
#include <stddef.h>
#include <stdint.h>
#include <stdio.h>
#include <stdlib.h>
#include <string.h>

typedef struct { uint32_t x, y, z; } dim3_t;
enum { OK = 0, OUT_OF_MEMORY = 2, FAILED = 1 };

static size_t live, peak, budget = (size_t)-1;
static int fail_malloc_at = -1, fail_host_at = -1, fail_copy_at = -1;   /* -1: none, 0: the next one */
static int refuse, last_error;
static char log_[1 << 20];
static size_t log_len;
static struct { const void* fn; const char* name; } kernels[8192];
static int n_kernels;
static const void* last_arg0[8192];

static int err(int e) {
  if (e) last_error = e;
  return e;
}
static int due(int* at) { return *at >= 0 && (*at)-- == 0; }

void fake_reset(void) {
  budget = (size_t)-1;
  fail_malloc_at = fail_host_at = fail_copy_at = -1;
  refuse = last_error = 0;
  log_len = 0;
  log_[0] = 0;
  peak = live;
}
void fake_set_budget(size_t b) { budget = b; }
void fake_fail_malloc(int n) { fail_malloc_at = n; }
void fake_fail_host(int n) { fail_host_at = n; }
void fake_fail_copy(int n) { fail_copy_at = n; }
void fake_refuse(int on) { refuse = on; }
size_t fake_live(void) { return live; }
size_t fake_peak(void) { return peak; }
const char* fake_log(void) { return log_; }
/* the first argument (a pointer) of the last launch of a kernel whose name holds `part` */
const void* fake_first_arg(const char* part) {
  for (int i = 0; i < n_kernels; ++i)
    if (last_arg0[i] && strstr(kernels[i].name, part)) return last_arg0[i];
  return NULL;
}

int hipMalloc(void** p, size_t n) {
  *p = NULL;
  if (due(&fail_malloc_at) || live + n > budget) return err(OUT_OF_MEMORY);
  char* m = aligned_alloc(256, (n + 256 + 255) / 256 * 256);
  if (!m) return err(OUT_OF_MEMORY);
  *(size_t*)m = n;
  memset(m + 256, 0xff, n);
  live += n;
  if (live > peak) peak = live;
  *p = m + 256;
  return OK;
}
int hipFree(void* p) {
  if (p) {
    char* m = (char*)p - 256;
    live -= *(size_t*)m;
    free(m);
  }
  return OK;
}
int hipHostMalloc(void** p, size_t n, unsigned flags) {
  (void)flags;
  *p = due(&fail_host_at) ? NULL : calloc(1, n);
  return *p ? OK : err(OUT_OF_MEMORY);
}
int hipHostFree(void* p) { free(p); return OK; }
int hipMemcpy(void* d, const void* s, size_t n, int k) {
  (void)k;
  if (due(&fail_copy_at)) return err(FAILED);
  memcpy(d, s, n);
  return OK;
}
int hipMemcpyAsync(void* d, const void* s, size_t n, int k, void* q) {
  (void)k, (void)q;
  memmove(d, s, n);
  return OK;
}
int hipMemcpy2DAsync(void* d, size_t dp, const void* s, size_t sp, size_t w, size_t h, int k, void* q) {
  (void)k, (void)q;
  for (size_t i = 0; i < h; ++i) memcpy((char*)d + i * dp, (const char*)s + i * sp, w);
  return OK;
}
int hipMemsetAsync(void* d, int v, size_t n, void* q) { (void)q; memset(d, v, n); return OK; }

static void note(const char* name) {
  int w = snprintf(log_ + log_len, sizeof log_ - log_len, "%s\n", name);
  if (w > 0 && log_len + w < sizeof log_) log_len += w;
}
static void launched(const void* fn, void** args) {
  for (int i = 0; i < n_kernels; ++i) {
    if (kernels[i].fn != fn) continue;
    const char* name = kernels[i].name;
    note(name);
    last_arg0[i] = args ? *(void**)args[0] : NULL;
    if (strstr(name, "mdpvi15ctl_init_kernel")) {   /* done_iter, flag */
      int64_t* ctl = *(int64_t**)args[0];
      ctl[0] = -1;
      ctl[1] = 0;
    } else if (refuse && strstr(name, "orbit_verdict_kernel")) {
      **(int64_t**)args[2] = -2;                      /* OrbitCtl::done of the host's copy: refused */
    } else if (refuse && strstr(name, "orbit_lds_kernel")) {
      **(int64_t**)args[3] = -2;
    }
    return;
  }
}
int hipLaunchKernel(const void* fn, dim3_t g, dim3_t b, void** args, size_t lds, void* s) {
  (void)g, (void)b, (void)lds, (void)s;
  launched(fn, args);
  return OK;
}
int __hipPushCallConfiguration(dim3_t g, dim3_t b, size_t lds, void* s) { (void)g, (void)b, (void)lds, (void)s; return OK; }
int __hipPopCallConfiguration(dim3_t* g, dim3_t* b, size_t* lds, void** s) {
  memset(g, 0, sizeof *g);
  memset(b, 0, sizeof *b);
  *lds = 0;
  *s = NULL;
  return OK;
}
void** __hipRegisterFatBinary(const void* d) { (void)d; static void* h[1]; return h; }
void __hipUnregisterFatBinary(void** m) { (void)m; }
void __hipRegisterFunction(void** m, const void* fn, char* dev, const char* name, unsigned t, void* a, void* b, void* c,
                           void* d, int* w) {
  (void)m, (void)dev, (void)t, (void)a, (void)b, (void)c, (void)d, (void)w;
  if (n_kernels < 8192) {
    kernels[n_kernels].fn = fn;
    kernels[n_kernels++].name = name;
  }
}
void __hipRegisterVar(void** m, void* v, char* h, char* n, int e, size_t s, int c, int g) {
  (void)m, (void)v, (void)h, (void)n, (void)e, (void)s, (void)c, (void)g;
}

int hipGetLastError(void) {
  int e = last_error;
  last_error = OK;
  return e;
}
const char* hipGetErrorString(int e) { return e == OUT_OF_MEMORY ? "out of memory" : "failed"; }
int hipGetDevice(int* d) { *d = 0; return OK; }
int hipDeviceGetAttribute(int* v, int a, int d) { (void)a, (void)d; *v = 256; return OK; }
int hipGetDevicePropertiesR0600(void* p, int d) { (void)p, (void)d; return FAILED; }
int hipGetSymbolAddress(void** p, const void* s) { (void)s; *p = NULL; return FAILED; }
int hipFuncSetAttribute(const void* f, int a, int v) { (void)f, (void)a, (void)v; return OK; }
int hipDeviceSynchronize(void) { return OK; }
static int handle(void** p) { *p = malloc(1); return OK; }
static int unhandle(void* p) { free(p); return OK; }
int hipEventCreate(void** e) { return handle(e); }
int hipEventCreateWithFlags(void** e, unsigned f) { (void)f; return handle(e); }
int hipEventDestroy(void* e) { return unhandle(e); }
int hipEventRecord(void* e, void* s) { (void)e, (void)s; return OK; }
int hipEventSynchronize(void* e) { (void)e; return OK; }
int hipEventElapsedTime(float* ms, void* a, void* b) { (void)a, (void)b; *ms = 0; return OK; }
int hipStreamCreateWithFlags(void** s, unsigned f) { (void)f; return handle(s); }
int hipStreamDestroy(void* s) { return unhandle(s); }
int hipStreamSynchronize(void* s) { (void)s; return OK; }
int hipStreamWaitEvent(void* s, void* e, unsigned f) { (void)s, (void)e, (void)f; return OK; }
int hipGraphCreate(void** g, unsigned f) { (void)f; return handle(g); }
int hipGraphDestroy(void* g) { return unhandle(g); }
int hipGraphAddKernelNode(void** n, void* g, const void* const* d, size_t nd, const void* p) {
  (void)g, (void)d, (void)nd, (void)p;
  *n = NULL;
  return OK;
}
int hipGraphInstantiate(void** x, void* g, void** n, char* l, size_t s) {
  (void)g, (void)n, (void)l, (void)s;
  note("hipGraphInstantiate");
  return handle(x);
}
int hipGraphLaunch(void* x, void* s) {
  (void)x, (void)s;
  note("hipGraphLaunch");
  return OK;
}
int hipGraphExecDestroy(void* x) { return unhandle(x); }
