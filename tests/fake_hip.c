/* A stand-in for the HIP runtime, for tests of the library's host code without a
 * GPU: device memory is host memory, launches are counted by kernel name and do
 * nothing, copies and streams are immediate.  fake_refuse(n) makes every hipMalloc
 * of exactly n bytes fail, fake_capacity(n) every one past n bytes in use. */
#include <stdint.h>
#include <stdio.h>
#include <stdlib.h>
#include <string.h>

typedef struct { unsigned x, y, z; } dim3;
typedef void *ptr;
enum { OK = 0, NO_MEMORY = 2, NOT_SUPPORTED = 801 };

static size_t refused, capacity = (size_t)-1, in_use, asked_n;
static size_t sizes[1 << 16];
static struct { ptr p; size_t n; } blocks[1 << 16];
static struct { const void *f; const char *name; int64_t launches; } kernels[4096];
static int n_kernels;

void fake_refuse(size_t n) { refused = n; }
void fake_capacity(size_t n) { capacity = n; }
size_t fake_in_use(void) { return in_use; }
/* hipMalloc calls of n bytes so far */
int64_t fake_asked(size_t n) {
  int64_t c = 0;
  for (size_t k = 0; k < asked_n; ++k) c += sizes[k] == n;
  return c;
}
/* launches so far of kernels whose (mangled) name contains s */
int64_t fake_launches(const char *s) {
  int64_t c = 0;
  for (int k = 0; k < n_kernels; ++k)
    if (strstr(kernels[k].name, s)) c += kernels[k].launches;
  return c;
}

int hipMalloc(ptr *p, size_t n) {
  if (asked_n < 1 << 16) sizes[asked_n++] = n;
  *p = NULL;
  if (n == refused || in_use + n > capacity) return NO_MEMORY;
  for (int k = 0; k < 1 << 16; ++k)
    if (!blocks[k].p) {
      *p = calloc(1, n);
      if (!*p) return NO_MEMORY;
      blocks[k].p = *p;
      blocks[k].n = n;
      in_use += n;
      return OK;
    }
  return NO_MEMORY;
}
int hipFree(ptr p) {
  for (int k = 0; p && k < 1 << 16; ++k)
    if (blocks[k].p == p) {
      in_use -= blocks[k].n;
      blocks[k].p = NULL;
      free(p);
      return OK;
    }
  if (p) abort(); /* not a live block */
  return OK;
}
int hipHostMalloc(ptr *p, size_t n, unsigned flags) { (void)flags; *p = calloc(1, n); return OK; }
int hipHostFree(ptr p) { free(p); return OK; }
int hipMemcpy(ptr d, const void *s, size_t n, int k) { (void)k; memmove(d, s, n); return OK; }
int hipMemcpyAsync(ptr d, const void *s, size_t n, int k, ptr st) {
  (void)st;
  return hipMemcpy(d, s, n, k);
}
int hipGetDevice(int *d) { *d = 0; return OK; }
int hipGetLastError(void) { return OK; }
const char *hipGetErrorString(int e) { return e == NO_MEMORY ? "out of memory" : "error"; }
int hipGetSymbolAddress(ptr *p, const void *sym) {
  static ptr mem;
  (void)sym;
  if (!mem) mem = calloc(1, 64 << 20);
  *p = mem;
  return OK;
}
int hipFuncSetAttribute(const void *f, int a, int v) { (void)f, (void)a, (void)v; return OK; }
int hipOccupancyMaxActiveBlocksPerMultiprocessor(int *n, const void *f, int t, size_t s) {
  (void)f, (void)t, (void)s;
  *n = 2;
  return OK;
}
int hipLaunchKernel(const void *f, dim3 g, dim3 b, ptr *args, size_t s, ptr st) {
  (void)g, (void)b, (void)args, (void)s, (void)st;
  for (int k = 0; k < n_kernels; ++k)
    if (kernels[k].f == f) {
      ++kernels[k].launches;
      return OK;
    }
  return NOT_SUPPORTED;
}
ptr *__hipRegisterFatBinary(const void *data) {
  static ptr module;
  (void)data;
  return &module;
}
void __hipUnregisterFatBinary(ptr *m) { (void)m; }
void __hipRegisterVar(ptr *m, ptr v, char *hn, char *dn, int e, size_t n, int c, int g) {
  (void)m, (void)v, (void)hn, (void)dn, (void)e, (void)n, (void)c, (void)g;
}
void __hipRegisterFunction(ptr *m, const void *f, char *dn, const char *name, unsigned t, ptr a,
                           ptr b, ptr c, ptr d, int *e) {
  (void)m, (void)dn, (void)t, (void)a, (void)b, (void)c, (void)d, (void)e;
  if (n_kernels < 4096) {
    kernels[n_kernels].f = f;
    kernels[n_kernels++].name = name;
  }
}
static dim3 cfg_g, cfg_b;
static size_t cfg_s;
static ptr cfg_st;
int __hipPushCallConfiguration(dim3 g, dim3 b, size_t s, ptr st) {
  cfg_g = g, cfg_b = b, cfg_s = s, cfg_st = st;
  return OK;
}
int __hipPopCallConfiguration(dim3 *g, dim3 *b, size_t *s, ptr *st) {
  *g = cfg_g, *b = cfg_b, *s = cfg_s, *st = cfg_st;
  return OK;
}
int hipStreamSynchronize(ptr s) { (void)s; return OK; }
int hipStreamCreateWithFlags(ptr *s, unsigned f) { (void)f; *s = (ptr)&cfg_st; return OK; }
int hipStreamDestroy(ptr s) { (void)s; return OK; }
int hipEventCreate(ptr *e) { *e = (ptr)&cfg_st; return OK; }
int hipEventDestroy(ptr e) { (void)e; return OK; }
int hipEventRecord(ptr e, ptr s) { (void)e, (void)s; return OK; }
int hipEventSynchronize(ptr e) { (void)e; return OK; }
int hipEventElapsedTime(float *ms, ptr a, ptr b) { (void)a, (void)b; *ms = 0; return OK; }
/* graphs: capture works and records nothing */
int hipStreamBeginCapture(ptr s, int m) { (void)s, (void)m; return OK; }
int hipStreamEndCapture(ptr s, ptr *g) { (void)s; *g = (ptr)&cfg_st; return OK; }
int hipGraphGetNodes(ptr g, ptr *n, size_t *c) { (void)g, (void)n; *c = 1; return OK; }
int hipGraphInstantiateWithFlags(ptr *x, ptr g, unsigned long long f) {
  (void)g, (void)f;
  *x = (ptr)&cfg_st;
  return OK;
}
int hipGraphDestroy(ptr g) { (void)g; return OK; }
int hipGraphExecDestroy(ptr x) { (void)x; return OK; }
int hipGraphLaunch(ptr x, ptr s) { (void)x, (void)s; return OK; }
