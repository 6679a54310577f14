/* A HIP runtime without a device, for tests of the library's host code: preloaded,
 * it serves allocations from reserved address space, counts them, accepts every
 * launch (recording the largest grid in work-items) and can be told to fail the
 * stream synchronisation.  Nothing runs: device memory reads as zeros. */
#define _GNU_SOURCE
#include <stdint.h>
#include <stdlib.h>
#include <string.h>
#include <sys/mman.h>

typedef struct { uint32_t x, y, z; } dim3_t;
enum { kMax = 4096 };
static struct { void* p; size_t n; } live[kMax];
static uint64_t held, most_items, launches, bad_frees;
static int sync_to_fail;

uint64_t stub_held(void) { return held; }
uint64_t stub_most_items(void) { return most_items; }
uint64_t stub_launches(void) { return launches; }
uint64_t stub_bad_frees(void) { return bad_frees; }
void stub_fail_sync(int n) { sync_to_fail = n; } /* the n-th from now on */
void stub_reset(void) { most_items = launches = bad_frees = 0; }

int hipGetDeviceCount(int* n) { *n = 1; return 0; }
int hipSetDevice(int d) { (void)d; return 0; }
int hipDeviceGetAttribute(int* v, int a, int d) { (void)a; (void)d; *v = 256; return 0; }
int hipGetLastError(void) { return 0; }
int hipMalloc(void** p, size_t n) {
  for (int i = 0; i < kMax; ++i)
    if (!live[i].p) {
      void* q = mmap(0, n, PROT_READ | PROT_WRITE, MAP_PRIVATE | MAP_ANONYMOUS | MAP_NORESERVE, -1, 0);
      if (q == MAP_FAILED) return 2; /* hipErrorOutOfMemory */
      live[i].p = *p = q;
      live[i].n = n;
      held += n;
      return 0;
    }
  return 2;
}
int hipFree(void* p) {
  if (!p) return 0;
  for (int i = 0; i < kMax; ++i)
    if (live[i].p == p) {
      munmap(p, live[i].n);
      held -= live[i].n;
      live[i].p = 0;
      return 0;
    }
  ++bad_frees;
  return 1;
}
int hipHostMalloc(void** p, size_t n, unsigned f) { (void)f; *p = calloc(1, n); return *p ? 0 : 2; }
int hipHostFree(void* p) { free(p); return 0; }
int hipMemcpy(void* d, const void* s, size_t n, int k) { (void)k; memcpy(d, s, n); return 0; }
int hipMemcpyAsync(void* d, const void* s, size_t n, int k, void* st) {
  (void)st;
  if (k == 2) memcpy(d, s, n); /* device to host */
  return 0;
}
int hipMemsetAsync(void* d, int v, size_t n, void* st) { (void)d; (void)v; (void)n; (void)st; return 0; }
int hipStreamSynchronize(void* st) { (void)st; return sync_to_fail > 0 && --sync_to_fail == 0 ? 999 : 0; }
int hipGetSymbolAddress(void** p, const void* s) { (void)s; return hipMalloc(p, 1 << 20); }
int hipEventCreate(void** e) { *e = malloc(1); return 0; }
int hipEventDestroy(void* e) { free(e); return 0; }
int hipEventRecord(void* e, void* st) { (void)e; (void)st; return 0; }
int hipEventElapsedTime(float* ms, void* a, void* b) { (void)a; (void)b; *ms = 0.f; return 0; }

static __thread struct { dim3_t g, b; size_t lds; void* st; } call;
int __hipPushCallConfiguration(dim3_t g, dim3_t b, size_t lds, void* st) {
  call.g = g; call.b = b; call.lds = lds; call.st = st;
  return 0;
}
int __hipPopCallConfiguration(dim3_t* g, dim3_t* b, size_t* lds, void** st) {
  *g = call.g; *b = call.b; *lds = call.lds; *st = call.st;
  return 0;
}
int hipLaunchKernel(const void* f, dim3_t g, dim3_t b, void** args, size_t lds, void* st) {
  (void)f; (void)args; (void)st;
  const uint64_t n = (uint64_t)g.x * b.x;
  if (n > most_items) most_items = n;
  ++launches;
  /* the limits of a launch: work-items of a dimension, workgroup size, LDS of a CU */
  if (n == 0 || n > 0xffffffffull || b.x > 1024 || lds > 160 * 1024) return 9; /* hipErrorInvalidConfiguration */
  return 0;
}
