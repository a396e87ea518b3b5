/* A HIP runtime of two devices in host memory, for tests of the library's host
 * code on a machine without a GPU: memory, streams and events know their device,
 * kernels do nothing, copies are made at once.  Load it with RTLD_GLOBAL before
 * the library. */
#include <pthread.h>
#include <stddef.h>
#include <stdlib.h>
#include <string.h>

enum { OK = 0, INVALID = 1, NOMEM = 2, HANDLE = 400, DEVICES = 2, SLOTS = 1 << 16 };
static __thread int cur;
static __thread int last;
static pthread_mutex_t mu = PTHREAD_MUTEX_INITIALIZER;
static struct { void* p; size_t n; int dev; } slot[SLOTS];
static size_t used[DEVICES], limit_bytes = (size_t)1 << 62;
static long mallocs, events, launches;
static int fail(int e) { return e ? (last = e) : 0; }

size_t stub_used(int dev) { return used[dev]; }
long stub_mallocs(void) { return mallocs; }
long stub_events(void) { return events; }
long stub_launches(void) { return launches; }
void stub_limit(size_t n) { limit_bytes = n; }

int hipGetDeviceCount(int* n) { *n = DEVICES; return OK; }
int hipGetDevice(int* d) { *d = cur; return OK; }
int hipSetDevice(int d) { if (d < 0 || d >= DEVICES) return fail(INVALID); cur = d; return OK; }
int hipGetLastError(void) { int e = last; last = 0; return e; }
const char* hipGetErrorString(int e) { (void)e; return "stub"; }

int hipMalloc(void** p, size_t n) {
  int rc = NOMEM;
  pthread_mutex_lock(&mu);
  ++mallocs;
  if (used[cur] + n <= limit_bytes)
    for (int i = 0; i < SLOTS; ++i)
      if (!slot[i].p) {
        if ((*p = slot[i].p = malloc(n ? n : 1))) {
          slot[i].n = n;
          slot[i].dev = cur;
          used[cur] += n;
          rc = OK;
        }
        break;
      }
  pthread_mutex_unlock(&mu);
  return fail(rc);
}
int hipFree(void* p) {
  int rc = p ? INVALID : OK;
  pthread_mutex_lock(&mu);
  for (int i = 0; p && i < SLOTS; ++i)
    if (slot[i].p == p) {
      used[slot[i].dev] -= slot[i].n;
      slot[i].p = NULL;
      free(p);
      rc = OK;
      break;
    }
  pthread_mutex_unlock(&mu);
  return fail(rc);
}
int hipHostMalloc(void** p, size_t n, unsigned f) { (void)f; return (*p = calloc(1, n ? n : 1)) ? OK : fail(NOMEM); }
int hipHostFree(void* p) { free(p); return OK; }
int hipHostGetDevicePointer(void** d, void* h, unsigned f) { (void)f; *d = h; return OK; }
int hipMemset(void* p, int v, size_t n) { memset(p, v, n); return OK; }
int hipMemsetAsync(void* p, int v, size_t n, void* s) { (void)s; memset(p, v, n); return OK; }
int hipMemcpy(void* d, const void* s, size_t n, int k) { (void)k; memmove(d, s, n); return OK; }
int hipMemcpyAsync(void* d, const void* s, size_t n, int k, void* st) { (void)k; (void)st; memmove(d, s, n); return OK; }
int hipGetSymbolAddress(void** p, const void* s) { (void)p; (void)s; return fail(INVALID); }

/* a stream or an event is its device; the null stream is the current one's */
static int dev_of(void* h) { return h ? *(int*)h : cur; }
static int make(void** h) { int* d = malloc(sizeof(int)); *d = cur; *h = d; return OK; }
int hipStreamCreateWithFlags(void** s, unsigned f) { (void)f; return make(s); }
int hipStreamDestroy(void* s) { free(s); return OK; }
int hipStreamSynchronize(void* s) { (void)s; return OK; }
int hipStreamWaitEvent(void* s, void* e, unsigned f) { (void)s; (void)e; (void)f; return OK; }
int hipDeviceSynchronize(void) { return OK; }
int hipEventCreate(void** e) { ++events; return make(e); }
int hipEventCreateWithFlags(void** e, unsigned f) { (void)f; ++events; return make(e); }
int hipEventDestroy(void* e) { free(e); return OK; }
int hipEventRecord(void* e, void* s) { return dev_of(e) == dev_of(s) ? OK : fail(HANDLE); }
int hipEventSynchronize(void* e) { (void)e; return OK; }
int hipEventElapsedTime(float* ms, void* a, void* b) { (void)a; (void)b; *ms = 1.0f; return OK; }
typedef struct { unsigned x, y, z; } dim3;
int __hipPushCallConfiguration(dim3 g, dim3 b, size_t n, void* s) {
  (void)g; (void)b; (void)n; (void)s;
  return OK;
}
int __hipPopCallConfiguration(dim3* g, dim3* b, size_t* n, void** s) {
  g->x = g->y = g->z = b->x = b->y = b->z = 1;
  *n = 0;
  *s = NULL;
  return OK;
}
int hipLaunchKernel(const void* f, dim3 g, dim3 b, void** args, size_t n, void* s) {
  (void)f; (void)g; (void)b; (void)args; (void)n; (void)s;
  ++launches;
  return OK;
}
