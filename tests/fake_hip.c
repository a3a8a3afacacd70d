/* A HIP runtime without a device, for tests of libtg.so's host code on the
 * CPU: "device" memory is ordinary zeroed memory, kernels do nothing (but
 * for the one that moves messages), and allocations and launches fail where a
 * real device would refuse them or where a test asks for it.  Loaded (RTLD_GLOBAL) before the library, its
 * definitions take the place of the runtime's.
 *
 * Copies and fills of more than BIG bytes are left out: what they move is
 * only read by kernels. */
#define _GNU_SOURCE
#define __HIP_PLATFORM_AMD__
#include <hip/hip_runtime_api.h>
#include <stdint.h>
#include <stdlib.h>
#include <string.h>
#include <sys/mman.h>
#include <time.h>

enum { BIG = 1 << 20 };

static uint64_t thread_limit = (uint64_t)1 << 32; /* a launch has fewer threads than this per dimension */
static size_t malloc_limit = (size_t)-1;          /* device allocations of this many bytes and more fail */
static int mallocs_left = -1;                     /* device allocations until one fails (-1: none does) */
static int host_mallocs_left = -1;                /* the same for pinned ones */
static size_t marked_copy = 0, marked_from = 0;   /* device-to-host copies of this size: bytes from .. on become 127 */
static int failing_syncs = 0;                     /* stream synchronisations still to fail */
static uint64_t launches, most_threads, live_mallocs;
static const void *release_kernel; /* a thread per distance up to 2^31, strides beyond: exempt from a lower limit */
static const void *message_kernel; /* k_message(dst, src, bytes, clocks) */
static uint64_t message_ticks;     /* the time its launches took, each block 100 ticks longer than the one before */
static __thread hipError_t last_error;

void fake_thread_limit(uint64_t n) { thread_limit = n; }
void fake_malloc_limit(size_t n) { malloc_limit = n; }
void fake_mallocs(int n) { mallocs_left = n; }
int fake_mallocs_left(void) { return mallocs_left; }
void fake_host_mallocs(int n) { host_mallocs_left = n; }
void fake_mark_copies(size_t bytes, size_t from) { marked_copy = bytes, marked_from = from; }
void fake_failing_syncs(int n) { failing_syncs = n; }
uint64_t fake_launches(void) { return launches; }
uint64_t fake_message_ticks(void) { return message_ticks; }
uint64_t fake_live_mallocs(void) { return live_mallocs; }
uint64_t fake_most_threads(void) { return most_threads; }

static hipError_t fail(hipError_t e) {
  last_error = e;
  return e;
}

/* memory: a header page holds the size */
static hipError_t map(void **p, size_t n) {
  char *m = mmap(NULL, n + 4096, PROT_READ | PROT_WRITE, MAP_PRIVATE | MAP_ANONYMOUS | MAP_NORESERVE, -1, 0);
  if (m == MAP_FAILED) return fail(hipErrorOutOfMemory);
  memcpy(m, &n, sizeof(n));
  *p = m + 4096;
  return hipSuccess;
}
static hipError_t unmap(void *p) {
  if (p) {
    size_t n;
    memcpy(&n, (char *)p - 4096, sizeof(n));
    munmap((char *)p - 4096, n + 4096);
  }
  return hipSuccess;
}
hipError_t hipMalloc(void **p, size_t n) {
  if (n >= malloc_limit || (mallocs_left >= 0 && mallocs_left-- == 0)) return fail(hipErrorOutOfMemory);
  ++live_mallocs;
  return map(p, n);
}
hipError_t hipFree(void *p) {
  if (p) --live_mallocs;
  return unmap(p);
}
hipError_t hipHostMalloc(void **p, size_t n, unsigned flags) {
  (void)flags;
  if (host_mallocs_left >= 0 && host_mallocs_left-- == 0) return fail(hipErrorOutOfMemory);
  return map(p, n);
}
hipError_t hipHostFree(void *p) { return unmap(p); }
hipError_t hipHostGetDevicePointer(void **d, void *h, unsigned flags) {
  (void)flags;
  *d = h;
  return hipSuccess;
}
hipError_t hipMemcpy(void *d, const void *s, size_t n, hipMemcpyKind k) {
  if (n <= BIG) memmove(d, s, n);
  if (k == hipMemcpyDeviceToHost && n == marked_copy) memset((char *)d + marked_from, 127, n - marked_from);
  return hipSuccess;
}
hipError_t hipMemcpyAsync(void *d, const void *s, size_t n, hipMemcpyKind k, hipStream_t st) {
  (void)st;
  return hipMemcpy(d, s, n, k);
}
hipError_t hipMemset(void *d, int v, size_t n) {
  if (n <= BIG) memset(d, v, n);
  return hipSuccess;
}
hipError_t hipMemsetAsync(void *d, int v, size_t n, hipStream_t st) {
  (void)st;
  return hipMemset(d, v, n);
}
hipError_t hipGetSymbolAddress(void **p, const void *sym) {
  (void)sym;
  return map(p, 64 << 20);
}

/* launches */
static __thread struct {
  dim3 grid, block;
  size_t shared;
  hipStream_t stream;
} conf;
hipError_t __hipPushCallConfiguration(dim3 grid, dim3 block, size_t shared, hipStream_t stream) {
  conf.grid = grid;
  conf.block = block;
  conf.shared = shared;
  conf.stream = stream;
  return hipSuccess;
}
hipError_t __hipPopCallConfiguration(dim3 *grid, dim3 *block, size_t *shared, hipStream_t *stream) {
  *grid = conf.grid;
  *block = conf.block;
  *shared = conf.shared;
  *stream = conf.stream;
  return hipSuccess;
}
hipError_t hipLaunchKernel(const void *f, dim3 g, dim3 b, void **args, size_t shared, hipStream_t st) {
  (void)st;
  const uint64_t x = (uint64_t)g.x * b.x, y = (uint64_t)g.y * b.y, z = (uint64_t)g.z * b.z;
  ++launches;
  if (x > most_threads) most_threads = x;
  if (!x || !y || !z || (uint64_t)b.x * b.y * b.z > 1024 || shared > 163840 ||
      x >= (f == release_kernel && thread_limit < (uint64_t)1 << 31 ? ((uint64_t)1 << 31) + 1 : thread_limit) ||
      y >= thread_limit || z >= thread_limit)
    return fail(hipErrorInvalidConfiguration);
  if (f == message_kernel) {
    memmove(*(char **)args[0], *(char **)args[1], *(int64_t *)args[2]);
    long long *clocks = *(long long **)args[3];
    if (clocks) {
      const uint64_t t0 = 1000 * launches;
      for (unsigned k = 0; k < g.x; ++k) clocks[2 * k] = t0 + k, clocks[2 * k + 1] = t0 + 100 * (k + 1);
      message_ticks += 100 * g.x;
    }
  }
  return hipSuccess;
}
void **__hipRegisterFatBinary(const void *data) {
  static void *handle;
  (void)data;
  return &handle;
}
void __hipUnregisterFatBinary(void **h) { (void)h; }
void __hipRegisterFunction(void **h, const void *f, char *a, const char *b, unsigned c, void *d, void *e, void *i,
                           void *j, int *k) {
  (void)h, (void)a, (void)c, (void)d, (void)e, (void)i, (void)j, (void)k;
  if (strstr(b, "k_message")) message_kernel = f;
  if (strstr(b, "k_ms_release_dist")) release_kernel = f;
}
void __hipRegisterVar(void **h, void *v, char *a, char *b, int c, size_t d, int e, int f) {
  (void)h, (void)v, (void)a, (void)b, (void)c, (void)d, (void)e, (void)f;
}

/* the device, streams and events */
hipError_t hipGetDevice(int *d) { return *d = 0, hipSuccess; }
hipError_t hipSetDevice(int d) { return d == 0 ? hipSuccess : fail(hipErrorInvalidDevice); }
hipError_t hipDeviceSynchronize(void) { return hipSuccess; }
hipError_t hipDeviceGetAttribute(int *v, hipDeviceAttribute_t a, int d) {
  (void)d;
  *v = a == hipDeviceAttributeMaxSharedMemoryPerBlock ? 163840 : 100000;
  return hipSuccess;
}
hipError_t hipGetDeviceProperties(hipDeviceProp_t *p, int d) {
  (void)d;
  memset(p, 0, sizeof(*p));
  strcpy(p->gcnArchName, "gfx950");
  return hipSuccess;
}
const char *hipGetErrorName(hipError_t e) { return e == hipSuccess ? "hipSuccess" : "a fake HIP error"; }
const char *hipGetErrorString(hipError_t e) { return hipGetErrorName(e); }
hipError_t hipGetLastError(void) {
  const hipError_t e = last_error;
  last_error = hipSuccess;
  return e;
}
static hipError_t handle(void **p) {
  *p = malloc(1);
  return hipSuccess;
}
hipError_t hipStreamCreateWithFlags(hipStream_t *s, unsigned f) { return (void)f, handle((void **)s); }
hipError_t hipStreamDestroy(hipStream_t s) { return free(s), hipSuccess; }
hipError_t hipStreamSynchronize(hipStream_t s) {
  (void)s;
  return failing_syncs > 0 && failing_syncs-- ? fail(hipErrorUnknown) : hipSuccess;
}
hipError_t hipStreamQuery(hipStream_t s) { return (void)s, hipSuccess; }
hipError_t hipStreamWaitEvent(hipStream_t s, hipEvent_t e, unsigned f) { return (void)s, (void)e, (void)f, hipSuccess; }
hipError_t hipEventCreate(hipEvent_t *e) { return handle((void **)e); }
hipError_t hipEventCreateWithFlags(hipEvent_t *e, unsigned f) { return (void)f, handle((void **)e); }
hipError_t hipEventDestroy(hipEvent_t e) { return free(e), hipSuccess; }
hipError_t hipEventRecord(hipEvent_t e, hipStream_t s) { return (void)e, (void)s, hipSuccess; }
hipError_t hipEventSynchronize(hipEvent_t e) { return (void)e, hipSuccess; }
hipError_t hipEventElapsedTime(float *ms, hipEvent_t a, hipEvent_t b) { return (void)a, (void)b, *ms = 0.f, hipSuccess; }
