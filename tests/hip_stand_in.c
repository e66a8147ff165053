/* A stand-in for the part of the HIP runtime that the library calls, for tests of its host code
 * without a GPU: device memory is host memory (cleared), copies are made at once, launches are
 * only reported.  Loaded before the library with its symbols global. */
#include <stdint.h>
#include <stdlib.h>
#include <string.h>
#include <sys/mman.h>

typedef struct { uint32_t x, y, z; } dim3_t;
typedef void (*launch_fn)(const char *name, uint32_t gx, uint32_t gy, uint32_t gz, uint32_t bx, size_t lds, void *stream, void **args);

enum { kMost = 512, kOutOfMemory = 2 };
static const void *g_func[kMost];
static char *g_name[kMost];
static int g_n;
static launch_fn g_on_launch;
static int g_fail = -1;         /* allocations until one fails, -1: none does */
static int g_fail_more;         /* and how many after it */
static uint64_t g_mallocs, g_frees, g_uploads, g_stream_syncs, g_device_syncs, g_largest;
static struct { dim3_t grid, block; size_t lds; void *stream; } g_call;

void stand_in_on_launch(launch_fn f) { g_on_launch = f; }
void stand_in_fail(int after, int more) { g_fail = after; g_fail_more = more; }
int stand_in_failing(void) { return g_fail >= 0; }   /* the allocation that is to fail has not come yet */
void stand_in_counts(uint64_t *out) {   /* allocations, frees, uploads, waits for a stream, waits for the device, largest allocation */
  out[0] = g_mallocs; out[1] = g_frees; out[2] = g_uploads; out[3] = g_stream_syncs; out[4] = g_device_syncs; out[5] = g_largest;
}

static int fails(void) {
  if (g_fail < 0) return 0;
  if (g_fail > 0) { --g_fail; return 0; }
  if (g_fail_more-- > 0) return 1;
  g_fail = -1;
  return 1;
}

void **__hipRegisterFatBinary(const void *data) { static void *module; (void)data; return &module; }
void __hipUnregisterFatBinary(void **m) { (void)m; }
void __hipRegisterFunction(void **m, const void *func, char *device_func, const char *name) {
  (void)m; (void)device_func;
  if (g_n < kMost) { g_func[g_n] = func; g_name[g_n++] = strdup(name); }
}
void __hipRegisterVar(void **m, void *var) { (void)m; (void)var; }
int __hipPushCallConfiguration(dim3_t grid, dim3_t block, size_t lds, void *stream) {
  g_call.grid = grid; g_call.block = block; g_call.lds = lds; g_call.stream = stream;
  return 0;
}
int __hipPopCallConfiguration(dim3_t *grid, dim3_t *block, size_t *lds, void **stream) {
  *grid = g_call.grid; *block = g_call.block; *lds = g_call.lds; *stream = g_call.stream;
  return 0;
}
int hipLaunchKernel(const void *func, dim3_t grid, dim3_t block, void **args, size_t lds, void *stream) {
  const char *name = "?";
  for (int k = 0; k < g_n; ++k)
    if (g_func[k] == func) name = g_name[k];
  if (g_on_launch) g_on_launch(name, grid.x, grid.y, grid.z, block.x, lds, stream, args);
  return 0;
}
/* cleared memory that takes no room until it is written (a device has more than this host); its size in front of it */
int hipMalloc(void **p, size_t n) {
  ++g_mallocs;
  if (n > g_largest) g_largest = n;
  *p = 0;
  if (fails()) return kOutOfMemory;
  size_t *m = mmap(0, n + 4096, PROT_READ | PROT_WRITE, MAP_PRIVATE | MAP_ANONYMOUS | MAP_NORESERVE, -1, 0);
  if (m == MAP_FAILED) return kOutOfMemory;
  *m = n + 4096;
  *p = (char *)m + 4096;
  return 0;
}
int hipFree(void *p) {
  ++g_frees;
  if (p) munmap((char *)p - 4096, *(size_t *)((char *)p - 4096));
  return 0;
}
int hipHostMalloc(void **p, size_t n, unsigned flags) { (void)flags; *p = calloc(1, n + 1); return 0; }
int hipHostFree(void *p) { free(p); return 0; }
int hipMemcpyAsync(void *to, const void *from, size_t n, int kind, void *stream) { (void)stream; g_uploads += kind == 1; memcpy(to, from, n); return 0; }
int hipStreamSynchronize(void *s) { (void)s; ++g_stream_syncs; return 0; }
static void *g_recorded;
void stand_in_record(void *stream) { g_recorded = stream; }   /* the stream that is being recorded, or null */
int hipStreamIsCapturing(void *stream, int *status) { *status = stream && stream == g_recorded; return 0; }
int hipDeviceSynchronize(void) { ++g_device_syncs; return 0; }
int hipEventCreateWithFlags(void **e, unsigned flags) { (void)flags; *e = malloc(1); return 0; }
int hipEventRecord(void *e, void *s) { (void)e; (void)s; return 0; }
int hipEventSynchronize(void *e) { (void)e; return 0; }
int hipFuncSetAttribute(const void *f, int attr, int value) { (void)f; (void)attr; (void)value; return 0; }
int hipGetDevice(int *d) { *d = 0; return 0; }
int hipSetDevice(int d) { (void)d; return 0; }
int hipGetLastError(void) { return 0; }
int hipGetSymbolAddress(void **p, const void *var) { static char memory[1 << 20]; (void)var; *p = memory; return 0; }
