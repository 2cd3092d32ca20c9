/* Stands in for the HIP runtime under libggarray.so, on the CPU: memory is the host's,
 * streams and events are nothing, and launches are recorded instead of run.  Loaded
 * before the library (RTLD_GLOBAL), so that its calls are found here.
 *
 * rec_names / rec_grids / rec_blocks: the launches since rec_clear, in order.
 * rec_capture(id): streams report that they record into graph `id` (0: none).
 * rec_fail(calls): the calls-th allocation from now fails (0: none). */
#include <stddef.h>
#include <stdint.h>
#include <stdlib.h>
#include <string.h>

typedef struct { uint32_t x, y, z; } dim3_t;
enum { MAXF = 4096, MAXL = 65536, kOutOfMemory = 2 };
static const void *f_host[MAXF];
static const char *f_name[MAXF];
static int n_f;
static const char *l_name[MAXL];
static uint32_t l_grid[MAXL], l_block[MAXL];
static int n_l;
static dim3_t c_grid, c_block;
static size_t c_shared;
static void *c_stream;
static uint64_t capture_id;
static int fail_in;

int rec_count(void) { return n_l; }
const char *rec_name(int i) { return l_name[i]; }
uint32_t rec_grid(int i) { return l_grid[i]; }
uint32_t rec_block(int i) { return l_block[i]; }
void rec_clear(void) { n_l = 0; }
void rec_capture(uint64_t id) { capture_id = id; }
void rec_fail(int calls) { fail_in = calls; }

/* operator new, which throws where memory is short: the largest request since rec_new_largest() was last asked. */
static size_t new_largest;
void *_Znwm(size_t n) {
  if (n > new_largest) new_largest = n;
  return malloc(n ? n : 1);
}
size_t rec_new_largest(void) {
  const size_t n = new_largest;
  new_largest = 0;
  return n;
}

void **__hipRegisterFatBinary(const void *data) { (void)data; return (void **)calloc(1, 64); }
void __hipUnregisterFatBinary(void **m) { (void)m; }
void __hipRegisterVar(void **m, void *v, char *a, char *b, int e, size_t s, int c, int g) {
  (void)m; (void)v; (void)a; (void)b; (void)e; (void)s; (void)c; (void)g;
}
void __hipRegisterFunction(void **m, const void *host, char *dev, const char *name, unsigned limit, void *a, void *b,
                           void *c, void *d, int *w) {
  (void)m; (void)dev; (void)limit; (void)a; (void)b; (void)c; (void)d; (void)w;
  if (n_f < MAXF) {
    f_host[n_f] = host;
    f_name[n_f++] = name;
  }
}
int __hipPushCallConfiguration(dim3_t grid, dim3_t block, size_t shared, void *stream) {
  c_grid = grid;
  c_block = block;
  c_shared = shared;
  c_stream = stream;
  return 0;
}
int __hipPopCallConfiguration(dim3_t *grid, dim3_t *block, size_t *shared, void **stream) {
  *grid = c_grid;
  *block = c_block;
  *shared = c_shared;
  *stream = c_stream;
  return 0;
}
static int launched(const void *f, dim3_t grid, dim3_t block) {
  const char *name = "?";
  for (int i = 0; i < n_f; ++i)
    if (f_host[i] == f) name = f_name[i];
  if (n_l < MAXL) {
    l_name[n_l] = name;
    l_grid[n_l] = grid.x;
    l_block[n_l++] = block.x;
  }
  return 0;
}
int hipLaunchKernel(const void *f, dim3_t grid, dim3_t block, void **args, size_t shared, void *stream) {
  (void)args; (void)shared; (void)stream;
  return launched(f, grid, block);
}
int hipExtLaunchKernel(const void *f, dim3_t grid, dim3_t block, void **args, size_t shared, void *stream, void *e0,
                       void *e1, int flags) {
  (void)args; (void)shared; (void)stream; (void)e0; (void)e1; (void)flags;
  return launched(f, grid, block);
}
int hipLaunchCooperativeKernel(const void *f, dim3_t grid, dim3_t block, void **args, unsigned shared, void *stream) {
  (void)args; (void)shared; (void)stream;
  return launched(f, grid, block);
}
int hipOccupancyMaxActiveBlocksPerMultiprocessor(int *n, const void *f, int block, size_t shared) {
  (void)f; (void)block; (void)shared;
  *n = 2;
  return 0;
}

static int take(void **p, size_t n) {
  if (fail_in && --fail_in == 0) return kOutOfMemory;
  *p = aligned_alloc(256, (n + 255) / 256 * 256 + 256);
  if (!*p) return kOutOfMemory;
  memset(*p, 0, n);
  return 0;
}
int hipMalloc(void **p, size_t n) { return take(p, n); }
int hipMallocAsync(void **p, size_t n, void *s) { (void)s; return take(p, n); }
int hipHostMalloc(void **p, size_t n, unsigned flags) { (void)flags; return take(p, n); }
int hipFree(void *p) { free(p); return 0; }
int hipFreeAsync(void *p, void *s) { (void)s; free(p); return 0; }
int hipHostFree(void *p) { free(p); return 0; }
int hipMemcpy(void *d, const void *s, size_t n, int kind) { (void)kind; memcpy(d, s, n); return 0; }
int hipMemcpyAsync(void *d, const void *s, size_t n, int kind, void *st) { (void)kind; (void)st; memcpy(d, s, n); return 0; }
int hipMemset(void *p, int v, size_t n) { memset(p, v, n); return 0; }
int hipMemsetAsync(void *p, int v, size_t n, void *s) { (void)s; memset(p, v, n); return 0; }
int hipMemsetD32Async(void *p, int v, size_t n, void *s) {
  (void)s;
  for (size_t i = 0; i < n; ++i) ((int *)p)[i] = v;
  return 0;
}
int hipStreamIsCapturing(void *s, int *st) { (void)s; *st = capture_id ? 1 : 0; return 0; }
int hipStreamGetCaptureInfo(void *s, int *st, unsigned long long *id) {
  (void)s;
  *st = capture_id ? 1 : 0;
  *id = capture_id;
  return 0;
}
static int handle(void **p) { *p = calloc(1, 64); return 0; }
int hipStreamCreateWithFlags(void **s, unsigned f) { (void)f; return handle(s); }
int hipEventCreate(void **e) { return handle(e); }
int hipEventCreateWithFlags(void **e, unsigned f) { (void)f; return handle(e); }
int hipStreamDestroy(void *s) { free(s); return 0; }
int hipEventDestroy(void *e) { free(e); return 0; }
int hipEventQuery(void *e) { (void)e; return 0; }
int hipEventRecord(void *e, void *s) { (void)e; (void)s; return 0; }
int hipEventSynchronize(void *e) { (void)e; return 0; }
int hipEventElapsedTime(float *ms, void *a, void *b) { (void)a; (void)b; *ms = 0; return 0; }
int hipStreamSynchronize(void *s) { (void)s; return 0; }
int hipDeviceSynchronize(void) { return 0; }
int hipGetDevice(int *d) { *d = 0; return 0; }
int hipDeviceGetAttribute(int *v, int a, int d) { (void)a; (void)d; *v = 256; return 0; }
int hipGetLastError(void) { return 0; }
const char *hipGetErrorName(int e) { (void)e; return "error"; }
int hipGetSymbolAddress(void **p, const void *symbol) {
  static char words[1 << 20];
  (void)symbol;
  *p = words;
  return 0;
}
