/* A stand-in for the HIP calls the library makes, loaded ahead of the real
 * runtime in a process of its own: launches run nothing, are counted and
 * named, and one of them can be made to fail.  The two kernels that write the
 * page table are carried out on host memory. */
#include <stddef.h>
#include <stdint.h>
#include <string.h>

enum { kMaxKernels = 4096, kMaxLog = 65536 };
static const void *host_fn[kMaxKernels];
static const char *dev_name[kMaxKernels];
static int n_kernels, n_log, fail_at = -1, last_error;
static int log_id[kMaxLog];
static uint32_t log_grid[kMaxLog];

void fake_reset(int at) {
  fail_at = at;
  n_log = last_error = 0;
}
int fake_launches(void) { return n_log; }
uint32_t fake_groups(int i) { return log_grid[i]; } /* workgroups of launch i */
const char *fake_kernel(int i) { return log_id[i] < 0 ? "" : dev_name[log_id[i]]; }

void **__hipRegisterFatBinary(const void *data) {
  static void *handle;
  (void)data;
  return &handle;
}
void __hipUnregisterFatBinary(void **h) { (void)h; }
void __hipRegisterVar(void **h, void *var, char *hv, char *dv, int ext, size_t size, int constant, int global) {
  (void)h, (void)var, (void)hv, (void)dv, (void)ext, (void)size, (void)constant, (void)global;
}
void __hipRegisterFunction(void **h, const void *host, char *dev, const char *name, unsigned limit, void *tid, void *bid,
                           void *bdim, void *gdim, int *wsize) {
  (void)h, (void)dev, (void)limit, (void)tid, (void)bid, (void)bdim, (void)gdim, (void)wsize;
  if (n_kernels < kMaxKernels) {
    host_fn[n_kernels] = host;
    dev_name[n_kernels++] = name;
  }
}

typedef struct { uint32_t x, y, z; } dims;
static dims grid_, block_;
static size_t shared_;
static void *stream_;
int __hipPushCallConfiguration(dims g, dims b, size_t s, void *st) {
  grid_ = g, block_ = b, shared_ = s, stream_ = st;
  return 0;
}
int __hipPopCallConfiguration(dims *g, dims *b, size_t *s, void **st) {
  *g = grid_, *b = block_, *s = shared_, *st = stream_;
  return 0;
}

/* the arguments of k_page_runs and k_step_begin, as csrc/kernels.h lays them out */
struct page_runs { int n, b[128], slot[128], page[128], count[128]; };
struct step_begin { int n_pos, b0, pos[64], n_pt, pt_b[64], pt_slot[64], pt_page[64]; };

int hipLaunchKernel(const void *fn, dims g, dims b, void **args, size_t shared, void *st) {
  (void)b, (void)shared, (void)st;
  int id = -1;
  for (int i = 0; i < n_kernels; ++i)
    if (host_fn[i] == fn) id = i;
  const int at = n_log;
  if (n_log < kMaxLog) {
    log_grid[n_log] = g.x * g.y * g.z;
    log_id[n_log++] = id;
  }
  if (at == fail_at) return last_error = 719; /* hipErrorLaunchFailure */
  if (id >= 0 && strstr(dev_name[id], "k_page_runs")) {
    const struct page_runs *r = args[0];
    int *table = *(int **)args[1], mpps = *(int *)args[2];
    for (int i = 0; i < r->n; ++i)
      for (int j = 0; j < r->count[i]; ++j) table[(size_t)r->b[i] * mpps + r->slot[i] + j] = r->page[i] + j;
  }
  if (id >= 0 && strstr(dev_name[id], "k_step_begin")) {
    const struct step_begin *s = args[0];
    int *table = *(int **)args[2], mpps = *(int *)args[3];
    for (int i = 0; i < s->n_pt; ++i) table[(size_t)s->pt_b[i] * mpps + s->pt_slot[i]] = s->pt_page[i];
  }
  return 0;
}
int hipGetLastError(void) {
  const int e = last_error;
  last_error = 0;
  return e;
}
const char *hipGetErrorString(int e) { return e ? "launch failed (stand-in runtime)" : "no error"; }
int hipMemsetAsync(void *p, int v, size_t n, void *st) { return (void)p, (void)v, (void)n, (void)st, 0; }
int hipMemcpyAsync(void *d, const void *s, size_t n, int kind, void *st) {
  return (void)d, (void)s, (void)n, (void)kind, (void)st, 0;
}
int hipGetDevice(int *d) { return *d = 0; }
int hipGetSymbolAddress(void **p, const void *sym) { return *p = (void *)sym, 0; }
static int thing;
int hipStreamCreateWithFlags(void **s, unsigned f) { return (void)f, *s = &thing, 0; }
int hipStreamDestroy(void *s) { return (void)s, 0; }
int hipStreamWaitEvent(void *s, void *e, unsigned f) { return (void)s, (void)e, (void)f, 0; }
int hipEventCreate(void **e) { return *e = &thing, 0; }
int hipEventCreateWithFlags(void **e, unsigned f) { return (void)f, *e = &thing, 0; }
int hipEventDestroy(void *e) { return (void)e, 0; }
int hipEventRecord(void *e, void *s) { return (void)e, (void)s, 0; }
int hipEventSynchronize(void *e) { return (void)e, 0; }
int hipEventElapsedTime(float *ms, void *a, void *b) { return (void)a, (void)b, *ms = 0, 0; }
