/* A HIP runtime of which only the host side exists: memory is host memory, a launch is written down
 * and its kernel never runs.  Loaded before libvf.so it stands in for the real runtime, so that the
 * library's own host code - what it allocates, which kernels it chooses, with which grids and
 * arguments - runs on a machine without a GPU, under allocation failures that a test asks for. */
#include <hip/hip_runtime_api.h>
#include <stdio.h>
#include <stdlib.h>
#include <string.h>

static hipError_t last_error = hipSuccess;
static size_t fail_lo = 1, fail_hi = 0;
static struct { const void *host; char name[200]; } kernels[512];
static int n_kernels;
static char log_text[1 << 20];
static size_t log_len;
static dim3 cfg_grid, cfg_block;
static size_t cfg_shared;
static hipStream_t cfg_stream;
static char static_array[1 << 20];
static int capturing;
static char refused[100];
static int refused_skip;

/* hipMalloc of lo..hi bytes fails from now on (lo > hi: none does) */
void stub_fail(size_t lo, size_t hi) { fail_lo = lo; fail_hi = hi; }
/* the launch after the next `skip` ones of kernels whose names hold `name` is refused (NULL: none is) */
void stub_fail_launch(const char *name, int skip) {
  snprintf(refused, sizeof refused, "%s", name ? name : "");
  refused_skip = skip;
}
/* every stream is being captured from now on (0: none is) */
void stub_capture(int on) { capturing = on; }
/* the launches so far, one "kernel grid weights" a line */
const char *stub_log(void) { return log_text; }
void stub_clear(void) { log_len = 0; log_text[0] = 0; }

static hipError_t err(hipError_t e) {
  if (e != hipSuccess) last_error = e;
  return e;
}
hipError_t hipGetLastError(void) {
  const hipError_t e = last_error;
  last_error = hipSuccess;
  return e;
}
hipError_t hipGetDeviceCount(int *n) { *n = 1; return hipSuccess; }
hipError_t hipGetDevice(int *d) { *d = 0; return hipSuccess; }
hipError_t hipSetDevice(int d) { return d == 0 ? hipSuccess : err(hipErrorInvalidDevice); }
hipError_t hipDeviceGetAttribute(int *v, hipDeviceAttribute_t a, int d) {
  (void)d;
  *v = a == hipDeviceAttributeMultiprocessorCount ? 256 : a == hipDeviceAttributeMaxSharedMemoryPerBlock ? 160 * 1024 : 0;
  return hipSuccess;
}
hipError_t hipMalloc(void **p, size_t n) {
  *p = NULL;
  if (n >= fail_lo && n <= fail_hi) return err(hipErrorOutOfMemory);
  *p = calloc(1, n);
  return *p ? hipSuccess : err(hipErrorOutOfMemory);
}
static int frees;
/* how many allocations have been given back */
int stub_frees(void) { return frees; }
hipError_t hipFree(void *p) { frees += p != NULL; free(p); return hipSuccess; }
hipError_t hipHostMalloc(void **p, size_t n, unsigned int f) { (void)f; *p = calloc(1, n); return hipSuccess; }
hipError_t hipHostFree(void *p) { free(p); return hipSuccess; }
hipError_t hipMemcpyAsync(void *d, const void *s, size_t n, hipMemcpyKind k, hipStream_t st) {
  (void)k; (void)st;
  memcpy(d, s, n);
  return hipSuccess;
}
hipError_t hipMemsetAsync(void *d, int v, size_t n, hipStream_t st) { (void)st; memset(d, v, n); return hipSuccess; }
hipError_t hipStreamSynchronize(hipStream_t s) { (void)s; return hipSuccess; }
hipError_t hipStreamIsCapturing(hipStream_t s, hipStreamCaptureStatus *st) {
  (void)s;
  *st = capturing ? hipStreamCaptureStatusActive : hipStreamCaptureStatusNone;
  return hipSuccess;
}
hipError_t hipEventCreate(hipEvent_t *e) { *e = (hipEvent_t)static_array; return hipSuccess; }
hipError_t hipEventCreateWithFlags(hipEvent_t *e, unsigned f) { (void)f; *e = NULL; return hipSuccess; }
hipError_t hipEventDestroy(hipEvent_t e) { (void)e; return hipSuccess; }
hipError_t hipEventRecord(hipEvent_t e, hipStream_t s) { (void)e; (void)s; return hipSuccess; }
hipError_t hipEventQuery(hipEvent_t e) { (void)e; return hipSuccess; }
hipError_t hipEventSynchronize(hipEvent_t e) { (void)e; return hipSuccess; }
hipError_t hipEventElapsedTime(float *ms, hipEvent_t a, hipEvent_t b) { (void)a; (void)b; *ms = 0; return hipSuccess; }
hipError_t hipFuncSetAttribute(const void *f, hipFuncAttribute a, int v) { (void)f; (void)a; (void)v; return hipSuccess; }
hipError_t hipFuncGetAttributes(struct hipFuncAttributes *a, const void *f) {
  (void)f;
  memset(a, 0, sizeof *a);
  a->sharedSizeBytes = 4096;
  return hipSuccess;
}
hipError_t hipOccupancyMaxActiveBlocksPerMultiprocessor(int *n, const void *f, int b, size_t s) {
  (void)f; (void)b; (void)s;
  *n = 1;
  return hipSuccess;
}
hipError_t hipGetSymbolAddress(void **p, const void *s) { (void)s; *p = static_array; return hipSuccess; }

/* what the compiler's host code calls */
void **__hipRegisterFatBinary(const void *d) { static void *handle; (void)d; return &handle; }
void __hipUnregisterFatBinary(void **h) { (void)h; }
void __hipRegisterVar(void **h, void *v, char *hv, char *dv, int e, size_t n, int c, int g) {
  (void)h; (void)v; (void)hv; (void)dv; (void)e; (void)n; (void)c; (void)g;
}
void __hipRegisterFunction(void **h, const void *host, char *dev, const char *name, unsigned lim, void *t, void *b, void *bd,
                           void *gd, int *w) {
  (void)h; (void)dev; (void)lim; (void)t; (void)b; (void)bd; (void)gd; (void)w;
  if (n_kernels == 512) abort();
  kernels[n_kernels].host = host;
  snprintf(kernels[n_kernels++].name, sizeof kernels[0].name, "%s", name);
}
hipError_t __hipPushCallConfiguration(dim3 g, dim3 b, size_t s, hipStream_t st) {
  cfg_grid = g; cfg_block = b; cfg_shared = s; cfg_stream = st;
  return hipSuccess;
}
hipError_t __hipPopCallConfiguration(dim3 *g, dim3 *b, size_t *s, hipStream_t *st) {
  *g = cfg_grid; *b = cfg_block; *s = cfg_shared; *st = cfg_stream;
  return hipSuccess;
}
hipError_t hipLaunchKernel(const void *f, dim3 g, dim3 b, void **args, size_t shared, hipStream_t st) {
  const char *name = "?";
  (void)shared; (void)st;
  for (int i = 0; i < n_kernels; ++i)
    if (kernels[i].host == f) name = kernels[i].name;
  /* the runtime's limit: less than 2^32 work-items in every dimension */
  if ((unsigned long long)g.x * b.x >> 32 || (unsigned long long)g.y * b.y >> 32 || (unsigned long long)g.z * b.z >> 32 ||
      !g.x || !g.y || !g.z)
    return err(hipErrorInvalidConfiguration);
  if (refused[0] && strstr(name, refused) && refused_skip-- == 0) {
    refused[0] = 0;
    return err(hipErrorLaunchFailure);
  }
  /* (the second argument of k_seq_step_held and k_seq_step_wide is their weights) */
  const void *weights = strstr(name, "k_seq_step_held") || strstr(name, "k_seq_step_wide") ? *(void **)args[1] : (void *)1;
  if (log_len + 300 < sizeof log_text)
    log_len += (size_t)snprintf(log_text + log_len, sizeof log_text - log_len, "%s %u %d\n", name, g.x, weights != NULL);
  return hipSuccess;
}
