/* A stand-in for the HIP runtime on the host, for tests of the library's host
 * code without a GPU: memory is host memory, kernels do nothing, streams,
 * events and graphs are numbers. Every call of interest is written to the log
 * (stub_log), one per line, and the n-th call of a named function can be made
 * to fail (stub_fail). Loaded with RTLD_GLOBAL before the library. */
#include <stdarg.h>
#include <stddef.h>
#include <stdio.h>
#include <stdlib.h>
#include <string.h>

typedef struct { unsigned x, y, z; } dim3_t;

static char log_[1 << 20];
static size_t used_;
static char fail_[64];
static int countdown_;
static long next_ = 1;
static struct { const void* fn; char name[256]; } kernels_[8192];
static int nkernels_;

const char* stub_log(void) { return log_; }
void stub_clear(void) { used_ = 0; log_[0] = 0; }
/* the n-th call from now on (1: the next) of `name` fails once */
void stub_fail(const char* name, int n) {
  snprintf(fail_, sizeof fail_, "%s", name);
  countdown_ = n;
}

static int call(const char* name, const char* fmt, ...) {
  int bad = 0;
  if (countdown_ > 0 && !strcmp(name, fail_) && --countdown_ == 0) bad = 1;
  if (used_ + 1024 < sizeof log_) {
    va_list ap;
    used_ += snprintf(log_ + used_, 128, "%s%s ", name, bad ? " FAILS" : "");
    va_start(ap, fmt);
    used_ += vsnprintf(log_ + used_, 512, fmt, ap);
    va_end(ap);
    log_[used_++] = '\n';
    log_[used_] = 0;
  }
  return bad ? 999 : 0;
}
static int make(const char* name, void** out) {
  *out = NULL;
  const long id = next_++;
  if (call(name, "%ld", id)) return 999;
  *out = (void*)id;
  return 0;
}

void** __hipRegisterFatBinary(const void* d) { static void* m; (void)d; return &m; }
void __hipUnregisterFatBinary(void** m) { (void)m; }
void __hipRegisterVar(void** m, void* v, char* a, char* b, int e, size_t s, int c, int g) {}
void __hipRegisterFunction(void** m, const void* fn, char* dev, const char* name, unsigned t, void* a,
                           void* b, void* c, void* d, int* w) {
  if (nkernels_ < 8192) {
    kernels_[nkernels_].fn = fn;
    snprintf(kernels_[nkernels_++].name, 256, "%s", name);
  }
}
static dim3_t cfg_grid_, cfg_block_;
static size_t cfg_lds_;
static void* cfg_stream_;
int __hipPushCallConfiguration(dim3_t g, dim3_t b, size_t lds, void* st) {
  cfg_grid_ = g; cfg_block_ = b; cfg_lds_ = lds; cfg_stream_ = st;
  return 0;
}
int __hipPopCallConfiguration(dim3_t* g, dim3_t* b, size_t* lds, void** st) {
  *g = cfg_grid_; *b = cfg_block_; *lds = cfg_lds_; *st = cfg_stream_;
  return 0;
}
int hipLaunchKernel(const void* fn, dim3_t g, dim3_t b, void** args, size_t lds, void* st) {
  const char* name = "?";
  for (int i = 0; i < nkernels_; ++i)
    if (kernels_[i].fn == fn) name = kernels_[i].name;
  return call("kernel", "%s %u %u %zu", name, g.x * g.y, b.x, lds);
}
int hipGetLastError(void) { return 0; }
const char* hipGetErrorString(int e) { return "error of the stand-in"; }
int hipGetDevice(int* d) { *d = 0; return 0; }
int hipSetDevice(int d) { return 0; }
int hipGetDeviceCount(int* n) { *n = 1; return 0; }
int hipGetDevicePropertiesR0600(void* p, int d) { return 999; }
int hipMalloc(void** p, size_t n) { *p = calloc(1, n ? n : 1); return *p ? 0 : 2; }
int hipFree(void* p) { free(p); return 0; }
int hipHostMalloc(void** p, size_t n, unsigned f) { return hipMalloc(p, n); }
int hipHostFree(void* p) { free(p); return 0; }
int hipGetSymbolAddress(void** p, const void* s) { *p = NULL; return 999; }
int hipMemcpy(void* d, const void* s, size_t n, int k) { memcpy(d, s, n); return 0; }
int hipMemcpyAsync(void* d, const void* s, size_t n, int k, void* st) {
  if (call("hipMemcpyAsync", "%zu", n)) return 999;
  memcpy(d, s, n);
  return 0;
}
int hipMemsetAsync(void* d, int v, size_t n, void* st) { memset(d, v, n); return 0; }
int hipStreamCreateWithFlags(void** s, unsigned f) { return make("hipStreamCreate", s); }
int hipStreamDestroy(void* s) { return call("hipStreamDestroy", "%ld", (long)s); }
int hipStreamSynchronize(void* s) { return call("hipStreamSynchronize", "%ld", (long)s); }
int hipStreamWaitEvent(void* s, void* e, unsigned f) {
  return call("hipStreamWaitEvent", "%ld %ld", (long)s, (long)e);
}
int hipStreamBeginCapture(void* s, int m) { return 0; }
int hipStreamEndCapture(void* s, void** g) { *g = (void*)next_++; return 0; }
int hipGraphInstantiate(void** x, void* g, void* n, char* b, size_t s) { return make("hipGraphInstantiate", x); }
int hipGraphDestroy(void* g) { return 0; }
int hipGraphExecDestroy(void* x) { return call("hipGraphExecDestroy", "%ld", (long)x); }
int hipGraphLaunch(void* x, void* s) { return call("hipGraphLaunch", "%ld %ld", (long)x, (long)s); }
int hipEventCreate(void** e) { return make("hipEventCreate", e); }
int hipEventCreateWithFlags(void** e, unsigned f) { return make("hipEventCreate", e); }
int hipEventDestroy(void* e) { return call("hipEventDestroy", "%ld", (long)e); }
int hipEventRecord(void* e, void* s) { return call("hipEventRecord", "%ld %ld", (long)e, (long)s); }
int hipEventSynchronize(void* e) { return call("hipEventSynchronize", "%ld", (long)e); }
int hipEventElapsedTime(float* ms, void* a, void* b) { *ms = 1.0f; return 0; }
