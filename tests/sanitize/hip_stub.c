/* A HIP runtime without a device, for the library's host code on the CPU: memory
 * is host memory, kernels do nothing but leave their names (and their blocks and
 * threads) in a log.  Built by tests/test_host_stub_cpu.py. */
#include <stdint.h>
#include <stdio.h>
#include <stdlib.h>
#include <string.h>

typedef int Err;
typedef struct {
  unsigned x, y, z;
} Dim;

static Dim grid_, block_;
static size_t shmem_;
static void* stream_;
Err __hipPushCallConfiguration(Dim g, Dim b, size_t s, void* t) {
  grid_ = g, block_ = b, shmem_ = s, stream_ = t;
  return 0;
}
Err __hipPopCallConfiguration(Dim* g, Dim* b, size_t* s, void** t) {
  *g = grid_, *b = block_, *s = shmem_, *t = stream_;
  return 0;
}

static struct {
  const void* fn;
  const char* name;
} kernels_[4096];
static int n_kernels_;
void** __hipRegisterFatBinary(const void* data) {
  static void* h;
  (void)data;
  return &h;
}
void __hipRegisterFunction(void** m, const void* fn, char* dev, const char* name, unsigned t, void* a, void* b,
                           void* c, void* d, int* e) {
  (void)m, (void)dev, (void)t, (void)a, (void)b, (void)c, (void)d, (void)e;
  if (n_kernels_ < 4096) kernels_[n_kernels_].fn = fn, kernels_[n_kernels_++].name = name;
}
void __hipRegisterVar(void) {}
void __hipUnregisterFatBinary(void** m) { (void)m; }

static char log_[1 << 20];
static size_t log_n_;
void stub_log_clear(void) { log_n_ = 0, log_[0] = 0; }
const char* stub_log(void) { return log_; }   /* "mangled-name blocks threads\n" per launch */
Err hipLaunchKernel(const void* fn, Dim g, Dim b, void** args, size_t shmem, void* stream) {
  const uint64_t threads = (uint64_t)b.x * b.y * b.z, blocks = (uint64_t)g.x * g.y * g.z;
  (void)args, (void)stream;
  if (threads == 0 || threads > 1024 || blocks == 0 || shmem > 160 * 1024) {
    fprintf(stderr, "[stub] launch outside the device's limits\n");
    return 1;
  }
  for (int i = 0; i < n_kernels_; ++i)
    if (kernels_[i].fn == fn && log_n_ + 512 < sizeof(log_))
      log_n_ += (size_t)snprintf(log_ + log_n_, 512, "%s %llu %llu\n", kernels_[i].name, (unsigned long long)blocks,
                                 (unsigned long long)threads);
  return 0;
}

static Err give(void** p, size_t n) {
  *p = calloc(1, n ? n : 1);
  return *p ? 0 : 2;
}
Err hipMalloc(void** p, size_t n) { return give(p, n); }
Err hipMallocAsync(void** p, size_t n, void* s) {
  (void)s;
  return give(p, n);
}
Err hipFree(void* p) {
  free(p);
  return 0;
}
Err hipFreeAsync(void* p, void* s) {
  (void)s;
  free(p);
  return 0;
}
Err hipMemcpy(void* d, const void* s, size_t n, int k) {
  (void)k;
  memcpy(d, s, n);
  return 0;
}
Err hipMemcpyAsync(void* d, const void* s, size_t n, int k, void* t) {
  (void)k, (void)t;
  memcpy(d, s, n);
  return 0;
}
Err hipMemset(void* d, int v, size_t n) {
  memset(d, v, n);
  return 0;
}
static char symbol_[1 << 20];
Err hipGetSymbolAddress(void** p, const void* s) {
  (void)s;
  *p = symbol_;
  return 0;
}
static int pool_;
Err hipDeviceGetDefaultMemPool(void** p, int d) {
  (void)d;
  *p = &pool_;
  return 0;
}
Err hipMemPoolSetAttribute(void* p, int a, void* v) {
  (void)p, (void)a, (void)v;
  return 0;
}
Err hipDeviceSynchronize(void) { return 0; }
Err hipStreamSynchronize(void* s) {
  (void)s;
  return 0;
}
Err hipFuncSetAttribute(const void* f, int a, int v) {
  (void)f, (void)a, (void)v;
  return 0;
}
Err hipGetDevice(int* d) {
  *d = 0;
  return 0;
}
Err hipSetDevice(int d) {
  (void)d;
  return 0;
}
Err hipGetLastError(void) { return 0; }
const char* hipGetErrorString(Err e) {
  (void)e;
  return "stub";
}
