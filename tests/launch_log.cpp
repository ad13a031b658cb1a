// A HIP runtime that launches nothing: every launch, event record and event wait of the library under test becomes a line
// of the file named by LAUNCH_LOG.  Loaded with global scope before the library, it takes the real runtime's place, so
// that the order a call enqueues its work in can be checked on a machine without a GPU.
//   L <stream> <kernel> <words of the first argument> | <words of the second>      W <stream> <event>      R <stream> <event>
#include <cstdint>
#include <cstdio>
#include <cstdlib>
#include <cstring>
#include <map>
#include <string>

struct dim3_ {
  uint32_t x, y, z;
};
typedef void *ptr;

static std::map<const void *, std::string> &names() {
  static std::map<const void *, std::string> m;
  return m;
}
static FILE *out() {
  static FILE *f = fopen(getenv("LAUNCH_LOG"), "w");
  return f;
}
static struct {
  dim3_ grid, block;
  size_t shared;
  ptr stream;
} config;
static uintptr_t next_handle = 0x10;

extern "C" {
ptr *__hipRegisterFatBinary(const void *) { return new ptr; }
void __hipUnregisterFatBinary(ptr *) {}
void __hipRegisterFunction(ptr *, const void *host, char *, const char *name, unsigned, ptr, ptr, ptr, ptr, int *) {
  names()[host] = name;
}
void __hipRegisterVar(ptr *, void *, char *, char *, int, size_t, int, int) {}
int __hipPushCallConfiguration(dim3_ grid, dim3_ block, size_t shared, ptr stream) {
  config = {grid, block, shared, stream};
  return 0;
}
int __hipPopCallConfiguration(dim3_ *grid, dim3_ *block, size_t *shared, ptr *stream) {
  *grid = config.grid;
  *block = config.block;
  *shared = config.shared;
  *stream = config.stream;
  return 0;
}
int hipLaunchKernel(const void *fn, dim3_, dim3_, void **args, size_t, ptr stream) {
  const std::string &name = names()[fn];
  fprintf(out(), "L %p %s", stream, name.c_str());
  // contraction kernels take a shape and an epilogue structure; of the others only the first word is looked at
  const bool gemm = name.find("gemm") != std::string::npos;
  for (int a = 0; a < (gemm ? 2 : 1); ++a) {
    for (int w = 0; w < (gemm ? 10 : 1); ++w) {
      uint64_t v;
      memcpy(&v, static_cast<const char *>(args[a]) + 8 * w, 8);
      fprintf(out(), " %llx", (unsigned long long)v);
    }
    fprintf(out(), " |");
  }
  fprintf(out(), "\n");
  fflush(out());
  return 0;
}
int hipEventRecord(ptr event, ptr stream) {
  fprintf(out(), "R %p %p\n", stream, event);
  fflush(out());
  return 0;
}
int hipStreamWaitEvent(ptr stream, ptr event, unsigned) {
  fprintf(out(), "W %p %p\n", stream, event);
  fflush(out());
  return 0;
}
int hipMemcpy(void *dst, const void *, size_t n, int) {  // the placement probe: block i on die i mod 8
  for (size_t i = 0; i < n / 4; ++i) static_cast<int32_t *>(dst)[i] = (int32_t)(i % 8);
  return 0;
}
int hipEventCreate(ptr *e) { return *e = (ptr)(next_handle += 0x10), 0; }
int hipEventCreateWithFlags(ptr *e, unsigned) { return hipEventCreate(e); }
int hipStreamCreateWithFlags(ptr *s, unsigned) { return hipEventCreate(s); }
int hipGetDeviceCount(int *n) { return *n = 1, 0; }
int hipGetDevice(int *d) { return *d = 0, 0; }
int hipOccupancyMaxActiveBlocksPerMultiprocessor(int *n, const void *, int, size_t) { return *n = 1, 0; }
int hipSetDevice(int) { return 0; }
int hipGetLastError() { return 0; }
int hipDeviceSynchronize() { return 0; }
int hipEventDestroy(ptr) { return 0; }
int hipEventElapsedTime(float *, ptr, ptr) { return 0; }
int hipEventSynchronize(ptr) { return 0; }
int hipFuncSetAttribute(const void *, int, int) { return 0; }
int hipGetSymbolAddress(ptr *, const void *) { return 1; }
int hipMemcpyAsync(void *, const void *, size_t, int, ptr) { return 0; }
int hipMemsetAsync(void *, int, size_t, ptr) { return 0; }
int hipStreamDestroy(ptr) { return 0; }
int hipStreamSynchronize(ptr) { return 0; }
}
