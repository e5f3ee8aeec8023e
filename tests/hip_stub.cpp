// Stands in for the HIP runtime on the CPU so that tests can run libmgc.so's
// host code without a GPU: "device" memory is host memory, two devices exist, the
// one-block byte copy is carried out at its launch and other kernels do nothing.
// A stream wait takes a while, as one on a GPU does, so that threads overlap.
// (The library's remaining imports are added as functions that return 0.)
#include <stdint.h>
#include <stdlib.h>
#include <string.h>
#include <time.h>

#include <map>
#include <mutex>
#include <string>

struct Dim3 {
  uint32_t x, y, z;
};
static std::mutex mu;
static std::map<const void*, std::string> kernels;
static thread_local int device = 0;
static thread_local struct {
  Dim3 grid, block;
  size_t lds;
  void* stream;
} config;

extern "C" {
void** __hipRegisterFatBinary(const void*) {
  static void* handle = nullptr;
  return &handle;
}
void __hipRegisterFunction(void**, const void* host, char*, const char* name, unsigned, void*,
                           void*, void*, void*, int*) {
  std::lock_guard<std::mutex> lk(mu);
  kernels[host] = name;
}
int __hipPushCallConfiguration(Dim3 grid, Dim3 block, size_t lds, void* stream) {
  config = {grid, block, lds, stream};
  return 0;
}
int __hipPopCallConfiguration(Dim3* grid, Dim3* block, size_t* lds, void** stream) {
  *grid = config.grid;
  *block = config.block;
  *lds = config.lds;
  *stream = config.stream;
  return 0;
}
int hipLaunchKernel(const void* f, Dim3, Dim3, void** args, size_t, void*) {
  std::string name;
  {
    std::lock_guard<std::mutex> lk(mu);
    name = kernels[f];
  }
  if (name.find("k_copy_bytes") != std::string::npos)
    memcpy(*static_cast<void**>(args[0]), *static_cast<void**>(args[1]),
           (size_t)*static_cast<int*>(args[2]));
  return 0;
}
int hipStreamSynchronize(void*) {
  const timespec t = {0, 200000};
  nanosleep(&t, nullptr);
  return 0;
}
int hipGetDeviceCount(int* n) {
  *n = 2;
  return 0;
}
int hipSetDevice(int d) {
  device = d;
  return 0;
}
int hipGetDevice(int* d) {
  *d = device;
  return 0;
}
int hipHostMalloc(void** p, size_t n, unsigned) {
  *p = calloc(n, 1);
  return 0;
}
int hipHostFree(void* p) {
  free(p);
  return 0;
}
int hipMalloc(void** p, size_t n) {
  *p = calloc(n, 1);
  return 0;
}
int hipFree(void* p) {
  free(p);
  return 0;
}
int hipHostGetDevicePointer(void** d, void* h, unsigned) {
  *d = h;
  return 0;
}
int hipGetSymbolAddress(void** p, const void*) {
  static char scratch[256];
  *p = scratch;
  return 0;
}
int hipMemcpy(void* d, const void* s, size_t n, int) {
  memcpy(d, s, n);
  return 0;
}
const char* hipGetErrorString(int) { return "stub"; }
}
