// A stand-in for the HIP runtime, for programs that link libkk.so without a GPU:
// the definitions here take the place of the runtime's.  Memory is host memory
// (zeroed), copies are memcpy, nothing runs.  Every kernel launch is recorded
// with its name, and refused if it asks for more than a gfx950 workgroup has
// (1024 threads, 160 KiB of LDS).
#pragma once
#include <hip/hip_runtime_api.h>

#include <cstdio>
#include <cstdlib>
#include <cstring>
#include <functional>
#include <map>
#include <string>
#include <vector>

struct Launch {
  std::string kernel;
  unsigned blocks, threads;
  size_t lds;
  void** args;  // valid during on_launch only
};
// filled before this program's own static objects are made
static std::map<const void*, std::string>& kernels() {
  static std::map<const void*, std::string> names;
  return names;
}
static std::vector<Launch> g_launches;
static std::function<double(const Launch&)> g_cost;  // ms that a launch is to take (0 without it)
static double g_clock = 0.0;

struct StubEvent {
  double at = 0.0;
};
static struct {
  dim3 grid, block;
  size_t lds;
  hipStream_t stream;
} g_config;

extern "C" {
void** __hipRegisterFatBinary(const void*) {
  static void* handle;
  return &handle;
}
void __hipRegisterFunction(void**, const void* host, char*, const char* name, unsigned, void*, void*, void*, void*,
                           int*) {
  kernels()[host] = name;
}
void __hipRegisterVar(void**, void*, char*, char*, int, size_t, int, int) {}
void __hipUnregisterFatBinary(void**) {}
hipError_t __hipPushCallConfiguration(dim3 grid, dim3 block, size_t lds, hipStream_t stream) {
  g_config = {grid, block, lds, stream};
  return hipSuccess;
}
hipError_t __hipPopCallConfiguration(dim3* grid, dim3* block, size_t* lds, hipStream_t* stream) {
  *grid = g_config.grid;
  *block = g_config.block;
  *lds = g_config.lds;
  *stream = g_config.stream;
  return hipSuccess;
}
static hipError_t g_last = hipSuccess;
hipError_t hipLaunchKernel(const void* f, dim3 grid, dim3 block, void** args, size_t lds, hipStream_t) {
  Launch l{kernels()[f], grid.x * grid.y * grid.z, block.x * block.y * block.z, lds, args};
  if (l.threads == 0 || l.threads > 1024 || l.lds > 160 * 1024 || l.blocks == 0) {
    printf("refused: %s, %u workgroups of %u threads, %zu bytes of LDS\n", l.kernel.c_str(), l.blocks, l.threads, lds);
    return g_last = hipErrorInvalidConfiguration;
  }
  if (g_cost) g_clock += g_cost(l);
  l.args = nullptr;
  g_launches.push_back(l);
  return hipSuccess;
}
hipError_t hipGetLastError() {
  const hipError_t e = g_last;
  g_last = hipSuccess;
  return e;
}
const char* hipGetErrorString(hipError_t e) { return e == hipSuccess ? "success" : "refused by the stand-in"; }
hipError_t hipMalloc(void** p, size_t n) { return (*p = calloc(n ? n : 1, 1)) ? hipSuccess : hipErrorOutOfMemory; }
hipError_t hipFree(void* p) {
  free(p);
  return hipSuccess;
}
hipError_t hipHostMalloc(void** p, size_t n, unsigned) { return hipMalloc(p, n); }
hipError_t hipHostFree(void* p) { return hipFree(p); }
hipError_t hipMemcpy(void* d, const void* s, size_t n, hipMemcpyKind) {
  memcpy(d, s, n);
  return hipSuccess;
}
hipError_t hipMemcpyAsync(void* d, const void* s, size_t n, hipMemcpyKind k, hipStream_t) { return hipMemcpy(d, s, n, k); }
hipError_t hipMemsetAsync(void* d, int v, size_t n, hipStream_t) {
  memset(d, v, n);
  return hipSuccess;
}
hipError_t hipMemGetInfo(size_t* avail, size_t* total) {
  *avail = *total = (size_t)288 << 30;
  return hipSuccess;
}
hipError_t hipGetDevice(int* d) {
  *d = 0;
  return hipSuccess;
}
hipError_t hipDeviceGetAttribute(int* v, hipDeviceAttribute_t, int) {
  *v = 256;
  return hipSuccess;
}
hipError_t hipGetSymbolAddress(void** p, const void*) { return hipMalloc(p, (size_t)16 << 20); }
hipError_t hipStreamCreateWithFlags(hipStream_t* s, unsigned) { return hipMalloc(reinterpret_cast<void**>(s), 1); }
hipError_t hipStreamDestroy(hipStream_t s) { return hipFree(s); }
hipError_t hipStreamSynchronize(hipStream_t) { return hipSuccess; }
hipError_t hipStreamWaitEvent(hipStream_t, hipEvent_t, unsigned) { return hipSuccess; }
hipError_t hipEventCreate(hipEvent_t* e) {
  *e = reinterpret_cast<hipEvent_t>(new StubEvent);
  return hipSuccess;
}
hipError_t hipEventCreateWithFlags(hipEvent_t* e, unsigned) { return hipEventCreate(e); }
hipError_t hipEventDestroy(hipEvent_t e) {
  delete reinterpret_cast<StubEvent*>(e);
  return hipSuccess;
}
hipError_t hipEventRecord(hipEvent_t e, hipStream_t) {
  reinterpret_cast<StubEvent*>(e)->at = g_clock;
  return hipSuccess;
}
hipError_t hipEventSynchronize(hipEvent_t) { return hipSuccess; }
hipError_t hipEventElapsedTime(float* ms, hipEvent_t a, hipEvent_t b) {
  *ms = (float)(reinterpret_cast<StubEvent*>(b)->at - reinterpret_cast<StubEvent*>(a)->at);
  return hipSuccess;
}
}

// launches recorded so far whose (mangled) kernel name holds `what`
static size_t launched(const char* what) {
  size_t n = 0;
  for (const Launch& l : g_launches) n += l.kernel.find(what) != std::string::npos;
  return n;
}
#define REQUIRE(x)                                              \
  do {                                                          \
    if (!(x)) {                                                 \
      printf("line %d: %s does not hold\n", __LINE__, #x);      \
      return 1;                                                 \
    }                                                           \
  } while (0)
