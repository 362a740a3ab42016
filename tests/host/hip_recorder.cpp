// A stand-in for the HIP runtime that launches nothing and writes down what it is asked: loaded in front of the library
// (RTLD_GLOBAL), it shows on a machine without a GPU which kernels a call submits, on which streams, behind which events.
#include <hip/hip_runtime_api.h>
#include <chrono>
#include <cstdio>
#include <map>
#include <mutex>
#include <string>
#include <thread>

static std::mutex mu;
static std::map<const void*, std::string> names;
static std::string text;
static long next_handle = 0x1000;
static int pause_us = 0;
struct Config { dim3 grid, block; size_t lds; hipStream_t st; };
static thread_local Config config;
static thread_local int caller = 0;

// One line per call: thread, what, stream, event, kernel, workgroups.
static void note(char what, const void* st, const void* ev, const void* kernel = nullptr, dim3 grid = dim3(0)) {
  {
    std::lock_guard<std::mutex> lock(mu);
    char line[160];
    std::snprintf(line, sizeof line, "%d %c %lx %lx %u ", caller, what, (long)st, (long)ev, grid.x * grid.y);
    text += line;
    text += kernel ? names[kernel] : "-";
    text += '\n';
  }
  if (pause_us) std::this_thread::sleep_for(std::chrono::microseconds(pause_us));
}
template <typename T>
static hipError_t make(T* out) {
  std::lock_guard<std::mutex> lock(mu);
  *out = reinterpret_cast<T>(next_handle += 0x10);
  return hipSuccess;
}

extern "C" {
// ---- for the test
void record_start(int pause) {
  std::lock_guard<std::mutex> lock(mu);
  text.clear();
  pause_us = pause;
}
void record_thread(int id) { caller = id; }
const char* record_text() { return text.c_str(); }

// ---- the runtime
void** __hipRegisterFatBinary(const void*) {
  static void* handle;
  return &handle;
}
void __hipUnregisterFatBinary(void**) {}
void __hipRegisterFunction(void**, const void* host, char*, const char* device, unsigned, void*, void*, void*, void*, int*) { names[host] = device; }
void __hipRegisterVar(void**, void*, char*, char*, int, size_t, int, int) {}
hipError_t __hipPushCallConfiguration(dim3 grid, dim3 block, size_t lds, hipStream_t st) {
  config = {grid, block, lds, st};
  return hipSuccess;
}
hipError_t __hipPopCallConfiguration(dim3* grid, dim3* block, size_t* lds, hipStream_t* st) {
  *grid = config.grid;
  *block = config.block;
  *lds = config.lds;
  *st = config.st;
  return hipSuccess;
}
hipError_t hipLaunchKernel(const void* f, dim3 grid, dim3, void**, size_t, hipStream_t st) {
  note('L', st, nullptr, f, grid);
  return hipSuccess;
}
hipError_t hipExtLaunchKernel(const void* f, dim3 grid, dim3, void**, size_t, hipStream_t st, hipEvent_t, hipEvent_t stop, int) {
  note('L', st, stop, f, grid);
  return hipSuccess;
}
hipError_t hipEventCreate(hipEvent_t* e) { return make(e); }
hipError_t hipEventCreateWithFlags(hipEvent_t* e, unsigned) {
  note('E', nullptr, nullptr);
  return make(e);
}
hipError_t hipEventDestroy(hipEvent_t) { return hipSuccess; }
hipError_t hipEventElapsedTime(float* ms, hipEvent_t, hipEvent_t) {
  *ms = 0;
  return hipSuccess;
}
hipError_t hipEventRecord(hipEvent_t e, hipStream_t st) {
  note('R', st, e);
  return hipSuccess;
}
hipError_t hipEventSynchronize(hipEvent_t) { return hipSuccess; }
hipError_t hipStreamCreateWithFlags(hipStream_t* st, unsigned) {
  note('S', nullptr, nullptr);
  return make(st);
}
hipError_t hipStreamWaitEvent(hipStream_t st, hipEvent_t e, unsigned) {
  note('W', st, e);
  return hipSuccess;
}
hipError_t hipFuncSetAttribute(const void*, hipFuncAttribute, int) { return hipSuccess; }
hipError_t hipGetDevice(int* d) {
  *d = 0;
  return hipSuccess;
}
hipError_t hipSetDevice(int) { return hipSuccess; }
hipError_t hipDeviceGetAttribute(int* v, hipDeviceAttribute_t, int) {
  *v = 100000;  // (only the wall clock's rate is asked for)
  return hipSuccess;
}
const char* hipGetErrorName(hipError_t) { return "error"; }
hipError_t hipGetLastError() { return hipSuccess; }
hipError_t hipGetSymbolAddress(void** p, const void*) {
  *p = nullptr;
  return hipSuccess;
}
hipError_t hipPointerGetAttributes(hipPointerAttribute_t* a, const void*) {
  *a = hipPointerAttribute_t{};
  return hipSuccess;
}
}
