// The HIP runtime calls that libd2moe makes, replaced by a log of what they
// would enqueue, so that a CPU test can see on which stream and after which
// event every copy and kernel goes.  Nothing is executed.  Loaded globally
// before the library, it takes the place of the runtime for it.
#include <hip/hip_runtime_api.h>

#include <map>
#include <string>

static std::string text;
static std::map<const void*, std::string> names;  // host stub -> device name
static uintptr_t pinned_from = 0, pinned_to = 0;  // the one pinned allocation

static void put(const char* op, const void* a, const void* b) {
  text += std::string(op) + " " + std::to_string((uintptr_t)a) + " " + std::to_string((uintptr_t)b) + "\n";
}

extern "C" {

const char* fake_log() { return text.c_str(); }
void fake_mark() { text += "mark 0 0\n"; }
void fake_pinned(uintptr_t from, uintptr_t to) { pinned_from = from, pinned_to = to; }

static struct { dim3 grid, block; size_t shared; hipStream_t stream; } config;
hipError_t __hipPushCallConfiguration(dim3 grid, dim3 block, size_t shared, hipStream_t s) {
  config = {grid, block, shared, s};
  return hipSuccess;
}
hipError_t __hipPopCallConfiguration(dim3* grid, dim3* block, size_t* shared, hipStream_t* s) {
  *grid = config.grid, *block = config.block, *shared = config.shared, *s = config.stream;
  return hipSuccess;
}
void** __hipRegisterFatBinary(const void*) {
  static void* module;
  return &module;
}
void __hipUnregisterFatBinary(void**) {}
void __hipRegisterFunction(void**, const void* host, char*, const char* name, unsigned, void*, void*,
                           dim3*, dim3*, int*) {
  names[host] = name;
}
void __hipRegisterVar(void**, void*, char*, char*, int, size_t, int, int) {}

hipError_t hipLaunchKernel(const void* f, dim3, dim3, void**, size_t, hipStream_t s) {
  put(("launch:" + names[f]).c_str(), s, nullptr);
  return hipSuccess;
}
hipError_t hipExtLaunchKernel(const void* f, dim3, dim3, void**, size_t, hipStream_t s, hipEvent_t,
                              hipEvent_t, int) {
  put(("launch:" + names[f]).c_str(), s, nullptr);
  return hipSuccess;
}
hipError_t hipMemcpyAsync(void*, const void*, size_t, hipMemcpyKind, hipStream_t s) {
  put("copy", s, nullptr);
  return hipSuccess;
}
hipError_t hipMemcpy2DAsync(void*, size_t, const void*, size_t, size_t, size_t, hipMemcpyKind,
                            hipStream_t s) {
  put("copy", s, nullptr);
  return hipSuccess;
}
hipError_t hipEventRecord(hipEvent_t e, hipStream_t s) {
  put("record", s, e);
  return hipSuccess;
}
hipError_t hipStreamWaitEvent(hipStream_t s, hipEvent_t e, unsigned) {
  put("wait", s, e);
  return hipSuccess;
}
hipError_t hipStreamCreateWithFlags(hipStream_t* s, unsigned) {
  static uintptr_t next = 50;
  *s = (hipStream_t)next++;
  return hipSuccess;
}
hipError_t hipEventCreateWithFlags(hipEvent_t* e, unsigned) {
  static uintptr_t next = 500;
  *e = (hipEvent_t)next++;
  return hipSuccess;
}
hipError_t hipGetLastError() { return hipSuccess; }
hipError_t hipGetDevice(int* d) {
  *d = 0;
  return hipSuccess;
}
hipError_t hipPointerGetAttributes(hipPointerAttribute_t* at, const void* p) {
  const uintptr_t u = (uintptr_t)p;
  *at = {};
  if (u < pinned_from || u >= pinned_to) return hipErrorInvalidValue;
  at->type = hipMemoryTypeHost;
  at->devicePointer = at->hostPointer = (void*)p;
  return hipSuccess;
}
hipError_t hipMemGetAddressRange(hipDeviceptr_t* base, size_t* size, hipDeviceptr_t p) {
  const uintptr_t u = (uintptr_t)p;
  if (u < pinned_from || u >= pinned_to) return hipErrorNotFound;
  *base = (hipDeviceptr_t)pinned_from, *size = pinned_to - pinned_from;
  return hipSuccess;
}
}
