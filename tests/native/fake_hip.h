// A HIP runtime for checks of the library's host code on the CPU: the functions that libhipsso.so
// calls, defined in the program that links it, so that they take the place of the real ones.
// Device memory is zeroed host memory that knows its device and its size; copies and fills are done
// at once and checked against it; kernels do nothing but what the check's `kernel` says; a call
// may be made to fail.
#pragma once

#define __HIP_PLATFORM_AMD__ 1
#include <hip/hip_runtime_api.h>

#include <cstdio>
#include <cstdlib>
#include <cstring>
#include <functional>
#include <map>
#include <mutex>
#include <string>
#include <vector>

namespace fake {

struct Block {
  size_t bytes;
  int device;
};
struct Launch {
  std::string name;
  dim3 grid;
  void** args;
  hipStream_t stream;
  template <class T>
  T arg(int i) const {
    return *static_cast<T*>(args[i]);
  }
};

struct State {
  std::recursive_mutex mu;
  int device = 0;
  std::map<char*, Block> device_memory;
  std::map<const void*, std::string> names;        // kernels
  std::map<std::string, int> launches;             // since the check last cleared it
  std::function<void(const Launch&)> kernel;
  std::map<hipStream_t, int> streams;              // -> device
  std::map<int, size_t> limit;                     // device -> bytes it has, none: no limit
  std::function<hipError_t(const char*)> fail;     // called first by calls that may be refused
  int allocations[8] = {};                         // by device
  std::map<hipStream_t, bool> busy;                // launches since the host last waited
  std::map<hipEvent_t, hipStream_t> recorded;
  std::vector<int> waited;                         // devices of the streams waited for
  int faults = 0;                                  // accesses outside of device memory
  std::vector<char> symbol = std::vector<char>(32 << 20);
};
inline State& state() {
  static State s;
  return s;
}

inline int device_of(hipStream_t s) {
  auto& st = state();
  auto it = st.streams.find(s);
  return it == st.streams.end() ? st.device : it->second;
}
inline hipError_t refused(const char* what) {
  return state().fail ? state().fail(what) : hipSuccess;
}
// The block that holds [p, p + bytes), or null.
inline const Block* holds(const void* p, size_t bytes) {
  auto& mem = state().device_memory;
  char* c = static_cast<char*>(const_cast<void*>(p));
  auto it = mem.upper_bound(c);
  if (it == mem.begin()) return nullptr;
  --it;
  return c + bytes <= it->first + it->second.bytes ? &it->second : nullptr;
}
inline void fault(const char* what, const void* p) {
  std::printf("fault: %s at %p\n", what, p);
  ++state().faults;
}
// A device address that a kernel or copy on stream s may use.
inline bool valid(const void* p, size_t bytes, hipStream_t s, const char* what) {
  const Block* b = holds(p, bytes);
  if (!b || b->device != device_of(s)) {
    fault(b ? "memory of another device" : what, p);
    return false;
  }
  return true;
}

}  // namespace fake

extern "C" {

void** __hipRegisterFatBinary(const void*) {
  static void* module;
  return &module;
}
void __hipUnregisterFatBinary(void**) {}
void __hipRegisterFunction(void**, const void* host, char*, const char* name, unsigned, void*,
                           void*, void*, void*, int*) {
  fake::state().names[host] = name;
}
void __hipRegisterVar(void**, void*, char*, char*, int, size_t, int, int) {}

static thread_local struct {
  dim3 grid, block;
  size_t shared;
  hipStream_t stream;
} fake_call;
hipError_t __hipPushCallConfiguration(dim3 grid, dim3 block, size_t shared, hipStream_t stream) {
  fake_call = {grid, block, shared, stream};
  return hipSuccess;
}
hipError_t __hipPopCallConfiguration(dim3* grid, dim3* block, size_t* shared, hipStream_t* stream) {
  *grid = fake_call.grid;
  *block = fake_call.block;
  *shared = fake_call.shared;
  *stream = fake_call.stream;
  return hipSuccess;
}
hipError_t hipLaunchKernel(const void* f, dim3 grid, dim3, void** args, size_t, hipStream_t s) {
  auto& st = fake::state();
  std::lock_guard<std::recursive_mutex> lock(st.mu);
  const std::string& name = st.names[f];
  ++st.launches[name];
  st.busy[s] = true;
  if (st.kernel) st.kernel({name, grid, args, s});
  return hipSuccess;
}

hipError_t hipGetLastError() { return hipSuccess; }
hipError_t hipGetDevice(int* d) {
  *d = fake::state().device;
  return hipSuccess;
}
hipError_t hipSetDevice(int d) {
  fake::state().device = d;
  return hipSuccess;
}
hipError_t hipStreamCreateWithFlags(hipStream_t* s, unsigned) {
  auto& st = fake::state();
  std::lock_guard<std::recursive_mutex> lock(st.mu);
  *s = reinterpret_cast<hipStream_t>(std::malloc(1));
  st.streams[*s] = st.device;
  return hipSuccess;
}
hipError_t hipStreamDestroy(hipStream_t s) {
  auto& st = fake::state();
  std::lock_guard<std::recursive_mutex> lock(st.mu);
  st.streams.erase(s);
  std::free(s);
  return hipSuccess;
}
hipError_t hipStreamGetDevice(hipStream_t s, hipDevice_t* d) {
  *d = fake::device_of(s);
  return hipSuccess;
}
hipError_t hipStreamSynchronize(hipStream_t s) {
  auto& st = fake::state();
  std::lock_guard<std::recursive_mutex> lock(st.mu);
  st.busy[s] = false;
  st.waited.push_back(fake::device_of(s));
  return hipSuccess;
}
hipError_t hipStreamWaitEvent(hipStream_t, hipEvent_t, unsigned) { return hipSuccess; }

hipError_t hipEventCreateWithFlags(hipEvent_t* e, unsigned) {
  const hipError_t r = fake::refused("event");
  if (r == hipSuccess) *e = reinterpret_cast<hipEvent_t>(std::malloc(1));
  return r;
}
hipError_t hipEventCreate(hipEvent_t* e) { return hipEventCreateWithFlags(e, 0); }
hipError_t hipEventDestroy(hipEvent_t e) {
  std::free(e);
  return hipSuccess;
}
hipError_t hipEventRecord(hipEvent_t e, hipStream_t s) {
  auto& st = fake::state();
  std::lock_guard<std::recursive_mutex> lock(st.mu);
  const hipError_t r = fake::refused("record");
  if (r == hipSuccess) st.recorded[e] = s;
  return r;
}
hipError_t hipEventSynchronize(hipEvent_t e) {
  auto& st = fake::state();
  std::lock_guard<std::recursive_mutex> lock(st.mu);
  if (st.recorded.count(e)) st.busy[st.recorded[e]] = false;
  return hipSuccess;
}
hipError_t hipEventElapsedTime(float* ms, hipEvent_t, hipEvent_t) {
  *ms = 0.0f;
  return hipSuccess;
}

hipError_t hipHostMalloc(void** p, size_t bytes, unsigned) {
  const hipError_t r = fake::refused("host memory");
  if (r == hipSuccess) *p = std::calloc(1, bytes);
  return r;
}
hipError_t hipHostFree(void* p) {
  std::free(p);
  return hipSuccess;
}

hipError_t hipMemPoolCreate(hipMemPool_t* pool, const hipMemPoolProps* props) {
  *pool = reinterpret_cast<hipMemPool_t>((size_t)props->location.id + 1);
  return hipSuccess;
}
hipError_t hipMemPoolDestroy(hipMemPool_t) { return hipSuccess; }
hipError_t hipMemPoolSetAttribute(hipMemPool_t, hipMemPoolAttr, void*) { return hipSuccess; }
hipError_t hipMemPoolTrimTo(hipMemPool_t, size_t) { return hipSuccess; }
hipError_t hipMallocFromPoolAsync(void** p, size_t bytes, hipMemPool_t pool, hipStream_t) {
  auto& st = fake::state();
  std::lock_guard<std::recursive_mutex> lock(st.mu);
  const hipError_t r = fake::refused("device memory");
  if (r != hipSuccess) return r;
  const int device = (int)reinterpret_cast<size_t>(pool) - 1;
  size_t held = bytes;
  for (const auto& b : st.device_memory)
    if (b.second.device == device) held += b.second.bytes;
  if (st.limit.count(device) && held > st.limit[device]) return hipErrorOutOfMemory;
  *p = std::calloc(1, bytes);
  st.device_memory[static_cast<char*>(*p)] = {bytes, device};
  ++st.allocations[device];
  return hipSuccess;
}
hipError_t hipMemGetInfo(size_t* left, size_t* total) {
  auto& st = fake::state();
  std::lock_guard<std::recursive_mutex> lock(st.mu);
  size_t held = 0;
  for (const auto& b : st.device_memory)
    if (b.second.device == st.device) held += b.second.bytes;
  *total = st.limit.count(st.device) ? st.limit[st.device] : (size_t)288 << 30;
  *left = *total - held;
  return hipSuccess;
}
hipError_t hipMemPoolGetAttribute(hipMemPool_t, hipMemPoolAttr, void* v) {   // nothing idle is kept
  *static_cast<uint64_t*>(v) = 0;
  return hipSuccess;
}
hipError_t hipFreeAsync(void* p, hipStream_t) {
  auto& st = fake::state();
  std::lock_guard<std::recursive_mutex> lock(st.mu);
  if (!st.device_memory.erase(static_cast<char*>(p))) {
    fake::fault("free of what is not an allocation", p);
    return hipErrorInvalidValue;
  }
  std::free(p);
  return hipSuccess;
}
hipError_t hipMemsetAsync(void* p, int v, size_t bytes, hipStream_t s) {
  auto& st = fake::state();
  std::lock_guard<std::recursive_mutex> lock(st.mu);
  if (bytes == 0) return hipSuccess;
  if (!fake::valid(p, bytes, s, "fill")) return hipErrorInvalidValue;
  std::memset(p, v, bytes);
  return hipSuccess;
}
hipError_t hipMemcpyAsync(void* to, const void* from, size_t bytes, hipMemcpyKind kind,
                          hipStream_t s) {
  auto& st = fake::state();
  std::lock_guard<std::recursive_mutex> lock(st.mu);
  const hipError_t r = fake::refused("copy");
  if (r != hipSuccess) return r;
  if (bytes == 0) return hipSuccess;
  if (kind != hipMemcpyHostToDevice && !fake::valid(from, bytes, s, "copy from"))
    return hipErrorInvalidValue;
  if (kind != hipMemcpyDeviceToHost && !fake::valid(to, bytes, s, "copy to"))
    return hipErrorInvalidValue;
  std::memcpy(to, from, bytes);
  return hipSuccess;
}
hipError_t hipMemcpy2DAsync(void* to, size_t to_pitch, const void* from, size_t from_pitch,
                            size_t width, size_t height, hipMemcpyKind kind, hipStream_t s) {
  for (size_t i = 0; i < height; ++i) {
    const hipError_t r = hipMemcpyAsync(static_cast<char*>(to) + i * to_pitch,
                                        static_cast<const char*>(from) + i * from_pitch, width,
                                        kind, s);
    if (r != hipSuccess) return r;
  }
  return hipSuccess;
}
hipError_t hipGetSymbolAddress(void** p, const void*) {
  *p = fake::state().symbol.data();
  return hipSuccess;
}

}  // extern "C"
