// A HIP runtime on host memory, for tests of the library's host side without a
// GPU: one device of 256 CUs with 160 KB of LDS, allocations from calloc,
// copies done at once, events always past.  Kernels do not run; their launches
// are logged.  Loaded with global symbols before the library, it answers the
// library's HIP calls.
#include <hip/hip_runtime.h>

#include <atomic>
#include <cstdlib>
#include <cstring>
#include <map>
#include <mutex>
#include <string>
#include <vector>

namespace {

struct Launch {
  char name[96];
  unsigned grid, block;
  unsigned long long lds;
  void* stream;
};

struct Config {
  dim3 grid, block;
  size_t lds;
  hipStream_t stream;
};

std::mutex mu;
std::map<const void*, std::string> names;
std::vector<Launch> launches;
std::atomic<long> fail_at{-1};  // this launch and those after it fail
std::atomic<uintptr_t> handles{0x1000};
std::map<void*, size_t> pinned;     // live pinned allocations
std::atomic<size_t> pinned_made{0};  // bytes of all so far
std::atomic<long> streams{0};        // live
thread_local std::vector<Config> configs;
thread_local hipError_t last_error = hipSuccess;

template <class T>
hipError_t handle(T* out) {
  *out = reinterpret_cast<T>(handles.fetch_add(16));
  return hipSuccess;
}

hipError_t memory(void** p, size_t n) {
  *p = std::calloc(1, n ? n : 1);
  return *p ? hipSuccess : hipErrorOutOfMemory;
}

}  // namespace

extern "C" {

// The log since the last call with clear set: at most max entries, the number of all.
size_t host_hip_launches(Launch* out, size_t max, int clear) {
  std::lock_guard<std::mutex> lk(mu);
  const size_t n = launches.size();
  for (size_t i = 0; i < n && i < max; ++i) out[i] = launches[i];
  if (clear) launches.clear();
  return n;
}
// Pinned bytes made so far and live now, live streams.
void host_hip_pinned(size_t* made, size_t* live, long* live_streams) {
  std::lock_guard<std::mutex> lk(mu);
  *made = pinned_made;
  *live = 0;
  for (auto& p : pinned) *live += p.second;
  *live_streams = streams;
}
// Launches fail from the k-th logged one on (-1: never).
void host_hip_fail_at(long k) { fail_at = k; }

void** __hipRegisterFatBinary(const void*) {
  static void* module;
  return &module;
}
void __hipUnregisterFatBinary(void**) {}
void __hipRegisterFunction(void**, const void* host, char*, const char* device, unsigned, uint3*,
                           uint3*, dim3*, dim3*, int*) {
  std::lock_guard<std::mutex> lk(mu);
  names[host] = device;
}
void __hipRegisterVar(void**, void*, char*, char*, int, size_t, int, int) {}
hipError_t __hipPushCallConfiguration(dim3 grid, dim3 block, size_t lds, hipStream_t stream) {
  configs.push_back({grid, block, lds, stream});
  return hipSuccess;
}
hipError_t __hipPopCallConfiguration(dim3* grid, dim3* block, size_t* lds, hipStream_t* stream) {
  *grid = configs.back().grid;
  *block = configs.back().block;
  *lds = configs.back().lds;
  *stream = configs.back().stream;
  configs.pop_back();
  return hipSuccess;
}
hipError_t hipLaunchKernel(const void* f, dim3 grid, dim3 block, void**, size_t lds,
                           hipStream_t stream) {
  std::lock_guard<std::mutex> lk(mu);
  if (fail_at >= 0 && (long)launches.size() >= fail_at)
    return last_error = hipErrorLaunchFailure;
  Launch l{};
  std::strncpy(l.name, names[f].c_str(), sizeof(l.name) - 1);
  l.grid = grid.x;
  l.block = block.x;
  l.lds = lds;
  l.stream = stream;
  launches.push_back(l);
  return hipSuccess;
}

hipError_t hipGetDevice(int* d) {
  *d = 0;
  return hipSuccess;
}
hipError_t hipSetDevice(int d) { return d == 0 ? hipSuccess : hipErrorInvalidDevice; }
hipError_t hipGetDevicePropertiesR0600(hipDeviceProp_tR0600* p, int) {
  std::memset(p, 0, sizeof(*p));
  p->multiProcessorCount = 256;
  p->sharedMemPerBlock = 160 * 1024;
  return hipSuccess;
}
hipError_t hipGetSymbolAddress(void** p, const void*) { return memory(p, 4096); }
hipError_t hipGetLastError() {
  const hipError_t e = last_error;
  last_error = hipSuccess;
  return e;
}
const char* hipGetErrorString(hipError_t) { return "host runtime error"; }
hipError_t hipDeviceSynchronize() { return hipSuccess; }

hipError_t hipMalloc(void** p, size_t n) { return memory(p, n); }
hipError_t hipHostMalloc(void** p, size_t n, unsigned) {
  const hipError_t e = memory(p, n);
  std::lock_guard<std::mutex> lk(mu);
  if (e == hipSuccess) pinned[*p] = n, pinned_made += n;
  return e;
}
hipError_t hipFree(void* p) {
  std::free(p);
  return hipSuccess;
}
hipError_t hipHostFree(void* p) {
  std::lock_guard<std::mutex> lk(mu);
  pinned.erase(p);
  std::free(p);
  return hipSuccess;
}
hipError_t hipMemGetInfo(size_t* f, size_t* t) {
  *f = *t = 8ull << 30;
  return hipSuccess;
}
hipError_t hipMemcpy(void* d, const void* s, size_t n, hipMemcpyKind) {
  std::memcpy(d, s, n);
  return hipSuccess;
}
hipError_t hipMemcpyAsync(void* d, const void* s, size_t n, hipMemcpyKind, hipStream_t) {
  std::memcpy(d, s, n);
  return hipSuccess;
}
hipError_t hipMemset(void* d, int v, size_t n) {
  std::memset(d, v, n);
  return hipSuccess;
}
hipError_t hipMemsetAsync(void* d, int v, size_t n, hipStream_t) { return hipMemset(d, v, n); }

hipError_t hipStreamCreateWithFlags(hipStream_t* s, unsigned) {
  ++streams;
  return handle(s);
}
hipError_t hipStreamDestroy(hipStream_t) {
  --streams;
  return hipSuccess;
}
hipError_t hipStreamSynchronize(hipStream_t) { return hipSuccess; }
hipError_t hipEventCreate(hipEvent_t* e) { return handle(e); }
hipError_t hipEventCreateWithFlags(hipEvent_t* e, unsigned) { return handle(e); }
hipError_t hipEventDestroy(hipEvent_t) { return hipSuccess; }
hipError_t hipEventQuery(hipEvent_t) { return hipSuccess; }
hipError_t hipEventRecord(hipEvent_t, hipStream_t) { return hipSuccess; }
hipError_t hipEventSynchronize(hipEvent_t) { return hipSuccess; }
hipError_t hipEventElapsedTime(float* ms, hipEvent_t, hipEvent_t) {
  *ms = 1.0f;
  return hipSuccess;
}

}  // extern "C"
