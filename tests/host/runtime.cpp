#include "runtime.h"

#include <cstdlib>
#include <cstring>
#include <functional>
#include <map>

#include "../../paper_1608_00139_amd/csrc/common.h"
#include "../../paper_1608_00139_amd/csrc/eps_solve.h"

namespace fake {
size_t limit = ~(size_t)0, live = 0;
std::vector<Emit> emits;
std::vector<std::string> launches;
template <class T>
struct Plain {  // memory that the refused allocations of the tests do not reach
  typedef T value_type;
  Plain() = default;
  template <class U>
  Plain(const Plain<U>&) {}
  T* allocate(size_t n) { return (T*)std::malloc(n * sizeof(T)); }
  void deallocate(T* p, size_t) { std::free(p); }
  template <class U>
  bool operator==(const Plain<U>&) const { return true; }
  template <class U>
  bool operator!=(const Plain<U>&) const { return false; }
};
static std::map<void*, size_t, std::less<void*>, Plain<std::pair<void* const, size_t>>> blocks;
}  // namespace fake

extern "C" {
hipError_t hipMalloc(void** p, size_t bytes) {
  if (bytes > fake::limit || fake::live > fake::limit - bytes) return hipErrorOutOfMemory;
  *p = std::calloc(1, bytes);  // (untouched pages stay unbacked)
  fake::blocks[*p] = bytes;
  fake::live += bytes;
  return hipSuccess;
}
hipError_t hipFree(void* p) {
  const auto it = fake::blocks.find(p);
  if (it == fake::blocks.end()) std::abort();
  fake::live -= it->second;
  fake::blocks.erase(it);
  std::free(p);
  return hipSuccess;
}
hipError_t hipHostMalloc(void** p, size_t bytes, unsigned) {
  *p = std::calloc(1, bytes);
  return hipSuccess;
}
hipError_t hipHostFree(void* p) {
  std::free(p);
  return hipSuccess;
}
hipError_t hipHostGetDevicePointer(void** d, void* h, unsigned) {
  *d = h;
  return hipSuccess;
}
hipError_t hipSetDevice(int) { return hipSuccess; }
hipError_t hipGetDeviceCount(int* n) {
  *n = 1;
  return hipSuccess;
}
hipError_t hipGetDevicePropertiesR0600(hipDeviceProp_t*, int) { return hipErrorInvalidValue; }
hipError_t hipMemset(void* p, int v, size_t bytes) {
  std::memset(p, v, bytes);
  return hipSuccess;
}
hipError_t hipMemsetAsync(void* p, int v, size_t bytes, hipStream_t) { return hipMemset(p, v, bytes); }
hipError_t hipMemcpyAsync(void* d, const void* s, size_t bytes, hipMemcpyKind, hipStream_t) {
  std::memcpy(d, s, bytes);
  return hipSuccess;
}
hipError_t hipStreamSynchronize(hipStream_t) { return hipSuccess; }
hipError_t hipStreamQuery(hipStream_t) { return hipSuccess; }
hipError_t hipDeviceSynchronize() { return hipSuccess; }
hipError_t hipEventCreate(hipEvent_t* e) {
  *e = (hipEvent_t)1;
  return hipSuccess;
}
hipError_t hipEventCreateWithFlags(hipEvent_t* e, unsigned) { return hipEventCreate(e); }
hipError_t hipEventDestroy(hipEvent_t) { return hipSuccess; }
hipError_t hipEventRecord(hipEvent_t, hipStream_t) { return hipSuccess; }
hipError_t hipEventQuery(hipEvent_t) { return hipSuccess; }
hipError_t hipEventSynchronize(hipEvent_t) { return hipSuccess; }
hipError_t hipEventElapsedTime(float* ms, hipEvent_t, hipEvent_t) {
  *ms = 1.f;
  return hipSuccess;
}
hipError_t hipGetLastError() { return hipSuccess; }
const char* hipGetErrorString(hipError_t) { return "error"; }
}

namespace dl {
static hipError_t noted(const char* name) {
  fake::launches.push_back(name);
  return hipSuccess;
}
hipError_t bool_kernels_init() { return hipSuccess; }
hipError_t eps_kernels_init() { return hipSuccess; }
hipError_t sg_lists_init() { return hipSuccess; }
void eps_release(EpsWorkspace*) {}
int64_t padded_size_for(int, int64_t n) { return (n + 255) / 256 * 256; }
int choose_nt_config(int, int64_t) { return 2; }
TileCfg nt_config(int, int) { return TileCfg{64, 64, 128, 256, 0}; }
hipError_t launch_ring_clear(unsigned long long*, int*, int, int, int, hipStream_t) { return noted("ring_clear"); }
hipError_t launch_ingest(int, const uint8_t*, int64_t, int, int, int8_t*, int8_t*, void*, void*, int,
                         unsigned long long*, hipStream_t) {
  return noted("ingest");
}
hipError_t launch_bytes_op(const int8_t*, const int8_t*, int, int, int, int, int8_t*, int8_t*, unsigned long long*,
                           hipStream_t, const StepGate&) {
  return noted("bytes_op");
}
hipError_t launch_layer_lists(const LayerLists& q, const int8_t*, hipStream_t) {
  *q.status_out = 2u;  // the series has repeated at step 2
  return noted("layer_lists");
}
hipError_t launch_hash_bool(uint8_t*, int64_t, int, int, unsigned, hipStream_t) { return noted("hash_bool"); }
hipError_t launch_group_step(int, const GroupDesc*, int, int, hipStream_t, const int*) { return noted("group_step"); }
hipError_t launch_emit(int, const void*, int Np, int, int n, uint8_t*, int64_t ldr, hipStream_t) {
  fake::emits.push_back({Np, n, ldr});
  return noted("emit");
}
hipError_t launch_emit_sum(const void*, int Np, int n, uint8_t*, int64_t ldr, unsigned long long*,
                           unsigned long long* sum, hipStream_t) {
  fake::emits.push_back({Np, n, ldr});
  *sum = 77;
  return noted("emit_sum");
}
}  // namespace dl
