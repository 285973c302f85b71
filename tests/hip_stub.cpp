// A HIP runtime without a GPU, for tests of the library's host code on the CPU: memory with a
// limit, copies on the host, launches that are recorded and not run.  Loaded with global symbols
// before the library, it takes the place of the runtime's own functions.
#define __HIP_PLATFORM_AMD__ 1
#include <hip/hip_runtime_api.h>
#include <sys/mman.h>

#include <cstring>
#include <map>
#include <vector>

namespace {
std::map<char*, size_t> blocks;
size_t live = 0, limit = (size_t)1 << 40;
hipError_t last = hipSuccess;
int device_of_pointers = 0;
long device_syncs = 0;
std::vector<char> table;  // what the last plain copy carried
std::vector<const void*> launched;       // functions
std::vector<unsigned long long> firsts;  // first 8 bytes of their arguments
dim3 grid, block;
size_t shared;
hipStream_t stream;

hipError_t result(hipError_t e) {
  if (e != hipSuccess) last = e;
  return e;
}
const std::pair<char* const, size_t>* block_of(const void* p) {
  auto it = blocks.upper_bound((char*)p);
  if (it == blocks.begin()) return nullptr;
  --it;
  return (const char*)p < it->first + it->second ? &*it : nullptr;
}
}  // namespace

extern "C" {

// ---- for the tests
void stub_limit(size_t bytes) { limit = bytes; }
size_t stub_live() { return live; }
void stub_pointers_on(int device) { device_of_pointers = device; }
long stub_device_syncs() { return device_syncs; }
size_t stub_table_bytes() { return table.size(); }
const void* stub_table() { return table.data(); }
void stub_forget_launches() { launched.clear(), firsts.clear(); }
size_t stub_launches() { return launched.size(); }
const void* stub_launched(size_t i) { return launched[i]; }
unsigned long long stub_first(size_t i) { return firsts[i]; }

// ---- the runtime
hipError_t hipMalloc(void** p, size_t n) {
  *p = nullptr;
  if (live + n > limit) return result(hipErrorOutOfMemory);
  void* m = mmap(nullptr, n, PROT_READ | PROT_WRITE, MAP_PRIVATE | MAP_ANONYMOUS | MAP_NORESERVE, -1, 0);
  if (m == MAP_FAILED) return result(hipErrorOutOfMemory);
  blocks[(char*)m] = n;
  live += n;
  *p = m;
  return hipSuccess;
}
hipError_t hipFree(void* p) {
  if (!p) return hipSuccess;
  auto it = blocks.find((char*)p);
  if (it == blocks.end()) return result(hipErrorInvalidValue);
  live -= it->second;
  munmap(p, it->second);
  blocks.erase(it);
  return hipSuccess;
}
hipError_t hipMemcpy(void* d, const void* s, size_t n, hipMemcpyKind) {
  table.assign((const char*)s, (const char*)s + n);
  std::memcpy(d, s, n);
  return hipSuccess;
}
hipError_t hipMemcpyAsync(void* d, const void* s, size_t n, hipMemcpyKind, hipStream_t) {
  std::memcpy(d, s, n);
  return hipSuccess;
}
hipError_t hipMemcpy2DAsync(void* d, size_t dp, const void* s, size_t sp, size_t w, size_t h, hipMemcpyKind k, hipStream_t) {
  if (k == hipMemcpyDeviceToDevice && !block_of(s)) return result(hipErrorInvalidValue);
  for (size_t y = 0; y < h; ++y) std::memcpy((char*)d + y * dp, (const char*)s + y * sp, w);
  return hipSuccess;
}
hipError_t hipMemset(void* d, int v, size_t n) { return std::memset(d, v, n), hipSuccess; }
hipError_t hipMemsetAsync(void* d, int v, size_t n, hipStream_t) { return std::memset(d, v, n), hipSuccess; }
hipError_t hipPointerGetAttributes(hipPointerAttribute_t* a, const void* p) {
  std::memset(a, 0, sizeof *a);
  a->type = block_of(p) ? hipMemoryTypeDevice : hipMemoryTypeUnregistered;
  a->device = block_of(p) ? device_of_pointers : 0;
  return hipSuccess;
}
hipError_t hipMemGetAddressRange(hipDeviceptr_t* base, size_t* size, hipDeviceptr_t p) {
  const auto* b = block_of(p);
  if (!b) return result(hipErrorNotFound);
  *base = b->first;
  *size = b->second;
  return hipSuccess;
}
hipError_t hipGetLastError() {
  const hipError_t e = last;
  last = hipSuccess;
  return e;
}
const char* hipGetErrorString(hipError_t) { return "error"; }
hipError_t hipGetDeviceCount(int* n) { return *n = 1, hipSuccess; }
hipError_t hipGetDevice(int* d) { return *d = 0, hipSuccess; }
hipError_t hipSetDevice(int) { return hipSuccess; }
hipError_t hipDeviceSynchronize() { return ++device_syncs, hipSuccess; }
hipError_t hipDeviceGetAttribute(int* v, hipDeviceAttribute_t, int) { return *v = 160 * 1024, hipSuccess; }
hipError_t hipGetDeviceProperties(hipDeviceProp_t* p, int) {  // R0600 in the headers
  std::memset(p, 0, sizeof *p);
  p->multiProcessorCount = 256;
  return hipSuccess;
}
hipError_t hipFuncGetAttributes(hipFuncAttributes*, const void*) { return hipSuccess; }
hipError_t hipFuncSetAttribute(const void*, hipFuncAttribute, int) { return hipSuccess; }
hipError_t hipGetSymbolAddress(void** p, const void*) { return *p = nullptr, hipSuccess; }
hipError_t hipStreamSynchronize(hipStream_t) { return hipSuccess; }
hipError_t hipStreamCreateWithFlags(hipStream_t* s, unsigned) { return *s = (hipStream_t)1, hipSuccess; }
hipError_t hipStreamDestroy(hipStream_t) { return hipSuccess; }
hipError_t hipStreamBeginCapture(hipStream_t, hipStreamCaptureMode) { return hipSuccess; }
hipError_t hipStreamEndCapture(hipStream_t, hipGraph_t* g) { return *g = (hipGraph_t)1, hipSuccess; }
hipError_t hipGraphInstantiate(hipGraphExec_t* e, hipGraph_t, hipGraphNode_t*, char*, size_t) {
  return *e = (hipGraphExec_t)1, hipSuccess;
}
hipError_t hipGraphLaunch(hipGraphExec_t, hipStream_t) { return hipSuccess; }
hipError_t hipGraphExecDestroy(hipGraphExec_t) { return hipSuccess; }
hipError_t hipGraphDestroy(hipGraph_t) { return hipSuccess; }
hipError_t hipEventCreate(hipEvent_t* e) { return *e = (hipEvent_t)1, hipSuccess; }
hipError_t hipEventDestroy(hipEvent_t) { return hipSuccess; }
hipError_t hipEventRecord(hipEvent_t, hipStream_t) { return hipSuccess; }
hipError_t hipEventSynchronize(hipEvent_t) { return hipSuccess; }
hipError_t hipEventElapsedTime(float* ms, hipEvent_t, hipEvent_t) { return *ms = 1.0f, hipSuccess; }
hipError_t hipLaunchKernel(const void* f, dim3, dim3, void** args, size_t, hipStream_t) {
  launched.push_back(f);
  unsigned long long first = 0;
  std::memcpy(&first, args[0], 8);
  firsts.push_back(first);
  return hipSuccess;
}
hipError_t __hipPushCallConfiguration(dim3 g, dim3 b, size_t s, hipStream_t st) {
  grid = g, block = b, shared = s, stream = st;
  return hipSuccess;
}
hipError_t __hipPopCallConfiguration(dim3* g, dim3* b, size_t* s, hipStream_t* st) {
  *g = grid, *b = block, *s = shared, *st = stream;
  return hipSuccess;
}
void** __hipRegisterFatBinary(const void*) {
  static void* handle;
  return &handle;
}
void __hipUnregisterFatBinary(void**) {}
void __hipRegisterFunction(void**, const void*, char*, const char*, unsigned, void*, void*, void*, void*, int*) {}
void __hipRegisterVar(void**, void*, char*, char*, int, size_t, int, int) {}

}  // extern "C"
