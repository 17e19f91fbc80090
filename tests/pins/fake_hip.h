// A stand-in for the HIP runtime: every call the library makes is written down, nothing runs.  An executable that includes
// this file and links libptchunk.so has the library call these functions instead of the runtime's, so that what is
// launched, on which stream and behind which event can be looked at without a GPU.  Memory is ordinary host memory.
#pragma once
#include <cxxabi.h>
#include <hip/hip_runtime_api.h>

#include <cstdint>
#include <cstdio>
#include <cstdlib>
#include <cstring>
#include <map>
#include <string>
#include <vector>

namespace fake {

struct Op {
  std::string what;          // "launch", "record", "wait", "copy", "sync stream", "sync event", "sync device", "destroy stream"
  std::string kernel;        // launch: name without namespace and template arguments
  uintptr_t stream = 0, event = 0;
  dim3 grid{0, 0, 0}, block{0, 0, 0};
  size_t lds = 0;
};

inline std::vector<Op> ops;
// filled by the library's constructors, before this executable's own
inline std::map<const void*, std::string>& kernels() { static auto* m = new std::map<const void*, std::string>; return *m; }
inline std::map<uintptr_t, std::pair<size_t, hipMemoryType>> memory;
inline std::map<uintptr_t, bool> capturing;       // streams under capture
inline uintptr_t next_handle = 0x1000;
inline std::string fail_kernel;                   // launches of this kernel fail once `fail_after` of them have passed
inline int fail_after = -1;
inline hipError_t last = hipSuccess;
inline int device = 0;

inline void note(const char* what, hipStream_t s = nullptr, hipEvent_t e = nullptr) {
  Op o;
  o.what = what; o.stream = (uintptr_t)s; o.event = (uintptr_t)e;
  ops.push_back(o);
}
inline hipError_t alloc(void** p, size_t n, hipMemoryType t) {
  const size_t size = n ? (n + 4095) / 4096 * 4096 : 4096;
  *p = aligned_alloc(4096, size);
  memset(*p, 0, size);
  memory[(uintptr_t)*p] = {n, t};
  return hipSuccess;
}
inline const std::pair<const uintptr_t, std::pair<size_t, hipMemoryType>>* find(const void* p) {
  auto it = memory.upper_bound((uintptr_t)p);
  if (it == memory.begin()) return nullptr;
  --it;
  return (uintptr_t)p < it->first + it->second.first ? &*it : nullptr;
}
// the operations since `from`, as text
inline std::string text(size_t from = 0) {
  std::string s;
  for (size_t i = from; i < ops.size(); ++i) {
    char b[256];
    const Op& o = ops[i];
    snprintf(b, sizeof b, "  %s %s stream %zx event %zx grid %u,%u block %u lds %zu\n", o.what.c_str(), o.kernel.c_str(), (size_t)o.stream,
             (size_t)o.event, o.grid.x, o.grid.y, o.block.x, o.lds);
    s += b;
  }
  return s;
}
inline std::vector<Op> launches(const char* kernel, size_t from = 0) {
  std::vector<Op> v;
  for (size_t i = from; i < ops.size(); ++i)
    if (ops[i].what == "launch" && ops[i].kernel == kernel) v.push_back(ops[i]);
  return v;
}
inline hipStream_t stream(uintptr_t id) { return (hipStream_t)id; }
inline void (*on_launch)(const Op&, void** args) = nullptr;      // looks at a launch's arguments

struct Call { dim3 grid, block; size_t lds; hipStream_t stream; };
inline std::vector<Call> calls;

}  // namespace fake

extern "C" {
void** __hipRegisterFatBinary(const void*) { static void* h; return &h; }
void __hipUnregisterFatBinary(void**) {}
void __hipRegisterFunction(void**, const void* host, char*, const char* name, unsigned, void*, void*, dim3*, dim3*, int*) {
  int st = 0;
  char* d = abi::__cxa_demangle(name, nullptr, nullptr, &st);
  std::string s = st == 0 && d ? d : name;
  free(d);
  const size_t at = s.find("k_");
  s = at == std::string::npos ? s : s.substr(at);
  fake::kernels()[host] = s.substr(0, s.find_first_of("<("));
}
void __hipRegisterVar(void**, void*, char*, const char*, int, size_t, int, int) {}
hipError_t __hipPushCallConfiguration(dim3 g, dim3 b, size_t lds, hipStream_t s) { fake::calls.push_back({g, b, lds, s}); return hipSuccess; }
hipError_t __hipPopCallConfiguration(dim3* g, dim3* b, size_t* lds, hipStream_t* s) {
  const fake::Call c = fake::calls.back();
  fake::calls.pop_back();
  *g = c.grid; *b = c.block; *lds = c.lds; *s = c.stream;
  return hipSuccess;
}
hipError_t hipLaunchKernel(const void* f, dim3 g, dim3 b, void** args, size_t lds, hipStream_t s) {
  fake::Op o;
  o.what = "launch"; o.kernel = fake::kernels()[f]; o.stream = (uintptr_t)s; o.grid = g; o.block = b; o.lds = lds;
  if (o.kernel == fake::fail_kernel && fake::fail_after >= 0 && fake::fail_after-- == 0) { fake::fail_after = 0; return fake::last = hipErrorLaunchFailure; }
  fake::ops.push_back(o);
  if (fake::on_launch) fake::on_launch(o, args);
  return hipSuccess;
}
hipError_t hipGetLastError(void) { const hipError_t e = fake::last; fake::last = hipSuccess; return e; }
const char* hipGetErrorString(hipError_t) { return "fake error"; }
hipError_t hipGetDevice(int* d) { *d = fake::device; return hipSuccess; }
hipError_t hipDeviceSynchronize(void) { fake::note("sync device"); return hipSuccess; }
hipError_t hipGetSymbolAddress(void** p, const void*) {
  static std::map<int, void*> mem;
  if (!mem[fake::device]) mem[fake::device] = calloc(1, 8 << 20);
  *p = mem[fake::device];
  return hipSuccess;
}
hipError_t hipMalloc(void** p, size_t n) { return fake::alloc(p, n, hipMemoryTypeDevice); }
hipError_t hipFree(void* p) { fake::memory.erase((uintptr_t)p); free(p); return hipSuccess; }
hipError_t hipHostMalloc(void** p, size_t n, unsigned) { return fake::alloc(p, n, hipMemoryTypeHost); }
hipError_t hipHostFree(void* p) { return hipFree(p); }
hipError_t hipHostGetDevicePointer(void** d, void* h, unsigned) { *d = h; return hipSuccess; }
hipError_t hipPointerGetAttributes(hipPointerAttribute_t* a, const void* p) {
  const auto* m = fake::find(p);
  if (!m) return fake::last = hipErrorInvalidValue;
  memset(a, 0, sizeof *a);
  a->type = m->second.second; a->devicePointer = const_cast<void*>(p); a->hostPointer = const_cast<void*>(p);
  return hipSuccess;
}
hipError_t hipMemGetAddressRange(hipDeviceptr_t* base, size_t* size, hipDeviceptr_t p) {
  const auto* m = fake::find(p);
  if (!m) return fake::last = hipErrorInvalidValue;
  *base = (hipDeviceptr_t)m->first; *size = m->second.first;
  return hipSuccess;
}
hipError_t hipMemcpy(void* d, const void* s, size_t n, hipMemcpyKind) { memcpy(d, s, n); fake::note("copy"); return hipSuccess; }
hipError_t hipMemcpyAsync(void* d, const void* s, size_t n, hipMemcpyKind, hipStream_t st) { memcpy(d, s, n); fake::note("copy", st); return hipSuccess; }
hipError_t hipMemset(void* d, int v, size_t n) { memset(d, v, n); return hipSuccess; }
hipError_t hipStreamCreateWithFlags(hipStream_t* s, unsigned) { *s = (hipStream_t)(fake::next_handle += 16); return hipSuccess; }
hipError_t hipStreamDestroy(hipStream_t s) { fake::note("destroy stream", s); return hipSuccess; }
hipError_t hipStreamSynchronize(hipStream_t s) {
  if (fake::capturing[(uintptr_t)s]) return fake::last = hipErrorStreamCaptureUnsupported;
  fake::note("sync stream", s);
  return hipSuccess;
}
hipError_t hipStreamWaitEvent(hipStream_t s, hipEvent_t e, unsigned) { fake::note("wait", s, e); return hipSuccess; }
hipError_t hipStreamIsCapturing(hipStream_t s, hipStreamCaptureStatus* c) {
  *c = fake::capturing[(uintptr_t)s] ? hipStreamCaptureStatusActive : hipStreamCaptureStatusNone;
  return hipSuccess;
}
hipError_t hipEventCreate(hipEvent_t* e) { *e = (hipEvent_t)(fake::next_handle += 16); return hipSuccess; }
hipError_t hipEventCreateWithFlags(hipEvent_t* e, unsigned) { return hipEventCreate(e); }
hipError_t hipEventDestroy(hipEvent_t) { return hipSuccess; }
hipError_t hipEventQuery(hipEvent_t) { return hipSuccess; }
hipError_t hipEventRecord(hipEvent_t e, hipStream_t s) { fake::note("record", s, e); return hipSuccess; }
hipError_t hipEventSynchronize(hipEvent_t e) { fake::note("sync event", nullptr, e); return hipSuccess; }
hipError_t hipEventElapsedTime(float* ms, hipEvent_t, hipEvent_t) { *ms = 1.0f; return hipSuccess; }
}  // extern "C"
