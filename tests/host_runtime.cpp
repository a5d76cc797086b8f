// A host-only stand-in for the HIP runtime, for tests of the library's host side without a
// GPU: memory is host memory, streams run at once, kernels are recorded and not run, except
// the copy of loaded blocks into their pool slots.  Allocations can be made to fail, and the
// device to report any number of compute units.
#include "internal.hpp"

#include <cstdlib>
#include <cstring>
#include <map>
#include <string>
#include <vector>

namespace {

std::map<const void*, std::string> names;
struct Launch {
  std::string name;
  unsigned long long grid, threads;
};
std::vector<Launch> launches;
std::map<void*, size_t> live;   // allocation -> bytes
int fail_in = 0, units = 256, run_copies = 1;
dim3 cfg_grid, cfg_block;
size_t cfg_lds;
hipStream_t cfg_stream;

hipError_t get(void** p, size_t n) {
  *p = nullptr;
  if (fail_in > 0 && --fail_in == 0) return hipErrorOutOfMemory;
  *p = std::calloc(n ? n : 1, 1);
  live[*p] = n;
  return hipSuccess;
}

// (freed memory stays mapped, filled with a pattern that no table holds)
hipError_t put(void* p) {
  auto it = live.find(p);
  if (it == live.end()) return p ? hipErrorInvalidValue : hipSuccess;
  std::memset(p, 0x5a, it->second);
  live.erase(it);
  return hipSuccess;
}

bool in_live(const void* p, size_t n) {
  for (auto& a : live)
    if ((const char*)p >= (const char*)a.first && (const char*)p + n <= (const char*)a.first + a.second) return true;
  return false;
}

long scatter_faults = 0, null_topologies = 0;

void scatter(const mrb::ScatterArgs& a) {
  const mrb::BlockDesc* d = (const mrb::BlockDesc*)(a.topo.base + a.topo.h.off_blk);
  if (!in_live(d, a.topo.h.n_blocks * sizeof *d)) {
    ++scatter_faults;
    return;
  }
  for (int b = 0; b < a.topo.h.n_blocks; ++b)
    std::memcpy(a.u + (size_t)d[b].slot * a.bsz, a.src + (size_t)b * a.bsz, a.bsz * sizeof(double));
}

}  // namespace

extern "C" {

// controls
void host_fail_allocation(int n) { fail_in = n; }   // the n-th allocation from now on fails
void host_compute_units(int n) { units = n; }
void host_run_copies(int on) { run_copies = on; }
long host_scatter_faults() { return scatter_faults; }   // block copies that read freed memory
long host_null_topologies() { return null_topologies; }   // refinements without a topology buffer
int host_launches() { return (int)launches.size(); }
const char* host_launch(int i, unsigned long long* grid, unsigned long long* threads) {
  *grid = launches[i].grid;
  *threads = launches[i].threads;
  return launches[i].name.c_str();
}
void host_clear() { launches.clear(); }

// the runtime
void** __hipRegisterFatBinary(const void*) { return nullptr; }
void __hipUnregisterFatBinary(void**) {}
void __hipRegisterFunction(void**, const void* f, char*, const char* name, unsigned, void*, void*, void*, void*, int*) {
  names[f] = name;
}
void __hipRegisterVar(void**, void*, char*, char*, int, size_t, int, int) {}
hipError_t __hipPushCallConfiguration(dim3 g, dim3 b, size_t lds, hipStream_t s) {
  cfg_grid = g;
  cfg_block = b;
  cfg_lds = lds;
  cfg_stream = s;
  return hipSuccess;
}
hipError_t __hipPopCallConfiguration(dim3* g, dim3* b, size_t* lds, hipStream_t* s) {
  *g = cfg_grid;
  *b = cfg_block;
  *lds = cfg_lds;
  *s = cfg_stream;
  return hipSuccess;
}
hipError_t hipLaunchKernel(const void* f, dim3 g, dim3 b, void** args, size_t, hipStream_t) {
  launches.push_back(Launch{names[f], g.x, b.x});
  // a launch holds fewer than 2^32 work items
  if ((unsigned long long)g.x * b.x > 0xffffffffull) return hipErrorInvalidConfiguration;
  if (names[f].find("k_refine") != std::string::npos && !((const mrb::RefineArgs*)args[0])->topo.base) ++null_topologies;
  if (run_copies && names[f].find("k_scatter") != std::string::npos) scatter(*(const mrb::ScatterArgs*)args[0]);
  return hipSuccess;
}
hipError_t hipLaunchCooperativeKernel(const void* f, dim3 g, dim3 b, void** args, unsigned lds, hipStream_t s) {
  return hipLaunchKernel(f, g, b, args, lds, s);
}
hipError_t hipOccupancyMaxActiveBlocksPerMultiprocessor(int* n, const void*, int, size_t) { return *n = 2, hipSuccess; }
hipError_t hipFuncSetAttribute(const void*, hipFuncAttribute, int) { return hipSuccess; }
hipError_t hipGetDevice(int* d) { return *d = 0, hipSuccess; }
hipError_t hipDeviceGetAttribute(int* v, hipDeviceAttribute_t, int) { return *v = units, hipSuccess; }
const char* hipGetErrorString(hipError_t) { return "error of the host runtime"; }
hipError_t hipGetLastError() { return hipSuccess; }
hipError_t hipGetSymbolAddress(void** p, const void*) {
  static char mem[mrb::kScratchBytes];
  return *p = mem, hipSuccess;
}
hipError_t hipMalloc(void** p, size_t n) { return get(p, n); }
hipError_t hipFree(void* p) { return put(p); }
hipError_t hipHostMalloc(void** p, size_t n, unsigned) { return get(p, n); }
hipError_t hipHostFree(void* p) { return put(p); }
hipError_t hipHostGetDevicePointer(void** d, void* h, unsigned) { return *d = h, hipSuccess; }
hipError_t hipMemcpy(void* d, const void* s, size_t n, hipMemcpyKind) { return std::memcpy(d, s, n), hipSuccess; }
hipError_t hipMemcpyAsync(void* d, const void* s, size_t n, hipMemcpyKind, hipStream_t) {
  return std::memcpy(d, s, n), hipSuccess;
}
hipError_t hipMemset(void* p, int v, size_t n) { return std::memset(p, v, n), hipSuccess; }
hipError_t hipMemsetAsync(void* p, int v, size_t n, hipStream_t) { return std::memset(p, v, n), hipSuccess; }
hipError_t hipStreamSynchronize(hipStream_t) { return hipSuccess; }
hipError_t hipStreamBeginCapture(hipStream_t, hipStreamCaptureMode) { return hipErrorNotSupported; }
hipError_t hipStreamEndCapture(hipStream_t, hipGraph_t*) { return hipErrorNotSupported; }
hipError_t hipGraphInstantiate(hipGraphExec_t*, hipGraph_t, hipGraphNode_t*, char*, size_t) { return hipErrorNotSupported; }
hipError_t hipGraphLaunch(hipGraphExec_t, hipStream_t) { return hipErrorNotSupported; }
hipError_t hipGraphDestroy(hipGraph_t) { return hipSuccess; }
hipError_t hipGraphExecDestroy(hipGraphExec_t) { return hipSuccess; }
hipError_t hipEventCreate(hipEvent_t* e) { return *e = (hipEvent_t)1, hipSuccess; }
hipError_t hipEventCreateWithFlags(hipEvent_t* e, unsigned) { return *e = (hipEvent_t)1, hipSuccess; }
hipError_t hipEventDestroy(hipEvent_t) { return hipSuccess; }
hipError_t hipEventRecord(hipEvent_t, hipStream_t) { return hipSuccess; }
hipError_t hipEventSynchronize(hipEvent_t) { return hipSuccess; }
hipError_t hipEventElapsedTime(float* ms, hipEvent_t, hipEvent_t) { return *ms = 1.0f, hipSuccess; }

}  // extern "C"
