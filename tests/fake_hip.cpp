// A stand-in for the HIP runtime, preloaded in front of it by CPU tests of the
// host orchestration: device memory is host memory with a settable capacity,
// calls are counted, and of the kernels only what the host reads back is done
// (kept ranks, statuses, sweeps); all other results are zero.
#define __HIP_PLATFORM_AMD__ 1
#include <hip/hip_runtime.h>

#include <algorithm>
#include <cstdlib>
#include <cstring>
#include <map>
#include <mutex>
#include <string>

#include "internal.h"

using namespace mps;

namespace {
std::mutex mtx;
std::map<void*, size_t> live;
std::map<const void*, std::string> kernels;
std::map<std::string, long long> blocks, launches;  // thread blocks and launches, by kernel name
size_t capacity = (size_t)1 << 34, used = 0;
long long mallocs = 0, frees = 0;
thread_local dim3 cfg_grid, cfg_block;
thread_local size_t cfg_shmem;
thread_local hipStream_t cfg_stream;
char symbol_memory[kScratchBytes];

void fused(const FusedGate& g) {
  g.dims[g.q + 1] = std::min(g.cap_k, 2 * std::min(g.dims[g.q], g.dims[g.q + 2]));
}
}  // namespace

extern "C" {

void fake_set_capacity(size_t bytes) { capacity = bytes; }
size_t fake_used() { return used; }
long long fake_mallocs() { return mallocs; }
long long fake_frees() { return frees; }
static long long count(const std::map<std::string, long long>& by_name, const char* kernel) {
  std::lock_guard<std::mutex> l(mtx);
  long long n = 0;
  for (auto& b : by_name)
    if (b.first.find(kernel) != std::string::npos) n += b.second;
  return n;
}
long long fake_blocks(const char* kernel) { return count(blocks, kernel); }
long long fake_launches(const char* kernel) { return count(launches, kernel); }

hipError_t hipMalloc(void** p, size_t n) {
  std::lock_guard<std::mutex> l(mtx);
  ++mallocs;
  *p = nullptr;
  if (used + n > capacity) return hipErrorOutOfMemory;
  *p = std::calloc(1, n);
  used += n;
  live[*p] = n;
  return hipSuccess;
}
hipError_t hipFree(void* p) {
  std::lock_guard<std::mutex> l(mtx);
  auto it = live.find(p);
  if (it == live.end()) return p ? hipErrorInvalidValue : hipSuccess;
  ++frees;
  used -= it->second;
  live.erase(it);
  std::free(p);
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
hipError_t hipMemsetAsync(void* d, int v, size_t n, hipStream_t) {
  std::memset(d, v, n);
  return hipSuccess;
}
hipError_t hipDeviceGetAttribute(int* v, hipDeviceAttribute_t, int) {
  *v = 160 * 1024;
  return hipSuccess;
}
hipError_t hipGetDevice(int* d) {
  *d = 0;
  return hipSuccess;
}
const char* hipGetErrorString(hipError_t) { return "fake"; }
hipError_t hipGetLastError() { return hipSuccess; }
hipError_t hipGetSymbolAddress(void** p, const void*) {
  *p = symbol_memory;
  return hipSuccess;
}
hipError_t hipFuncSetAttribute(const void*, hipFuncAttribute, int) { return hipSuccess; }
hipError_t hipStreamCreateWithFlags(hipStream_t* s, unsigned) {
  *s = (hipStream_t)std::malloc(1);
  return hipSuccess;
}
hipError_t hipStreamDestroy(hipStream_t s) {
  std::free((void*)s);
  return hipSuccess;
}
hipError_t hipStreamSynchronize(hipStream_t) { return hipSuccess; }
hipError_t hipStreamWaitEvent(hipStream_t, hipEvent_t, unsigned) { return hipSuccess; }
hipError_t hipEventCreate(hipEvent_t* e) {
  *e = (hipEvent_t)std::malloc(1);
  return hipSuccess;
}
hipError_t hipEventCreateWithFlags(hipEvent_t* e, unsigned) { return hipEventCreate(e); }
hipError_t hipEventDestroy(hipEvent_t e) {
  std::free((void*)e);
  return hipSuccess;
}
hipError_t hipEventRecord(hipEvent_t, hipStream_t) { return hipSuccess; }
hipError_t hipEventElapsedTime(float* ms, hipEvent_t, hipEvent_t) {
  *ms = 0.f;
  return hipSuccess;
}

void** __hipRegisterFatBinary(const void*) { return (void**)std::malloc(8); }
void __hipUnregisterFatBinary(void**) {}
void __hipRegisterVar(void**, void*, char*, char*, int, size_t, int, int) {}
void __hipRegisterFunction(void**, const void* host, char*, const char* name, unsigned, void*, void*, void*, void*,
                           int*) {
  std::lock_guard<std::mutex> l(mtx);
  kernels[host] = name;
}
hipError_t __hipPushCallConfiguration(dim3 grid, dim3 block, size_t shmem, hipStream_t s) {
  cfg_grid = grid;
  cfg_block = block;
  cfg_shmem = shmem;
  cfg_stream = s;
  return hipSuccess;
}
hipError_t __hipPopCallConfiguration(dim3* grid, dim3* block, size_t* shmem, hipStream_t* s) {
  *grid = cfg_grid;
  *block = cfg_block;
  *shmem = cfg_shmem;
  *s = cfg_stream;
  return hipSuccess;
}

hipError_t hipLaunchKernel(const void* f, dim3 grid, dim3, void** args, size_t, hipStream_t) {
  std::string name;
  {
    std::lock_guard<std::mutex> l(mtx);
    name = kernels[f];
    blocks[name] += (long long)grid.x * grid.y * grid.z;
    ++launches[name];
  }
  auto is = [&](const char* k) { return name.find(k) != std::string::npos; };
  if (is("15finalize_kernel")) {
    const FinItem* it = *(const FinItem**)args[0];
    for (unsigned b = 0; b < grid.x; ++b) {
      *it[b].k_out = std::min(it[b].cap, it[b].n);
      *it[b].scale_out = 1.0;
      *it[b].disc_out = 0.0;
      *it[b].status_out = 0;
    }
  } else if (is("14lq_rank_kernel")) {
    const LqFinItem* it = *(const LqFinItem**)args[0];
    for (unsigned b = 0; b < grid.x; ++b) {
      *it[b].k_out = std::min(it[b].cap, it[b].n);
      *it[b].scale_out = 1.0;
      *it[b].disc_out = 0.0;
      *it[b].status_out = 0;
    }
  } else if (is("19jacobi_small_kernel") || is("20jacobi_single_kernel")) {
    const JacItem* it = *(const JacItem**)args[0];
    for (unsigned b = 0; b < grid.x; ++b) *it[b].sweeps_done = 1;
  } else if (is("19gate2q_fused_kernel")) {
    fused(*(const FusedGate*)args[0]);
  } else if (is("17fused_step_kernel")) {
    const FusedRun* runs = *(const FusedRun**)args[0];
    const int64_t step = *(const int64_t*)args[1];
    for (unsigned b = 0; b < grid.x; ++b) {
      const FusedRun& r = runs[b];
      const int64_t gi = r.g0 + step;
      if (gi >= r.g1 || r.q1[gi] < 0) continue;
      FusedGate g{};
      g.dims = r.dims;
      g.q = r.q0[gi];
      g.cap_k = r.cap[g.q + 1];
      fused(g);
    }
  }
  return hipSuccess;
}

hipError_t hipStreamBeginCapture(hipStream_t, hipStreamCaptureMode) { return hipErrorNotSupported; }
hipError_t hipStreamEndCapture(hipStream_t, hipGraph_t*) { return hipErrorNotSupported; }
hipError_t hipMemcpy2DAsync(void*, size_t, const void*, size_t, size_t, size_t, hipMemcpyKind, hipStream_t) {
  return hipErrorNotSupported;
}

}  // extern "C"
