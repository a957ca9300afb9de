// The HIP and kernel-launch functions that the library's host code calls, on host
// memory: for CPU builds of jx_abi.cpp and jx_server.cpp (included after this file
// by a check program, so that it sees their types).  Launches run nothing; they
// are recorded, and a check may let them block or fail.
#pragma once
#include <hip/hip_runtime_api.h>

#include <atomic>
#include <cstdio>
#include <cstdlib>
#include <cstring>
#include <string>
#include <vector>

#include "jx_internal.h"

namespace fake {
constexpr int kCus = 256;
struct Launch {
  std::string kind;  // "batch" or "fused"
  jx::LaunchCfg cfg;
  int mode = 0, n = 0, T = 0;
  int waves_per_env = 1;
};
std::vector<Launch> launches;                // single-threaded checks only
double (*elapsed_ms)() = nullptr;            // what the next event pair measured
std::atomic<bool> events_done{true};         // false: launches stay in flight
std::atomic<int> fail_uploads{0};            // so many of the next uploads fail
int fails = 0;
}  // namespace fake

#define CHECK(c, ...)                           \
  do {                                          \
    if (!(c)) {                                 \
      std::fprintf(stderr, "FAIL %d: ", __LINE__); \
      std::fprintf(stderr, __VA_ARGS__);        \
      std::fprintf(stderr, "\n");               \
      ++fake::fails;                            \
    }                                           \
  } while (0)

extern "C" {
hipError_t hipGetDeviceCount(int* n) { *n = 1; return hipSuccess; }
hipError_t hipSetDevice(int) { return hipSuccess; }
hipError_t hipGetDeviceProperties(hipDeviceProp_t* p, int) {
  std::memset(p, 0, sizeof(*p));
  p->multiProcessorCount = fake::kCus;
  std::strcpy(p->gcnArchName, "host");
  return hipSuccess;
}
const char* hipGetErrorString(hipError_t) { return "host error"; }
hipError_t hipGetLastError() { return hipSuccess; }
hipError_t hipMalloc(void** p, size_t n) { *p = std::calloc(n ? n : 1, 1); return *p ? hipSuccess : hipErrorOutOfMemory; }
hipError_t hipFree(void* p) { std::free(p); return hipSuccess; }
hipError_t hipHostMalloc(void** p, size_t n, unsigned) { return hipMalloc(p, n); }
hipError_t hipHostFree(void* p) { return hipFree(p); }
hipError_t hipHostGetDevicePointer(void** d, void* h, unsigned) { *d = h; return hipSuccess; }
hipError_t hipMemset(void* p, int v, size_t n) { std::memset(p, v, n); return hipSuccess; }
hipError_t hipMemcpy(void* d, const void* s, size_t n, hipMemcpyKind) { std::memcpy(d, s, n); return hipSuccess; }
hipError_t hipMemcpyAsync(void* d, const void* s, size_t n, hipMemcpyKind, hipStream_t) {
  int left = fake::fail_uploads.load();
  while (left > 0 && !fake::fail_uploads.compare_exchange_weak(left, left - 1)) {
  }
  if (left > 0) return hipErrorUnknown;
  std::memcpy(d, s, n);
  return hipSuccess;
}
hipError_t hipDeviceSynchronize() { return hipSuccess; }
hipError_t hipStreamCreateWithFlags(hipStream_t* s, unsigned) { *s = nullptr; return hipSuccess; }
hipError_t hipStreamDestroy(hipStream_t) { return hipSuccess; }
hipError_t hipStreamSynchronize(hipStream_t) { return hipSuccess; }
hipError_t hipEventCreate(hipEvent_t* e) { *e = nullptr; return hipSuccess; }
hipError_t hipEventCreateWithFlags(hipEvent_t* e, unsigned) { *e = nullptr; return hipSuccess; }
hipError_t hipEventDestroy(hipEvent_t) { return hipSuccess; }
hipError_t hipEventRecord(hipEvent_t, hipStream_t) { return hipSuccess; }
hipError_t hipEventQuery(hipEvent_t) { return fake::events_done.load() ? hipSuccess : hipErrorNotReady; }
hipError_t hipEventElapsedTime(float* ms, hipEvent_t, hipEvent_t) {
  *ms = fake::elapsed_ms ? (float)fake::elapsed_ms() : 1.f;
  return hipSuccess;
}
int roctxRangePushA(const char*) { return 0; }
int roctxRangePop() { return 0; }
}

#ifndef FAKE_THREADS  // (the server launches from its own threads: not recorded there)
#define FAKE_RECORD(...) fake::launches.push_back(__VA_ARGS__)
#else
#define FAKE_RECORD(...) (void)0
#endif

namespace jx {
int launch_batch(const DevState& s, const DevIo& io, const LaunchCfg& lc, int, int max_w, int64_t frames_bytes, int n_cu,
                 uint32_t, void*) {
  const bool frames = io.mode != MODE_RESET && io.obs != nullptr && io.dbg == nullptr;
  FAKE_RECORD({"batch", lc, io.mode, s.n, 1, step_waves_per_env(lc, io.mode, frames, s.n, frames_bytes, max_w, n_cu)});
  (void)frames, (void)max_w, (void)frames_bytes, (void)n_cu, (void)lc, (void)s;
  return 0;
}
int launch_rollout_fused(const DevState& s, const uint8_t*, uint8_t*, int64_t, float*, uint8_t*, uint8_t*, int T,
                         const LaunchCfg& lc, int, int n_cu, int64_t, uint32_t, void*) {
  FAKE_RECORD({"fused", lc, MODE_STEP, s.n, T, fused_waves_per_env(lc, s.n, n_cu)});
  (void)s, (void)T, (void)lc, (void)n_cu;
  return 0;
}
int launch_clear_queues(uint32_t*, void*) { return 0; }
int launch_serve(const DevState*, const DevIo*, const ServeItem*, int, uint32_t*, uint32_t, int, int, void*) { return 0; }
int scratch_device_address(int, uint32_t** out) {
  static uint32_t words[kScratchWords];
  *out = words;
  return 0;
}
const char* kernel_error_string(int) { return "host error"; }
}  // namespace jx
