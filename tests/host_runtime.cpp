// A stand-in for the HIP runtime and the kernel launchers, for tests of the
// library's host code (rpd_api.cpp, proj_plan.cpp) without a GPU. Launches
// are recorded instead of run. Of the kernels, only the two that count
// positions leave something behind: the count, in device memory and, where the
// launch asks for it, in host memory, when the stream is waited for or another
// counting kernel is enqueued behind it (no earlier here).
//
// As in the runtime, an error stays the thread's last error until
// hipGetLastError takes it, a call that succeeds does not clear it, and a
// launcher returns it although its kernel has been enqueued.
#include <cstdlib>
#include <cstring>
#include <deque>
#include <string>

#include "rpd_launch.h"

namespace {

hipError_t g_last = hipSuccess;
std::string g_log;
std::deque<int> g_counts;   // what the counting kernels find, in the order of their launches

struct Pending {
  int32_t* at;
  int32_t value;
};
std::deque<Pending> g_pending;   // stores of enqueued kernels

hipError_t set(hipError_t e) {
  if (e != hipSuccess) g_last = e;
  return e;
}

hipError_t take_last() {
  const hipError_t e = g_last;
  g_last = hipSuccess;
  return e;
}

void complete() {
  for (const Pending& p : g_pending) *p.at = p.value;
  g_pending.clear();
}

hipError_t count_kernel(int32_t* dev, int32_t* host) {
  complete();
  const int n = g_counts.empty() ? 0 : g_counts.front();
  if (!g_counts.empty()) g_counts.pop_front();
  g_pending.push_back({dev, n});
  if (host) g_pending.push_back({host, n});
  return take_last();
}

}  // namespace

// ------------------------------------------------ what a test sets and reads --

extern "C" {
int host_fail_malloc = 0, host_fail_capturing = 0;   // the call returns this error
void host_reset() {
  g_last = hipSuccess;
  g_log.clear();
  g_counts.clear();
  host_fail_malloc = host_fail_capturing = 0;
}
void host_set_last_error(int e) { g_last = static_cast<hipError_t>(e); }
void host_add_count(int n) { g_counts.push_back(n); }
const char* host_log() { return g_log.c_str(); }
}

// ------------------------------------------------------------------ runtime --

extern "C" {
hipError_t hipGetLastError() { return take_last(); }
const char* hipGetErrorString(hipError_t e) { return e == hipSuccess ? "no error" : "an error"; }
hipError_t hipStreamIsCapturing(hipStream_t, hipStreamCaptureStatus* s) {
  *s = hipStreamCaptureStatusNone;
  return set(static_cast<hipError_t>(host_fail_capturing));
}
hipError_t hipThreadExchangeStreamCaptureMode(hipStreamCaptureMode*) { return hipSuccess; }
hipError_t hipHostMalloc(void** p, size_t n, unsigned) {
  if (host_fail_malloc) return set(static_cast<hipError_t>(host_fail_malloc));
  *p = calloc(1, n);
  return hipSuccess;
}
hipError_t hipStreamSynchronize(hipStream_t) {
  g_log += "sync ";
  complete();
  return hipSuccess;
}
hipError_t hipMemcpyAsync(void* dst, const void* src, size_t n, hipMemcpyKind, hipStream_t) {
  g_log += "copy ";
  complete();
  memcpy(dst, src, n);
  return hipSuccess;
}
hipError_t hipEventRecord(hipEvent_t, hipStream_t) { return hipSuccess; }
hipError_t hipGetDevice(int* d) {
  *d = 0;
  return hipSuccess;
}
hipError_t hipGetSymbolAddress(void** p, const void* symbol) {
  *p = const_cast<void*>(symbol);
  return hipSuccess;
}
}

// ----------------------------------------------------------------- launches --

namespace rpd {
namespace {
hipError_t note(const char* what, long long n) {
  g_log += what;
  g_log += std::to_string(n) + " ";
  return take_last();
}
}  // namespace

hipError_t launch_compact(const Launch& a, bool, int, int32_t* host_n, hipStream_t) {
  g_log += "compact ";
  return count_kernel(a.n_masked, host_n);
}
hipError_t launch_lazy_next(const Launch& a, int, int, int, int32_t* host_m, hipStream_t) {
  g_log += "next ";
  return count_kernel(a.lazy.m, host_m);
}
bool compact_fused(const Launch&) { return false; }
hipError_t launch_norm_rows(const Launch& a, hipStream_t) { return note("norm", a.max_masked); }
hipError_t launch_proj_stream(const Launch& a, hipStream_t) { return note("stream", a.max_masked); }
hipError_t launch_proj_big(const Launch& a, hipStream_t) { return note("big", a.max_masked); }
hipError_t launch_proj_f32(const Launch& a, hipStream_t) { return note("f32_", a.max_masked); }
hipError_t launch_reduce_score(const Launch& a, hipStream_t) { return note("reduce", a.max_masked); }
hipError_t launch_lazy_reduce(const Launch&, int, int m_cap, const ProjPlan*, hipStream_t) {
  return note("walk", m_cap);
}
hipError_t launch_lazy_score(const Launch& a, hipStream_t) { return note("score", a.max_masked); }
hipError_t launch_commit(const Launch&, hipStream_t) { return note("commit", 0); }
hipError_t launch_apply_commit(long long, uint8_t*, int32_t*, const uint8_t*, const int32_t*, int32_t*, int, int32_t*,
                               hipStream_t) {
  return take_last();
}
hipError_t launch_gate_commit(const Launch&, const int32_t*, const float*, const float*, hipStream_t) {
  return take_last();
}
}  // namespace rpd
