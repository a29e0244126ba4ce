// A HIP runtime of host memory, and kernel launchers that only count: the host runtime
// (runtime.cpp, baselines.cpp) runs on it without a device.  It keeps what is allocated and
// what is in flight on which stream, refuses streams, events and graphs of another device than
// the current one, and makes the k-th fallible call fail on request.
#pragma once
#include <cstdio>
#include <cstdlib>
#include <cstring>
#include <map>
#include <set>
#include <string>
#include <vector>

#include "runtime.h"

namespace fake {
struct Stream {
  int dev = 0;
  int work = 0;  // launches not yet waited for
  std::set<Stream*> joined;
};
struct Event {
  int dev = 0;
  Stream* src = nullptr;
};
struct Graph {
  int dev = 0;
  Stream* on = nullptr;  // of its last replay
};
inline int device = 0;
inline hipError_t last = hipSuccess;
inline int64_t calls = 0, fail_at = -1;
inline bool capturing = false;
inline std::set<Stream*> streams;
inline std::map<int, Stream*> null_streams;
inline std::map<void*, size_t> ordered, plain, pinned;  // hipMallocAsync, hipMalloc, hipHostMalloc
inline int other_device = 0;  // launches, records and replays refused as another device's
inline int destroyed_in_flight = 0;  // graphs

inline hipError_t fail(hipError_t e) { return last = e; }
inline bool inject() { return ++calls == fail_at; }
inline Stream* stream(hipStream_t st) {
  if (st) return (Stream*)st;
  Stream*& s = null_streams[device];
  if (!s) {
    s = new Stream;
    s->dev = device;
    streams.insert(s);
  }
  return s;
}
inline void work(hipStream_t st) {
  Stream* s = stream(st);
  if (s->dev != device) {
    ++other_device;
    fail(hipErrorInvalidHandle);
  } else if (!capturing) {
    ++s->work;
  }
}
inline int in_flight() {
  int n = 0;
  for (Stream* s : streams) n += s->work;
  return n;
}
inline hipError_t allocate(std::map<void*, size_t>& m, void** p, size_t n) {
  if (inject()) return fail(hipErrorOutOfMemory);
  *p = calloc(1, n ? n : 1);
  m[*p] = n;
  return hipSuccess;
}
inline hipError_t release(std::map<void*, size_t>& m, void* p) {
  if (!m.erase(p)) return fail(hipErrorInvalidValue);
  free(p);
  return hipSuccess;
}
inline int failures = 0;
}  // namespace fake

#define CHECK(c, ...)                  \
  do {                                 \
    if (!(c)) {                        \
      std::printf("FAIL %s: ", #c);    \
      std::printf(__VA_ARGS__);        \
      std::printf("\n");               \
      ++fake::failures;                \
    }                                  \
  } while (0)

extern "C" {
hipError_t hipGetDevice(int* d) { *d = fake::device; return hipSuccess; }
hipError_t hipGetLastError() {
  if (fake::inject()) fake::last = hipErrorInvalidValue;  // another caller's error, still pending
  const hipError_t e = fake::last;
  fake::last = hipSuccess;
  return e;
}
const char* hipGetErrorString(hipError_t) { return "injected"; }
hipError_t hipMalloc(void** p, size_t n) { return fake::allocate(fake::plain, p, n); }
hipError_t hipFree(void* p) { return fake::release(fake::plain, p); }
hipError_t hipMallocAsync(void** p, size_t n, hipStream_t) { return fake::allocate(fake::ordered, p, n); }
hipError_t hipFreeAsync(void* p, hipStream_t) { return fake::release(fake::ordered, p); }
hipError_t hipHostMalloc(void** p, size_t n, unsigned) { return fake::allocate(fake::pinned, p, n); }
hipError_t hipHostFree(void* p) { return fake::release(fake::pinned, p); }
hipError_t hipMemcpyAsync(void* d, const void* s, size_t n, hipMemcpyKind, hipStream_t) {
  if (fake::inject()) return fake::fail(hipErrorInvalidValue);
  std::memcpy(d, s, n);
  return hipSuccess;
}
hipError_t hipMemsetAsync(void* d, int v, size_t n, hipStream_t) {
  if (fake::inject()) return fake::fail(hipErrorInvalidValue);
  std::memset(d, v, n);
  return hipSuccess;
}
hipError_t hipStreamCreateWithFlags(hipStream_t* st, unsigned) {
  auto* s = new fake::Stream;
  s->dev = fake::device;
  fake::streams.insert(s);
  *st = (hipStream_t)s;
  return hipSuccess;
}
hipError_t hipStreamDestroy(hipStream_t st) {
  fake::streams.erase((fake::Stream*)st);
  for (fake::Stream* s : fake::streams) s->joined.erase((fake::Stream*)st);
  delete (fake::Stream*)st;
  return hipSuccess;
}
hipError_t hipStreamSynchronize(hipStream_t st) {
  fake::Stream* s = fake::stream(st);
  s->work = 0;
  for (fake::Stream* j : s->joined) j->work = 0;
  s->joined.clear();
  return fake::inject() ? fake::fail(hipErrorUnknown) : hipSuccess;
}
hipError_t hipSetDevice(int d) { fake::device = d; return hipSuccess; }
hipError_t hipDeviceSynchronize() {
  for (fake::Stream* s : fake::streams)
    if (s->dev == fake::device) s->work = 0;
  return hipSuccess;
}
hipError_t hipStreamIsCapturing(hipStream_t, hipStreamCaptureStatus* c) {
  *c = hipStreamCaptureStatusNone;
  return hipSuccess;
}
hipError_t hipStreamWaitEvent(hipStream_t st, hipEvent_t e, unsigned) {
  auto* ev = (fake::Event*)e;
  if (ev->src) fake::stream(st)->joined.insert(ev->src);
  return hipSuccess;
}
hipError_t hipStreamBeginCapture(hipStream_t, hipStreamCaptureMode) {
  if (fake::inject()) return fake::fail(hipErrorInvalidValue);
  fake::capturing = true;
  return hipSuccess;
}
hipError_t hipStreamEndCapture(hipStream_t, hipGraph_t* g) {
  fake::capturing = false;
  auto* x = new fake::Graph;
  x->dev = fake::device;
  *g = (hipGraph_t)x;
  return hipSuccess;
}
hipError_t hipGraphInstantiate(hipGraphExec_t* x, hipGraph_t g, hipGraphNode_t*, char*, size_t) {
  if (fake::inject()) return fake::fail(hipErrorOutOfMemory);
  *x = (hipGraphExec_t) new fake::Graph(*(fake::Graph*)g);
  return hipSuccess;
}
hipError_t hipGraphLaunch(hipGraphExec_t x, hipStream_t st) {
  if (fake::inject()) return fake::fail(hipErrorOutOfMemory);
  if (((fake::Graph*)x)->dev != fake::device) ++fake::other_device;
  ((fake::Graph*)x)->on = fake::stream(st);
  ++fake::stream(st)->work;
  return hipSuccess;
}
hipError_t hipGraphDestroy(hipGraph_t g) { delete (fake::Graph*)g; return hipSuccess; }
hipError_t hipGraphExecDestroy(hipGraphExec_t x) {
  fake::Stream* on = ((fake::Graph*)x)->on;
  if (on && on->work) ++fake::destroyed_in_flight;
  delete (fake::Graph*)x;
  return hipSuccess;
}
hipError_t hipEventCreateWithFlags(hipEvent_t* e, unsigned) {
  auto* ev = new fake::Event;
  ev->dev = fake::device;
  *e = (hipEvent_t)ev;
  return hipSuccess;
}
hipError_t hipEventDestroy(hipEvent_t e) { delete (fake::Event*)e; return hipSuccess; }
hipError_t hipEventRecord(hipEvent_t e, hipStream_t st) {
  auto* ev = (fake::Event*)e;
  if (ev->dev != fake::stream(st)->dev) {
    ++fake::other_device;
    return fake::fail(hipErrorInvalidHandle);
  }
  ev->src = fake::stream(st);
  return hipSuccess;
}
hipError_t hipEventSynchronize(hipEvent_t) { return hipSuccess; }
hipError_t hipEventElapsedTime(float* ms, hipEvent_t, hipEvent_t) { *ms = 0.0f; return hipSuccess; }
hipError_t hipDeviceGetDefaultMemPool(hipMemPool_t*, int) { return hipErrorNotSupported; }
hipError_t hipMemPoolSetAttribute(hipMemPool_t, hipMemPoolAttr, void*) { return hipSuccess; }
}

namespace et {
typedef const TestDesc* D;
typedef const int64_t* O;
void launch_clear_flags(hipStream_t st, D, O, int) { fake::work(st); }
void launch_colpart(int64_t, hipStream_t st, D, O, int) { fake::work(st); }
void launch_colmean(int64_t, hipStream_t st, D, O, int) { fake::work(st); }
void launch_stage(int64_t, hipStream_t st, D, O, int) { fake::work(st); }
void launch_gram(int, bool, int64_t, hipStream_t st, D, O, int, bool) { fake::work(st); }
void launch_gram_finish(int64_t, hipStream_t st, D, O, int, bool) { fake::work(st); }
void launch_gram_sums(int, int64_t, hipStream_t st, D, O, int) { fake::work(st); }
void launch_rowsum(int64_t, hipStream_t st, D, O, int) { fake::work(st); }
void launch_observed(hipStream_t st, D, O, int) { fake::work(st); }
void launch_center(bool, int64_t, hipStream_t st, D, O, int) { fake::work(st); }
void launch_member(int64_t, hipStream_t st, D, O, int, bool) { fake::work(st); }
void launch_member_public(int64_t, int64_t, uint64_t, int64_t, int64_t, uint32_t*, hipStream_t st) { fake::work(st); }
void launch_member_import(int64_t, hipStream_t st, D, const uint32_t*) { fake::work(st); }
void launch_perm(int, int64_t, hipStream_t st, D, O, int, const int32_t*) { fake::work(st); }
void launch_pstat(int64_t, hipStream_t st, D, O, int) { fake::work(st); }
void launch_cross_final(hipStream_t st, D) { fake::work(st); }
void launch_unpack(bool, int64_t, hipStream_t st, D, void*, void*, void*) { fake::work(st); }
void launch_rowmap(const uint32_t*, int64_t, int64_t, int64_t, int64_t, int32_t*, hipStream_t st) { fake::work(st); }
void launch_sum_flags(D, int, const int32_t*, hipStream_t st) { fake::work(st); }
void launch_collect(D, int, int64_t, int64_t, double*, int32_t*, hipStream_t st) { fake::work(st); }
void launch_count(const double*, int64_t, const int32_t*, double*, DevResult*, hipStream_t st) { fake::work(st); }
void launch_precomp(bool, D, int64_t, int64_t, double*, hipStream_t st) { fake::work(st); }
void launch_precomp_stat(D, int64_t, int64_t, const double*, double*, hipStream_t st) { fake::work(st); }
void launch_permgen(int64_t, uint64_t, int64_t, int64_t, int64_t, int32_t*, hipStream_t st) { fake::work(st); }
void launch_hsic_perms(int64_t, int64_t, uint64_t, int64_t, int64_t, int64_t, uint16_t*, uint16_t*, hipStream_t st) { fake::work(st); }
void launch_hsic_prep(bool, D, int64_t, int64_t, int64_t, void*, double*, double*, double*, int32_t*, hipStream_t st) { fake::work(st); }
int64_t hsic_parts(bool, int64_t n) { return n; }
void launch_hsic_terms(bool, D, const void*, int64_t, int64_t, const uint16_t*, const uint16_t*, int64_t, double*, hipStream_t st) { fake::work(st); }
void launch_hsic_stat(const double*, int64_t, int64_t, int64_t, const uint16_t*, const double*, const double*, int64_t, const double*, double*, hipStream_t st) { fake::work(st); }
void launch_put_desc(const TestDesc&, O, TestDesc*, int64_t*, hipStream_t st) { fake::work(st); }
}  // namespace et
