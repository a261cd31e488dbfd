// A HIP runtime of the host alone, for tests of the library's host code: the
// functions that the library calls, over counters, a card of a chosen size and
// a list of the launches.  Nothing runs on a device, and no address that it
// gives out is ever read or written.
#pragma once

#include <hip/hip_runtime.h>
#include <stdio.h>
#include <stdlib.h>
#include <string.h>

#include <map>
#include <string>
#include <vector>

#include "../../include/ccc.h"
#include "../../paper_1705_08213_amd/csrc/kernels.h"

namespace fake {

struct Launch {
  std::string kernel;  // mangled name
  dim3 grid, block;
  hipStream_t stream;
  ccc::Pair2Args pair;      // of the 2-way kernels
  ccc::OperandJob job;      // of the operand pass
  int64_t base = 0, count = 0;  // of the kernels over 3-way units
};

// (registered before main, by the sources' own initialisers)
inline std::map<const void*, std::string>& names() {
  static std::map<const void*, std::string> m;
  return m;
}
inline std::vector<Launch> launches;
inline std::map<uintptr_t, size_t> allocated;
inline std::map<hipStream_t, unsigned long long> capture;  // capture id of a stream
struct Object {
  void* p;
  hipHostFn_t fn;
};
inline std::map<unsigned long long, std::vector<Object*>> graphs;  // user objects by capture id
inline void destroy_graph(unsigned long long id) {
  for (Object* o : graphs[id]) {
    o->fn(o->p);
    delete o;
  }
  graphs.erase(id);
}
inline size_t card = size_t(288) << 30, used = 0;
inline uintptr_t next = uintptr_t(1) << 40;
inline long mallocs = 0, failed = 0, frees = 0, syncs = 0;
inline hipError_t last = hipSuccess;

inline hipError_t give(hipError_t e) {
  if (e != hipSuccess) last = e;
  return e;
}
inline bool is(const Launch& l, const char* part) {
  return l.kernel.find(part) != std::string::npos;
}
inline hipStream_t stream(int k) { return reinterpret_cast<hipStream_t>(uintptr_t(0x1000 + 64 * k)); }

}  // namespace fake

extern "C" {

void** __hipRegisterFatBinary(const void*) { return nullptr; }
void __hipUnregisterFatBinary(void**) {}
void __hipRegisterFunction(void**, const void* host, char*, const char* name, unsigned, void*, void*,
                           void*, void*, int*) {
  fake::names()[host] = name;
}
void __hipRegisterVar(void**, void*, char*, char*, int, size_t, int, int) {}

static thread_local struct {
  dim3 grid, block;
  size_t shared;
  hipStream_t stream;
} pushed;
hipError_t __hipPushCallConfiguration(dim3 g, dim3 b, size_t s, hipStream_t st) {
  pushed = {g, b, s, st};
  return hipSuccess;
}
hipError_t __hipPopCallConfiguration(dim3* g, dim3* b, size_t* s, hipStream_t* st) {
  *g = pushed.grid;
  *b = pushed.block;
  *s = pushed.shared;
  *st = pushed.stream;
  return hipSuccess;
}

hipError_t hipLaunchKernel(const void* f, dim3 g, dim3 b, void** args, size_t, hipStream_t st) {
  fake::Launch l;
  l.kernel = fake::names()[f];
  l.grid = g;
  l.block = b;
  l.stream = st;
  memset(static_cast<void*>(&l.pair), 0, sizeof l.pair);
  memset(static_cast<void*>(&l.job), 0, sizeof l.job);
  if (fake::is(l, "mfma2_") || fake::is(l, "pop2_kernel"))
    memcpy(static_cast<void*>(&l.pair), args[0], sizeof l.pair);
  if (fake::is(l, "15operands_kernel")) memcpy(static_cast<void*>(&l.job), args[0], sizeof l.job);
  if (fake::is(l, "Triple3Args")) {
    memcpy(&l.base, args[2], 8);
    memcpy(&l.count, args[3], 8);
  }
  fake::launches.push_back(l);
  // the runtime's limits: fewer than 2^32 work-items along a dimension
  const bool ok = g.x && g.y && g.z && (uint64_t)g.x * b.x < (uint64_t(1) << 32) &&
                  (uint64_t)g.y * b.y < (uint64_t(1) << 32) && b.x * b.y * b.z <= 1024;
  return fake::give(ok ? hipSuccess : hipErrorInvalidConfiguration);
}

hipError_t hipMalloc(void** p, size_t bytes) {
  ++fake::mallocs;
  if (bytes > fake::card - fake::used) {
    ++fake::failed;
    return fake::give(hipErrorOutOfMemory);
  }
  *p = reinterpret_cast<void*>(fake::next);
  fake::allocated[fake::next] = bytes;
  fake::next += (bytes + 4095) / 4096 * 4096;
  fake::used += bytes;
  return hipSuccess;
}
hipError_t hipFree(void* p) {
  if (!p) return hipSuccess;
  ++fake::frees;
  auto it = fake::allocated.find(reinterpret_cast<uintptr_t>(p));
  if (it == fake::allocated.end()) return fake::give(hipErrorInvalidValue);
  fake::used -= it->second;
  fake::allocated.erase(it);
  return hipSuccess;
}
hipError_t hipMemGetInfo(size_t* free_, size_t* total) {
  *free_ = fake::card - fake::used;
  *total = fake::card;
  return hipSuccess;
}
hipError_t hipDeviceSynchronize(void) {
  ++fake::syncs;
  return hipSuccess;
}
hipError_t hipGetLastError(void) {
  const hipError_t e = fake::last;
  fake::last = hipSuccess;
  return e;
}
hipError_t hipGetDevice(int* d) {
  *d = 0;
  return hipSuccess;
}
hipError_t hipSetDevice(int) { return hipSuccess; }
hipError_t hipDeviceGetAttribute(int* v, hipDeviceAttribute_t, int) {
  *v = 256;
  return hipSuccess;
}
hipError_t hipGetSymbolAddress(void** p, const void*) {
  *p = reinterpret_cast<void*>(uintptr_t(1) << 36);
  return hipSuccess;
}
hipError_t hipMemcpy(void*, const void*, size_t, hipMemcpyKind) { return hipSuccess; }

hipError_t hipStreamIsCapturing(hipStream_t s, hipStreamCaptureStatus* st) {
  *st = fake::capture.count(s) ? hipStreamCaptureStatusActive : hipStreamCaptureStatusNone;
  return hipSuccess;
}
hipError_t hipStreamGetCaptureInfo(hipStream_t s, hipStreamCaptureStatus* st,
                                   unsigned long long* id) {
  hipStreamIsCapturing(s, st);
  *id = fake::capture.count(s) ? fake::capture[s] : 0;
  return hipSuccess;
}
hipError_t hipStreamGetCaptureInfo_v2(hipStream_t s, hipStreamCaptureStatus* st,
                                      unsigned long long* id, hipGraph_t* g,
                                      const hipGraphNode_t** deps, size_t* n) {
  hipStreamGetCaptureInfo(s, st, id);
  *g = reinterpret_cast<hipGraph_t>(uintptr_t(*id));
  *deps = nullptr;
  *n = 0;
  return hipSuccess;
}
hipError_t hipUserObjectCreate(hipUserObject_t* o, void* p, hipHostFn_t fn, unsigned, unsigned) {
  *o = reinterpret_cast<hipUserObject_t>(new fake::Object{p, fn});
  return hipSuccess;
}
hipError_t hipGraphRetainUserObject(hipGraph_t g, hipUserObject_t o, unsigned, unsigned) {
  fake::graphs[reinterpret_cast<uintptr_t>(g)].push_back(reinterpret_cast<fake::Object*>(o));
  return hipSuccess;
}
hipError_t hipUserObjectRelease(hipUserObject_t, unsigned) { return hipSuccess; }
hipError_t hipThreadExchangeStreamCaptureMode(hipStreamCaptureMode*) { return hipSuccess; }
hipError_t hipStreamCreateWithFlags(hipStream_t* s, unsigned) {
  static int k = 1000;
  *s = fake::stream(k++);
  return hipSuccess;
}
hipError_t hipStreamDestroy(hipStream_t) { return hipSuccess; }
hipError_t hipStreamBeginCapture(hipStream_t, hipStreamCaptureMode) { return hipSuccess; }
hipError_t hipStreamEndCapture(hipStream_t, hipGraph_t* g) {
  *g = reinterpret_cast<hipGraph_t>(uintptr_t(0x77));
  return hipSuccess;
}
hipError_t hipStreamWaitEvent(hipStream_t, hipEvent_t, unsigned) { return hipSuccess; }
hipError_t hipGraphInstantiate(hipGraphExec_t* e, hipGraph_t, hipGraphNode_t*, char*, size_t) {
  *e = reinterpret_cast<hipGraphExec_t>(uintptr_t(0x78));
  return hipSuccess;
}
hipError_t hipGraphLaunch(hipGraphExec_t, hipStream_t) { return hipSuccess; }
hipError_t hipGraphDestroy(hipGraph_t) { return hipSuccess; }
hipError_t hipGraphExecDestroy(hipGraphExec_t) { return hipSuccess; }
hipError_t hipEventCreate(hipEvent_t* e) {
  *e = nullptr;
  return hipSuccess;
}
hipError_t hipEventCreateWithFlags(hipEvent_t* e, unsigned) { return hipEventCreate(e); }
hipError_t hipEventDestroy(hipEvent_t) { return hipSuccess; }
hipError_t hipEventRecord(hipEvent_t, hipStream_t) { return hipSuccess; }
hipError_t hipEventSynchronize(hipEvent_t) { return hipSuccess; }
hipError_t hipEventElapsedTime(float* ms, hipEvent_t, hipEvent_t) {
  *ms = 0.f;
  return hipSuccess;
}

}  // extern "C"
