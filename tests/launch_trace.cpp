// Host stand-in for the HIP runtime calls that libqn makes (built and loaded by
// launch_trace.py ahead of the library).  Launches, copies and events do
// nothing; every launch and every raised LDS limit is a line of a log:
//   raise DEVICE KERNEL
//   launch DEVICE GRID BLOCK LDS SPAN KERNEL
// SPAN: for k_fast_rows the largest distance, in bytes, of a workgroup's rows
// from its first one (input or output), which the kernel holds in 32 bits.
#include <cxxabi.h>
#include <hip/hip_runtime.h>

#include <algorithm>
#include <cstdio>
#include <cstdlib>
#include <map>
#include <string>

#include "qn_internal.h"

namespace {
std::map<const void*, std::string> names;
std::string text;
int device = 0;
struct Config {
  dim3 grid, block;
  size_t lds;
  hipStream_t st;
} config;

const std::string& name_of(const void* f) {
  static const std::string unknown = "?";
  auto it = names.find(f);
  return it == names.end() ? unknown : it->second;
}

long long rows_span(const qn::RowArgs& a) {
  auto off = [&](int r, long long s1, long long s0, long long ys) {
    const int pl = r / a.oy;
    return (pl / a.om) * s1 + (pl % a.om) * s0 + (r - pl * (long long)a.oy) * ys;
  };
  long long span = 0;
  for (int r0 = 0; r0 < a.rows; r0 += a.lines) {
    const int r1 = std::min(r0 + a.lines, a.rows) - 1;
    const long long in = off(r1, a.is1, a.is0, a.iys) - off(r0, a.is1, a.is0, a.iys);
    const long long out = off(r1, a.s1, a.s0, a.ys) - off(r0, a.s1, a.s0, a.ys);
    span = std::max({span, 8 * in, 8 * out});
  }
  return span;
}
}  // namespace

extern "C" {
const char* trace_text() { return text.c_str(); }
void trace_clear() { text.clear(); }
void trace_device(int d) { device = d; }
int trace_argument_bytes(int kind) {
  return kind == 0 ? sizeof(qn::EpiArgs) : kind == 1 ? sizeof(qn::LineArgs) : sizeof(qn::RowArgs);
}

void** __hipRegisterFatBinary(const void*) {
  static void* module;
  return &module;
}
void __hipUnregisterFatBinary(void**) {}
void __hipRegisterVar(void**, void*, char*, char*, int, size_t, int, int) {}
void __hipRegisterFunction(void**, const void* host, char*, const char* dev, unsigned, void*, void*,
                           dim3*, dim3*, int*) {
  int st = 0;
  char* d = abi::__cxa_demangle(dev, nullptr, nullptr, &st);
  names[host] = d ? d : dev;
  std::free(d);
}
hipError_t __hipPushCallConfiguration(dim3 g, dim3 b, size_t lds, hipStream_t st) {
  config = {g, b, lds, st};
  return hipSuccess;
}
hipError_t __hipPopCallConfiguration(dim3* g, dim3* b, size_t* lds, hipStream_t* st) {
  *g = config.grid;
  *b = config.block;
  *lds = config.lds;
  *st = config.st;
  return hipSuccess;
}
hipError_t hipLaunchKernel(const void* f, dim3 g, dim3 b, void** args, size_t lds, hipStream_t) {
  const std::string& n = name_of(f);
  long long span = 0;
  if (n.find("k_fast_rows<") != std::string::npos)
    span = rows_span(*static_cast<const qn::RowArgs*>(args[0]));
  char buf[160];
  std::snprintf(buf, sizeof buf, "launch %d %lld %d %zu %lld ", device,
                (long long)g.x * g.y * g.z, (int)(b.x * b.y * b.z), lds, span);
  text += buf + n + "\n";
  return hipSuccess;
}
hipError_t hipFuncSetAttribute(const void* f, hipFuncAttribute, int) {
  text += "raise " + std::to_string(device) + " " + name_of(f) + "\n";
  return hipSuccess;
}
hipError_t hipGetDevice(int* d) {
  *d = device;
  return hipSuccess;
}
const char* hipGetErrorString(hipError_t) { return "error"; }
hipError_t hipGetLastError() { return hipSuccess; }
hipError_t hipGetSymbolAddress(void** p, const void*) {
  *p = reinterpret_cast<void*>(1 << 20);
  return hipSuccess;
}
hipError_t hipHostMalloc(void** p, size_t n, unsigned) {
  *p = std::calloc(n, 1);
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
hipError_t hipMemcpyAsync(void*, const void*, size_t, hipMemcpyKind, hipStream_t) { return hipSuccess; }
hipError_t hipEventCreate(hipEvent_t* e) {
  *e = reinterpret_cast<hipEvent_t>(1);
  return hipSuccess;
}
hipError_t hipEventCreateWithFlags(hipEvent_t* e, unsigned) { return hipEventCreate(e); }
hipError_t hipEventDestroy(hipEvent_t) { return hipSuccess; }
hipError_t hipEventRecord(hipEvent_t, hipStream_t) { return hipSuccess; }
hipError_t hipEventSynchronize(hipEvent_t) { return hipSuccess; }
hipError_t hipEventElapsedTime(float* ms, hipEvent_t, hipEvent_t) {
  *ms = 1.f;
  return hipSuccess;
}
hipError_t hipStreamCreateWithFlags(hipStream_t* s, unsigned) {
  *s = reinterpret_cast<hipStream_t>(1);
  return hipSuccess;
}
hipError_t hipStreamDestroy(hipStream_t) { return hipSuccess; }
hipError_t hipStreamSynchronize(hipStream_t) { return hipSuccess; }
hipError_t hipStreamWaitEvent(hipStream_t, hipEvent_t, unsigned) { return hipSuccess; }
hipError_t hipStreamBeginCapture(hipStream_t, hipStreamCaptureMode) { return hipSuccess; }
hipError_t hipStreamEndCapture(hipStream_t, hipGraph_t* g) {
  *g = reinterpret_cast<hipGraph_t>(1);
  return hipSuccess;
}
hipError_t hipGraphInstantiate(hipGraphExec_t* e, hipGraph_t, hipGraphNode_t*, char*, size_t) {
  *e = reinterpret_cast<hipGraphExec_t>(1);
  return hipSuccess;
}
hipError_t hipGraphLaunch(hipGraphExec_t, hipStream_t) { return hipSuccess; }
hipError_t hipGraphExecDestroy(hipGraphExec_t) { return hipSuccess; }
hipError_t hipGraphDestroy(hipGraph_t) { return hipSuccess; }
}
