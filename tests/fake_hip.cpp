// A stand-in for the HIP runtime, for tests that look at what the library enqueues and in which order: loaded in front of the library,
// it takes the place of every runtime function that the library calls, writes launches, event records and stream waits to a log and
// runs nothing.  fake_hip_fail makes the n-th call of a function fail.
#include <cstdint>
#include <cstdio>
#include <cstring>
#include <map>
#include <string>

namespace {
struct Dim3 { uint32_t x, y, z; };
struct Config { Dim3 grid, block; size_t lds; void* stream; };
std::map<const void*, std::string> kernels;
std::string logged;
Config pushed;
int last_error = 0;
uintptr_t next_handle = 0x1000;
std::map<std::string, long> calls, fail_at;
constexpr int kFailure = 999;

int call(const char* fn) {
  const long n = ++calls[fn];
  auto f = fail_at.find(fn);
  if (f == fail_at.end() || f->second != n) return 0;
  last_error = kFailure;
  return kFailure;
}
void put(const char* what, const void* a, const char* b, int rc) {
  char line[1024];
  snprintf(line, sizeof line, "%s %zx %s %d\n", what, (size_t)a, b, rc);
  logged += line;
}
std::string hex(const void* p) { char t[32]; snprintf(t, sizeof t, "%zx", (size_t)p); return t; }
}  // namespace

extern "C" {
const char* fake_hip_log() { return logged.c_str(); }
void fake_hip_reset() { logged.clear(); calls.clear(); fail_at.clear(); last_error = 0; }
void fake_hip_fail(const char* fn, long n) { fail_at[fn] = n; }

void** __hipRegisterFatBinary(const void*) { static void* module; return &module; }
void __hipUnregisterFatBinary(void**) {}
void __hipRegisterFunction(void**, const void* host, char*, const char* name, unsigned, void*, void*, void*, void*, int*) { kernels[host] = name; }
void __hipRegisterVar(void**, void*, char*, char*, int, size_t, int, int) {}
int __hipPushCallConfiguration(Dim3 grid, Dim3 block, size_t lds, void* stream) { pushed = {grid, block, lds, stream}; return 0; }
int __hipPopCallConfiguration(Dim3* grid, Dim3* block, size_t* lds, void** stream) {
  *grid = pushed.grid; *block = pushed.block; *lds = pushed.lds; *stream = pushed.stream;
  return 0;
}
int hipLaunchKernel(const void* f, Dim3, Dim3, void**, size_t, void* stream) {
  const int rc = call("hipLaunchKernel");
  put("launch", stream, kernels.count(f) ? kernels[f].c_str() : "?", rc);
  return rc;
}
int hipEventRecord(void* event, void* stream) { const int rc = call("hipEventRecord"); put("record", stream, hex(event).c_str(), rc); return rc; }
int hipStreamWaitEvent(void* stream, void* event, unsigned) { const int rc = call("hipStreamWaitEvent"); put("wait", stream, hex(event).c_str(), rc); return rc; }
int hipEventCreate(void** e) { const int rc = call("hipEventCreate"); *e = rc ? nullptr : (void*)(next_handle += 16); return rc; }
int hipEventCreateWithFlags(void** e, unsigned) { const int rc = call("hipEventCreateWithFlags"); *e = rc ? nullptr : (void*)(next_handle += 16); return rc; }
int hipStreamCreateWithFlags(void** s, unsigned) { const int rc = call("hipStreamCreateWithFlags"); *s = rc ? nullptr : (void*)(next_handle += 16); return rc; }
int hipEventDestroy(void*) { return 0; }
int hipEventSynchronize(void*) { return 0; }
int hipEventElapsedTime(float* ms, void*, void*) { *ms = 0; return 0; }
int hipStreamSynchronize(void*) { return 0; }
int hipGetDevice(int* d) { *d = 0; return 0; }
int hipGetSymbolAddress(void** p, const void*) { *p = (void*)0x100000; return 0; }
int hipGetLastError() { const int e = last_error; last_error = 0; return e; }
const char* hipGetErrorString(int) { return "fake error"; }
}
