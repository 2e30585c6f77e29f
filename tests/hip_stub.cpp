// A HIP runtime that runs nothing: preloaded before librid.so, it serves the
// library's host code on a machine without a GPU.  Device memory is host
// memory, kernel launches are logged by name and may be told to fail, and so
// may allocations.  What a call would launch, allocate and report can then be
// tested on the CPU.  Host compiler only.
#include <cstddef>
#include <cstdint>
#include <cstdlib>
#include <cstring>
#include <map>
#include <string>

namespace {
struct Dim3 {
  uint32_t x, y, z;
};
struct Config {
  Dim3 grid, block;
  size_t lds;
  void* stream;
};
constexpr int kOk = 0, kOutOfMemory = 2, kLaunchFailure = 719;
thread_local Config config;
thread_local int last_error = kOk;
std::map<const void*, std::string>& names() {
  static std::map<const void*, std::string> m;
  return m;
}
std::string log_text, fail_launch;
int allocations = 0;
bool fail_alloc = false;

int launch(const void* f) {
  auto it = names().find(f);
  const std::string n = it == names().end() ? "?" : it->second;
  if (!fail_launch.empty() && n.find(fail_launch) != std::string::npos) {
    fail_launch.clear();
    return last_error = kLaunchFailure;
  }
  log_text += n + "\n";
  return kOk;
}
}  // namespace

extern "C" {
// the log of kernel names since the last call (valid until the next one)
const char* stub_take_log() {
  static std::string taken;
  taken.swap(log_text);
  log_text.clear();
  return taken.c_str();
}
// the next launch of a kernel whose name holds `part` fails
void stub_fail_next_launch(const char* part) { fail_launch = part; }
void stub_fail_allocations(int on) { fail_alloc = on != 0; }
int stub_allocations() { return allocations; }

void** __hipRegisterFatBinary(const void*) {
  static void* h;
  return &h;
}
void __hipUnregisterFatBinary(void**) {}
void __hipRegisterFunction(void**, const void* host, char*, const char* name, unsigned, void*,
                           void*, void*, void*, int*) {
  names()[host] = name;
}
void __hipRegisterVar(void**, void*, char*, char*, int, size_t, int, int) {}
int __hipPushCallConfiguration(Dim3 g, Dim3 b, size_t lds, void* st) {
  config = Config{g, b, lds, st};
  return kOk;
}
int __hipPopCallConfiguration(Dim3* g, Dim3* b, size_t* lds, void** st) {
  *g = config.grid;
  *b = config.block;
  *lds = config.lds;
  *st = config.stream;
  return kOk;
}
int hipLaunchKernel(const void* f, Dim3, Dim3, void**, size_t, void*) { return launch(f); }
int hipExtLaunchKernel(const void* f, Dim3, Dim3, void**, size_t, void*, void*, void*, int) {
  return launch(f);
}
int hipMalloc(void** p, size_t n) {
  if (fail_alloc) return last_error = kOutOfMemory;
  ++allocations;
  *p = std::calloc(1, n ? n : 1);
  return *p ? kOk : kOutOfMemory;
}
int hipFree(void* p) {
  std::free(p);
  return kOk;
}
int hipMemcpy(void* d, const void* s, size_t n, int) {
  std::memcpy(d, s, n);
  return kOk;
}
int hipMemcpyAsync(void* d, const void* s, size_t n, int, void*) {
  std::memcpy(d, s, n);
  return kOk;
}
int hipMemset(void* d, int v, size_t n) {
  std::memset(d, v, n);
  return kOk;
}
int hipGetLastError() {
  const int e = last_error;
  last_error = kOk;
  return e;
}
const char* hipGetErrorString(int) { return "stub error"; }
int hipDeviceSynchronize() { return kOk; }
int hipStreamSynchronize(void*) { return kOk; }
int hipFuncSetAttribute(const void*, int, int) { return kOk; }
int hipGetDevice(int* d) {
  *d = 0;
  return kOk;
}
int hipSetDevice(int) { return kOk; }
}
