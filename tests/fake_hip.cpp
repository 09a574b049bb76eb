// The part of the HIP runtime that libcitrus.so calls, for tests of its host side on a machine without a GPU.  Loaded in front
// of the real library: every launch is recorded (kernel, grid, workgroup, LDS) and none is made; the n-th can be told to fail.  A
// grid of 2^32 or more work-items in a dimension is refused, as the runtime refuses it.
#include <cxxabi.h>
#include <stdint.h>
#include <stdio.h>
#include <stdlib.h>
#include <string.h>

#include <map>
#include <string>

struct dim3 {
  uint32_t x, y, z;
};

namespace {
std::map<const void*, std::string> names;
std::string log_text;
dim3 call_grid, call_block;
size_t call_shared;
void* call_stream;
int launches = 0, fail_at = -1, last_error = 0, compute_units = 256;
alignas(256) char device_array[256];

void note(const char* what, const std::string& text) { log_text += std::string(what) + " " + text + "\n"; }
std::string kernel_name(const void* host) {
  const auto it = names.find(host);
  if (it == names.end()) return "?";
  int status = 0;
  char* d = abi::__cxa_demangle(it->second.c_str(), nullptr, nullptr, &status);
  std::string s = status == 0 ? d : it->second;
  free(d);
  return s;
}
}  // namespace

extern "C" {
void fake_reset(int n) { log_text.clear(); launches = 0; fail_at = n; last_error = 0; }
void fake_compute_units(int n) { compute_units = n; }  // before the first call
const char* fake_log() { return log_text.c_str(); }

void** __hipRegisterFatBinary(const void*) { static void* handle; return &handle; }
void __hipUnregisterFatBinary(void**) {}
void __hipRegisterFunction(void**, const void* host, char* name, const char*, unsigned, void*, void*, void*, void*, int*) { names[host] = name; }
void __hipRegisterVar(void**, void*, char*, char*, int, size_t, int, int) {}
int __hipPushCallConfiguration(dim3 grid, dim3 block, size_t shared, void* stream) {
  call_grid = grid; call_block = block; call_shared = shared; call_stream = stream;
  return 0;
}
int __hipPopCallConfiguration(dim3* grid, dim3* block, size_t* shared, void** stream) {
  *grid = call_grid; *block = call_block; *shared = call_shared; *stream = call_stream;
  return 0;
}
int hipLaunchKernel(const void* host, dim3 grid, dim3 block, void**, size_t shared, void*) {
  const bool refused = uint64_t{grid.x} * block.x >> 32 || uint64_t{grid.y} * block.y >> 32 || uint64_t{grid.z} * block.z >> 32;
  if (launches++ == fail_at || refused) return last_error = 9;  // hipErrorInvalidConfiguration
  char buf[128];
  snprintf(buf, sizeof buf, "[%u %u %u] [%u %u %u] %zu ", grid.x, grid.y, grid.z, block.x, block.y, block.z, shared);
  note("launch", buf + kernel_name(host));
  return 0;
}
int hipGetLastError() { const int e = last_error; last_error = 0; return e; }
int hipFuncSetAttribute(const void* host, int, int value) { note("lds", std::to_string(value) + " " + kernel_name(host)); return 0; }
int hipGetDevice(int* device) { *device = 0; return 0; }
int hipDeviceGetAttribute(int* value, int, int) { *value = compute_units; return 0; }
int hipGetSymbolAddress(void** address, const void*) { *address = device_array; return 0; }
int hipEventRecord(void*, void*) { return 0; }
int hipStreamWaitEvent(void*, void*, unsigned) { return 0; }
int hipStreamSynchronize(void*) { return 0; }
}
