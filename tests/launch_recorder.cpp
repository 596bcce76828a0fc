// A stand-in for the part of the HIP runtime that the library calls: it launches nothing and writes down
// what would have been launched.  Loaded with RTLD_GLOBAL in front of the library (tests/launch_recorder.py),
// its symbols are the ones the library binds to, so that the route of a call can be checked without a GPU.
#include <cxxabi.h>
#include <stdint.h>
#include <stdlib.h>

#include <map>
#include <string>

namespace {
struct Dim3 {
  uint32_t x, y, z;
};
struct Config {
  Dim3 grid, block;
  size_t shared;
  void* stream;
} config;
std::map<const void*, std::string> kernels;  // host stub -> demangled device name
std::string launched, names;
void* handle = nullptr;
int error = 0;

void line(std::string& to, const std::string& name, uint32_t grid, uint32_t block) {
  to += name + '\t' + std::to_string(grid) + '\t' + std::to_string(block) + '\n';
}
}  // namespace

extern "C" {
void** __hipRegisterFatBinary(const void*) { return &handle; }
void __hipUnregisterFatBinary(void**) {}
void __hipRegisterVar(void**, void*, char*, char*, int, size_t, int, int) {}
void __hipRegisterFunction(void**, const void* stub, char*, const char* name, unsigned, void*, void*, void*, void*, int*) {
  int status = 0;
  char* const text = abi::__cxa_demangle(name, nullptr, nullptr, &status);
  kernels[stub] = status == 0 ? text : name;
  free(text);
  line(names, kernels[stub], 0, 0);
}
int __hipPushCallConfiguration(Dim3 grid, Dim3 block, size_t shared, void* stream) {
  config = {grid, block, shared, stream};
  return 0;
}
int __hipPopCallConfiguration(Dim3* grid, Dim3* block, size_t* shared, void** stream) {
  *grid = config.grid;
  *block = config.block;
  *shared = config.shared;
  *stream = config.stream;
  return 0;
}
int hipLaunchKernel(const void* stub, Dim3 grid, Dim3 block, void**, size_t, void*) {
  if (grid.x == 0 || (uint64_t)grid.x * block.x >= 1ull << 32) return error = 9;  // (what the runtime refuses)
  line(launched, kernels.count(stub) ? kernels[stub] : "?", grid.x, block.x);
  return 0;
}
int hipGetLastError() {
  const int e = error;
  error = 0;
  return e;
}
int hipGetDevice(int* device) { return *device = 0; }
int hipDeviceGetAttribute(int* value, int, int) {
  *value = 256;  // (the library asks for the number of CUs only)
  return 0;
}
int hipGetSymbolAddress(void** address, const void*) {
  *address = (void*)0x100000;
  return 0;
}
// the launches since the last call, one line each: kernel, workgroups, threads
const char* recorder_take() {
  static std::string out;
  out.swap(launched);
  launched.clear();
  return out.c_str();
}
const char* recorder_kernels() { return names.c_str(); }
}
