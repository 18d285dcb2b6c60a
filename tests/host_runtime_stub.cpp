// Stands in for the HIP runtime in a process without a GPU: the library's host code runs, every call is
// written to a log, allocations and captures can be made to fail.  Errors stay until hipGetLastError reads
// them, as in the runtime.  Loaded ahead of the library, so that its symbols are found first.
#include <cstdint>
#include <cstdio>
#include <map>
#include <string>

namespace {
std::map<const void*, std::string> g_names;
std::string g_log;
int g_error = 0, g_fail_malloc = 0, g_capturing = 0, g_fail_query = 0;
uint64_t g_next = 0x700000000000ull;
struct Dim3 { uint32_t x, y, z; };
struct Config { Dim3 grid, block; size_t shared; void* stream; } g_config;

template <class... T>
void note(const char* format, T... values) {
  char line[4096];
  std::snprintf(line, sizeof line, format, values...);
  g_log += line;
  g_log += '\n';
}
int fail(int error) { return g_error = error; }
}  // namespace

extern "C" {
void stub_set(int fail_malloc, int capturing, int fail_query) { g_fail_malloc = fail_malloc; g_capturing = capturing; g_fail_query = fail_query; }
const char* stub_take_log() { static std::string out; out.swap(g_log); g_log.clear(); return out.c_str(); }

int hipGetDevice(int* dev) { *dev = 0; return 0; }
int hipMalloc(void** ptr, size_t bytes) {
  note("malloc %zu", bytes);
  if (g_fail_malloc) return fail(2);
  *ptr = reinterpret_cast<void*>(g_next);
  g_next += (bytes + 4095) & ~size_t(4095);
  return 0;
}
int hipFree(void*) { note("%s", "free"); return 0; }
int hipMemsetAsync(void*, int, size_t bytes, void*) { note("memset %zu", bytes); return 0; }
int hipStreamSynchronize(void*) { note("%s", "synchronize"); return 0; }
int hipStreamIsCapturing(void*, int* status) { if (g_fail_query) return fail(906); *status = g_capturing; return 0; }
int hipGetLastError() { const int e = g_error; g_error = 0; return e; }
const char* hipGetErrorString(int) { return "stub error"; }
int hipGetSymbolAddress(void** ptr, const void*) { *ptr = reinterpret_cast<void*>(0x600000000000ull); return 0; }
int hipFuncSetAttribute(const void*, int, int) { return 0; }
int hipLaunchKernel(const void* f, Dim3 grid, Dim3, void**, size_t, void*) {
  note("launch %s %u %u %u", g_names[f].c_str(), grid.x, grid.y, grid.z);
  return 0;
}
void** __hipRegisterFatBinary(const void*) { static void* handle = nullptr; return &handle; }
void __hipUnregisterFatBinary(void**) {}
void __hipRegisterFunction(void**, const void* host, char*, const char* device, unsigned, void*, void*, void*, void*, int*) { g_names[host] = device; }
void __hipRegisterVar(void**, void*, char*, char* device, int, size_t bytes, int, int) { note("variable %s %zu", device, bytes); }
int __hipPushCallConfiguration(Dim3 grid, Dim3 block, size_t shared, void* stream) { g_config = {grid, block, shared, stream}; return 0; }
int __hipPopCallConfiguration(Dim3* grid, Dim3* block, size_t* shared, void** stream) {
  *grid = g_config.grid; *block = g_config.block; *shared = g_config.shared; *stream = g_config.stream;
  return 0;
}
}
