// A HIP runtime without a GPU, for tests of the library's host code: "device" memory is host memory, kernel launches are
// noted by name and not carried out, and the library's host allocations can be made to fail.  Built as
// libamdhip64.so.7 and found before the real one (see __init__.py); defines just what libbca.so uses.
#include <hip/hip_runtime_api.h>

#include <cstdlib>
#include <cstring>
#include <iterator>
#include <map>
#include <new>
#include <string>
#include <vector>

namespace {
std::map<const void*, std::string>& names() {
  static std::map<const void*, std::string> m;
  return m;
}
struct Launch {
  const void* kernel;
  unsigned grid;
  size_t lds;
  std::vector<char> arg;
};
std::vector<Launch>& launches() {
  static std::vector<Launch> v;
  return v;
}
bool g_fail = false;
unsigned long long g_mallocs = 0, g_frees = 0;
std::string g_watched;  // kernels of whose argument number g_arg the first g_arg_bytes bytes are kept
unsigned g_arg = 0, g_arg_bytes = 0;
int g_cus = 256;
size_t g_static_lds = 0;
struct Config {
  dim3 grid, block;
  size_t lds;
  hipStream_t stream;
} g_config;
}  // namespace

// The library resolves these to the runtime's copy, which comes before the standard library in its list.
void* operator new(size_t n) {
  void* p = g_fail ? nullptr : malloc(n ? n : 1);
  if (!p) throw std::bad_alloc();
  return p;
}
void* operator new(size_t n, const std::nothrow_t&) noexcept { return g_fail ? nullptr : malloc(n ? n : 1); }
void operator delete(void* p) noexcept { free(p); }
void operator delete(void* p, size_t) noexcept { free(p); }
void operator delete(void* p, const std::nothrow_t&) noexcept { free(p); }

extern "C" {

// ---- for the tests
void fake_fail_host_allocations(int on) { g_fail = on != 0; }
unsigned long long fake_device_allocations() { return g_mallocs; }
unsigned long long fake_device_frees() { return g_frees; }
void fake_set_cus(int n) { g_cus = n; }
void fake_set_static_lds(unsigned n) { g_static_lds = n; }  // what every kernel is said to have
unsigned fake_num_launches() { return (unsigned)launches().size(); }
const char* fake_launch_name(unsigned i) { return names()[launches()[i].kernel].c_str(); }
unsigned fake_launch_grid(unsigned i) { return launches()[i].grid; }
unsigned fake_launch_lds(unsigned i) { return (unsigned)launches()[i].lds; }
void fake_watch(const char* kernel, unsigned arg, unsigned n_bytes) { g_watched = kernel, g_arg = arg, g_arg_bytes = n_bytes; }
const char* fake_launch_arg(unsigned i) { return launches()[i].arg.empty() ? nullptr : launches()[i].arg.data(); }
unsigned fake_num_kernels() { return (unsigned)names().size(); }
const char* fake_kernel_name(unsigned i) { return std::next(names().begin(), i)->second.c_str(); }  // every kernel the library has
void fake_forget_launches() { launches().clear(); }

// ---- the runtime
void** __hipRegisterFatBinary(const void*) {
  static void* handle;
  return &handle;
}
void __hipUnregisterFatBinary(void**) {}
void __hipRegisterFunction(void**, const void* host, char*, const char* device, unsigned, void*, void*, void*, void*, int*) {
  names()[host] = device;
}
void __hipRegisterVar(void**, void*, char*, char*, int, size_t, int, int) {}
hipError_t __hipPushCallConfiguration(dim3 grid, dim3 block, size_t lds, hipStream_t stream) {
  g_config = {grid, block, lds, stream};
  return hipSuccess;
}
hipError_t __hipPopCallConfiguration(dim3* grid, dim3* block, size_t* lds, hipStream_t* stream) {
  *grid = g_config.grid, *block = g_config.block, *lds = g_config.lds, *stream = g_config.stream;
  return hipSuccess;
}
hipError_t hipLaunchKernel(const void* f, dim3 grid, dim3, void** args, size_t lds, hipStream_t) {
  const bool failing = g_fail;  // the note is the test's, not the library's
  g_fail = false;
  launches().push_back({f, grid.x, lds, {}});
  if (g_arg_bytes != 0 && names()[f].find(g_watched) != std::string::npos)
    launches().back().arg.assign((const char*)args[g_arg], (const char*)args[g_arg] + g_arg_bytes);
  g_fail = failing;
  return hipSuccess;
}
hipError_t hipMalloc(void** p, size_t n) {
  ++g_mallocs;
  *p = aligned_alloc(4096, (n + 4095) / 4096 * 4096 + 4096);
  return *p ? hipSuccess : hipErrorOutOfMemory;
}
hipError_t hipFree(void* p) {
  g_frees += p != nullptr;
  free(p);
  return hipSuccess;
}
hipError_t hipMemcpy(void* d, const void* s, size_t n, hipMemcpyKind) {
  memcpy(d, s, n);
  return hipSuccess;
}
hipError_t hipMemset(void* d, int x, size_t n) {
  memset(d, x, n);
  return hipSuccess;
}
hipError_t hipGetSymbolAddress(void** p, const void* symbol) {
  *p = const_cast<void*>(symbol);
  return hipSuccess;
}
hipError_t hipSetDevice(int) { return hipSuccess; }
hipError_t hipGetDevice(int* d) {
  *d = 0;
  return hipSuccess;
}
hipError_t hipGetDeviceCount(int* n) {
  *n = 1;
  return hipSuccess;
}
hipError_t hipGetDeviceProperties(hipDeviceProp_t* prop, int) {
  memset(prop, 0, sizeof *prop);
  prop->warpSize = 64, prop->multiProcessorCount = g_cus;
  return hipSuccess;
}
hipError_t hipDeviceGetAttribute(int* x, hipDeviceAttribute_t, int) {
  *x = g_cus;
  return hipSuccess;
}
hipError_t hipFuncGetAttributes(hipFuncAttributes* a, const void*) {
  memset(a, 0, sizeof *a);
  a->sharedSizeBytes = g_static_lds;
  return hipSuccess;
}
hipError_t hipDeviceSynchronize() { return hipSuccess; }
hipError_t hipGetLastError() { return hipSuccess; }
const char* hipGetErrorString(hipError_t) { return "fake"; }
hipError_t hipEventCreate(hipEvent_t* e) {
  *e = (hipEvent_t)malloc(1);
  return hipSuccess;
}
hipError_t hipEventDestroy(hipEvent_t e) {
  free((void*)e);
  return hipSuccess;
}
hipError_t hipEventRecord(hipEvent_t, hipStream_t) { return hipSuccess; }
hipError_t hipEventSynchronize(hipEvent_t) { return hipSuccess; }
hipError_t hipEventElapsedTime(float* t, hipEvent_t, hipEvent_t) {
  *t = 0.f;
  return hipSuccess;
}
}
