// A stand-in for the HIP runtime calls that libltmp2 makes, for host tests of
// its launches, allocations and streams without a GPU: device memory is lazily
// backed host memory, kernels do not run, and every launch, allocation, stream
// creation and memory error is appended to the file FAKE_HIP_LOG.  Loaded with
// RTLD_GLOBAL ahead of the library, it takes precedence over the real runtime.
//
// FAKE_HIP_PRIORITY / FAKE_HIP_CU_MASK: priority and first mask word reported
// for streams that the library did not create.
#include <sys/mman.h>

#include <cstdint>
#include <cstdio>
#include <cstdlib>
#include <cstring>
#include <map>
#include <set>
#include <string>

namespace {

struct Dim3 {
  uint32_t x, y, z;
};

FILE* log_file() {
  static FILE* f = std::fopen(std::getenv("FAKE_HIP_LOG"), "a");
  return f;
}

std::map<const void*, std::string>& names() {
  static std::map<const void*, std::string> m;
  return m;
}
std::map<void*, size_t>& sizes() {
  static std::map<void*, size_t> m;
  return m;
}
std::set<void*>& own_streams() {
  static std::set<void*> s;
  return s;
}

Dim3 g_grid, g_block;
size_t g_shared;
void* g_stream;
uintptr_t g_next = 0x1000;

void* handle() { return reinterpret_cast<void*>(g_next += 16); }

int new_stream(void** s, const char* how) {
  own_streams().insert(*s = handle());
  std::fprintf(log_file(), "stream %s\n", how);
  std::fflush(log_file());
  return 0;
}

}  // namespace

extern "C" {

void** __hipRegisterFatBinary(const void*) {
  static void* h = nullptr;
  return &h;
}
void __hipUnregisterFatBinary(void**) {}
void __hipRegisterFunction(void**, const void* host, char*, const char* name, unsigned, void*,
                           void*, void*, void*, int*) {
  names()[host] = name;
}
void __hipRegisterVar(void**, void*, char*, char*, int, size_t, int, int) {}
int __hipPushCallConfiguration(Dim3 grid, Dim3 block, size_t shared, void* stream) {
  g_grid = grid;
  g_block = block;
  g_shared = shared;
  g_stream = stream;
  return 0;
}
int __hipPopCallConfiguration(Dim3* grid, Dim3* block, size_t* shared, void** stream) {
  *grid = g_grid;
  *block = g_block;
  *shared = g_shared;
  *stream = g_stream;
  return 0;
}
int hipLaunchKernel(const void* f, Dim3 grid, Dim3 block, void**, size_t shared, void* stream) {
  std::fprintf(log_file(), "launch %s %u %u %u %u %zu %p\n", names()[f].c_str(), grid.x, grid.y,
               grid.z, block.x, shared, stream);
  std::fflush(log_file());
  return 0;
}

int hipMalloc(void** p, size_t n) {
  void* q = mmap(nullptr, n, PROT_READ | PROT_WRITE, MAP_PRIVATE | MAP_ANONYMOUS | MAP_NORESERVE,
                 -1, 0);
  if (q == MAP_FAILED) return 2;
  sizes()[*p = q] = n;
  std::fprintf(log_file(), "malloc %zu\n", n);
  std::fflush(log_file());
  return 0;
}
int hipFree(void* p) {
  if (p) munmap(p, sizes()[p]), sizes().erase(p);
  return 0;
}
int hipMemcpy(void* d, const void* s, size_t n, int) {
  std::memcpy(d, s, n);
  return 0;
}
int hipMemcpyAsync(void* d, const void* s, size_t n, int, void*) {
  std::memcpy(d, s, n);
  return 0;
}
int hipMemsetAsync(void*, int, size_t, void*) { return 0; }  // fresh memory is zero

int hipStreamCreate(void** s) { return new_stream(s, "plain"); }
int hipStreamCreateWithFlags(void** s, unsigned flags) {
  return new_stream(s, flags == 1 ? "nonblocking" : "flags");
}
int hipStreamDestroy(void*) { return 0; }
int hipStreamSynchronize(void*) { return 0; }
int hipStreamWaitEvent(void*, void*, unsigned) { return 0; }
int hipStreamGetPriority(void* s, int* p) {
  const char* e = std::getenv("FAKE_HIP_PRIORITY");
  *p = e && !own_streams().count(s) ? std::atoi(e) : 0;
  return 0;
}
int hipExtStreamGetCUMask(void* s, uint32_t words, uint32_t* mask) {
  if (words < 8) return 1;
  for (uint32_t k = 0; k < words; ++k) mask[k] = k < 8 ? 0xffffffffu : 0u;
  const char* e = std::getenv("FAKE_HIP_CU_MASK");
  if (e && !own_streams().count(s)) mask[0] = uint32_t(std::strtoul(e, nullptr, 0));
  return 0;
}
int hipStreamBeginCapture(void*, int) { return 0; }
int hipStreamEndCapture(void*, void** g) {
  *g = handle();
  return 0;
}
int hipGraphInstantiate(void** e, void*, void**, char*, size_t) {
  *e = handle();
  return 0;
}
int hipGraphLaunch(void*, void*) { return 0; }
int hipGraphDestroy(void*) { return 0; }
int hipGraphExecDestroy(void*) { return 0; }

int hipEventCreate(void** e) {
  *e = handle();
  return 0;
}
int hipEventCreateWithFlags(void** e, unsigned) {
  *e = handle();
  return 0;
}
int hipEventDestroy(void*) { return 0; }
int hipEventRecord(void*, void*) { return 0; }
int hipEventElapsedTime(float* ms, void*, void*) {
  *ms = 0.f;
  return 0;
}
int hipFuncSetAttribute(const void*, int, int) { return 0; }
int hipOccupancyMaxActiveBlocksPerMultiprocessor(int* n, const void*, int, size_t) {
  *n = 1;
  return 0;
}
int hipGetDevice(int* d) {
  *d = 0;
  return 0;
}
int hipGetLastError() { return 0; }
const char* hipGetErrorString(int) { return "fake HIP error"; }
int hipGetSymbolAddress(void** p, const void*) {
  *p = nullptr;
  return 1;
}
}
