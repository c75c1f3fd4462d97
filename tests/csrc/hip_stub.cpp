// A HIP runtime without a device, for tests of the library's host code: memory
// is host memory, kernels are counted by name and not run, streams, events and
// graphs are handles without a meaning (work of a capture is counted once, its
// replays are not).  Loaded with RTLD_GLOBAL before the library, so that the
// library's HIP calls bind to it.  Own control: stub_* below.
#include <cstdint>
#include <cstdlib>
#include <cstring>
#include <map>
#include <string>

namespace {
struct Dim3 {
  uint32_t x, y, z;
};
struct Launch {
  Dim3 grid, block;
  size_t shmem;
  void* stream;
} pushed;
std::map<const void*, std::string>& names() {
  static std::map<const void*, std::string> m;
  return m;
}
std::map<std::string, long>& counts() {
  static std::map<std::string, long> m;
  return m;
}
long mallocs = 0, fail_at = 0;
constexpr int kOutOfMemory = 2;
int handle;

int launch(const void* f, void** args) {
  const std::string& n = names()[f];
  ++counts()[n];
  if (n.find("k_set_int") != std::string::npos) {  // the error flags of a factorisation
    int* p = *static_cast<int**>(args[0]);
    p[0] = *static_cast<int*>(args[1]);
    p[1] = 0;
  }
  return 0;
}
}  // namespace

extern "C" {
// the n-th allocation of device memory from now on fails (0: none)
void stub_fail_at(long n) {
  mallocs = 0;
  fail_at = n;
}
long stub_mallocs() { return mallocs; }
void stub_clear_counts() { counts().clear(); }
// launches of the kernels whose (mangled) name holds `part`
long stub_launches(const char* part) {
  long s = 0;
  for (const auto& c : counts())
    if (c.first.find(part) != std::string::npos) s += c.second;
  return s;
}

void** __hipRegisterFatBinary(const void*) {
  static void* m = &handle;
  return &m;
}
void __hipRegisterFunction(void**, const void* f, char*, const char* name, unsigned, void*, void*, void*, void*, int*) {
  names()[f] = name;
}
void __hipRegisterVar(void**, void*, char*, char*, int, size_t, int, int) {}
void __hipUnregisterFatBinary(void**) {}
int __hipPushCallConfiguration(Dim3 g, Dim3 b, size_t shmem, void* s) {
  pushed = {g, b, shmem, s};
  return 0;
}
int __hipPopCallConfiguration(Dim3* g, Dim3* b, size_t* shmem, void** s) {
  *g = pushed.grid;
  *b = pushed.block;
  *shmem = pushed.shmem;
  *s = pushed.stream;
  return 0;
}
int hipLaunchKernel(const void* f, Dim3, Dim3, void** args, size_t, void*) { return launch(f, args); }
int hipExtLaunchKernel(const void* f, Dim3, Dim3, void** args, size_t, void*, void*, void*, int) {
  return launch(f, args);
}

int hipMalloc(void** p, size_t n) {
  if (++mallocs == fail_at) return kOutOfMemory;
  *p = std::calloc(1, n);
  return *p ? 0 : kOutOfMemory;
}
int hipFree(void* p) {
  std::free(p);
  return 0;
}
int hipHostMalloc(void** p, size_t n, unsigned) {
  *p = std::calloc(1, n);
  return *p ? 0 : kOutOfMemory;
}
int hipHostFree(void* p) {
  std::free(p);
  return 0;
}
int hipMemcpyAsync(void* d, const void* s, size_t n, int, void*) {
  std::memcpy(d, s, n);
  return 0;
}
int hipMemsetAsync(void* d, int v, size_t n, void*) {
  std::memset(d, v, n);
  return 0;
}

static int give(void** p) {
  *p = &handle;
  return 0;
}
int hipEventCreate(void** e) { return give(e); }
int hipEventCreateWithFlags(void** e, unsigned) { return give(e); }
int hipEventDestroy(void*) { return 0; }
// every interval shorter than the one before, so that a timed search takes
// whatever it times last
int hipEventElapsedTime(float* ms, void*, void*) {
  static float t = 1000.0f;
  *ms = t *= 0.999f;
  return 0;
}
int hipEventRecord(void*, void*) { return 0; }
int hipEventSynchronize(void*) { return 0; }
int hipStreamCreateWithFlags(void** s, unsigned) { return give(s); }
int hipStreamDestroy(void*) { return 0; }
int hipStreamSynchronize(void*) { return 0; }
int hipStreamWaitEvent(void*, void*, unsigned) { return 0; }
int hipStreamBeginCapture(void*, int) { return 0; }
int hipStreamEndCapture(void*, void** g) { return give(g); }
int hipStreamIsCapturing(void*, int* status) {
  *status = 0;
  return 0;
}
int hipThreadExchangeStreamCaptureMode(int*) { return 0; }
int hipGraphInstantiate(void** e, void*, void**, char*, size_t) { return give(e); }
int hipGraphLaunch(void*, void*) { return 0; }
int hipGraphDestroy(void*) { return 0; }
int hipGraphExecDestroy(void*) { return 0; }
int hipGetDevice(int* d) {
  *d = 0;
  return 0;
}
int hipGetDevicePropertiesR0600(void* p, int) {
  std::memset(p, 0, 1472);  // sizeof(hipDeviceProp_t)
  return 0;
}
int hipGetSymbolAddress(void** p, const void*) { return give(p); }
int hipGetLastError() { return 0; }
const char* hipGetErrorString(int) { return "stub"; }
}
