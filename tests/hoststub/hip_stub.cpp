// A HIP runtime that computes nothing, for tests of librel's host side without a
// GPU: memory up to a limit, kernel launches noted by name, streams that the test
// declares destroyed. Loaded before librel with global symbols, it takes the
// runtime's place there.
#define __HIP_PLATFORM_AMD__
#include <hip/hip_runtime_api.h>
#include <sys/mman.h>

#include <cstring>
#include <map>
#include <set>
#include <string>

namespace {
struct Config { dim3 grid, block; size_t shm; hipStream_t stream; };
Config g_config;
std::map<const void*, std::string> g_names;
std::map<void*, size_t> g_live;
std::set<void*> g_dead;
size_t g_limit = ~size_t(0), g_used = 0;
int g_frees = 0, g_dead_uses = 0;
bool g_capture = false;
std::string g_log;

hipError_t use(hipStream_t s) {
  if (g_dead.count(s)) ++g_dead_uses;
  return hipSuccess;
}
}  // namespace

extern "C" {

void stub_limit(size_t bytes) { g_limit = bytes; }
size_t stub_used() { return g_used; }
int stub_frees() { return g_frees; }
int stub_dead_uses() { return g_dead_uses; }
void stub_kill(void* stream) { g_dead.insert(stream); }
void stub_revive(void* stream) { g_dead.erase(stream); }
void stub_capture(int on) { g_capture = on != 0; }
void stub_clear_log() { g_log.clear(); }
const char* stub_log() { return g_log.c_str(); }  // "kernel workgroups\n" per launch

void** __hipRegisterFatBinary(const void*) { static void* h; return &h; }
void __hipUnregisterFatBinary(void**) {}
void __hipRegisterFunction(void**, const void* f, char*, const char* name, unsigned, void*, void*, void*, void*, int*) { g_names[f] = name; }
void __hipRegisterVar(void**, void*, char*, char*, int, size_t, int, int) {}
hipError_t __hipPushCallConfiguration(dim3 g, dim3 b, size_t m, hipStream_t s) { g_config = {g, b, m, s}; return hipSuccess; }
hipError_t __hipPopCallConfiguration(dim3* g, dim3* b, size_t* m, hipStream_t* s) {
  *g = g_config.grid; *b = g_config.block; *m = g_config.shm; *s = g_config.stream;
  return hipSuccess;
}
hipError_t hipLaunchKernel(const void* f, dim3 g, dim3, void**, size_t, hipStream_t s) {
  g_log += g_names[f] + " " + std::to_string(g.x) + "\n";
  return use(s);
}

hipError_t hipMalloc(void** p, size_t n) {
  if (g_used + n > g_limit) return hipErrorOutOfMemory;
  void* q = mmap(nullptr, n ? n : 1, PROT_READ | PROT_WRITE, MAP_PRIVATE | MAP_ANONYMOUS | MAP_NORESERVE, -1, 0);
  if (q == MAP_FAILED) return hipErrorOutOfMemory;
  g_live[q] = n;
  g_used += n;
  *p = q;
  return hipSuccess;
}
hipError_t hipFree(void* p) {
  auto it = g_live.find(p);
  if (it == g_live.end()) return p ? hipErrorInvalidValue : hipSuccess;
  munmap(p, it->second ? it->second : 1);
  g_used -= it->second;
  g_live.erase(it);
  ++g_frees;
  return hipSuccess;
}
hipError_t hipHostMalloc(void** p, size_t n, unsigned) { *p = calloc(1, n); return hipSuccess; }
hipError_t hipHostFree(void* p) { free(p); return hipSuccess; }
hipError_t hipMemcpy(void* d, const void* s, size_t n, hipMemcpyKind) { memcpy(d, s, n); return hipSuccess; }
hipError_t hipMemcpyAsync(void* d, const void* s, size_t n, hipMemcpyKind, hipStream_t st) { memcpy(d, s, n); return use(st); }
hipError_t hipGetSymbolAddress(void** p, const void*) { static char word[64]; *p = word; return hipSuccess; }

hipError_t hipGetDeviceCount(int* n) { *n = 1; return hipSuccess; }
hipError_t hipSetDevice(int) { return hipSuccess; }
hipError_t hipGetDevicePropertiesR0600(hipDeviceProp_tR0600* p, int) {
  memset(p, 0, sizeof *p);
  p->multiProcessorCount = 256;
  p->sharedMemPerBlock = 65536;
  return hipSuccess;
}
hipError_t hipGetLastError() { return hipSuccess; }
const char* hipGetErrorString(hipError_t) { return "stub"; }
hipError_t hipFuncSetAttribute(const void*, hipFuncAttribute, int) { return hipSuccess; }

hipError_t hipStreamCreateWithFlags(hipStream_t* s, unsigned) { *s = (hipStream_t)malloc(8); return hipSuccess; }
hipError_t hipStreamDestroy(hipStream_t) { return hipSuccess; }
hipError_t hipStreamSynchronize(hipStream_t s) { return use(s); }
hipError_t hipStreamWaitEvent(hipStream_t s, hipEvent_t, unsigned) { return use(s); }
hipError_t hipStreamIsCapturing(hipStream_t s, hipStreamCaptureStatus* st) {
  *st = g_capture ? hipStreamCaptureStatusActive : hipStreamCaptureStatusNone;
  return use(s);
}
hipError_t hipEventCreate(hipEvent_t* e) { *e = (hipEvent_t)malloc(8); return hipSuccess; }
hipError_t hipEventCreateWithFlags(hipEvent_t* e, unsigned) { return hipEventCreate(e); }
hipError_t hipEventDestroy(hipEvent_t) { return hipSuccess; }
hipError_t hipEventRecord(hipEvent_t, hipStream_t s) { return use(s); }
hipError_t hipEventElapsedTime(float* ms, hipEvent_t, hipEvent_t) { *ms = 0; return hipSuccess; }

hipError_t hipStreamBeginCapture(hipStream_t, hipStreamCaptureMode) { return hipSuccess; }
hipError_t hipStreamEndCapture(hipStream_t, hipGraph_t* g) { *g = (hipGraph_t)malloc(8); return hipSuccess; }
hipError_t hipGraphInstantiate(hipGraphExec_t* e, hipGraph_t, hipGraphNode_t*, char*, size_t) { *e = (hipGraphExec_t)malloc(8); return hipSuccess; }
hipError_t hipGraphLaunch(hipGraphExec_t, hipStream_t s) { return use(s); }
hipError_t hipGraphExecDestroy(hipGraphExec_t) { return hipSuccess; }
hipError_t hipGraphDestroy(hipGraph_t) { return hipSuccess; }

}  // extern "C"
