// A stand-in for the HIP runtime that runs no kernels: device memory is host
// memory, launches are written down.  Tests load the product library against
// it to check, without a GPU, what the host side allocates, clears and
// launches, on which device and stream.
//
// Two devices.  Every new allocation is filled with 0xCD.  The start-of-pass
// kernels' clearing of the words they are given is carried out, as far as
// their arguments say; a loss leaves its sums filled with 0xEE, as one that
// was overtaken by another might.  Everything else a kernel would do is left
// out.  In a captured stream nothing is carried out; a loss there counts as
// cleared when its capture clears the sums before it.
#include <hip/hip_runtime_api.h>

#include <cstdint>
#include <cstdio>
#include <cstdlib>
#include <cstring>
#include <map>
#include <set>
#include <string>
#include <vector>

namespace {

struct Alloc { size_t bytes; int device; };
struct Launch {
  std::string name;
  int device;
  unsigned grid[3], block[3];
  size_t lds;
  void* stream;
  uint64_t arg[4];  // see `words`
};
std::map<char*, Alloc> allocs;
std::map<const void*, std::string> names;
std::vector<Launch> launches;
std::vector<int> set_log;
std::set<void*> capturing;
int current = 0;
std::vector<std::pair<uint64_t, uint64_t>> captured_clears;  // first byte, bytes
// a loss's sums: eight doubles 128 bytes apart, after the first the count of finished workgroups
template <typename F> void loss_bytes(uint64_t sums, F f) {
  for (int k = 0; k < 8; ++k)
    for (int i = 0; i < (k == 0 ? 12 : 8); ++i) f(((char*)sums)[128 * k + i]);
}
size_t limit = SIZE_MAX;
char* symbol[2];
struct Config { dim3 grid, block; size_t lds; hipStream_t stream; };
std::vector<Config> configs;

size_t held_bytes = 0;

}  // namespace

extern "C" {

// ------------------------------------------------------------ what tests read
int fake_current() { return current; }
void fake_set_current(int d) { current = d; }
void fake_limit(size_t bytes) { limit = bytes; }
void fake_capture(void* stream, int on) { captured_clears.clear(); if (on) capturing.insert(stream); else capturing.erase(stream); }
size_t fake_held() { return held_bytes; }
// bytes of the allocation that holds p (0: none) and its device
size_t fake_alloc(void* p, int* device, char** base) {
  auto it = allocs.upper_bound((char*)p);
  if (it == allocs.begin()) return 0;
  --it;
  if ((char*)p >= it->first + it->second.bytes) return 0;
  *device = it->second.device;
  *base = it->first;
  return it->second.bytes;
}
int fake_allocs() { return (int)allocs.size(); }
int fake_alloc_device(int i) { auto it = allocs.begin(); std::advance(it, i); return it->second.device; }
int fake_launches() { return (int)launches.size(); }
void fake_clear_launches() { launches.clear(); }
const char* fake_launch(int i, int* device, void** stream, uint64_t* lds, uint64_t* threads, uint64_t* groups, uint64_t* arg) {
  const Launch& l = launches[i];
  *device = l.device; *stream = l.stream; *lds = l.lds;
  *threads = l.block[0]; *groups = (uint64_t)l.grid[0] * l.grid[1];
  memcpy(arg, l.arg, sizeof(l.arg));
  return l.name.c_str();
}

// ------------------------------------------------------------ the runtime
hipError_t hipGetDeviceCount(int* n) { *n = 2; return hipSuccess; }
hipError_t hipSetDevice(int d) { if (d < 0 || d > 1) return hipErrorInvalidDevice; current = d; return hipSuccess; }
hipError_t hipGetDevice(int* d) { *d = current; return hipSuccess; }
hipError_t hipGetDevicePropertiesR0600(hipDeviceProp_tR0600* p, int) {
  memset(p, 0, sizeof(*p));
  p->multiProcessorCount = 256;
  strcpy(p->gcnArchName, "gfx950");
  return hipSuccess;
}
hipError_t hipDeviceGetAttribute(int* v, hipDeviceAttribute_t, int) { *v = 163840; return hipSuccess; }
hipError_t hipFuncSetAttribute(const void*, hipFuncAttribute, int) { return hipSuccess; }
hipError_t hipOccupancyMaxActiveBlocksPerMultiprocessor(int* n, const void*, int block, size_t lds) {
  const int by_threads = 2048 / block, by_lds = lds ? (int)(163840 / lds) : by_threads;
  *n = by_threads < by_lds ? by_threads : by_lds;
  return hipSuccess;
}
hipError_t hipMalloc(void** p, size_t n) {
  *p = nullptr;
  if (held_bytes + n > limit) return hipErrorOutOfMemory;
  char* q = (char*)aligned_alloc(256, (n + 255) / 256 * 256);
  if (!q) return hipErrorOutOfMemory;
  memset(q, 0xCD, n);
  allocs[q] = {n, current};
  held_bytes += n;
  *p = q;
  return hipSuccess;
}
hipError_t hipFree(void* p) {
  if (!p) return hipSuccess;
  auto it = allocs.find((char*)p);
  if (it == allocs.end()) return hipErrorInvalidValue;
  held_bytes -= it->second.bytes;
  allocs.erase(it);
  free(p);
  return hipSuccess;
}
hipError_t hipMemcpy(void* d, const void* s, size_t n, hipMemcpyKind) { memcpy(d, s, n); return hipSuccess; }
hipError_t hipMemcpyAsync(void* d, const void* s, size_t n, hipMemcpyKind, hipStream_t) { memcpy(d, s, n); return hipSuccess; }
hipError_t hipMemset(void* d, int v, size_t n) { memset(d, v, n); return hipSuccess; }
hipError_t hipGetSymbolAddress(void** p, const void*) {
  if (!symbol[current]) symbol[current] = (char*)calloc(1, (size_t)32 << 20);
  *p = symbol[current];
  return hipSuccess;
}
hipError_t hipStreamCreateWithFlags(hipStream_t* s, unsigned) { *s = (hipStream_t)malloc(8); return hipSuccess; }
hipError_t hipStreamDestroy(hipStream_t s) { free(s); return hipSuccess; }
hipError_t hipStreamSynchronize(hipStream_t) { return hipSuccess; }
hipError_t hipStreamIsCapturing(hipStream_t s, hipStreamCaptureStatus* st) {
  *st = capturing.count(s) ? hipStreamCaptureStatusActive : hipStreamCaptureStatusNone;
  return hipSuccess;
}
hipError_t hipStreamBeginCapture(hipStream_t s, hipStreamCaptureMode) { capturing.insert(s); return hipSuccess; }
hipError_t hipStreamEndCapture(hipStream_t s, hipGraph_t* g) { capturing.erase(s); *g = (hipGraph_t)malloc(8); return hipSuccess; }
hipError_t hipGraphInstantiate(hipGraphExec_t* e, hipGraph_t, hipGraphNode_t*, char*, size_t) { *e = (hipGraphExec_t)malloc(8); return hipSuccess; }
hipError_t hipGraphLaunch(hipGraphExec_t, hipStream_t) { return hipSuccess; }
hipError_t hipGraphExecDestroy(hipGraphExec_t e) { free(e); return hipSuccess; }
hipError_t hipGraphDestroy(hipGraph_t g) { free(g); return hipSuccess; }
hipError_t hipEventCreate(hipEvent_t* e) { *e = (hipEvent_t)malloc(8); return hipSuccess; }
hipError_t hipEventDestroy(hipEvent_t e) { free(e); return hipSuccess; }
hipError_t hipEventRecord(hipEvent_t, hipStream_t) { return hipSuccess; }
hipError_t hipEventSynchronize(hipEvent_t) { return hipSuccess; }
hipError_t hipEventElapsedTime(float* t, hipEvent_t, hipEvent_t) { *t = 1.0f; return hipSuccess; }
hipError_t hipGetLastError() { return hipSuccess; }
const char* hipGetErrorString(hipError_t) { return "error of the stand-in"; }

void** __hipRegisterFatBinary(const void*) { static void* h; return &h; }
void __hipUnregisterFatBinary(void**) {}
void __hipRegisterFunction(void**, const void* host, char*, const char* name, unsigned, void*, void*, dim3*, dim3*, int*) {
  names[host] = name;
}
void __hipRegisterVar(void**, void*, char*, char*, int, size_t, int, int) {}
hipError_t __hipPushCallConfiguration(dim3 g, dim3 b, size_t lds, hipStream_t s) { configs.push_back({g, b, lds, s}); return hipSuccess; }
hipError_t __hipPopCallConfiguration(dim3* g, dim3* b, size_t* lds, hipStream_t* s) {
  Config c = configs.back();
  configs.pop_back();
  *g = c.grid; *b = c.block; *lds = c.lds; *s = c.stream;
  return hipSuccess;
}
hipError_t hipLaunchKernel(const void* f, dim3 g, dim3 b, void** args, size_t lds, hipStream_t s) {
  Launch l{names[f], current, {g.x, g.y, g.z}, {b.x, b.y, b.z}, lds, s, {}};
  auto word = [&](int i) { uint64_t v; memcpy(&v, args[i], 8); return v; };
  auto has = [&](const char* n) { return l.name.find(n) != std::string::npos; };
  if (has("k_begin_batch") || (has("k_begin") && !has("batch"))) {  // (arguments or table, words, how many)
    l.arg[0] = word(1); l.arg[1] = word(2);
    auto in = allocs.upper_bound((char*)l.arg[0]);
    const char* at = (char*)l.arg[0];
    const bool held = in != allocs.begin() && at + l.arg[1] * 4 <= std::prev(in)->first + std::prev(in)->second.bytes;
    const bool sym = symbol[current] && at >= symbol[current] && at + l.arg[1] * 4 <= symbol[current] + ((size_t)32 << 20);
    if (!held && !sym) { fprintf(stderr, "a pass start clears words that are not allocated\n"); abort(); }
    if (capturing.count(s)) captured_clears.push_back({l.arg[0], l.arg[1] * 4});
    else memset((void*)l.arg[0], 0, l.arg[1] * 4);
  } else if (has("k_loss") && !has("batch")) {  // image, target, n, adjoint, sums, loss
    l.arg[0] = word(4);
    l.arg[1] = 1;  // the sums are zero
    if (capturing.count(s)) {
      l.arg[1] = 0;
      for (auto& c : captured_clears) l.arg[1] |= c.first <= l.arg[0] && c.first + c.second >= l.arg[0] + 7 * 128 + 8;
    } else {
      loss_bytes(l.arg[0], [&](char& b) { l.arg[1] &= b == 0; b = (char)0xEE; });
    }
  }
  launches.push_back(l);
  return hipSuccess;
}

}  // extern "C"
