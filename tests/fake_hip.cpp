// A HIP runtime without a GPU, for tests of the library's host code: the entry points
// that libgrlbm.so imports, under the runtime's soname.  Device memory is host memory
// from a card of fake_card() bytes; copies are done at once; kernels are not run.  Every
// call of interest is noted as one line of text: what, the stream, the calling thread
// (0 is the one that called fake_reset) and its arguments.
//
// Compiled with FAIL_NEW it is another library instead: an operator new whose calls fail on
// request.
#ifdef FAIL_NEW
#include <cstdlib>
#include <new>

static int fail_after = -1;
extern "C" void fake_fail_new(int after) { fail_after = after; }
extern "C" int fake_new_left() { return fail_after; }
void* operator new(std::size_t n) {
  if (fail_after == 0) throw std::bad_alloc();
  if (fail_after > 0) --fail_after;
  return std::malloc(n);
}
void operator delete(void* p) noexcept { std::free(p); }
void operator delete(void* p, std::size_t) noexcept { std::free(p); }
#else
#include <hip/hip_runtime_api.h>

#include <algorithm>
#include <cstdio>
#include <cstdlib>
#include <cstring>
#include <map>
#include <mutex>
#include <set>
#include <string>
#include <thread>
#include <vector>

namespace {

std::recursive_mutex mu;
std::vector<std::string> notes;
std::map<const void*, std::string> kernels;
std::map<char*, size_t> device, pinned;
std::set<void*> capture;
std::map<std::thread::id, int> threads;
size_t card = size_t(1) << 32, used = 0;
size_t allocs = 0;
std::string fail_kernel;
int fail_after = -1, slots = 1 << 20;
void (*on_sync)(void*) = nullptr;
thread_local hipError_t last = hipSuccess;
thread_local hipStreamCaptureMode mode = hipStreamCaptureModeGlobal;
thread_local std::vector<size_t> config;
thread_local int current = 0;

int me() {
  const auto it = threads.emplace(std::this_thread::get_id(), (int)threads.size());
  return it.first->second;
}
void note(const char* what, const void* stream, const std::string& rest = "") {
  char b[96];
  snprintf(b, sizeof b, "%s stream=%zx thread=%d ", what, (size_t)stream, me());
  notes.push_back(b + rest);
}
std::string num(const char* k, size_t v) {
  char b[48];
  snprintf(b, sizeof b, "%s=%zx ", k, v);
  return b;
}
hipError_t err(hipError_t e) {
  if (e != hipSuccess) last = e;
  return e;
}
// A call that is forbidden while a stream is being captured in global mode breaks that
// capture, unless the calling thread is in relaxed mode.
bool forbidden(const char* what) {
  if (capture.empty() || mode == hipStreamCaptureModeRelaxed) return false;
  note("BROKEN-CAPTURE", nullptr, what);
  return true;
}
const std::pair<char* const, size_t>* range(std::map<char*, size_t>& m, const void* p) {
  auto it = m.upper_bound((char*)p);
  if (it == m.begin()) return nullptr;
  --it;
  return (char*)p < it->first + it->second ? &*it : nullptr;
}

}  // namespace

extern "C" {

void fake_reset(size_t bytes) {
  std::lock_guard<std::recursive_mutex> l(mu);
  notes.clear();
  threads.clear();
  me();
  if (bytes) card = bytes;
  fail_kernel.clear();
  fail_after = -1;
}
size_t fake_used() { return used; }
size_t fake_allocs() { return allocs; }
void fake_capture(void* s, int on) {
  std::lock_guard<std::recursive_mutex> l(mu);
  if (on) {
    capture.insert(s);
  } else {
    capture.erase(s);
  }
}
// The launch after `after` further ones of kernels whose name holds `name` fails.
void fake_fail(const char* name, int after) {
  std::lock_guard<std::recursive_mutex> l(mu);
  fail_kernel = name;
  fail_after = after;
}
void fake_slots(int n) { slots = n; }  // pinned allocations that can still be had
void fake_on_sync(void (*fn)(void*)) { on_sync = fn; }
const char* fake_notes() {
  static std::string all;
  std::lock_guard<std::recursive_mutex> l(mu);
  all.clear();
  for (const auto& n : notes) all += n + "\n";
  return all.c_str();
}

void** __hipRegisterFatBinary(const void*) {
  static void* h = nullptr;
  return &h;
}
void __hipUnregisterFatBinary(void**) {}
void __hipRegisterFunction(void**, const void* fn, char*, const char* name, unsigned, void*, void*, void*, void*, int*) {
  std::lock_guard<std::recursive_mutex> l(mu);
  kernels[fn] = name;
}
void __hipRegisterVar(void**, void*, char*, char*, int, size_t, int, int) {}
hipError_t __hipPushCallConfiguration(dim3 g, dim3 b, size_t lds, hipStream_t s) {
  config = {g.x, g.y, g.z, b.x, b.y, b.z, lds, (size_t)s};
  return hipSuccess;
}
hipError_t __hipPopCallConfiguration(dim3* g, dim3* b, size_t* lds, hipStream_t* s) {
  *g = dim3(config[0], config[1], config[2]);
  *b = dim3(config[3], config[4], config[5]);
  *lds = config[6];
  *s = (hipStream_t)config[7];
  return hipSuccess;
}
hipError_t hipLaunchKernel(const void* fn, dim3 g, dim3 b, void** args, size_t lds, hipStream_t s) {
  std::lock_guard<std::recursive_mutex> l(mu);
  const std::string& name = kernels[fn];
  // more threads than 32 bits count cannot be launched
  if ((uint64_t)g.x * b.x > 0xffffffffull) return err(hipErrorInvalidConfiguration);
  if (!fail_kernel.empty() && name.find(fail_kernel) != std::string::npos && fail_after-- == 0)
    return err(hipErrorLaunchFailure);
  note("launch", s, name + " " + num("grid", g.x) + num("block", b.x) + num("lds", lds) +
                        num("a0", *(size_t*)args[0]) + num("a1", *(size_t*)args[1]));
  return hipSuccess;
}
hipError_t hipMalloc(void** p, size_t n) {
  std::lock_guard<std::recursive_mutex> l(mu);
  if (forbidden("hipMalloc")) return err(hipErrorStreamCaptureUnsupported);
  if (used + n > card) return err(hipErrorOutOfMemory);
  char* b = (char*)aligned_alloc(256, (n + 255) / 256 * 256);
  memset(b, 0, n);
  device[b] = n;
  used += n;
  ++allocs;
  note("malloc", nullptr, num("p", (size_t)b) + num("bytes", n));
  *p = b;
  return hipSuccess;
}
hipError_t hipFree(void* p) {
  std::lock_guard<std::recursive_mutex> l(mu);
  if (!p) return hipSuccess;
  used -= device.at((char*)p);
  device.erase((char*)p);
  note("free", nullptr, num("p", (size_t)p));
  free(p);
  return hipSuccess;
}
hipError_t hipMemGetInfo(size_t* f, size_t* t) {
  *f = card - used;
  *t = card;
  return hipSuccess;
}
hipError_t hipHostMalloc(void** p, size_t n, unsigned) {
  std::lock_guard<std::recursive_mutex> l(mu);
  if (slots <= 0) return err(hipErrorOutOfMemory);
  --slots;
  *p = malloc(n);
  pinned[(char*)*p] = n;
  return hipSuccess;
}
hipError_t hipHostFree(void* p) {
  std::lock_guard<std::recursive_mutex> l(mu);
  pinned.erase((char*)p);
  free(p);
  return hipSuccess;
}
hipError_t hipPointerGetAttributes(hipPointerAttribute_t* a, const void* p) {
  std::lock_guard<std::recursive_mutex> l(mu);
  memset(a, 0, sizeof *a);
  if (range(device, p)) {
    a->type = hipMemoryTypeDevice;
  } else if (range(pinned, p)) {
    a->type = hipMemoryTypeHost;
  } else {
    return err(hipErrorInvalidValue);
  }
  return hipSuccess;
}
hipError_t hipMemcpyAsync(void* d, const void* s, size_t n, hipMemcpyKind kind, hipStream_t st) {
  {
    std::lock_guard<std::recursive_mutex> l(mu);
    note("copy", st, num("dst", (size_t)d) + num("src", (size_t)s) + num("bytes", n) + num("kind", kind));
  }
  memcpy(d, s, n);
  return hipSuccess;
}
hipError_t hipMemsetAsync(void* d, int v, size_t n, hipStream_t) {
  memset(d, v, n);
  return hipSuccess;
}
hipError_t hipStreamCreate(hipStream_t* s) {
  static size_t next = 0x1000;
  std::lock_guard<std::recursive_mutex> l(mu);
  *s = (hipStream_t)(next += 0x10);
  return hipSuccess;
}
hipError_t hipStreamDestroy(hipStream_t) { return hipSuccess; }
hipError_t hipStreamSynchronize(hipStream_t s) {
  {
    std::lock_guard<std::recursive_mutex> l(mu);
    note("sync", s);
  }
  if (on_sync) on_sync(s);
  return hipSuccess;
}
hipError_t hipDeviceSynchronize() {
  std::lock_guard<std::recursive_mutex> l(mu);
  note("device-sync", nullptr);
  return hipSuccess;
}
hipError_t hipStreamIsCapturing(hipStream_t s, hipStreamCaptureStatus* st) {
  std::lock_guard<std::recursive_mutex> l(mu);
  *st = capture.count(s) ? hipStreamCaptureStatusActive : hipStreamCaptureStatusNone;
  return hipSuccess;
}
hipError_t hipThreadExchangeStreamCaptureMode(hipStreamCaptureMode* m) {
  std::swap(*m, mode);
  return hipSuccess;
}
hipError_t hipStreamBeginCapture(hipStream_t s, hipStreamCaptureMode) {
  std::lock_guard<std::recursive_mutex> l(mu);
  if (capture.count(s)) return err(hipErrorIllegalState);
  capture.insert(s);
  note("begin-capture", s);
  return hipSuccess;
}
hipError_t hipStreamEndCapture(hipStream_t s, hipGraph_t* g) {
  std::lock_guard<std::recursive_mutex> l(mu);
  capture.erase(s);
  *g = (hipGraph_t)malloc(1);
  note("end-capture", s);
  return hipSuccess;
}
hipError_t hipGraphInstantiate(hipGraphExec_t* e, hipGraph_t, hipGraphNode_t*, char*, size_t) {
  *e = (hipGraphExec_t)malloc(1);
  return hipSuccess;
}
hipError_t hipGraphDestroy(hipGraph_t g) {
  free(g);
  return hipSuccess;
}
hipError_t hipGraphExecDestroy(hipGraphExec_t e) {
  std::lock_guard<std::recursive_mutex> l(mu);
  note("destroy-graph", nullptr, num("exec", (size_t)e));
  free(e);
  return hipSuccess;
}
hipError_t hipGraphLaunch(hipGraphExec_t e, hipStream_t s) {
  std::lock_guard<std::recursive_mutex> l(mu);
  note("graph", s, num("exec", (size_t)e));
  return hipSuccess;
}
hipError_t hipEventCreate(hipEvent_t* e) {
  *e = (hipEvent_t)malloc(1);
  return hipSuccess;
}
hipError_t hipEventCreateWithFlags(hipEvent_t* e, unsigned) { return hipEventCreate(e); }
hipError_t hipEventDestroy(hipEvent_t e) {
  free(e);
  return hipSuccess;
}
hipError_t hipEventRecord(hipEvent_t, hipStream_t) { return hipSuccess; }
hipError_t hipEventSynchronize(hipEvent_t) { return hipSuccess; }
hipError_t hipEventElapsedTime(float* ms, hipEvent_t, hipEvent_t) {
  *ms = 1.0f;
  return hipSuccess;
}
hipError_t hipGetDevice(int* d) {
  *d = current;
  return hipSuccess;
}
hipError_t hipSetDevice(int d) {
  current = d;
  return hipSuccess;
}
hipError_t hipDeviceGetAttribute(int* v, hipDeviceAttribute_t, int) {
  *v = 256;
  return hipSuccess;
}
hipError_t hipGetSymbolAddress(void** p, const void*) {
  static char* b = (char*)calloc(1, 9 << 20 << 1);
  *p = b;
  return hipSuccess;
}
hipError_t hipGetLastError() {
  const hipError_t e = last;
  last = hipSuccess;
  return e;
}
const char* hipGetErrorString(hipError_t) { return "fake error"; }

}  // extern "C"
#endif
