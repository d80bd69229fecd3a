// grlbm_copy.hip -- host data in and out: large copies through pinned slots by several
// host threads, and the check of initial fields.
//
// A copy of pageable memory by one thread runs at what that thread copies and, into
// memory just allocated, at what the kernel zeroes pages: 124 MB of populations took 13 ms
// to read out (9.5 GB/s), most of it on the host.  Here up to kCopyThreads threads each
// move every so-many-th chunk through two pinned slots, so that DMA, the copies between
// slot and user memory and the page faults overlap (124 MB now 3.9-6 ms out, 3.2 ms in
// instead of 5; the check of a 96^3 field and its copy 1.5 ms instead of 2.9).
#include <hip/hip_runtime.h>

#include <algorithm>
#include <cmath>
#include <cstring>
#include <thread>

#include "grlbm_internal.h"

namespace grlbm {

namespace {

constexpr size_t kChunk = size_t(2) << 20;      // bytes of a slot
constexpr size_t kThreadedBytes = 2 * kChunk;   // smaller copies stay with the runtime
constexpr int kCopyThreads = 4;
constexpr int kMaxSlots = 16;                   // pinned memory: at most 32 MiB in a process

struct Slot {
  void* buf = nullptr;
  hipEvent_t done = nullptr;
  int device = 0;
};

// Idle slots, kept while a context or a batch lives.
std::mutex g_mu;
Slot g_idle[kMaxSlots];
int g_nidle = 0;
int g_slots = 0;  // idle and in use
int g_users = 0;

void free_slot(Slot& s) {
  if (s.done) (void)hipEventDestroy(s.done);
  if (s.buf) (void)hipHostFree(s.buf);
  --g_slots;
}

// A slot of the current device `dev`; buf is nullptr if none can be had.
Slot take_slot(int dev) {
  std::lock_guard<std::mutex> lock(g_mu);
  for (int i = 0; i < g_nidle; ++i)
    if (g_idle[i].device == dev) {
      std::swap(g_idle[i], g_idle[--g_nidle]);
      return g_idle[g_nidle];
    }
  Slot s;
  if (g_slots >= kMaxSlots) return s;
  s.device = dev;
  ++g_slots;
  if (hipHostMalloc(&s.buf, kChunk, hipHostMallocDefault) != hipSuccess ||
      hipEventCreateWithFlags(&s.done, hipEventDisableTiming) != hipSuccess) {
    (void)hipGetLastError();
    free_slot(s);
    return Slot();
  }
  return s;
}

void give_slot(Slot& s) {
  if (!s.buf) return;
  std::lock_guard<std::mutex> lock(g_mu);
  if (g_users > 0) {
    g_idle[g_nidle++] = s;
  } else {
    free_slot(s);
  }
}

// fn(i) for i in [0, n), n <= kCopyThreads, each in a thread of its own (the last in this
// one).  Where a thread cannot be had, for want of one or of memory, its part runs here.
template <typename Fn>
void in_threads(int n, Fn fn) {
  std::thread ts[kCopyThreads];
  int i = 0;
  for (; i + 1 < n; ++i) {
    try {
      ts[i] = std::thread(fn, i);
    } catch (...) {
      break;
    }
  }
  const int started = i;
  for (; i < n; ++i) fn(i);
  for (i = 0; i < started; ++i) ts[i].join();
}

// The chunks i, i + n, ... of a copy, through two slots in turn.
hipError_t move_chunks(char* dev, char* host, size_t bytes, bool out, hipStream_t s, int device, int i, int n) {
  hipError_t e = hipSetDevice(device);
  Slot slots[2] = {take_slot(device), take_slot(device)};
  size_t off[2] = {0, 0}, len[2] = {0, 0};  // what a slot's copy in flight moves
  auto finish = [&](int k) {
    if (len[k] == 0) return;
    if (e == hipSuccess) e = hipEventSynchronize(slots[k].done);
    if (e == hipSuccess && out) std::memcpy(host + off[k], slots[k].buf, len[k]);
    len[k] = 0;
  };
  int k = 0;
  for (size_t at = (size_t)i * kChunk; at < bytes && e == hipSuccess; at += (size_t)n * kChunk) {
    const size_t m = std::min(kChunk, bytes - at);
    if (!slots[k].buf) {  // no pinned memory: the runtime's own way
      e = out ? hipMemcpyAsync(host + at, dev + at, m, hipMemcpyDeviceToHost, s)
              : hipMemcpyAsync(dev + at, host + at, m, hipMemcpyHostToDevice, s);
      if (e == hipSuccess) e = hipStreamSynchronize(s);
      continue;
    }
    finish(k);
    if (e != hipSuccess) break;
    if (!out) std::memcpy(slots[k].buf, host + at, m);
    e = out ? hipMemcpyAsync(slots[k].buf, dev + at, m, hipMemcpyDeviceToHost, s)
            : hipMemcpyAsync(dev + at, slots[k].buf, m, hipMemcpyHostToDevice, s);
    if (e == hipSuccess) e = hipEventRecord(slots[k].done, s);
    off[k] = at;
    len[k] = m;
    k ^= 1;
  }
  finish(k);
  finish(k ^ 1);
  if (e != hipSuccess) (void)hipStreamSynchronize(s);  // nothing uses a slot that goes back
  give_slot(slots[0]);
  give_slot(slots[1]);
  return e;
}

// Memory that the runtime knows (pinned, managed, another device's): it moves that itself,
// without a copy by the host.
bool known(const void* host) {
  hipPointerAttribute_t a{};
  if (hipPointerGetAttributes(&a, host) != hipSuccess) {
    (void)hipGetLastError();
    return false;
  }
  return a.type != hipMemoryTypeUnregistered;
}

hipError_t copy(void* dev, void* host, size_t bytes, bool out, hipStream_t s) {
  if (bytes < kThreadedBytes || known(host)) {
    const hipError_t e = out ? hipMemcpyAsync(host, dev, bytes, hipMemcpyDeviceToHost, s)
                             : hipMemcpyAsync(dev, host, bytes, hipMemcpyHostToDevice, s);
    return e == hipSuccess ? hipStreamSynchronize(s) : e;
  }
  int device = 0;
  hipError_t e = hipGetDevice(&device);
  if (e != hipSuccess) return e;
  // hipStreamPerThread is another stream in each worker, which would not wait for what
  // the caller has enqueued: its copies stay in this thread
  const int n = s == hipStreamPerThread ? 1 : (int)std::min<size_t>(kCopyThreads, (bytes + kChunk - 1) / kChunk);
  hipError_t each[kCopyThreads] = {};
  in_threads(n, [&](int i) { each[i] = move_chunks((char*)dev, (char*)host, bytes, out, s, device, i, n); });
  for (int i = 0; i < n; ++i)
    if (each[i] != hipSuccess) return each[i];
  return hipSuccess;
}

}  // namespace

void copy_users(int change) {
  std::lock_guard<std::mutex> lock(g_mu);
  g_users += change;
  if (g_users > 0) return;
  while (g_nidle > 0) free_slot(g_idle[--g_nidle]);
}

hipError_t copy_out(void* host, const void* dev, size_t bytes, hipStream_t s) {
  return copy(const_cast<void*>(dev), host, bytes, true, s);
}

hipError_t copy_in(void* dev, const void* host, size_t bytes, hipStream_t s) {
  return copy(dev, const_cast<void*>(host), bytes, false, s);
}

lbm_status check_fields(const lbm_params* p, const double* Q) {
  const int64_t N = (int64_t)p->nx * p->ny * p->nz;
  const double g1 = p->gamma - 1.0;
  auto pressure = [&](int64_t n) {
    const double m0 = Q[N + n], m1 = Q[2 * N + n], m2 = Q[3 * N + n];
    return g1 * (Q[4 * N + n] - 0.5 * (m0 * m0 + m1 * m1 + m2 * m2) / Q[n]);
  };
  // runs of cells by one thread each, without a branch per cell; first[i] is the first
  // run of thread i that holds an unphysical cell
  constexpr int64_t kRun = 4096;
  const int64_t runs = (N + kRun - 1) / kRun;
  const int threads = (int)std::min<int64_t>(kCopyThreads, (runs + 7) / 8);
  int64_t first[kCopyThreads] = {runs, runs, runs, runs};
  static_assert(kCopyThreads == 4, "one entry of first for each thread");
  in_threads(threads, [&](int i) {
    for (int64_t r = runs * i / threads; r < runs * (i + 1) / threads; ++r) {
      const int64_t end = std::min(N, (r + 1) * kRun);
      int bad = 0;
      for (int64_t n = r * kRun; n < end; ++n) {
        const double rho = Q[n], m0 = Q[N + n], m1 = Q[2 * N + n], m2 = Q[3 * N + n], E = Q[4 * N + n];
        // zero unless one of them is not finite
        const double z = (rho - rho) + (m0 - m0) + (m1 - m1) + (m2 - m2) + (E - E);
        bad |= (int)!(z == 0.0) | (int)!(rho > 0.0) | (int)!(pressure(n) > 0.0);
      }
      if (bad) {
        first[i] = r;
        return;
      }
    }
  });
  const int64_t r = *std::min_element(first, first + kCopyThreads);
  for (int64_t n = r * kRun; r < runs && n < std::min(N, (r + 1) * kRun); ++n) {
    for (int k = 0; k < 5; ++k)
      if (!std::isfinite(Q[k * N + n]))
        return fail(LBM_EINVAL, "initial fields are not finite at cell %lld", (long long)n);
    if (!(Q[n] > 0.0))
      return fail(LBM_EINVAL, "initial density %g at cell %lld is not positive", Q[n], (long long)n);
    if (!(pressure(n) > 0.0))
      return fail(LBM_EINVAL, "initial pressure %g at cell %lld is not positive", pressure(n), (long long)n);
  }
  return LBM_OK;
}

}  // namespace grlbm
