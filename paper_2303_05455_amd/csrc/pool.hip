// Device buffers of the library's objects and calls, kept for the next one.
//
// hipMalloc and hipFree take about 10 us each for small buffers and 100 to
// 600 us for large ones, and a context has some thirty of them, so creating
// and destroying one, or one call's scratch, could take longer than its
// kernels: a refinement run of 48,600 points (three contexts and a kNN graph)
// took 12.1 ms and takes 10.2 with the buffers kept, an inverted-file graph of
// 200,000 points 19.9 and 16.4.  A released buffer therefore waits here for a
// request of its size class on its device.
//
// Lifetime: every object and call works on one stream, and dev_free_all
// synchronises it before it takes the buffers, so no kernel or copy still uses
// one that is handed out again (a stream that cannot be waited for, or that
// captures: hipFree, as ever).  The null stream is one of each device: it is the
// buffers' device whose stream is waited for, whichever is current.  Not the
// whole device: hipDeviceSynchronize breaks
// the graph captures of other threads.  What waits is bounded (kMaxIdle),
// buffers above kMaxBlock never wait, a buffer that was not asked for again
// during kMaxAge releases is given back to the device, when an allocation
// fails all of them are before it is tried again, and so they are by ivhd_trim.
#include <algorithm>
#include <mutex>
#include <new>
#include <unordered_map>
#include <vector>

#include "ivhd_internal.h"

namespace ivhd {
namespace {

constexpr size_t kMaxBlock = size_t{128} << 20;
constexpr size_t kMaxIdle = size_t{512} << 20;
constexpr uint64_t kMaxAge = 64;

struct Block {
  void *p;
  size_t bytes;   // a size class
  int device;
  uint64_t since;   // the release that brought it here
};

// never destroyed: objects may be released while the process ends
struct Pool {
  std::mutex mu;
  std::unordered_map<void *, Block> used;   // pooled buffers handed out
  std::vector<Block> idle;                  // oldest first
  size_t idle_bytes = 0;
  uint64_t releases = 0;
};
Pool &pool() {
  static Pool *P = new Pool();
  return *P;
}

// eight classes to each power of two, 512 bytes at least
size_t size_class(size_t bytes) {
  if (bytes <= 512) return 512;
  size_t step = 64;
  while (step * 16 < bytes) step *= 2;
  return (bytes + step - 1) / step * step;
}

void give_back(const std::vector<Block> &blocks) {
  for (const Block &b : blocks) (void)hipFree(b.p);
}

// what waits, out of the pool
void take_idle(Pool &P, std::vector<Block> &idle) {
  std::lock_guard<std::mutex> lk(P.mu);
  idle.swap(P.idle);
  P.idle_bytes = 0;
}

// the calls below without their guards against std::bad_alloc

hipError_t get(void **p, size_t bytes) {
  int device = 0;
  hipError_t e = hipGetDevice(&device);
  if (e != hipSuccess) return e;
  Pool &P = pool();
  const bool pooled = bytes <= kMaxBlock;
  if (pooled) {
    bytes = size_class(bytes);
    std::lock_guard<std::mutex> lk(P.mu);
    for (size_t i = P.idle.size(); i-- > 0;)   // the last released first
      if (P.idle[i].device == device && P.idle[i].bytes == bytes) {
        P.used.emplace(P.idle[i].p, P.idle[i]);
        *p = P.idle[i].p;
        P.idle_bytes -= bytes;
        P.idle.erase(P.idle.begin() + (ptrdiff_t)i);
        return hipSuccess;
      }
  }
  e = hipMalloc(p, bytes);
  if (e == hipErrorOutOfMemory) {
    (void)hipGetLastError();
    std::vector<Block> idle;
    take_idle(P, idle);
    if (idle.empty()) return e;
    give_back(idle);
    e = hipMalloc(p, bytes);
  }
  if (e == hipSuccess && pooled) {
    std::lock_guard<std::mutex> lk(P.mu);
    P.used.emplace(*p, Block{*p, bytes, device, 0});   // without its entry a buffer goes back to the device
  }
  return e;
}

// waits for the stream (of that device, if it is the null stream); false when it cannot be waited for
bool wait_for(hipStream_t stream, int device, int current) {
  if (device != current && hipSetDevice(device) != hipSuccess) return false;
  hipStreamCaptureStatus capturing = hipStreamCaptureStatusNone;
  const bool done = hipStreamIsCapturing(stream, &capturing) == hipSuccess &&
                    capturing == hipStreamCaptureStatusNone && hipStreamSynchronize(stream) == hipSuccess;
  return (device == current || hipSetDevice(current) == hipSuccess) && done;
}

void put(void *const *bufs, size_t n, hipStream_t stream) {
  Pool &P = pool();
  std::vector<Block> back;
  std::vector<int> devices;   // of the buffers: one, as a rule
  {
    std::lock_guard<std::mutex> lk(P.mu);
    for (size_t i = 0; i < n; ++i) {
      const auto it = bufs[i] ? P.used.find(bufs[i]) : P.used.end();
      if (it != P.used.end() && std::find(devices.begin(), devices.end(), it->second.device) == devices.end())
        devices.push_back(it->second.device);
    }
  }
  int current = 0;
  bool idle = hipGetDevice(&current) == hipSuccess;
  for (const int d : devices) idle = idle && wait_for(stream, d, current);
  if (!idle) (void)hipGetLastError();
  {
    std::lock_guard<std::mutex> lk(P.mu);
    P.idle.reserve(P.idle.size() + n);
    back.reserve(P.idle.size() + 2 * n);
    ++P.releases;
    for (size_t i = 0; i < n; ++i) {
      if (!bufs[i]) continue;
      const auto it = P.used.find(bufs[i]);
      if (it == P.used.end() || !idle) {
        back.push_back(Block{bufs[i], 0, 0, 0});
        if (it != P.used.end()) P.used.erase(it);
        continue;
      }
      it->second.since = P.releases;
      P.idle.push_back(it->second);
      P.idle_bytes += it->second.bytes;
      P.used.erase(it);
    }
    size_t drop = 0;
    while (drop < P.idle.size() && (P.idle_bytes > kMaxIdle || P.releases - P.idle[drop].since > kMaxAge)) {
      P.idle_bytes -= P.idle[drop].bytes;
      back.push_back(P.idle[drop++]);
    }
    P.idle.erase(P.idle.begin(), P.idle.begin() + (ptrdiff_t)drop);
  }
  give_back(back);   // hipFree synchronises by itself
}

}  // namespace

hipError_t pool_get(void **p, size_t bytes) {
  *p = nullptr;
  try {
    return get(p, bytes);
  } catch (const std::bad_alloc &) {
    if (*p) return hipSuccess;   // allocated, without an entry
    return hipErrorOutOfMemory;
  }
}

void dev_free_all(void *const *bufs, size_t n, hipStream_t stream) {
  bool any = false;
  for (size_t i = 0; i < n; ++i) any = any || bufs[i];
  if (!any) return;
  try {
    put(bufs, n, stream);
  } catch (const std::bad_alloc &) {   // nothing was moved: back to the device, which needs no memory
    Pool &P = pool();
    for (size_t i = 0; i < n; ++i) {
      if (!bufs[i]) continue;
      {
        std::lock_guard<std::mutex> lk(P.mu);
        P.used.erase(bufs[i]);
      }
      (void)hipFree(bufs[i]);
    }
  }
}

}  // namespace ivhd

extern "C" int ivhd_trim(void) {
  std::vector<ivhd::Block> idle;
  ivhd::take_idle(ivhd::pool(), idle);
  ivhd::give_back(idle);
  return IVHD_OK;
}
