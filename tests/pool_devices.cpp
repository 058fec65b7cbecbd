// Host check of the device buffer pool (pool.hip) against a stand-in for the
// HIP runtime with two devices: a buffer that work still uses must not be
// handed out; and without host memory nothing is thrown or lost.  Built and run
// by test_pool_devices.py.
#include <cstdio>
#include <cstdlib>
#include <map>
#include <new>
#include <set>

#include "knn_internal.h"

namespace {
int g_device = 0;
bool g_capturing = false;
bool g_no_memory = false;   // operator new throws
std::map<void *, int> g_of;                              // allocation -> device
std::map<std::pair<int, hipStream_t>, std::set<void *>> g_busy;   // (device, stream): what queued work uses

void check(bool ok, const char *what) {
  if (ok) return;
  std::printf("FAILED: %s\n", what);
  std::exit(1);
}
bool busy(void *p) {
  for (const auto &q : g_busy)
    if (q.second.count(p)) return true;
  return false;
}
hipStream_t stream_no(int k) { return reinterpret_cast<hipStream_t>(static_cast<uintptr_t>(k)); }
}  // namespace

void *operator new(size_t n) {
  void *p = g_no_memory ? nullptr : std::malloc(n);
  if (!p) throw std::bad_alloc();
  return p;
}
void operator delete(void *p) noexcept { std::free(p); }
void operator delete(void *p, size_t) noexcept { std::free(p); }

namespace ivhd {
int fail(int code, const char *, ...) { return code; }
}  // namespace ivhd

extern "C" {
const char *hipGetErrorString(hipError_t) { return ""; }
hipError_t hipGetDevice(int *d) {
  *d = g_device;
  return hipSuccess;
}
hipError_t hipSetDevice(int d) {
  if (d < 0 || d > 1) return hipErrorInvalidDevice;
  g_device = d;
  return hipSuccess;
}
hipError_t hipMalloc(void **p, size_t bytes) {
  const bool none = g_no_memory;   // the device has memory of its own
  g_no_memory = false;
  *p = std::malloc(bytes);
  g_of[*p] = g_device;
  g_no_memory = none;
  return hipSuccess;
}
hipError_t hipFree(void *p) {   // waits for the device of the buffer
  check(g_of.count(p) == 1, "freed what is allocated");
  for (auto &q : g_busy)
    if (q.first.first == g_of[p]) q.second.clear();
  g_of.erase(p);
  std::free(p);
  return hipSuccess;
}
hipError_t hipStreamSynchronize(hipStream_t s) {
  for (auto &q : g_busy)
    if (q.first.second == s && (s || q.first.first == g_device)) q.second.clear();
  return hipSuccess;
}
hipError_t hipStreamIsCapturing(hipStream_t, hipStreamCaptureStatus *st) {
  *st = g_capturing ? hipStreamCaptureStatusActive : hipStreamCaptureStatusNone;
  return hipSuccess;
}
hipError_t hipGetLastError() { return hipSuccess; }
}

int main() {
  // the buffers' device and the one current at the release, on the null and a named stream
  for (int of = 0; of < 2; ++of)
    for (int at = 0; at < 2; ++at)
      for (int st = 0; st < 2; ++st) {
        const hipStream_t s = stream_no(16 * st);
        (void)hipSetDevice(of);
        void *b[3] = {};
        check(ivhd::pool_get(&b[0], 1000) == hipSuccess && ivhd::pool_get(&b[2], 5000) == hipSuccess, "allocates");
        check(!busy(b[0]) && !busy(b[2]), "an unused buffer is handed out");
        g_busy[{of, s}] = {b[0], b[2]};
        (void)hipSetDevice(at);
        ivhd::dev_free_all(b, 3, s);
        check(g_device == at, "the current device stays");
        for (int dev = 0; dev < 2; ++dev) {
          (void)hipSetDevice(dev);
          void *p = nullptr;
          check(ivhd::pool_get(&p, 1000) == hipSuccess && g_of[p] == dev, "a buffer of the current device");
          check(!busy(p), "no buffer that queued work still uses");
          ivhd::dev_free(p, s);
        }
      }
  // a capturing stream: given back to the device, not kept
  (void)hipSetDevice(0);
  void *p = nullptr;
  check(ivhd::pool_get(&p, 77777) == hipSuccess, "allocates");
  g_capturing = true;
  ivhd::dev_free(p, stream_no(16));
  check(g_of.count(p) == 0, "freed while a capture is on");
  g_capturing = false;
  // no host memory: a failure code, and a release that gives the buffer back
  {
    ivhd::Scratch S(stream_no(16));
    float *q = nullptr, *r = nullptr;
    check(S.get(&q, 3000000, "a buffer") == IVHD_OK, "allocates");
    const size_t had = g_of.size();
    g_no_memory = true;
    check(S.get(&r, 100, "another") == IVHD_ENOMEM && r == nullptr && g_of.size() == had, "refuses without host memory");
    S.~Scratch();
    g_no_memory = false;
    new (&S) ivhd::Scratch(stream_no(16));
    check(g_of.count(q) == 0, "released without host memory");
    void *again = nullptr;
    check(ivhd::pool_get(&again, 12000000) == hipSuccess && g_of.count(again) == 1, "allocates again");
    ivhd::dev_free(again, stream_no(16));
  }
  // trimmed: what waits goes back, what is in use does not
  void *held = nullptr, *idle = nullptr;
  (void)hipSetDevice(1);
  check(ivhd::pool_get(&held, 4000) == hipSuccess && ivhd::pool_get(&idle, 9000) == hipSuccess, "allocates");
  ivhd::dev_free(idle, nullptr);
  check(g_of.count(idle) == 1, "a released buffer waits");
  check(ivhd_trim() == IVHD_OK && g_of.size() == 1 && g_of.count(held) == 1, "only the buffer in use is left");
  ivhd::dev_free(held, nullptr);
  ivhd::Carve many;
  void *parts[20];
  for (void *&part : parts) many.add(reinterpret_cast<unsigned char **>(&part), 10);
  ivhd::Scratch S;
  check(many.get(S, "too many") == IVHD_ESTATE, "more parts than there is room for");
  std::printf("ok\n");
  return 0;
}
