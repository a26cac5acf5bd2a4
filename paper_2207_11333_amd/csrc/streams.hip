// The library's own streams: second streams of contexts, lanes of servers, copy
// streams of graph stores.  They are kept when their owner goes and handed to the
// next one: after hipStreamDestroy of a synchronised stream the ROCm 7.0 runtime has
// written to host memory that it had freed with it (two words of a 912-byte array that
// the caller allocated next, in 4 of 9 processes; in none of 9 with the stream kept).
// As many are held as were in use at one time, up to kSlots.
#include "common.hpp"

#include <mutex>

namespace hgnn {

namespace {

constexpr int kSlots = 256;
struct Slot {
  hipStream_t stream;
  int dev;
  bool used;
};
std::mutex g_mu;
Slot g_slot[kSlots] = {}; // the first g_n, in the order of creation
int g_n = 0;

void drop(int i) {
  for (--g_n; i < g_n; ++i) g_slot[i] = g_slot[i + 1];
}

} // namespace

// The oldest idle one of the current device: it was created when the fewest streams
// shared its hardware queue.  One that the runtime no longer knows (after a device
// reset) is dropped.
hipError_t stream_acquire(hipStream_t *out) {
  *out = nullptr;
  int dev = 0;
  hipError_t e = hipGetDevice(&dev);
  if (e != hipSuccess) return e;
  std::lock_guard<std::mutex> lk(g_mu);
  for (int i = 0; i < g_n;) {
    Slot &t = g_slot[i];
    if (t.used || t.dev != dev) {
      ++i;
      continue;
    }
    e = hipStreamQuery(t.stream);
    if (e == hipSuccess || e == hipErrorNotReady) {
      t.used = true;
      *out = t.stream;
      return hipSuccess;
    }
    (void)hipGetLastError();
    drop(i);
  }
  e = hipStreamCreateWithFlags(out, hipStreamNonBlocking);
  if (e == hipSuccess && g_n < kSlots) g_slot[g_n++] = {*out, dev, true};
  return e;
}

// One that a caller's open capture still holds is not used again.
void stream_release(hipStream_t s) {
  if (!s) return;
  hipStreamCaptureStatus st = hipStreamCaptureStatusNone;
  const bool ok = hipStreamIsCapturing(s, &st) == hipSuccess && st == hipStreamCaptureStatusNone;
  std::lock_guard<std::mutex> lk(g_mu);
  for (int i = 0; i < g_n; ++i)
    if (g_slot[i].stream == s) {
      g_slot[i].used = false;
      if (ok) return;
      drop(i);
      break;
    }
  (void)hipStreamDestroy(s);
}

} // namespace hgnn
