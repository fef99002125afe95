// host_read.h -- device fields to host arrays, in chunks through pinned memory.
//
// A copy into pageable memory is staged by the runtime on one thread, waits
// for each chunk, and faults in the pages of a fresh array as it goes: 168 MB
// of moments (256 x 160 x 128) took 15.5 ms.  Here the chunks go through a
// ring of pinned buffers at the link's rate (57 GB/s, 3 ms), and a few helper
// threads copy them on, each into planes of its own.  While the GPU still
// works on the steps before the read, they touch the pages of the result,
// which is most of what a copy into a fresh array costs (one thread: 5 GB/s
// fresh, 60 GB/s touched).  200 steps and a read into fresh arrays: 256 x 160 x
// 128 FP32 39.2 -> 26.0 ms, 192 x 192 x 130 FP16 35.8 -> 23.2 ms.
#pragma once

#include <hip/hip_runtime.h>

#include <algorithm>
#include <atomic>
#include <condition_variable>
#include <cstdint>
#include <cstring>
#include <mutex>
#include <thread>
#include <vector>

namespace lbk {

// Pinned memory is allocated and freed whatever another thread captures: a
// capture in the global mode, torch's default, would otherwise be invalidated by
// the first large read, or the destruction, of a domain beside it.
class CaptureRelaxed {
 public:
  CaptureRelaxed() { swapped_ = hipThreadExchangeStreamCaptureMode(&mode_) == hipSuccess; }
  ~CaptureRelaxed() {
    if (swapped_) (void)hipThreadExchangeStreamCaptureMode(&mode_);
  }
  CaptureRelaxed(const CaptureRelaxed &) = delete;
  CaptureRelaxed &operator=(const CaptureRelaxed &) = delete;

 private:
  hipStreamCaptureMode mode_ = hipStreamCaptureModeRelaxed;
  bool swapped_;
};

// Pinned ring and events of one domain, made at its first large read and
// given back with it: at most SLOTS * SLOT_BYTES.
struct HostRing {
  static constexpr int SLOTS = 4;
  static constexpr size_t SLOT_BYTES = size_t(4) << 20;
  char *mem[SLOTS] = {};
  hipEvent_t ev[SLOTS] = {};
  // false: no pinned memory; the caller copies without it.  The events belong
  // to the stream's device, whichever is current.
  bool ready(hipStream_t s) {
    if (ev[SLOTS - 1]) return true;
    const CaptureRelaxed relaxed;
    int current = 0, device = 0;
    if (hipGetDevice(&current) != hipSuccess || hipStreamGetDevice(s, &device) != hipSuccess) {
      (void)hipGetLastError();
      return false;
    }
    if (device != current && hipSetDevice(device) != hipSuccess) return false;
    const bool ok = make();
    if (device != current) (void)hipSetDevice(current);
    return ok;
  }
  HostRing() = default;
  HostRing(const HostRing &) = delete;
  HostRing &operator=(const HostRing &) = delete;
  ~HostRing() {
    const CaptureRelaxed relaxed;
    for (int i = 0; i < SLOTS; ++i) {
      if (ev[i]) (void)hipEventDestroy(ev[i]);
      if (mem[i]) (void)hipHostFree(mem[i]);
    }
  }

 private:
  bool make() {
    for (int i = 0; i < SLOTS; ++i) {
      if (!mem[i] && hipHostMalloc((void **)&mem[i], SLOT_BYTES, hipHostMallocDefault) != hipSuccess) {
        mem[i] = nullptr;
        (void)hipGetLastError();
        return false;
      }
      if (!ev[i] && hipEventCreateWithFlags(&ev[i], hipEventDisableTiming) != hipSuccess) {
        ev[i] = nullptr;
        (void)hipGetLastError();
        return false;
      }
    }
    return true;
  }
};

// Helper threads of one read.  Chunk c of every plane lies at slot c % SLOTS
// once published; a slot is free again when every helper is past its chunk.
class HostCopiers {
 public:
  // planes of n doubles at h[k]; plane k of chunk c (cnt doubles, node n0) is
  // at slot + k * cnt
  HostCopiers(const HostRing &ring, double *const *h, int planes, long long n, long long chunk)
      : ring_(ring), h_(h, h + planes), n_(n), chunk_(chunk) {
    const int want = disjoint() ? std::min(planes, 4) : 1;
    step_ = want;
    done_ = std::vector<std::atomic<long long>>(want);
    for (auto &d : done_) d.store(0);
    th_.reserve((size_t)want);
    try {
      for (int w = 0; w < want; ++w) th_.emplace_back([this, w] { work(w); });
    } catch (...) {  // too few threads: the caller copies the rest
    }
  }
  ~HostCopiers() {
    {
      std::lock_guard<std::mutex> g(m_);
      stop_.store(true);
    }
    cv_.notify_all();
    for (auto &t : th_) t.join();
  }
  HostCopiers(const HostCopiers &) = delete;
  HostCopiers &operator=(const HostCopiers &) = delete;

  // chunks [0, upto) are in their slots
  void publish(long long upto) {
    {
      std::lock_guard<std::mutex> g(m_);
      published_.store(upto, std::memory_order_release);
    }
    cv_.notify_all();
    for (size_t w = th_.size(); w < done_.size(); ++w)
      for (long long c = done_[w].load(); c < upto; ++c) {
        copy((int)w, c);
        done_[w].store(c + 1);
      }
  }
  // returns once the first `upto` chunks have left their slots
  void wait(long long upto) {
    for (auto &d : done_)
      while (d.load(std::memory_order_acquire) < upto) std::this_thread::yield();
  }

 private:
  // arrays that overlap are copied in order by one thread
  bool disjoint() const {
    for (size_t a = 0; a < h_.size(); ++a)
      for (size_t b = a + 1; b < h_.size(); ++b)
        if (h_[a] < h_[b] + n_ && h_[b] < h_[a] + n_) return false;
    return true;
  }
  void copy(int w, long long c) const {
    const long long n0 = c * chunk_, cnt = std::min(chunk_, n_ - n0);
    const double *s = (const double *)ring_.mem[c % HostRing::SLOTS];
    for (size_t k = (size_t)w; k < h_.size(); k += (size_t)step_)
      std::memcpy(h_[k] + n0, s + (long long)k * cnt, (size_t)cnt * 8);
  }
  void work(int w) {
    // one write per page, until there is something to copy; of nothing, so
    // that a read that fails leaves the arrays as they were (an addition: a load
    // and a store would fault twice, into the shared page of zeros first)
    for (size_t k = (size_t)w; k < h_.size(); k += (size_t)step_)
      for (long long i = 0; i < n_; i += 512) {
        if (published_.load(std::memory_order_acquire) || stop_.load()) goto copies;
        __asm__ volatile("lock; addq $0, %0" : "+m"(*(uint64_t *)(h_[k] + i)));
      }
  copies:
    {
      std::unique_lock<std::mutex> g(m_);
      cv_.wait(g, [this] { return published_.load() > 0 || stop_.load(); });
    }
    const long long chunks = (n_ + chunk_ - 1) / chunk_;
    for (long long c = 0; c < chunks; ++c) {
      while (published_.load(std::memory_order_acquire) <= c) {
        if (stop_.load()) return;
        std::this_thread::yield();
      }
      copy(w, c);
      done_[(size_t)w].store(c + 1, std::memory_order_release);
    }
  }

  const HostRing &ring_;
  std::vector<double *> h_;
  long long n_, chunk_;
  int step_ = 1;
  std::vector<std::atomic<long long>> done_;
  std::atomic<long long> published_{0};
  std::atomic<bool> stop_{false};
  std::mutex m_;
  std::condition_variable cv_;
  std::vector<std::thread> th_;
};

// Below this many bytes the chunks' threads and events cost more than the
// plain copy.
constexpr size_t HOST_RING_MIN_BYTES = size_t(8) << 20;

// `planes` fields of n doubles each into h[0 .. planes).  launch(n0, cnt)
// enqueues on s the kernel that writes nodes n0 .. n0 + cnt - 1 of all planes
// to stage[planes][cnt]; stage holds max_cnt nodes of them.  Synchronises.
template <class Launch>
hipError_t read_fields(HostRing &ring, double *const *h, int planes, long long n, double *stage,
                       long long max_cnt, hipStream_t s, Launch launch) {
  hipError_t e = hipSuccess;
  if ((size_t)n * planes * 8 < HOST_RING_MIN_BYTES || !ring.ready(s)) {
    for (long long n0 = 0; n0 < n; n0 += max_cnt) {
      const long long cnt = std::min(max_cnt, n - n0);
      launch(n0, cnt);
      if ((e = hipGetLastError()) != hipSuccess) return e;
      for (int k = 0; k < planes; ++k)
        if ((e = hipMemcpyAsync(h[k] + n0, stage + k * cnt, (size_t)cnt * 8, hipMemcpyDeviceToHost,
                                s)) != hipSuccess)
          return e;
      if ((e = hipStreamSynchronize(s)) != hipSuccess) return e;
    }
    return e;
  }
  const long long chunk =
      std::min<long long>(max_cnt, (long long)(HostRing::SLOT_BYTES / 8) / planes / 512 * 512);
  const long long chunks = (n + chunk - 1) / chunk;
  HostCopiers copiers(ring, h, planes, n, chunk);
  long long sent = 0;
  for (long long c = 0; c < chunks; ++c) {
    // keep the stream SLOTS - 1 chunks ahead of the one awaited
    for (; sent < chunks && sent < c + HostRing::SLOTS - 1; ++sent) {
      const int slot = (int)(sent % HostRing::SLOTS);
      const long long n0 = sent * chunk, cnt = std::min(chunk, n - n0);
      copiers.wait(sent - HostRing::SLOTS + 1);
      launch(n0, cnt);
      if ((e = hipGetLastError()) != hipSuccess) break;
      if ((e = hipMemcpyAsync(ring.mem[slot], stage, (size_t)cnt * planes * 8,
                              hipMemcpyDeviceToHost, s)) != hipSuccess ||
          (e = hipEventRecord(ring.ev[slot], s)) != hipSuccess)
        break;
    }
    if (e == hipSuccess) e = hipEventSynchronize(ring.ev[c % HostRing::SLOTS]);
    if (e != hipSuccess) break;
    copiers.publish(c + 1);
  }
  if (e == hipSuccess) copiers.wait(chunks);
  else (void)hipStreamSynchronize(s);  // nothing of the call is left in flight
  return e;
}

}  // namespace lbk
