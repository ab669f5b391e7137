// Large host <-> device transfers with conversion between FP64 host arrays and
// the planes' precision.
//
// One host thread that converts into a fresh vector, a copy from or to pageable
// memory, and a result array whose pages are touched for the first time bound
// these calls, at 57 GB/s of PCIe a few milliseconds' worth.  From kStageMin values
// on the copies go through a ring of pinned slots while several threads convert the
// other slots, so conversion, first touch and copy overlap.  Measured, before ->
// now: 7.1 M and 21.2 M values of a 192^3 FP32 fluid read 57 -> 25.6 ms (21.8 of
// them for the first array, whose pages fault one by one), 21.2 M set 30 -> 8.4 ms;
// 2.1 M values on a context of their own, the ring's making included, 3.4 -> 2.1 ms
// up and 3.1 -> 1.8 ms down; 1.2 M 1.9 -> 1.7 and 1.8 -> 1.5, so the line lies at 2^20.
//
// The rings belong to the process: a transfer leases one of its device's, and the
// idle ones go when the last context does.  Making one takes 0.13-0.4 ms.  Threads
// live for one call.  Smaller transfers keep the plain path, whose cost is below
// that of starting the threads (0.11 ms).
#pragma once
#include <hip/hip_runtime.h>
#include <sched.h>

#include <algorithm>
#include <atomic>
#include <cmath>
#include <mutex>
#include <thread>
#include <type_traits>
#include <vector>

namespace epdlb {

constexpr size_t kStageMin = 1024 * 1024;  // values
constexpr size_t kStageSlotBytes = 1u << 20;  // 256 KiB slots: 9.2 ms where these take 5.2
constexpr int kStageSlots = 16;
constexpr int kStageMaxThreads = 8;
constexpr size_t kStageIdle = 2;

// The thread's current device while it lives; the one before is put back.
class DeviceScope {
 public:
  explicit DeviceScope(int device) {
    if (hipGetDevice(&before_) != hipSuccess) return;
    set_ = device != before_ && hipSetDevice(device) == hipSuccess;
  }
  ~DeviceScope() {
    if (set_) (void)hipSetDevice(before_);
  }
  DeviceScope(const DeviceScope&) = delete;
  DeviceScope& operator=(const DeviceScope&) = delete;

 private:
  int before_ = 0;
  bool set_ = false;
};

struct HostStage {
  int device = 0;
  unsigned char* pin = nullptr;
  hipEvent_t ev[kStageSlots] = {};

  // false (and nothing held) when the pinned ring or an event cannot be had.
  // The events are made on the ring's device, whichever the caller's current one
  // is: an event is recorded only on streams of its own device.
  bool ensure() {
    if (pin) return true;
    const DeviceScope on(device);
    void* p = nullptr;
    if (hipHostMalloc(&p, kStageSlotBytes * kStageSlots, hipHostMallocDefault) != hipSuccess) {
      (void)hipGetLastError();
      return false;
    }
    pin = static_cast<unsigned char*>(p);
    for (hipEvent_t& e : ev)
      if (hipEventCreateWithFlags(&e, hipEventDisableTiming) != hipSuccess) {
        (void)hipGetLastError();
        release();
        return false;
      }
    return true;
  }
  void release() {
    for (hipEvent_t& e : ev) {
      if (e) (void)hipEventDestroy(e);
      e = nullptr;
    }
    if (pin) (void)hipHostFree(pin);
    pin = nullptr;
  }
};

// The rings of this process.  Contexts hold a StageUser for as long as they live.
class StagePool {
 public:
  static StagePool& get() {
    static StagePool* p = new StagePool;  // never destroyed: contexts may outlive static objects
    return *p;
  }
  void attach() {
    std::lock_guard<std::mutex> g(m_);
    ++users_;
  }
  void detach() {
    std::vector<HostStage> drop;
    {
      std::lock_guard<std::mutex> g(m_);
      if (--users_ == 0) drop.swap(idle_);
    }
    for (HostStage& s : drop) s.release();
  }
  // An idle ring of the device, else a new one; pin == nullptr when none can be had.
  HostStage take(int device) {
    {
      std::lock_guard<std::mutex> g(m_);
      for (size_t i = 0; i < idle_.size(); ++i)
        if (idle_[i].device == device) {
          const HostStage s = idle_[i];
          idle_.erase(idle_.begin() + long(i));
          return s;
        }
    }
    HostStage s;
    s.device = device;
    (void)s.ensure();
    return s;
  }
  void give(HostStage s) {
    if (!s.pin) return;
    {
      std::lock_guard<std::mutex> g(m_);
      size_t same = 0;
      for (const HostStage& o : idle_) same += o.device == s.device;
      if (users_ > 0 && same < kStageIdle) {
        idle_.push_back(s);
        return;
      }
    }
    s.release();
  }

 private:
  StagePool() { idle_.reserve(64); }
  std::mutex m_;
  std::vector<HostStage> idle_;
  int users_ = 0;
};
struct StageUser {
  StageUser() { StagePool::get().attach(); }
  ~StageUser() { StagePool::get().detach(); }
  StageUser(const StageUser&) = delete;
  StageUser& operator=(const StageUser&) = delete;
};
// One transfer's ring.  A transfer that failed may leave copies in flight into
// it: the stream is waited for, and no other transfer gets the ring.
struct StageLease {
  HostStage st;
  hipStream_t s;
  bool bad = false;
  StageLease(int device, hipStream_t stream) : st(StagePool::get().take(device)), s(stream) {}
  ~StageLease() {
    if (bad)
      st.release();
    else
      StagePool::get().give(st);
  }
  hipError_t failed(hipError_t e) {
    bad = true;
    (void)hipStreamSynchronize(s);
    return e;
  }
};

// Threads of one transfer: the CPUs this process may use, at most kStageMaxThreads.
inline int stage_threads() {
  cpu_set_t set;
  CPU_ZERO(&set);
  int n = 1;
  if (sched_getaffinity(0, sizeof(set), &set) == 0) n = CPU_COUNT(&set);
  return std::max(1, std::min(n, kStageMaxThreads));
}

// Workers of one transfer, joined when it ends by whatever way.  No exception
// leaves it: with no thread to be had, run() is false and the caller takes the
// plain path.
struct StageWorkers {
  std::thread th[kStageMaxThreads];
  int n = 0;
  std::atomic<bool> stop{false};
  template <class F> bool run(F&& f) {
    const int want = stage_threads();
    try {
      for (; n < want; ++n) th[n] = std::thread(f);
    } catch (...) {  // no thread to be had
    }
    return n > 0;
  }
  void join() {
    for (int i = 0; i < n; ++i) th[i].join();
    n = 0;
  }
  ~StageWorkers() {
    stop.store(true);
    join();
  }
};

inline void stage_pause(int& spins) {
  if (++spins < 64)
    __builtin_ia32_pause();
  else
    std::this_thread::yield();
}

// dst[i] = conv(i, src[i]) for i < count, src on the device; returns when dst
// is whole.  *done = false: not taken (no ring or threads), nothing written.
template <typename T, class Conv>
hipError_t staged_download(int device, hipStream_t s, double* dst, const T* src, size_t count, Conv conv,
                           bool* done) {
  *done = false;
  StageLease lease(device, s);
  HostStage& st = lease.st;
  if (!st.pin) return hipSuccess;
  constexpr size_t per = kStageSlotBytes / sizeof(T);
  const long chunks = long((count + per - 1) / per);
  std::atomic<long> next{0}, landed{0};           // chunks handed to workers, chunks in their slots
  std::atomic<int> busy[kStageSlots];             // 1: a slot holds values not yet converted
  for (auto& b : busy) b.store(0);
  StageWorkers w;
  const bool ok = w.run([&] {
    for (;;) {
      const long c = next.fetch_add(1);
      if (c >= chunks) return;
      int spins = 0;
      while (landed.load(std::memory_order_acquire) <= c) {
        if (w.stop.load()) return;
        stage_pause(spins);
      }
      const T* h = reinterpret_cast<const T*>(st.pin + size_t(c % kStageSlots) * kStageSlotBytes);
      const size_t i0 = size_t(c) * per, i1 = std::min(count, i0 + per);
      for (size_t i = i0; i < i1; ++i) dst[i] = double(conv(i, h[i - i0]));
      busy[c % kStageSlots].store(0, std::memory_order_release);
    }
  });
  if (!ok) return hipSuccess;
  *done = true;
  constexpr long ahead = kStageSlots / 2;  // copies in flight
  for (long c = 0; c < chunks + ahead; ++c) {
    if (c < chunks) {
      const int slot = int(c % kStageSlots);
      int spins = 0;
      while (busy[slot].load(std::memory_order_acquire)) stage_pause(spins);
      busy[slot].store(1, std::memory_order_relaxed);
      const size_t i0 = size_t(c) * per, m = std::min(count, i0 + per) - i0;
      hipError_t e = hipMemcpyAsync(st.pin + size_t(slot) * kStageSlotBytes, src + i0, m * sizeof(T),
                                    hipMemcpyDeviceToHost, s);
      if (e == hipSuccess) e = hipEventRecord(st.ev[slot], s);
      if (e != hipSuccess) return lease.failed(e);
    }
    if (c >= ahead) {
      const hipError_t e = hipEventSynchronize(st.ev[(c - ahead) % kStageSlots]);
      if (e != hipSuccess) return lease.failed(e);
      landed.store(c - ahead + 1, std::memory_order_release);
    }
  }
  w.join();
  return hipSuccess;
}

// dst[i] = conv(i, src[i]) for i < count, dst on the device; returns when the
// copies are done.  *finite: whether every src value is finite.
template <typename T, class Conv>
hipError_t staged_upload(int device, hipStream_t s, T* dst, const double* src, size_t count, Conv conv,
                         bool* finite, bool* done) {
  *done = false;
  StageLease lease(device, s);
  HostStage& st = lease.st;
  if (!st.pin) return hipSuccess;
  constexpr size_t per = kStageSlotBytes / sizeof(T);
  const long chunks = long((count + per - 1) / per);
  std::atomic<long> next{0}, freed{0};  // chunks handed to workers, chunks whose copy is done
  std::atomic<bool> fin{true};
  std::atomic<long> ready[kStageSlots];  // last chunk converted into the slot
  for (auto& r : ready) r.store(-1);
  StageWorkers w;
  const bool ok = w.run([&] {
    for (;;) {
      const long c = next.fetch_add(1);
      if (c >= chunks) return;
      int spins = 0;
      while (freed.load(std::memory_order_acquire) <= c - kStageSlots) {
        if (w.stop.load()) return;
        stage_pause(spins);
      }
      T* h = reinterpret_cast<T*>(st.pin + size_t(c % kStageSlots) * kStageSlotBytes);
      const size_t i0 = size_t(c) * per, i1 = std::min(count, i0 + per);
      bool f = true;
      for (size_t i = i0; i < i1; ++i) {
        f &= std::isfinite(src[i]);
        h[i - i0] = T(conv(i, src[i]));
      }
      if (!f) fin.store(false, std::memory_order_relaxed);
      ready[c % kStageSlots].store(c, std::memory_order_release);
    }
  });
  if (!ok) return hipSuccess;
  *done = true;
  constexpr long ahead = kStageSlots / 2;
  for (long c = 0; c < chunks + ahead; ++c) {
    if (c < chunks) {
      const int slot = int(c % kStageSlots);
      int spins = 0;
      while (ready[slot].load(std::memory_order_acquire) != c) stage_pause(spins);
      const size_t i0 = size_t(c) * per, m = std::min(count, i0 + per) - i0;
      hipError_t e = hipMemcpyAsync(dst + i0, st.pin + size_t(slot) * kStageSlotBytes, m * sizeof(T),
                                    hipMemcpyHostToDevice, s);
      if (e == hipSuccess) e = hipEventRecord(st.ev[slot], s);
      if (e != hipSuccess) return lease.failed(e);
    }
    if (c >= ahead) {
      const hipError_t e = hipEventSynchronize(st.ev[(c - ahead) % kStageSlots]);
      if (e != hipSuccess) return lease.failed(e);
      freed.store(c - ahead + 1, std::memory_order_release);
    }
  }
  w.join();
  *finite = fin.load();
  return hipSuccess;
}

// The conversion that leaves a value as it is but for its type.
struct AsIs {
  template <class X> X operator()(size_t, X v) const { return v; }
};
// FP64 planes take FP64 host arrays as they lie.
template <typename T, class Conv> constexpr bool direct_copy() {
  return std::is_same<T, double>::value && std::is_same<Conv, AsIs>::value;
}

// Host FP64 values -> device planes of T, each through conv(index, value);
// returns when the host array is free again.
template <typename T, class Conv>
hipError_t host_upload(int device, hipStream_t s, T* dst, const double* src, size_t count, Conv conv) {
  if (count >= kStageMin) {
    bool done = false, finite = true;
    const hipError_t e = staged_upload(device, s, dst, src, count, conv, &finite, &done);
    if (e != hipSuccess || done) return e;
  }
  std::vector<T> h;
  const void* from = src;
  if constexpr (!direct_copy<T, Conv>()) {
    h.resize(count);
    for (size_t i = 0; i < count; ++i) h[i] = T(conv(i, src[i]));
    from = h.data();
  }
  const hipError_t e = hipMemcpyAsync(dst, from, count * sizeof(T), hipMemcpyHostToDevice, s);
  const hipError_t w = hipStreamSynchronize(s);
  return e != hipSuccess ? e : w;
}

// Device planes of T -> host FP64 values through conv(index, value).
template <typename T, class Conv>
hipError_t host_download(int device, hipStream_t s, double* dst, const T* src, size_t count, Conv conv) {
  if (count >= kStageMin) {
    bool done = false;
    const hipError_t e = staged_download(device, s, dst, src, count, conv, &done);
    if (e != hipSuccess || done) return e;
  }
  std::vector<T> h;
  void* to = dst;
  if constexpr (!direct_copy<T, Conv>()) {
    h.resize(count);
    to = h.data();
  }
  const hipError_t e = hipMemcpyAsync(to, src, count * sizeof(T), hipMemcpyDeviceToHost, s);
  const hipError_t w = hipStreamSynchronize(s);
  if (e != hipSuccess || w != hipSuccess) return e != hipSuccess ? e : w;
  if constexpr (!direct_copy<T, Conv>())
    for (size_t i = 0; i < count; ++i) dst[i] = double(conv(i, h[i]));
  return hipSuccess;
}

}  // namespace epdlb
