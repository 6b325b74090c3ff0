// Scalars that kernels hand to the host (norms' partial sums, Hessenberg columns).
#pragma once

#include <hip/hip_runtime.h>

#include <chrono>
#include <cstdint>
#include <string>
#include <thread>
#include <utility>

#include "../../include/mrcm.h"
#include "device.h"
#include "internal.h"

namespace mrcm {

// A pinned buffer that kernels store into (publish) and one host thread watches:
// post(n, s) marks the first n places unset before the kernels that write them are
// launched on stream s, wait returns once all of them are set.  A copy to the host and a
// stream synchronisation take 14.7 us from the launch of a 2 us kernel, stores from
// the device and a watch 11.1 us, and those are stores of the step's last kernel, not a
// launch more (the host waits once per Arnoldi step, for j + 2 values; eight
// right-hand sides made eight copies).  Solves against copies: 64 x 64 in FP64
// 535 -> 474 us, 220 x 60 2.68 -> 2.40 ms, 512 x 512 with eight right-hand sides 3.28 -> 2.92
// ms, the batched solves of three grids 6.50 -> 3.17 ms.  The unset mark is a
// signalling NaN, which no arithmetic produces; should a place never change,
// the wait ends with the stream's work.
// A wait gives its core away every kSpins looks and asks the stream only once in
// kAskEvery: with neither, the waits of 16 threads on 16 cores kept each other's
// launches, and the runtime's threads, off the cores (64 x 64 solves, wall time per solve
// over all threads: 0.60 to 1.3 ms, against 0.23 to 0.61 with copies and
// synchronisations and 0.17 to 0.25 now; one thread 0.48, 0.77, 0.43 to 0.45; 64
// looks instead of 256 cost a small 3-D solve 1%, 1060 and 1070 us).
struct Mailbox {
  static constexpr int kPlaces = kMaxVecBlocks + 256;
  static constexpr uint64_t kUnset = 0x7ff4a5c3e1d2b697ull;
  static constexpr unsigned kSpins = 256;
  static constexpr std::chrono::microseconds kAskEvery{1000};
  double* h = nullptr;  // the same address on the host and the device; owned
  int posted = 0;

  Mailbox() = default;
  Mailbox(Mailbox&& o) noexcept : h(o.h), posted(o.posted) {
    o.h = nullptr;
    o.posted = 0;
  }
  Mailbox& operator=(Mailbox&& o) noexcept {
    std::swap(h, o.h);
    std::swap(posted, o.posted);
    return *this;
  }
  ~Mailbox() {
    if (h) (void)hipHostFree(h);
  }

  static void check(hipError_t e, const char* what) {
    if (e != hipSuccess)
      throw Error(e == hipErrorOutOfMemory ? MRCM_ENOMEM : MRCM_EDEVICE,
                  std::string(what) + ": " + hipGetErrorString(e));
  }
  void create() {
    if (h) return;
    check(hipHostMalloc((void**)&h, sizeof(double) * kPlaces,
                        hipHostMallocMapped | hipHostMallocCoherent),
          "hipHostMalloc");
  }
  // A post that nobody waited for (the caller left by an error) may still be answered:
  // the stream is drained first, so that the old scalars are not taken for the new ones.
  double* post(int n, hipStream_t s) {
    if (posted > 0) check(hipStreamSynchronize(s), "hipStreamSynchronize");
    uint64_t* q = reinterpret_cast<uint64_t*>(h);
    for (int i = 0; i < n; ++i) __atomic_store_n(q + i, kUnset, __ATOMIC_RELAXED);
    __atomic_thread_fence(__ATOMIC_SEQ_CST);
    posted = n;
    return h;
  }
  const double* wait(hipStream_t s) {
    using clock = std::chrono::steady_clock;
    if (posted == 0) throw Error(MRCM_EDEVICE, "no scalars to wait for");
    const uint64_t* q = reinterpret_cast<const uint64_t*>(h);
    int i = 0;
    auto set = [&]() {
      while (i < posted && __atomic_load_n(q + i, __ATOMIC_RELAXED) != kUnset) ++i;
      return i == posted;
    };
    auto ask = clock::now() + kAskEvery;
    for (unsigned spin = 1; !set(); ++spin) {
      __builtin_ia32_pause();
      if (spin % kSpins != 0) continue;
      std::this_thread::yield();
      if (clock::now() < ask) continue;
      const hipError_t e = hipStreamQuery(s);
      if (e == hipErrorNotReady) {
        ask = clock::now() + kAskEvery;
        continue;
      }
      check(e, "hipStreamQuery");
      if (set()) break;
      throw Error(MRCM_EDEVICE, "a kernel's scalars did not arrive");
    }
    __atomic_thread_fence(__ATOMIC_ACQUIRE);
    posted = 0;
    return h;
  }
};

}  // namespace mrcm
