// Just enough of the HIP device language to compile a kernel with the host compiler and run one
// workgroup with a thread per lane, in any order of its wavefronts: threadIdx and blockIdx,
// __syncthreads (wavefronts that have returned count as arrived, as on the hardware), and the
// cross-lane operations of a full wavefront.  __shared__ memory holds, before a workgroup starts,
// words that read as a large double or as the integer 5.
#pragma once

#include <math.h>
#include <stdint.h>

#include <condition_variable>
#include <functional>
#include <mutex>
#include <thread>
#include <vector>

#define __global__
#define __device__
#define __host__
#define __shared__ static __attribute__((section("lds")))
#define __forceinline__ inline
#define __launch_bounds__(...)

struct Index3 {
  unsigned x = 0, y = 0, z = 0;
};
inline thread_local Index3 threadIdx, blockIdx, blockDim;

extern uint64_t __start_lds[], __stop_lds[];

namespace host_hip {

// A barrier for `n` threads, some of which may leave for good.
class Barrier {
 public:
  explicit Barrier(int n) : left_(n) {}
  void wait() {
    std::unique_lock<std::mutex> l(m_);
    const long turn = turn_;
    ++here_;
    if (!open()) cv_.wait(l, [&] { return turn != turn_; });
  }
  void leave() {
    std::lock_guard<std::mutex> l(m_);
    --left_;
    --running_;
    open();
  }
  bool all_waiting() {   // every thread that has not left
    std::lock_guard<std::mutex> l(m_);
    return here_ == running_;
  }
  void start() {
    std::lock_guard<std::mutex> l(m_);
    ++running_;
  }

 private:
  bool open() {
    if (here_ == 0 || here_ < left_) return false;
    here_ = 0;
    ++turn_;
    cv_.notify_all();
    return true;
  }
  std::mutex m_;
  std::condition_variable cv_;
  int left_, here_ = 0, running_ = 0;
  long turn_ = 0;
};

struct Wave {
  Barrier bar{64};
  uint64_t slot[64];
};
// Where set, atomic additions are put here and made later: the memory that other workgroups see
// at the same time is then changed by plain stores alone.
inline std::vector<std::pair<unsigned long long*, unsigned long long>>* deferred = nullptr;
inline thread_local Wave* wave;
inline thread_local Barrier* block;

// Every lane's value, at the same point of all 64 lanes.
template <class F>
auto exchange(uint64_t v, F f) {
  wave->slot[threadIdx.x % 64] = v;
  wave->bar.wait();
  auto r = f(wave->slot);
  wave->bar.wait();
  return r;
}

// Workgroup `b` of a kernel: `first` wavefronts at once, the others once those wait at a
// barrier of the workgroup (or have returned) and between() has run.
inline void run_block(unsigned b, int threads, int first, const std::function<void()>& between,
                      const std::function<void()>& kernel) {
  for (uint64_t* p = __start_lds; p < __stop_lds; ++p) *p = 0x4629000000000005ull;
  Barrier bar(threads);
  std::vector<Wave> waves(threads / 64);
  std::vector<std::thread> pool;
  auto start = [&](int lo, int hi) {
    for (int t = lo; t < hi; ++t) {
      bar.start();
      pool.emplace_back([&, t] {
        threadIdx.x = t;
        blockIdx.x = b;
        blockDim.x = threads;
        wave = &waves[t / 64];
        block = &bar;
        kernel();
        block->leave();
      });
    }
  };
  start(0, 64 * first);
  if (64 * first < threads) {
    while (!bar.all_waiting()) std::this_thread::yield();
    between();
    start(64 * first, threads);
  }
  for (auto& t : pool) t.join();
}

}  // namespace host_hip

inline void __syncthreads() { host_hip::block->wait(); }
inline unsigned __lane_id() { return threadIdx.x % 64; }
inline int __popcll(uint64_t v) { return __builtin_popcountll(v); }
inline uint64_t __umul64hi(uint64_t a, uint64_t b) {
  return (uint64_t)(((unsigned __int128)a * b) >> 64);
}
inline unsigned long long __ballot(bool p) {
  return host_hip::exchange(p, [](const uint64_t* s) {
    unsigned long long m = 0;
    for (int i = 0; i < 64; ++i) m |= (unsigned long long)(s[i] != 0) << i;
    return m;
  });
}
inline double __shfl_xor(double v, int o, int = 64) {
  uint64_t u = __builtin_bit_cast(uint64_t, v);
  const int src = (threadIdx.x % 64) ^ o;
  return __builtin_bit_cast(double, host_hip::exchange(u, [=](const uint64_t* s) { return s[src]; }));
}
inline void atomicAdd(unsigned long long* p, unsigned long long v) {
  if (host_hip::deferred) host_hip::deferred->emplace_back(p, v);   // one thread's, in the kernels used
  else __atomic_fetch_add(p, v, 5);
}
inline void atomicOr(unsigned* p, unsigned v) { __atomic_fetch_or(p, v, 5); }

// Row shifts and row_bcast:15 of the data-parallel primitives; a source outside the row or a row
// outside the mask leaves `old` (0 with bound_ctrl).
inline int host_update_dpp(int old, int v, int ctrl, int row_mask, int, bool bound) {
  const int lane = threadIdx.x % 64, row = lane / 16;
  int src = -1;
  if (ctrl > 0x110 && ctrl < 0x120) src = lane % 16 >= ctrl - 0x110 ? lane - (ctrl - 0x110) : -1;
  if (ctrl == 0x142) src = row > 0 ? 16 * row - 1 : -1;
  const bool on = (row_mask >> row) & 1;
  return host_hip::exchange((uint32_t)v, [=](const uint64_t* s) {
    return !on ? old : src >= 0 ? (int)(uint32_t)s[src] : bound ? 0 : old;
  });
}
inline int host_readlane(int v, int lane) {
  return host_hip::exchange((uint32_t)v, [=](const uint64_t* s) { return (int)(uint32_t)s[lane]; });
}
#define __builtin_amdgcn_update_dpp host_update_dpp
#define __builtin_amdgcn_readlane host_readlane
