// What the single-launch kernels share (the tridiagonalisation, the Lanczos
// steps): all work-groups resident together, exchanging vectors through device
// memory inside one launch.
//
// A vector is published with accesses that are coherent over the XCDs by
// themselves (agent-scope atomics of 8 bytes), every step into fresh memory that
// was filled with a value no arithmetic produces; a reader polls the entries it
// needs until they differ from it. So a step costs one trip from writer to reader
// and no cache is written back or invalidated. A wait that exceeds its bound
// raises *err and ends the work-group, and with it, in time, the others.
#ifndef GEVP_EXCHANGE_H
#define GEVP_EXCHANGE_H
#include <algorithm>
#include <condition_variable>
#include <mutex>

#include "common.h"

namespace {
constexpr unsigned long long HOLE = 0x7ff8a5c35a3cf00dull;  // a NaN with a payload of its own
__device__ __forceinline__ void publish(unsigned long long* dst, double v) {
  unsigned long long u = __double_as_longlong(v);
  u = u == HOLE ? 0x7ff8000000000000ull : u;
  __hip_atomic_store(dst, u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
__device__ __forceinline__ unsigned long long peek(const unsigned long long* src) {
  return __hip_atomic_load(src, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
__global__ __launch_bounds__(256) void k_fill_holes(unsigned long long* x, int64_t words, int* err) {
  const int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x;
  if (i == 0 && err) *err = 0;
  for (int64_t k = i; k < words; k += (int64_t)gridDim.x * 256) x[k] = HOLE;
}

// sum over the wave, the same in every lane: within rows of 16 lanes, then
// across the rows, by lane shifts of the vector unit
template <int CTRL, int ROWS>
__device__ __forceinline__ double dpp_move(double v) {
  const unsigned long long u = __double_as_longlong(v);
  const unsigned lo = __builtin_amdgcn_update_dpp(0, (unsigned)u, CTRL, ROWS, 0xf, true);
  const unsigned hi = __builtin_amdgcn_update_dpp(0, (unsigned)(u >> 32), CTRL, ROWS, 0xf, true);
  return __longlong_as_double(((unsigned long long)hi << 32) | lo);
}
__device__ __forceinline__ double wave_total(double v) {
  v += dpp_move<0x111, 0xf>(v);  // row_shr 1, 2, 4, 8
  v += dpp_move<0x112, 0xf>(v);
  v += dpp_move<0x114, 0xf>(v);
  v += dpp_move<0x118, 0xf>(v);
  v += dpp_move<0x142, 0xa>(v);  // lane 15 of rows 0 and 2 to the next row
  v += dpp_move<0x143, 0xc>(v);  // lane 31 to the upper half
  const unsigned long long u = __double_as_longlong(v);
  const unsigned lo = __builtin_amdgcn_readlane((unsigned)u, 63);
  const unsigned hi = __builtin_amdgcn_readlane((unsigned)(u >> 32), 63);
  return __longlong_as_double(((unsigned long long)hi << 32) | lo);
}

// Sums over the wave of 16 values a lane: the lane returns the total of value
// 4 * (lane / 16) + (lane & 3).  The first two levels exchange halves of the
// values as they add them, the last two rotate within rows of 16 lanes.
__device__ __forceinline__ double2 swap_halves32(double a, double b) {
  const unsigned long long ua = __double_as_longlong(a), ub = __double_as_longlong(b);
  const auto lo = __builtin_amdgcn_permlane32_swap((unsigned)ua, (unsigned)ub, false, false);
  const auto hi = __builtin_amdgcn_permlane32_swap((unsigned)(ua >> 32), (unsigned)(ub >> 32), false, false);
  return make_double2(__longlong_as_double(((unsigned long long)hi[0] << 32) | lo[0]),
                      __longlong_as_double(((unsigned long long)hi[1] << 32) | lo[1]));
}
__device__ __forceinline__ double2 swap_halves16(double a, double b) {
  const unsigned long long ua = __double_as_longlong(a), ub = __double_as_longlong(b);
  const auto lo = __builtin_amdgcn_permlane16_swap((unsigned)ua, (unsigned)ub, false, false);
  const auto hi = __builtin_amdgcn_permlane16_swap((unsigned)(ua >> 32), (unsigned)(ub >> 32), false, false);
  return make_double2(__longlong_as_double(((unsigned long long)hi[0] << 32) | lo[0]),
                      __longlong_as_double(((unsigned long long)hi[1] << 32) | lo[1]));
}
__device__ __forceinline__ double wave_totals16(const double (&v)[16]) {
  double a[8], b[4];
#pragma unroll
  for (int k = 0; k < 8; ++k) {
    const double2 t = swap_halves32(v[k], v[k + 8]);
    a[k] = t.x + t.y;
  }
#pragma unroll
  for (int k = 0; k < 4; ++k) {
    const double2 t = swap_halves16(a[k], a[k + 4]);
    b[k] = t.x + t.y;
    b[k] += dpp_move<0x128, 0xf>(b[k]);  // row_ror 8, 4, 2, 1
    b[k] += dpp_move<0x124, 0xf>(b[k]);
    b[k] += dpp_move<0x122, 0xf>(b[k]);
    b[k] += dpp_move<0x121, 0xf>(b[k]);
  }
  const int l = threadIdx.x & 3;
  const double x = l & 1 ? b[1] : b[0], y = l & 1 ? b[3] : b[2];
  return l & 2 ? y : x;
}

}  // namespace

constexpr int EXCHANGE_SPINS = 1 << 18;  // polls before a wait gives up: some tenths of a second

namespace {
inline gevp_status fill_holes(gevp_ctx* c, unsigned long long* x, int64_t words, int* err) {
  hipLaunchKernelGGL(k_fill_holes, dim3((unsigned)std::min<int64_t>((words + 255) / 256, 4096)), dim3(256), 0,
                     c->stream, x, words, err);
  GEVP_HIP_TRY(hipGetLastError());
  return GEVP_OK;
}
}  // namespace

// The compute units of a device that such launches of this process may count on: a
// launch takes as many as it has work-groups before it starts and gives them back
// when it has ended, so that launches of several threads never each hold a part of
// what the others wait for.  It waits in turn, asleep, and for no longer than the
// launches before it run: a share is taken only when the stream has nothing else
// left to do, and a holder never waits for a second one.  (It is not left to chance
// which kernel runs: the results would then depend, in their last bits, on who else
// is running.)
class LaunchTurn {
 public:
  LaunchTurn(gevp_ctx* c, int64_t groups) : d_(device(c->device)) {
    (void)hipStreamSynchronize(c->stream);
    const int cus = gevp_device_cus(c->device);
    share_ = (int)std::min<int64_t>(groups, cus);
    std::unique_lock<std::mutex> lock(d_.mu);
    const unsigned long long ticket = d_.next++;
    d_.cv.wait(lock, [&] { return ticket == d_.serving && d_.used + share_ <= cus; });
    d_.used += share_;
    ++d_.serving;
    lock.unlock();
    d_.cv.notify_all();
  }
  ~LaunchTurn() {
    {
      std::lock_guard<std::mutex> lock(d_.mu);
      d_.used -= share_;
    }
    d_.cv.notify_all();
  }
  LaunchTurn(const LaunchTurn&) = delete;
  LaunchTurn& operator=(const LaunchTurn&) = delete;

 private:
  struct Device {
    std::mutex mu;
    std::condition_variable cv;
    int used = 0;
    unsigned long long next = 0, serving = 0;
  };
  static Device& device(int i) {
    static Device all[64];
    return all[i >= 0 && i < 64 ? i : 0];
  }
  Device& d_;
  int share_;
};

inline int exchange_spins(const gevp_ctx* c) {
  const int n = (c->parent ? c->parent : c)->polls;
  return n < 0 ? EXCHANGE_SPINS : n;
}

// whether this handle's stream may take such a launch now: not where one gave up or
// other work is meant to run beside (nor under capture, which a call that waits for
// its outcome ends in any case)
inline bool resident_allowed(gevp_ctx* c) {
  return !c->shared_gpu && !stream_capturing(c);
}

// whether all work-groups of a launch fit the device at once. An ordinary launch
// is enough then: kernels of other streams end by themselves, so all become
// resident. (A cooperative launch gives the process one more hardware queue for
// good, which slowed batches on eight streams from 94 to 139 ms.)
template <class F>
bool resident_fits(gevp_ctx* c, F f, int threads, int64_t groups) {
  int per_cu = 0, cus = 0;
  if (hipOccupancyMaxActiveBlocksPerMultiprocessor(&per_cu, f, threads, 0) != hipSuccess ||
      hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, c->device) != hipSuccess) {
    (void)hipGetLastError();
    return false;
  }
  return (int64_t)per_cu * cus >= groups;
}

#endif
