// static_bot.hip -- the fast greedy heuristic (Alg. 2) on a static set of
// bags of tasks, and the cloud-wide reward of a placement (Eqs. (14)-(16)
// summed: beta_vc per VM used in a VC, minus beta_tc per VM bought in the
// paid cloud, minus gamma_vc per VM left idle in a VC; the example of
// Sec. VII).
//
// Two forms.  Many scenarios: one lane per scenario (static_lane_*, below).
// Few: one wavefront per scenario, one lane per vehicular cloud (K <= 64).  A
// task's VC is the lowest lane of the ballot "free >= need": the first VC in
// the cloud's order with room, found in one instruction instead of Alg. 2's
// scan.  Tasks are read 64 at a time (one coalesced load), broadcast from
// their lane with readlane, and their placements written back by the lane
// that read them.  The tasks of one scenario are placed in order (each
// depends on the VMs the earlier ones took); scenarios run in parallel.
#include "device.hpp"
#include "kernels.hpp"

namespace mdpvi {

namespace {

constexpr int kStaticWaves = 4;                   // scenarios per workgroup
constexpr int32_t kStaticMaxUnits = 1 << 30;      // largest capacity or task need
constexpr int32_t kPlacePaid = -1;
constexpr int32_t kPlaceEmpty = -2;

__device__ __forceinline__ long long wave_sum(long long v) {
  for (int off = kWave / 2; off > 0; off >>= 1) v += __shfl_xor(v, off, kWave);
  return v;
}

// Reward of the totals, products rounded before the subtractions (no
// contraction), left to right.
__device__ __forceinline__ double cloud_reward(long long vc, long long paid, long long idle,
                                               double bvc, double btc, double gvc) {
  const double a = __dmul_rn(bvc, static_cast<double>(vc));
  const double b = __dmul_rn(btc, static_cast<double>(paid));
  const double c = __dmul_rn(gvc, static_cast<double>(idle));
  return __dsub_rn(__dsub_rn(a, b), c);
}

__device__ __forceinline__ void write_totals(long long b, long long vc, long long paid, long long idle,
                                             double bvc, double btc, double gvc,
                                             long long* totals, double* reward, int32_t* status) {
  totals[3 * b + 0] = vc;
  totals[3 * b + 1] = paid;
  totals[3 * b + 2] = idle;
  reward[b] = cloud_reward(vc, paid, idle, bvc, btc, gvc);
  status[b] = 0;
}

// 0, or 1 if a capacity of the scenario is out of [0, 2^30], or 2 if a task
// need is out of [0, 2^30] (checked before any output is written).
__device__ __forceinline__ int32_t check_inputs(int lane, int K, long long T, const int32_t* cb,
                                                const int32_t* nb) {
  const int32_t c = lane < K ? cb[lane] : 0;
  if (__ballot(c < 0 || c > kStaticMaxUnits)) return 1;
  for (long long t0 = 0; t0 < T; t0 += kWave) {
    const long long t = t0 + lane;
    const int32_t n = t < T ? nb[t] : 0;
    if (__ballot(n < 0 || n > kStaticMaxUnits)) return 2;
  }
  return 0;
}

__global__ __launch_bounds__(kWave* kStaticWaves) void static_first_fit_kernel(
    long long B, int K, long long T, const int32_t* __restrict__ caps, const int32_t* __restrict__ need,
    double bvc, double btc, double gvc, int32_t* __restrict__ place, int32_t* __restrict__ used,
    long long* __restrict__ totals, double* __restrict__ reward, int32_t* __restrict__ status) {
  const int lane = threadIdx.x % kWave;
  const long long b = static_cast<long long>(blockIdx.x) * kStaticWaves + threadIdx.x / kWave;
  if (b >= B) return;  // the whole wavefront leaves together
  const int32_t* cb = caps + b * K;
  const int32_t* nb = need + b * T;
  const int32_t bad = check_inputs(lane, K, T, cb, nb);
  if (bad) {
    if (lane == 0) status[b] = bad;
    return;
  }
  const int32_t cap = lane < K ? cb[lane] : 0;
  int32_t free = lane < K ? cap : -1;  // lanes past the last VC never have room
  long long paid = 0;                  // wavefront-uniform
  for (long long t0 = 0; t0 < T; t0 += kWave) {
    const long long t = t0 + lane;
    const int32_t mine = t < T ? nb[t] : 0;
    int32_t my_place = kPlaceEmpty;
    const int cnt = static_cast<int>(T - t0 < kWave ? T - t0 : kWave);
    for (int i = 0; i < cnt; ++i) {
      const int32_t n = __builtin_amdgcn_readlane(mine, i);
      if (n > 0) {
        const unsigned long long fits = __ballot(free >= n);
        int32_t where = kPlacePaid;
        if (fits) {
          where = static_cast<int32_t>(__builtin_ctzll(fits));
          if (lane == where) free -= n;
        } else {
          paid += n;
        }
        if (lane == i) my_place = where;
      }
    }
    if (t < T) place[b * T + t] = my_place;
  }
  const long long u = lane < K ? cap - free : 0;
  const long long f = lane < K ? free : 0;
  if (lane < K) used[b * K + lane] = static_cast<int32_t>(u);
  const long long vc = wave_sum(u), idle = wave_sum(f);
  if (lane == 0) write_totals(b, vc, paid, idle, bvc, btc, gvc, totals, reward, status);
}

// Score a given placement: place[t] = VC index, kPlacePaid, or anything for
// an empty slot (need 0).  Status 3: a VC over its capacity; 4: a place code
// out of [-1, K) on a task; nothing but the status is written then.
__global__ __launch_bounds__(kWave* kStaticWaves) void static_score_kernel(
    long long B, int K, long long T, const int32_t* __restrict__ caps, const int32_t* __restrict__ need,
    const int32_t* __restrict__ place, double bvc, double btc, double gvc, int32_t* __restrict__ used,
    long long* __restrict__ totals, double* __restrict__ reward, int32_t* __restrict__ status) {
  const int lane = threadIdx.x % kWave;
  const long long b = static_cast<long long>(blockIdx.x) * kStaticWaves + threadIdx.x / kWave;
  if (b >= B) return;
  const int32_t* cb = caps + b * K;
  const int32_t* nb = need + b * T;
  const int32_t* pb = place + b * T;
  int32_t bad = check_inputs(lane, K, T, cb, nb);
  if (bad) {
    if (lane == 0) status[b] = bad;
    return;
  }
  const int32_t cap = lane < K ? cb[lane] : 0;
  long long u = 0, paid = 0;
  bool range_bad = false;
  for (long long t0 = 0; t0 < T; t0 += kWave) {
    const long long t = t0 + lane;
    const int32_t n = t < T ? nb[t] : 0;
    const int32_t p = t < T && n > 0 ? pb[t] : kPlaceEmpty;
    range_bad = range_bad || (n > 0 && (p < kPlacePaid || p >= K));
    if (n > 0 && p == kPlacePaid) paid += n;
    const int cnt = static_cast<int>(T - t0 < kWave ? T - t0 : kWave);
    for (int i = 0; i < cnt; ++i) {
      const int32_t ni = __builtin_amdgcn_readlane(n, i);
      const int32_t pi = __builtin_amdgcn_readlane(p, i);
      if (ni > 0 && lane == pi) u += ni;
    }
  }
  paid = wave_sum(paid);
  if (__ballot(range_bad)) bad = 4;
  else if (__ballot(lane < K && u > cap)) bad = 3;
  if (bad) {
    if (lane == 0) status[b] = bad;
    return;
  }
  if (lane < K) used[b * K + lane] = static_cast<int32_t>(u);
  const long long vc = wave_sum(u), idle = wave_sum(lane < K ? cap - u : 0);
  if (lane == 0) write_totals(b, vc, paid, idle, bvc, btc, gvc, totals, reward, status);
}

// ------------------------------------------------- one lane per scenario
//
// A wavefront per scenario leaves lanes past K idle and spends its time on
// the serial steps of every task: 964 us for a million scenarios of 11 VCs and
// 55 tasks (0.6 TB/s).  With one lane per scenario the same steps place 64
// tasks at a time: the free VMs of a scenario's VCs are the lane's registers
// (KB of them, those past K never have room), a task's VC is the last match of
// a scan from the highest VC down, and tasks and placements pass through LDS,
// 64 scenarios by up to 64 tasks, so that global memory is read and written a
// row (one scenario) at a time.  Rows of 65 words: lane l's task i lies in bank
// l + i.  A million such scenarios take 207 us and their scoring 183 us, bound by
// the 5 vector instructions per VC and task (two wavefronts per SIMD, as many
// as the LDS holds at 12 VCs); taking the first match with masks of the wavefront instead
// (4 vector instructions, but a chain of scalar ones) took 214 us.

constexpr int kLaneTasks = 64;
constexpr int kLaneStride = kLaneTasks + 1;

// Rows [0, rows) of a [rows][n] block at src (row pitch `pitch`), columns
// [c0, c0 + n), n <= 64, to or from tile rows; `rows` wavefront-uniform.
// Loaded straight into LDS, all rows in flight at once (the caller
// waits with tile_wait): through registers, 8 rows at a time, each batch waited
// for memory and a million scenarios took 278 us.
template <int STRIDE>
__device__ __forceinline__ void tile_in(int32_t* tile, const int32_t* src, long long pitch, int rows, int n) {
  if (static_cast<int>(threadIdx.x) < n) {
    const int32_t* p = src + threadIdx.x;
    for (int r = 0; r < rows; ++r)
      __builtin_amdgcn_global_load_lds(
          (const __attribute__((address_space(1))) void*)(p + r * pitch),
          (__attribute__((address_space(3))) void*)(tile + r * STRIDE), 4, 0, 0);
  }
}
__device__ __forceinline__ void tile_wait() {
  __builtin_amdgcn_s_waitcnt(0);
  __syncthreads();
}
// `good`: bit r set where row r may be written.
template <int STRIDE>
__device__ __forceinline__ void tile_out(const int32_t* tile, int32_t* dst, long long pitch, int rows, int n,
                                         unsigned long long good) {
  const int lane = threadIdx.x;
  int r = 0;
  for (; r + 8 <= rows; r += 8) {
    if ((good >> r & 0xffull) != 0xffull) break;   // row by row from here on
    int32_t v[8];
#pragma unroll
    for (int q = 0; q < 8; ++q) v[q] = tile[(r + q) * STRIDE + lane];
    if (lane < n) {
#pragma unroll
      for (int q = 0; q < 8; ++q) dst[(r + q) * pitch + lane] = v[q];
    }
  }
  for (; r < rows; ++r)
    if ((good >> r & 1ull) && lane < n) dst[r * pitch + lane] = tile[r * STRIDE + lane];
}

__device__ __forceinline__ bool units_ok(int32_t n) { return n >= 0 && n <= kStaticMaxUnits; }

// Loads the scenarios' capacities (ctile, cap) and checks capacities and
// needs; returns the lane's status (1, 2 or 0).  After it tile holds the
// first chunk of needs.
template <int KB>
__device__ __forceinline__ int32_t lane_inputs(int32_t* tile, int32_t* ctile, const int32_t* cb, const int32_t* nb,
                                               int K, long long T, int rows, int32_t (&cap)[KB]) {
  const int lane = threadIdx.x;
  const long long chunks = (T + kLaneTasks - 1) / kLaneTasks;
  bool need_bad = false;
  tile_in<KB + 1>(ctile, cb, K, rows, K);
  // chunk 0 last, so that the tile holds it afterwards
  for (long long c = chunks - 1; c >= 0; --c) {
    const int n = static_cast<int>(T - c * kLaneTasks < kLaneTasks ? T - c * kLaneTasks : kLaneTasks);
    if (c < chunks - 1) __syncthreads();
    tile_in<kLaneStride>(tile, nb + c * kLaneTasks, T, rows, n);
    tile_wait();
    for (int i = 0; i < n; ++i) need_bad = need_bad || !units_ok(tile[lane * kLaneStride + i]);
  }
  if (chunks == 0) tile_wait();
  int32_t bad = 0;
#pragma unroll
  for (int k = 0; k < KB; ++k) {
    cap[k] = k < K ? ctile[lane * (KB + 1) + k] : -1;
    if (k < K && !units_ok(cap[k])) bad = 1;
  }
  return lane >= rows ? 0 : bad ? bad : need_bad ? 2 : 0;
}

template <int KB>
__global__ __launch_bounds__(kWave) void static_lane_first_fit_kernel(
    long long B, int K, long long T, const int32_t* __restrict__ caps, const int32_t* __restrict__ need,
    double bvc, double btc, double gvc, int32_t* __restrict__ place, int32_t* __restrict__ used,
    long long* __restrict__ totals, double* __restrict__ reward, int32_t* __restrict__ status) {
  __shared__ int32_t tile[kWave * kLaneStride], ctile[kWave * (KB + 1)];
  const int lane = threadIdx.x;
  const long long b0 = static_cast<long long>(blockIdx.x) * kWave;
  const int rows = static_cast<int>(B - b0 < kWave ? B - b0 : kWave);
  const int32_t* nb = need + b0 * T;
  int32_t free[KB];
  const int32_t bad = lane_inputs<KB>(tile, ctile, caps + b0 * K, nb, K, T, rows, free);
  const bool live = lane < rows && bad == 0;
  const unsigned long long good = __ballot(live);
  long long vc = 0, paid = 0;
  for (long long t0 = 0; t0 < T; t0 += kLaneTasks) {
    const int n = static_cast<int>(T - t0 < kLaneTasks ? T - t0 : kLaneTasks);
    if (t0 > 0) {
      __syncthreads();
      tile_in<kLaneStride>(tile, nb + t0, T, rows, n);
      tile_wait();
    }
    for (int i = 0; i < n; ++i) {
      const int32_t want = tile[lane * kLaneStride + i];
      int32_t where = kPlacePaid;
#pragma unroll
      for (int k = KB - 1; k >= 0; --k) where = free[k] >= want ? k : where;
#pragma unroll
      for (int k = 0; k < KB; ++k) free[k] -= where == k ? want : 0;
      vc += where >= 0 ? want : 0;
      paid += where < 0 ? want : 0;
      tile[lane * kLaneStride + i] = want > 0 ? where : kPlaceEmpty;
    }
    __syncthreads();
    tile_out<kLaneStride>(tile, place + b0 * T + t0, T, rows, n, good);
  }
  long long idle = 0;
#pragma unroll
  for (int k = 0; k < KB; ++k) {
    if (k < K) {
      idle += free[k];
      ctile[lane * (KB + 1) + k] -= free[k];   // used = capacity - free
    }
  }
  __syncthreads();
  tile_out<KB + 1>(ctile, used + b0 * K, K, rows, K, good);
  if (live) write_totals(b0 + lane, vc, paid, idle, bvc, btc, gvc, totals, reward, status);
  else if (lane < rows) status[b0 + lane] = bad;
}

// The score of a given placement, one lane per scenario: the VMs taken on a
// VC leave a column of free VMs in LDS that the lane alone updates (a task
// beyond them marks the scenario instead, so that 32 bits hold them).  Its
// outputs follow the last task, so the needs are checked on the way.  Chunks
// of 32 tasks (half the LDS of 64: eight wavefronts per CU instead of four).
constexpr int kScoreTasks = 32;
constexpr int kScoreStride = kScoreTasks + 1;

template <int KB>
__global__ __launch_bounds__(kWave) void static_lane_score_kernel(
    long long B, int K, long long T, const int32_t* __restrict__ caps, const int32_t* __restrict__ need,
    const int32_t* __restrict__ place, double bvc, double btc, double gvc, int32_t* __restrict__ used,
    long long* __restrict__ totals, double* __restrict__ reward, int32_t* __restrict__ status) {
  constexpr int kIn = kWave * (2 * kScoreStride > KB + 1 ? 2 * kScoreStride : KB + 1);
  __shared__ int32_t in[kIn];             // the capacities, then a chunk of needs and of places
  __shared__ uint32_t left[KB * kWave];   // free VMs of (VC, lane)
  int32_t* need_t = in;
  int32_t* place_t = in + kWave * kScoreStride;
  const int lane = threadIdx.x;
  const long long b0 = static_cast<long long>(blockIdx.x) * kWave;
  const int rows = static_cast<int>(B - b0 < kWave ? B - b0 : kWave);
  const int32_t* nb = need + b0 * T;
  const int32_t* pb = place + b0 * T;
  tile_in<KB + 1>(in, caps + b0 * K, K, rows, K);
  tile_wait();
  int32_t cap[KB];
  bool cap_bad = false, need_bad = false, range_bad = false, over = false;
#pragma unroll
  for (int k = 0; k < KB; ++k) {
    if (k < K) {
      cap[k] = in[lane * (KB + 1) + k];
      cap_bad = cap_bad || !units_ok(cap[k]);
      left[k * kWave + lane] = static_cast<uint32_t>(cap[k]);
    }
  }
  long long vc = 0, paid = 0;
  for (long long t0 = 0; t0 < T; t0 += kScoreTasks) {
    const int n = static_cast<int>(T - t0 < kScoreTasks ? T - t0 : kScoreTasks);
    __syncthreads();
    tile_in<kScoreStride>(need_t, nb + t0, T, rows, n);
    tile_in<kScoreStride>(place_t, pb + t0, T, rows, n);
    tile_wait();
    for (int i = 0; i < n; ++i) {
      const int32_t want = need_t[lane * kScoreStride + i];
      const int32_t p = place_t[lane * kScoreStride + i];
      const bool task = want > 0, on = task && p >= 0 && p < K;
      need_bad = need_bad || !units_ok(want);
      range_bad = range_bad || (task && (p < kPlacePaid || p >= K));
      const int at = (on ? p : 0) * kWave + lane;
      const uint32_t f = left[at];
      const bool fits = on && f >= static_cast<uint32_t>(want);
      over = over || (on && !fits);
      left[at] = f - (fits ? static_cast<uint32_t>(want) : 0u);
      vc += on ? want : 0;
      paid += task && p == kPlacePaid ? want : 0;
    }
  }
  const int32_t bad = cap_bad ? 1 : need_bad ? 2 : range_bad ? 4 : over ? 3 : 0;
  const bool live = lane < rows && bad == 0;
  const unsigned long long good = __ballot(live);
  __syncthreads();
  long long idle = 0;
#pragma unroll
  for (int k = 0; k < KB; ++k) {
    if (k < K) {
      const int32_t f = static_cast<int32_t>(left[k * kWave + lane]);
      idle += f;
      in[lane * (KB + 1) + k] = cap[k] - f;
    }
  }
  __syncthreads();
  tile_out<KB + 1>(in, used + b0 * K, K, rows, K, good);
  if (live) write_totals(b0 + lane, vc, paid, idle, bvc, btc, gvc, totals, reward, status);
  else if (lane < rows) status[b0 + lane] = bad;
}

dim3 static_grid(long long B) { return dim3(static_cast<uint32_t>((B + kStaticWaves - 1) / kStaticWaves)); }

// Scenarios from which the lane form runs: its wavefronts take as long
// however few they are (5 us more than an empty call at 11 VCs and 55 tasks,
// 40 at 40 and 80), the wavefront form about 1.0 and 1.6 ns per scenario once
// it fills the chip.  Both forms at 16,384 and 65,536 scenarios, with the
// call's host part of 18 us: 23 and 25 against 23 and 74 us (11 VCs, 55 tasks),
// 59 and 63 against 32 and 107 us (40, 80).
constexpr long long kLaneScenarios = 32768;

// ... and for placing, whose lanes scan every VC for every task: from 25 VCs on
// the wavefronts' time passes the other form's for 32,768 scenarios (1.06 of
// it at 32 VCs and 200 tasks, 0.8 at 49,152); from 33 on it does so wherever the
// last of the 1,280 wavefronts that LDS holds at a time are few (40 VCs, 200
// tasks: 0.84 of it at 65,536, 1.26 at 98,304, 0.86 at 262,144), which the
// line bounds to a third of them; beyond 48 it is never faster (64 VCs, 200
// tasks: 1.9 at 32,768, 1.14 at 262,144).
bool lane_first_fit(long long B, int K) {
  const long long from = K <= 24 ? kLaneScenarios : K <= 32 ? 49152 : K <= 48 ? 163840 : (1ll << 62);
  return B >= from;
}

// CALL(most VCs of the kernel); LAST for those beyond 32, or 48.
#define MDPVI_STATIC_K(K_, CALL, LAST) \
  if ((K_) <= 4) CALL(4);              \
  else if ((K_) <= 8) CALL(8);         \
  else if ((K_) <= 12) CALL(12);       \
  else if ((K_) <= 16) CALL(16);       \
  else if ((K_) <= 24) CALL(24);       \
  else if ((K_) <= 32) CALL(32);       \
  else if ((K_) <= 48) CALL(48);       \
  else CALL(LAST)

}  // namespace

hipError_t launch_static_first_fit(long long B, int K, long long T, const int32_t* caps, const int32_t* need,
                                   double bvc, double btc, double gvc, int32_t* place, int32_t* used,
                                   long long* totals, double* reward, int32_t* status, hipStream_t s) {
  if (B == 0) return hipSuccess;
  if (lane_first_fit(B, K)) {
#define MDPVI_CALL(KB_)                                                                                             \
  hipLaunchKernelGGL((static_lane_first_fit_kernel<KB_>), dim3(static_cast<uint32_t>((B + kWave - 1) / kWave)),     \
                     dim3(kWave), 0, s, B, K, T, caps, need, bvc, btc, gvc, place, used, totals, reward, status)
    MDPVI_STATIC_K(K, MDPVI_CALL, 48);
#undef MDPVI_CALL
    return hipGetLastError();
  }
  hipLaunchKernelGGL(static_first_fit_kernel, static_grid(B), dim3(kWave * kStaticWaves), 0, s, B, K, T,
                     caps, need, bvc, btc, gvc, place, used, totals, reward, status);
  return hipGetLastError();
}

hipError_t launch_static_score(long long B, int K, long long T, const int32_t* caps, const int32_t* need,
                               const int32_t* place, double bvc, double btc, double gvc, int32_t* used,
                               long long* totals, double* reward, int32_t* status, hipStream_t s) {
  if (B == 0) return hipSuccess;
  if (B >= kLaneScenarios) {
#define MDPVI_CALL(KB_)                                                                                         \
  hipLaunchKernelGGL((static_lane_score_kernel<KB_>), dim3(static_cast<uint32_t>((B + kWave - 1) / kWave)),     \
                     dim3(kWave), 0, s, B, K, T, caps, need, place, bvc, btc, gvc, used, totals, reward, status)
    MDPVI_STATIC_K(K, MDPVI_CALL, 64);
#undef MDPVI_CALL
    return hipGetLastError();
  }
  hipLaunchKernelGGL(static_score_kernel, static_grid(B), dim3(kWave * kStaticWaves), 0, s, B, K, T,
                     caps, need, place, bvc, btc, gvc, used, totals, reward, status);
  return hipGetLastError();
}

}  // namespace mdpvi
