// orbit.hpp -- value iteration and fixed-policy evaluation on the orbits of
// the host permutations.
//
// All hosts share one capacity and one set of rates, so permuting the hosts
// maps the chain onto itself.  Value iteration: an iterate that is invariant
// under host permutations (V^0 = 0, any constant, any earlier solution) stays
// so, and a Jacobi sweep needs one backup per orbit and class instead of one
// per state.  Evaluation: so too where the policy's target load (the
// occupancy of the host it places on, or none) is the same over each orbit;
// which of several equally loaded hosts it names does not matter.
// The orbits of the (C+1)^K occupancies are the multisets of K digits in
// 0..C, binom(C+K, K) of them (8,008 against 1,771,561 at K = 6, C = 10).
// Value iteration's sums are exact or independent of the host order
// (stay_sum), so its orbit iterates are the full sweeps' bit for bit;
// evaluation's differ from them in the rounding of its FP64 sums.
//
// An orbit is named by its rank in the combinatorial number system: with
// the digits ascending, n_0 <= .. <= n_{K-1},
//   rank = sum_i binom(n_i + i, i + 1).
// A table holds, per orbit, the ranks its backup reads (layout row by row,
// n entries each):
//   rows 0..K-1        one unit less on the host of position k (itself at n_k = 0)
//   rows K..2K-1       the host of position k emptied
//   rows (2+e)K + k    a class-e task placed on the host of position k (n, the
//                      -inf entry of the arrival terms, where it has no room)
#pragma once

#include <type_traits>

#include "device.hpp"

namespace mdpvi {

constexpr uint32_t kOrbitMax = 1u << 20;       // orbits the form covers
constexpr uint32_t kOrbitBinom = 2048;         // entries of the rank table (K (C+1))
constexpr int kOrbitBlock = 128;               // threads of a sweep workgroup
constexpr uint32_t kOrbitGrid = 1024;          // most workgroups of a sweep
constexpr int kOrbitChunk = 32;                // sweeps of a chunk (a multiple of kResSlots)
constexpr int kOrbitFirst = 8;                 // ... of a solve's first one (likewise)
constexpr int kOrbitLdsBlock = 1024;           // most threads of an LDS-resident solve
constexpr int kOrbitSmallBlock = 256;          // ... of a batch's instances of at most as many lanes
constexpr int kOrbitBigBlock = 512;            // ... of its larger ones
constexpr size_t kOrbitLds = 156 * 1024;       // its dynamic LDS (the kernels hold up to 4 KB more)

// The two operations: the stored type of the iterates.
struct OrbitVi {
  using T = float;
  static constexpr bool kEval = false;
};
struct OrbitEval {
  using T = double;
  static constexpr bool kEval = true;
};

// What the check of a start (and a policy) found, as bits; the host's copy of
// OrbitCtl::done says it too.
constexpr uint32_t kOrbitDiffers = 1, kOrbitNoRoom = 2;   // not invariant; an infeasible action
constexpr long long kOrbitDoneRefused = -2, kOrbitDoneInfeasible = -3;
constexpr uint32_t kOrbitCheckGrid = 8192;                // most workgroups of the check

// Control words of an orbit solve, in device memory and, as the host's copy,
// in pinned host memory.
struct OrbitCtl {
  long long done;      // -1 while running, else the index of the final iterate; host copy
                       // also kOrbitDoneRefused or kOrbitDoneInfeasible
  double residual;     // its residual
  long long base;      // sweeps done before the chunk that runs (device copy)
  double tol;          // the stopping tolerance (device copy)
  long long refused;   // the check's bits (device copy)
  long long pad[11];
};

struct OrbitShape {
  int32_t K, C, J, R;
  int32_t L;              // value slots (and lanes) per orbit: J rounded up to 1, 2, 4 or 8
  int32_t dig_bits;       // bits per digit in dig: 8, or 4 beyond 8 hosts
  int32_t wide;           // 1: table entries of 32 bits, 0: of 16
  uint32_t n;             // orbits
  uint64_t n_occ;
  FastDiv divR;
  const uint32_t* binom;  // [K][C+1]: binom(v + i, i + 1)
  const uint64_t* dig;    // [n]: the ascending digits, packed
  const uint32_t* rep;    // [n]: the occupancy index of the representative
  const void* tab;        // [(2 + J) K][n]
};

// The parameters an orbit backup needs.
struct OrbitParams {
  double p[kMaxJ], r_place[kMaxJ], r_reject[kMaxJ];
  double mu_L, nu_L, hold, gamma;
  int32_t size[kMaxJ];
};

// The buffers of a solve.
struct OrbitWork {
  void* V[2];          // iterates [n][L]
  double* A[2];        // their arrival terms [n + 1], the last -inf
  uint32_t* act;       // evaluation [n][L]: rank the arrival leads to, top bit: placed on a host
  double* res;         // residual words: kResSlots slots of kOrbitGrid
  OrbitCtl* ctl;
  uint32_t* found;     // a single instance's check: a workgroup's bits each
};

// One instance of a batch (orbit_batch.hip).
struct OrbitInst {
  OrbitShape S;
  OrbitParams P;
  OrbitWork W;          // W.res: launched sweeps only
  int64_t offset;       // its first state in the concatenated arrays
  uint32_t grid;        // workgroups of its sweeps
  int32_t inst;         // its index in the batch
};

// W as the sweep of (chunk) index i reads and writes it.
__host__ __device__ inline OrbitWork orbit_work(const OrbitWork& W, long long i) {
  OrbitWork w = W;
  if (i & 1) {
    w.V[0] = W.V[1];
    w.V[1] = W.V[0];
    w.A[0] = W.A[1];
    w.A[1] = W.A[0];
  }
  return w;
}

// x[e] for a lane's e < L, x the same for the wavefront.  Every entry goes
// through a scalar register and a select: indexed by lane, the parameters
// would be kept in scratch memory.
__device__ __forceinline__ double pick(const double (&x)[kMaxJ], int e, int L) {
  double v = 0.0;
#pragma unroll
  for (int i = 0; i < kMaxJ; ++i)
    if (i < L) {
      const long long b = __double_as_longlong(x[i]);
      const unsigned lo = static_cast<unsigned>(__builtin_amdgcn_readfirstlane(static_cast<int>(b)));
      const unsigned hi = static_cast<unsigned>(__builtin_amdgcn_readfirstlane(static_cast<int>(b >> 32)));
      const double s = __longlong_as_double(static_cast<long long>(static_cast<unsigned long long>(hi) << 32 | lo));
      v = e == i ? s : v;
    }
  return v;
}

// Digits of occupancy o (KX = K hosts, or 16 for any K up to 16: the digits
// beyond K are zero).
template <int KX>
__device__ __forceinline__ void orbit_digits(const OrbitShape& S, uint32_t o, int (&n)[KX]) {
#pragma unroll
  for (int k = 0; k < KX; ++k) {
    if (KX <= 8 || k < S.K) {
      const uint32_t q = fast_div(o, S.divR);
      n[k] = static_cast<int>(o - q * static_cast<uint32_t>(S.R));
      o = q;
    } else {
      n[k] = 0;
    }
  }
}

// Rank of the digits n (sorted here; padding digits sort to the front).  B:
// the rank table in LDS.
template <int KX>
__device__ __forceinline__ uint32_t orbit_rank(const OrbitShape& S, const uint32_t* B, int (&n)[KX]) {
#pragma unroll
  for (int a = 0; a < KX - 1; ++a) {
#pragma unroll
    for (int b = 0; b < KX - 1 - a; ++b) {
      const int lo = min(n[b], n[b + 1]), hi = max(n[b], n[b + 1]);
      n[b] = lo;
      n[b + 1] = hi;
    }
  }
  uint32_t r = 0;
#pragma unroll
  for (int k = 0; k < KX; ++k) {
    const int pos = KX <= 8 ? k : k - (KX - S.K);   // padding digits are zero and add nothing
    if (KX <= 8 || pos >= 0) r += B[pos * S.R + n[k]];
  }
  return r;
}

// Readers of the arrays of a backup: raw buffer views of global memory (one
// 32-bit lane offset per load, uniform row offsets in scalar registers) or LDS.
template <typename Idx>
struct TabView {
  BufView v;
  __device__ __forceinline__ uint32_t operator()(uint32_t lane, uint32_t row) const {
    if constexpr (sizeof(Idx) == 2)
      return static_cast<uint16_t>(__builtin_amdgcn_raw_buffer_load_b16(v.r, lane * 2u, row * 2u, 0));
    else
      return __builtin_amdgcn_raw_buffer_load_b32(v.r, lane * 4u, row * 4u, 0);
  }
};
template <typename Idx>
__device__ __forceinline__ TabView<Idx> tab_view(const OrbitShape& S) {
  return {make_view(S.tab, static_cast<uint32_t>(sizeof(Idx)) * S.n * static_cast<uint32_t>((2 + S.J) * S.K))};
}
template <typename T>
struct GlobalView {
  BufView v;
  __device__ __forceinline__ T operator()(uint32_t i) const {
    if constexpr (sizeof(T) == 4)
      return __builtin_bit_cast(T, __builtin_amdgcn_raw_buffer_load_b32(v.r, i * 4u, 0, 0));
    else
      return __builtin_bit_cast(T, __builtin_amdgcn_raw_buffer_load_b64(v.r, i * 8u, 0, 0));
  }
};
template <typename T>
__device__ __forceinline__ GlobalView<T> global_view(const void* p, uint32_t n) {
  return {make_view(p, n * static_cast<uint32_t>(sizeof(T)))};
}
template <typename T>
struct LdsView {
  const T* p;
  __device__ __forceinline__ T operator()(uint32_t i) const { return p[i]; }
};

// What one lane's backup (class e of orbit r) reads.  KX = K hosts, or 16 for
// any K of 9..16 (the positions beyond K read the orbit itself with weight 0
// and the -inf entry).
template <class Op, int KX>
struct OrbitIdx {
  uint32_t rel[KX], rst[KX];
  uint32_t plc[Op::kEval ? 1 : KX];   // evaluation: the orbit's act word
  uint64_t dig;
};

template <class Op, int KX, class Tab>
__device__ __forceinline__ void orbit_load_idx(const OrbitShape& S, Tab tab, GlobalView<uint64_t> dig,
                                               GlobalView<uint32_t> act, uint32_t r, uint32_t e,
                                               OrbitIdx<Op, KX>& x) {
  const int K = KX <= 8 ? KX : S.K;
  const uint32_t rp = e * static_cast<uint32_t>(K) * S.n + r;
#pragma unroll
  for (int k = 0; k < KX; ++k) x.rel[k] = k < K ? tab(r, static_cast<uint32_t>(k) * S.n) : r;
  if constexpr (Op::kEval) {
    x.plc[0] = act(r * static_cast<uint32_t>(S.L) + e);
  } else {
#pragma unroll
    for (int k = 0; k < KX; ++k) x.plc[k] = k < K ? tab(rp, static_cast<uint32_t>(2 * K + k) * S.n) : S.n;
  }
#pragma unroll
  for (int k = 0; k < KX; ++k) x.rst[k] = k < K ? tab(r, static_cast<uint32_t>(K + k) * S.n) : r;
  x.dig = dig(r);
}

template <int KX>
__device__ __forceinline__ int orbit_digit(uint64_t dig, int k) {
  return KX <= 8 ? static_cast<int>((dig >> (8 * k)) & 0xffu) : static_cast<int>((dig >> (4 * k)) & 0xfu);
}

// max() without the quieting of fmax: neither operand is a signalling NaN.
__device__ __forceinline__ double orbit_max(double a, double b) {
  double r;
  asm("v_max_f64 %0, %1, %2" : "=v"(r) : "v"(a), "v"(b));
  return r;
}

// The new value of (r, e).  Value iteration: the arithmetic of backup_arrival
// (sweep_impl.hpp).
template <class Op, int KX, int L, class VV, class AV>
__device__ __forceinline__ typename Op::T orbit_backup(const OrbitShape& S, const OrbitIdx<Op, KX>& x, VV V, AV A,
                                                       uint32_t r, uint32_t e, double r_place, double r_reject,
                                                       const OrbitParams& P, typename Op::T& own) {
  using T = typename Op::T;
  constexpr int NA = Op::kEval ? 1 : KX;
  const int K = KX <= 8 ? KX : S.K;
  own = V(r * L + e);
  T vd[KX], vr[KX];
  double aa[NA], a_rej = 0.0;
#pragma unroll
  for (int k = 0; k < KX; ++k) vd[k] = V(x.rel[k] * L + e);
  if constexpr (Op::kEval) {
    aa[0] = A(x.plc[0] & 0x7fffffffu);
  } else {
    a_rej = A(r);
#pragma unroll
    for (int k = 0; k < KX; ++k) aa[k] = A(x.plc[k]);
  }
#pragma unroll
  for (int k = 0; k < KX; ++k) vr[k] = V(x.rst[k] * L + e);
  int load = 0;
#pragma unroll
  for (int k = 0; k < KX; ++k) load += orbit_digit<KX>(x.dig, k);
  const double fu = static_cast<double>(S.K * S.C - load);   // free units
  double sum = fu * static_cast<double>(own), rs = 0.0, ab = aa[0];
#pragma unroll
  for (int k = 0; k < KX; ++k)
    sum = fma(static_cast<double>(orbit_digit<KX>(x.dig, k)), static_cast<double>(vd[k]), sum);
#pragma unroll
  for (int k = 1; k < NA; ++k) ab = orbit_max(ab, aa[k]);
#pragma unroll
  for (int k = 0; k < KX; ++k) rs += k < K ? static_cast<double>(vr[k]) : 0.0;
  const double D = fma(P.nu_L, rs, P.mu_L * sum);   // stay_sum
  double best;
  if constexpr (Op::kEval)
    best = fma(P.gamma, ab, fma(-P.hold, fu, x.plc[0] >> 31 ? r_place : r_reject));
  else
    best = orbit_max(fma(P.gamma, a_rej, fma(-P.hold, fu, r_reject)), fma(P.gamma, ab, fma(-P.hold, fu, r_place)));
  return static_cast<T>(fma(P.gamma, D, best));
}

// v of lane E of the group of L neighbouring lanes.
template <int L, int E>
__device__ __forceinline__ int group_lane_b32(int b) {
  if constexpr (L == 2)
    return __builtin_amdgcn_mov_dpp(b, E == 0 ? 0xA0 : 0xF5, 0xf, 0xf, true);   // quad_perm
  else if constexpr (L == 4)
    return __builtin_amdgcn_mov_dpp(b, 0x55 * E, 0xf, 0xf, true);
  else
    return __shfl(b, (static_cast<int>(threadIdx.x) % kWave & ~(L - 1)) + E, kWave);
}
template <int L, int E, typename T>
__device__ __forceinline__ T group_lane(T v) {
  if constexpr (L == 1) {
    return v;
  } else if constexpr (sizeof(T) == 4) {
    return __builtin_bit_cast(T, group_lane_b32<L, E>(__builtin_bit_cast(int, v)));
  } else {
    const long long b = __builtin_bit_cast(long long, v);
    const unsigned lo = static_cast<unsigned>(group_lane_b32<L, E>(static_cast<int>(b)));
    const unsigned hi = static_cast<unsigned>(group_lane_b32<L, E>(static_cast<int>(b >> 32)));
    return __builtin_bit_cast(T, static_cast<long long>(static_cast<unsigned long long>(hi) << 32 | lo));
  }
}

// The arrival term of an orbit from the new values of its lanes: the FMA
// chain of backup_arrival.
template <int L, int E = 0, typename T>
__device__ __forceinline__ double orbit_arrival(T vn, int J, const OrbitParams& P, double a = 0.0) {
  const T v = group_lane<L, E>(vn);
  if (E < J) a = fma(P.p[E], static_cast<double>(v), a);
  if constexpr (E + 1 < L) return orbit_arrival<L, E + 1>(vn, J, P, a);
  return a;
}

// Largest of the wavefront's v (not NaN) in lane 63: row shifts, then the
// rows' last lanes broadcast on.
template <int CTRL, int ROWS>
__device__ __forceinline__ double dpp_max_step(double v) {
  const long long b = __double_as_longlong(v);
  const int lo = static_cast<int>(b), hi = static_cast<int>(b >> 32);
  const int lo2 = __builtin_amdgcn_update_dpp(lo, lo, CTRL, ROWS, 0xf, false);
  const int hi2 = __builtin_amdgcn_update_dpp(hi, hi, CTRL, ROWS, 0xf, false);
  return orbit_max(v, __longlong_as_double(static_cast<long long>(
                          (static_cast<unsigned long long>(static_cast<unsigned>(hi2)) << 32) |
                          static_cast<unsigned>(lo2))));
}
__device__ __forceinline__ double wave_max_last(double v) {
  v = dpp_max_step<0x111, 0xf>(v);   // row_shr:1
  v = dpp_max_step<0x112, 0xf>(v);   // row_shr:2
  v = dpp_max_step<0x114, 0xf>(v);   // row_shr:4
  v = dpp_max_step<0x118, 0xf>(v);   // row_shr:8
  v = dpp_max_step<0x142, 0xa>(v);   // row_bcast:15
  v = dpp_max_step<0x143, 0xc>(v);   // row_bcast:31
  return v;
}

}  // namespace mdpvi
