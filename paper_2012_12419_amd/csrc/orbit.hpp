// orbit.hpp -- value iteration on the orbits of the host permutations.
//
// All hosts share one capacity and one set of rates, so permuting the hosts
// maps the chain onto itself: an iterate that is invariant under host
// permutations (V^0 = 0, any constant, any earlier solution) stays so, and a
// Jacobi sweep needs one backup per orbit and class instead of one per state.
// The orbits of the (C+1)^K occupancies are the multisets of K digits in
// 0..C, binom(C+K, K) of them (8,008 against 1,771,561 at K = 6, C = 10).
// Every sum of a backup is exact or independent of the host order
// (stay_sum), so the orbit iterates are the full sweeps' bit for bit.
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

#include "device.hpp"

namespace mdpvi {

constexpr uint32_t kOrbitMax = 1u << 20;       // orbits the form covers
constexpr uint32_t kOrbitBinom = 2048;         // entries of the rank table (K (C+1))
constexpr int kOrbitBlock = 128;               // threads of a sweep workgroup
constexpr uint32_t kOrbitGrid = 1024;          // most workgroups of a sweep
constexpr int kOrbitChunk = 32;                // sweeps of a chunk (a multiple of kResSlots)
constexpr int kOrbitLdsBlock = 1024;           // most threads of an LDS-resident solve
constexpr size_t kOrbitLds = 160 * 1024 - 2048;   // its dynamic LDS

// Control words of an orbit solve, in device memory and, as the host's copy,
// in pinned host memory.
struct OrbitCtl {
  long long done;      // -1 while running, else the index of the final iterate
  double residual;     // its residual (the host's copy only)
  long long flag;      // 1: the starting iterate is not invariant
  long long base;      // sweeps done before the chunk that runs (device copy)
  double tol;          // the stopping tolerance (device copy)
  long long pad[11];
};

struct OrbitShape {
  int32_t K, C, J, R;
  int32_t L;              // value slots (and lanes) per orbit: J rounded up to 1, 2, 4 or 8
  int32_t dig_bits;       // bits per digit in dig: 8, or 4 beyond 8 hosts
  int32_t wide;           // 1: table entries of 32 bits, 0: of 16
  uint32_t n;             // orbits
  uint64_t n_occ;
  const uint32_t* binom;  // [K][C+1]: binom(v + i, i + 1)
  const uint64_t* dig;    // [n]: the ascending digits, packed
  const uint32_t* rep;    // [n]: the occupancy index of the representative
  const void* tab;        // [(2 + J) K][n]
};

// The parameters an orbit backup needs (a by-value kernel argument).
struct OrbitParams {
  double p[kMaxJ], r_place[kMaxJ], r_reject[kMaxJ];
  double mu_L, nu_L, hold, gamma;
};

__device__ __forceinline__ double pick(const double (&x)[kMaxJ], int e, int L) {
  double v = x[0];
#pragma unroll
  for (int i = 1; i < kMaxJ; ++i)
    if (i < L) v = e == i ? x[i] : v;
  return v;
}

// Rank of the digits of occupancy o (KX hosts; KX = 16: any K up to 16, the
// digits beyond K read as zero and sorted to the front).  B: the rank table
// in LDS.
template <int KX>
__device__ __forceinline__ uint32_t orbit_rank(int K, int R, FastDiv divR, const uint32_t* B, uint32_t o) {
  int n[KX];
#pragma unroll
  for (int k = 0; k < KX; ++k) {
    if (KX <= 8 || k < K) {
      const uint32_t q = fast_div(o, divR);
      n[k] = static_cast<int>(o - q * static_cast<uint32_t>(R));
      o = q;
    } else {
      n[k] = 0;
    }
  }
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
    const int pos = KX <= 8 ? k : k - (KX - K);   // padding digits are zero and add nothing
    if (KX <= 8 || pos >= 0) r += B[pos * R + n[k]];
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
struct F32View {
  BufView v;
  __device__ __forceinline__ float operator()(uint32_t i) const { return ld_f32(v, i * 4u, 0); }
};
struct F64View {
  BufView v;
  __device__ __forceinline__ double operator()(uint32_t i) const { return ld_f64(v, i * 8u, 0); }
};
template <typename T>
struct LdsView {
  const T* p;
  __device__ __forceinline__ T operator()(uint32_t i) const { return p[i]; }
};

// One lane's part of an orbit backup: class e of orbit r.  KX = K hosts, or
// 16 for any K of 9..16 (the positions beyond K read the orbit itself with
// weight 0 and the -inf entry).
template <int KX>
struct OrbitIdx {
  uint32_t rel[KX], rst[KX], plc[KX];
};

template <int KX, class Tab>
__device__ __forceinline__ void orbit_load_idx(const OrbitShape& S, Tab tab, uint32_t r, int e, OrbitIdx<KX>& x) {
  const int K = KX <= 8 ? KX : S.K;
  const uint32_t rp = static_cast<uint32_t>(e * K) * S.n + r;
#pragma unroll
  for (int k = 0; k < KX; ++k) x.rel[k] = k < K ? tab(r, static_cast<uint32_t>(k) * S.n) : r;
#pragma unroll
  for (int k = 0; k < KX; ++k) x.plc[k] = k < K ? tab(rp, static_cast<uint32_t>(2 * K + k) * S.n) : S.n;
#pragma unroll
  for (int k = 0; k < KX; ++k) x.rst[k] = k < K ? tab(r, static_cast<uint32_t>(K + k) * S.n) : r;
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

// The new value of (r, e): the arithmetic of backup_arrival (sweep_impl.hpp).
template <int KX, int L, class VV, class AV>
__device__ __forceinline__ float orbit_backup(const OrbitShape& S, const OrbitIdx<KX>& x, uint64_t dig, VV V, AV A,
                                              uint32_t r, uint32_t e, double r_place, double r_reject,
                                              const OrbitParams& P, float& own) {
  const int K = KX <= 8 ? KX : S.K;
  own = V(r * L + e);
  const double a_rej = A(r);
  float vd[KX], vr[KX];
  double aa[KX];
#pragma unroll
  for (int k = 0; k < KX; ++k) vd[k] = V(x.rel[k] * L + e);
#pragma unroll
  for (int k = 0; k < KX; ++k) aa[k] = A(x.plc[k]);
#pragma unroll
  for (int k = 0; k < KX; ++k) vr[k] = V(x.rst[k] * L + e);
  int load = 0;
#pragma unroll
  for (int k = 0; k < KX; ++k) load += orbit_digit<KX>(dig, k);
  const double fu = static_cast<double>(S.K * S.C - load);   // free units
  double sum = fu * static_cast<double>(own), rs = 0.0, ab = aa[0];
#pragma unroll
  for (int k = 0; k < KX; ++k)
    sum = fma(static_cast<double>(orbit_digit<KX>(dig, k)), static_cast<double>(vd[k]), sum);
#pragma unroll
  for (int k = 1; k < KX; ++k) ab = orbit_max(ab, aa[k]);
#pragma unroll
  for (int k = 0; k < KX; ++k) rs += k < K ? static_cast<double>(vr[k]) : 0.0;
  const double D = fma(P.nu_L, rs, P.mu_L * sum);   // stay_sum
  const double best = orbit_max(fma(P.gamma, a_rej, fma(-P.hold, fu, r_reject)),
                                fma(P.gamma, ab, fma(-P.hold, fu, r_place)));
  return static_cast<float>(fma(P.gamma, D, best));
}

// v of lane `e` of the group of L neighbouring lanes.
template <int L, int E>
__device__ __forceinline__ float group_lane(float v) {
  if constexpr (L == 1) return v;
  const int b = __float_as_int(v);
  if constexpr (L == 2)
    return __int_as_float(__builtin_amdgcn_mov_dpp(b, E == 0 ? 0xA0 : 0xF5, 0xf, 0xf, true));   // quad_perm
  else if constexpr (L == 4)
    return __int_as_float(__builtin_amdgcn_mov_dpp(b, 0x55 * E, 0xf, 0xf, true));
  else
    return __shfl(v, (static_cast<int>(threadIdx.x) % kWave & ~(L - 1)) + E, kWave);
}

template <int L, int E>
__device__ __forceinline__ double arrival_chain(float vn, int J, const OrbitParams& P, double a) {
  const float v = group_lane<L, E>(vn);
  if (E < J) a = fma(P.p[E], static_cast<double>(v), a);
  if constexpr (E + 1 < L) return arrival_chain<L, E + 1>(vn, J, P, a);
  return a;
}

// The arrival term of an orbit from the new values of its lanes: the FMA
// chain of backup_arrival.
template <int L>
__device__ __forceinline__ double orbit_arrival(float vn, int J, const OrbitParams& P) {
  return arrival_chain<L, 0>(vn, J, P, 0.0);
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
