// orbit_impl.hpp -- the workgroup bodies of the orbit form, shared by the
// single-instance kernels (orbit.hip) and the batched ones (orbit_batch.hip).
#pragma once

#include "orbit.hpp"

namespace mdpvi {

// The rank table into LDS (all threads of the workgroup).
__device__ __forceinline__ void orbit_stage_binom(const OrbitShape& S, uint32_t* B) {
  for (int i = threadIdx.x; i < S.K * S.R; i += blockDim.x) B[i] = S.binom[i];
  __syncthreads();
}

// Orbit r unranked, and the ranks of the orbits its backup reads, into the
// table (KX: any K up to it).
template <int KX, typename Idx>
__device__ __forceinline__ void orbit_table(const OrbitShape& S, const OrbitParams& P, const uint32_t* B, uint32_t r,
                                            uint64_t* __restrict__ dig, uint32_t* __restrict__ rep,
                                            Idx* __restrict__ tab) {
  const int K = S.K, R = S.R;
  int n[KX];
  uint32_t left = r;
  int v = S.C;
  uint64_t packed = 0;
  uint32_t o = 0;
#pragma unroll
  for (int i = KX - 1; i >= 0; --i) {
    n[i] = 0;
    if (i < K) {
      while (B[i * R + v] > left) --v;   // B[i R] = 0: ends at v = 0
      left -= B[i * R + v];
      n[i] = v;
      packed |= static_cast<uint64_t>(v) << (S.dig_bits * i);
      o = o * static_cast<uint32_t>(R) + static_cast<uint32_t>(v);
    }
  }
  dig[r] = packed;
  rep[r] = o;
#pragma unroll
  for (int k = 0; k < KX; ++k) {
    if (k < K) {
      // one unit less: the first position of the run of equal digits moves
      int p = k;
#pragma unroll
      for (int i = KX - 1; i >= 0; --i)
        if (i < k && n[i] == n[k]) p = i;
      const uint32_t rel = n[k] > 0 ? r - B[p * R + n[k]] + B[p * R + n[k] - 1] : r;
      tab[static_cast<size_t>(k) * S.n + r] = static_cast<Idx>(rel);
      // emptied: the positions below k move up by one
      uint32_t q = 0;
#pragma unroll
      for (int i = 0; i < KX; ++i) {
        if (i < K && i < k) q += B[(i + 1) * R + n[i]];
        if (i < K && i > k) q += B[i * R + n[i]];
      }
      tab[static_cast<size_t>(K + k) * S.n + r] = static_cast<Idx>(q);
      // a class-e task placed: the positions above k with a smaller digit
      // than the new one move down
      for (int e = 0; e < S.J; ++e) {
        const int w = n[k] + P.size[e];
        uint32_t t = S.n;
        if (w <= S.C) {
          t = 0;
          int at = k;
#pragma unroll
          for (int i = 0; i < KX; ++i) {
            if (i < K && i != k) {
              if (i > k && n[i] < w) {
                t += B[(i - 1) * R + n[i]];
                at = i;
              } else {
                t += B[i * R + n[i]];
              }
            }
          }
          t += B[at * R + w];
        }
        tab[static_cast<size_t>((2 + e) * K + k) * S.n + r] = static_cast<Idx>(t);
      }
    }
  }
}

// Orbit r's start: its representative's values and their arrival term; for
// an evaluation also the orbit its policy's arrival leads to.  (An infeasible
// action, which the check reports, reads as the paid cloud here.)
template <class Op>
__device__ __forceinline__ void orbit_begin(const OrbitShape& S, const OrbitParams& P, const OrbitWork& W,
                                            const typename Op::T* __restrict__ V, const uint8_t* __restrict__ pi,
                                            uint32_t r) {
  using T = typename Op::T;
  T* Vr = static_cast<T*>(W.V[0]);
  const uint32_t o = S.rep[r];
  double a = 0.0;
  for (int e = 0; e < S.L; ++e) {
    const uint32_t at = r * static_cast<uint32_t>(S.L) + e;
    const uint64_t s = o + static_cast<uint64_t>(e) * S.n_occ;
    const T v = e < S.J ? V[s] : T(0);
    Vr[at] = v;
    if (e < S.J) a = fma(P.p[e], static_cast<double>(v), a);
    if constexpr (Op::kEval) {
      uint32_t act = r;
      const int x = e < S.J ? pi[s] : S.K;
      if (x < S.K) {
        const size_t w = static_cast<size_t>((2 + e) * S.K + x) * S.n + r;
        const uint32_t t = S.wide ? static_cast<const uint32_t*>(S.tab)[w] : static_cast<const uint16_t*>(S.tab)[w];
        if (t != S.n) act = t | 0x80000000u;
      }
      W.act[at] = act;
    }
  }
  W.A[0][r] = a;
}

// n[x] for a host x, -1 for any other action.
template <int KX>
__device__ __forceinline__ int orbit_load(const OrbitShape& S, const int (&n)[KX], int x) {
  int load = -1;
#pragma unroll
  for (int k = 0; k < KX; ++k) load = (KX <= 8 || k < S.K) && k == x ? n[k] : load;
  return load;
}

// The start (value iteration's bit for bit) and an evaluation's target load of
// occupancy o, every class, against those of the occupancy with the first two
// neighbouring digits out of order exchanged: where all agree, each occupancy
// agrees with its orbit's representative, which has none (and mostly the two
// are near each other in memory).  Also the actions' room.  The bits found.
template <class Op, int KX>
__device__ __forceinline__ uint32_t orbit_check(const OrbitShape& S, const OrbitParams& P,
                                                const typename Op::T* __restrict__ V, const uint8_t* __restrict__ pi,
                                                uint32_t o) {
  int n[KX];
  orbit_digits<KX>(S, o, n);
  int at = -1, lo = 0, hi = 0;   // the place, and the digits there and behind it
  uint32_t stride = 1, other = o;
#pragma unroll
  for (int k = 0; k < KX - 1; ++k) {
    if ((KX <= 8 || k < S.K - 1) && at < 0 && n[k] > n[k + 1]) {
      at = k;
      lo = n[k];
      hi = n[k + 1];
      other = o + static_cast<uint32_t>(lo - hi) * stride * static_cast<uint32_t>(S.R - 1);
    }
    stride *= static_cast<uint32_t>(S.R);
  }
  bool differs = false, infeasible = false;
  for (int e = 0; e < S.J; ++e) {
    const uint64_t cls = static_cast<uint64_t>(e) * S.n_occ;
    if constexpr (Op::kEval) {
      const int x = pi[o + cls], load = orbit_load<KX>(S, n, x);
      infeasible = infeasible || x > S.K || (x < S.K && load + P.size[e] > S.C);
      if (at >= 0) {
        const int y = pi[other + cls];
        const int there = y == at ? hi : y == at + 1 ? lo : orbit_load<KX>(S, n, y);
        differs = differs || load != there || V[o + cls] != V[other + cls];
      }
    } else {
      differs = differs || (at >= 0 && __float_as_uint(V[o + cls]) != __float_as_uint(V[other + cls]));
    }
  }
  return (differs || infeasible ? kOrbitDiffers : 0u) | (infeasible ? kOrbitNoRoom : 0u);
}

// The bits of all threads of the workgroup (every thread calls it).
__device__ __forceinline__ uint32_t orbit_found(uint32_t bits) {
  __shared__ uint32_t all;
  if (threadIdx.x == 0) all = 0;
  __syncthreads();
  const uint32_t wave = (__ballot(bits & kOrbitDiffers) ? kOrbitDiffers : 0u) | (__ballot(bits & kOrbitNoRoom) ? kOrbitNoRoom : 0u);
  if (wave && threadIdx.x % kWave == 0) atomicOr(&all, wave);
  __syncthreads();
  return all;
}

// The bits of n workgroups' words.
__device__ __forceinline__ uint32_t orbit_found(const uint32_t* words, uint32_t n) {
  uint32_t bits = 0;
  for (uint32_t i = threadIdx.x; i < n; i += blockDim.x) bits |= words[i];
  return orbit_found(bits);
}

// Every class of occupancy o := its orbit's value.
template <class T, int KX>
__device__ __forceinline__ void orbit_expand(const OrbitShape& S, const uint32_t* B, const T* __restrict__ Vr,
                                             T* __restrict__ V, uint32_t o) {
  int n[KX];
  orbit_digits<KX>(S, o, n);
  const uint32_t r = orbit_rank<KX>(S, B, n);
  for (int e = 0; e < S.J; ++e)
    V[o + static_cast<uint64_t>(e) * S.n_occ] = Vr[r * static_cast<uint32_t>(S.L) + e];
}

// One sweep over the orbits, W.V[0], W.A[0] -> W.V[1], W.A[1], by workgroup
// `block` of `grid`, L lanes per orbit (one per class): the orbits of its lanes and every grid-th such group after
// them.  A sweep of a few thousand orbits is bound by latency (8,008 orbits
// at K = 6, C = 10 are two wavefronts per CU), so its loads form two dependent
// steps only, table rows and then values, and nothing waits for the stop
// test: the tolerance and the previous sweep's residual words are loaded
// first, the backup runs, and only the stores wait for the verdict.  Every
// workgroup leaves its largest |V' - V| in its own word of slot i mod 4; the
// next sweep's workgroups each read all of them (at most kOrbitGrid).  A
// stopped sweep passes the residual on, so that every later one stops too,
// and its first workgroup calls stopped(residual).
template <class Op, int K, int L, typename Idx, class Stopped>
__device__ __forceinline__ void orbit_sweep(const OrbitShape& S, const OrbitParams& P, const OrbitWork& W, int i,
                                            uint32_t block, uint32_t grid, Stopped stopped) {
  using T = typename Op::T;
  __shared__ double part[kOrbitBlock / kWave];
  __shared__ int go[kOrbitBlock / kWave], bad[kOrbitBlock / kWave];
  constexpr uint32_t kWords = kOrbitGrid / kOrbitBlock;
  const BufView prev = make_view(W.res + static_cast<size_t>((i + kResSlots - 1) % kResSlots) * kOrbitGrid,
                                 kOrbitGrid * 8u);
  const double tol = load_agent(&W.ctl->tol);
  double pw[kWords];
#pragma unroll
  for (uint32_t w = 0; w < kWords; ++w)
    pw[w] = w * kOrbitBlock < grid ? ld_f64(prev, threadIdx.x * 8u, w * kOrbitBlock * 8u) : 0.0;
  const int lane = threadIdx.x % kWave;
  const int wid = threadIdx.x / kWave;
  const uint32_t e = threadIdx.x % L;
  const uint32_t ec = e < static_cast<uint32_t>(S.J) ? e : 0;
  const double r_place = pick(P.r_place, ec, L), r_reject = pick(P.r_reject, ec, L);
  const TabView<Idx> tab = tab_view<Idx>(S);
  const GlobalView<T> vin = global_view<T>(W.V[0], S.n * L);
  const GlobalView<double> ain = global_view<double>(W.A[0], S.n + 1);
  const GlobalView<uint64_t> dig = global_view<uint64_t>(S.dig, S.n);
  const GlobalView<uint32_t> act = global_view<uint32_t>(W.act, S.n * L);
  const BufView vout = make_view(W.V[1], S.n * L * static_cast<uint32_t>(sizeof(T)));
  const BufView aout = make_view(W.A[1], S.n * 8u);
  constexpr uint32_t per = kOrbitBlock / L;
  double dmax = 0.0;
  bool nan = false;
  bool tested = false;
  for (uint32_t base = block * per; base < S.n; base += grid * per) {
    const uint32_t r = base + threadIdx.x / L;
    const uint32_t rc = r < S.n ? r : S.n - 1;
    OrbitIdx<Op, K> x;
    orbit_load_idx<Op, K>(S, tab, dig, act, rc, ec, x);
    T own;
    const T vn = orbit_backup<Op, K, L>(S, x, vin, ain, rc, ec, r_place, r_reject, P, own);
    const double anew = orbit_arrival<L>(vn, S.J, P);
    const double d = fabs(static_cast<double>(vn) - static_cast<double>(own));
    nan = nan || d != d;
    dmax = orbit_max(dmax, d);
    if (!tested) {   // the verdict on the sweep before, once per workgroup
      tested = true;
      bool up = false, bd = false;
#pragma unroll
      for (uint32_t w = 0; w < kWords; ++w) {
        up = up || pw[w] >= tol;
        bd = bd || pw[w] != pw[w];
      }
      const bool wu = __ballot(up) != 0, wb = __ballot(bd) != 0;
      if (lane == 0) {
        go[wid] = wu;
        bad[wid] = wb;
      }
      __syncthreads();
      bool any = false, anyb = false;
#pragma unroll
      for (int w = 0; w < kOrbitBlock / kWave; ++w) {
        any = any || go[w];
        anyb = anyb || bad[w];
      }
      if (!any || anyb) {
        // stopped: every word of this slot becomes the last residual
        double pm = pw[0];
#pragma unroll
        for (uint32_t w = 1; w < kWords; ++w) pm = (pw[w] > pm || pw[w] != pw[w]) ? pw[w] : pm;
        pm = wave_max(pm);
        if (lane == 0) part[wid] = pm;
        __syncthreads();
        if (threadIdx.x == 0) {
#pragma unroll
          for (int w = 0; w < kOrbitBlock / kWave; ++w) pm = (part[w] > pm || part[w] != part[w]) ? part[w] : pm;
          W.res[static_cast<size_t>(i % kResSlots) * kOrbitGrid + block] = pm;
          if (block == 0) stopped(pm);
        }
        return;
      }
    }
    if (r < S.n && e < static_cast<uint32_t>(S.J)) {
      if constexpr (sizeof(T) == 4)
        st_f32(vout, vn, (r * L + e) * 4u, 0);
      else
        st_f64(vout, vn, (r * L + e) * 8u, 0);
      if (e == 0) st_f64(aout, anew, r * 8u, 0);
    }
  }
  dmax = wave_max_last(dmax);
  const bool wn = __ballot(nan) != 0;
  if (lane == kWave - 1) part[wid] = wn ? NAN : dmax;
  __syncthreads();
  if (threadIdx.x == 0) {
    double m = part[0];
#pragma unroll
    for (int w = 1; w < kOrbitBlock / kWave; ++w) m = (part[w] > m || part[w] != part[w]) ? part[w] : m;
    W.res[static_cast<size_t>(i % kResSlots) * kOrbitGrid + block] = m;
  }
}

// Up to `most` sweeps by the calling workgroup (at most NB threads) with both
// iterates and both arrays of arrival terms in LDS: one barrier per sweep, no
// launch.  Lane t owns the classes of orbits t / L, t / L + threads / L, ..;
// with HOIST > 0 the table rows of its (at most HOIST) orbits stay in
// registers, else they are read from the caches every sweep.  it0: sweeps
// done before.  Thread 0 calls ended(sweeps, residual, stopped).
template <class Op, int K, int L, int HOIST, int NB, class Ended>
__device__ __forceinline__ void orbit_lds(const OrbitShape& S, const OrbitParams& P, const OrbitWork& W0,
                                          long long it0, long long most, double tol, double* lds, Ended ended) {
  using T = typename Op::T;
  const OrbitWork W = orbit_work(W0, it0);
  __shared__ int up[3], bad[3];
  __shared__ double part[NB / kWave];
  const TabView<uint16_t> tab = tab_view<uint16_t>(S);
  const GlobalView<uint64_t> dig = global_view<uint64_t>(S.dig, S.n);
  const GlobalView<uint32_t> act = global_view<uint32_t>(W.act, S.n * L);
  const uint32_t n = S.n, na = n + 1;
  double* Aa = lds;
  double* Ab = Aa + na;
  T* Va = reinterpret_cast<T*>(Ab + na);
  T* Vb = Va + n * L;
  const T* Vg = static_cast<const T*>(W.V[0]);
  const double* Ag = W.A[0];
  for (uint32_t i = threadIdx.x; i < n * L; i += blockDim.x) {
    Va[i] = Vg[i];
    Vb[i] = T(0);
  }
  for (uint32_t i = threadIdx.x; i < na; i += blockDim.x) {
    Aa[i] = Ag[i];
    Ab[i] = -INFINITY;   // entry n stays -inf
  }
  if (threadIdx.x < 3) {
    up[threadIdx.x] = 0;
    bad[threadIdx.x] = 0;
  }
  const int lane = threadIdx.x % kWave;
  const uint32_t e = threadIdx.x % L;
  const uint32_t ec = e < static_cast<uint32_t>(S.J) ? e : 0;
  const double r_place = pick(P.r_place, ec, L), r_reject = pick(P.r_reject, ec, L);
  const uint32_t per = blockDim.x / L;
  const uint32_t first = threadIdx.x / L;
  constexpr int H = HOIST > 0 ? HOIST : 1;
  OrbitIdx<Op, K> hx[H];
  if constexpr (HOIST > 0) {
#pragma unroll
    for (int h = 0; h < HOIST; ++h) {
      const uint32_t r = first + h * per;
      orbit_load_idx<Op, K>(S, tab, dig, act, r < n ? r : n - 1, ec, hx[h]);
    }
  }
  __syncthreads();
  double dmax = 0.0;
  long long it = 0;
  bool stop = false;
  int slot = 0;
  while (it < most) {
    dmax = 0.0;
    bool nan = false;
    auto one = [&](uint32_t r, const OrbitIdx<Op, K>& x) {
      T own;
      const T vn = orbit_backup<Op, K, L>(S, x, LdsView<T>{Va}, LdsView<double>{Aa}, r < n ? r : n - 1, ec, r_place,
                                          r_reject, P, own);
      const double anew = orbit_arrival<L>(vn, S.J, P);
      const double d = fabs(static_cast<double>(vn) - static_cast<double>(own));
      dmax = orbit_max(dmax, d);
      nan = nan || d != d;
      if (r < n && e < static_cast<uint32_t>(S.J)) {
        Vb[r * L + e] = vn;
        if (e == 0) Ab[r] = anew;
      }
    };
    if constexpr (HOIST > 0) {
#pragma unroll
      for (int h = 0; h < HOIST; ++h) one(first + h * per, hx[h]);
    } else {
      for (uint32_t base = 0; base < n; base += per) {
        const uint32_t r = base + first;
        OrbitIdx<Op, K> x;
        orbit_load_idx<Op, K>(S, tab, dig, act, r < n ? r : n - 1, ec, x);
        one(r, x);
      }
    }
    if (nan) dmax = NAN;
    if (__ballot(!(dmax < tol)) != 0 && lane == 0) up[slot] = 1;
    if (__ballot(nan) != 0 && lane == 0) bad[slot] = 1;
    __syncthreads();
    const bool more = up[slot] != 0 && bad[slot] == 0;
    ++it;
    double* ta = Aa;
    Aa = Ab;
    Ab = ta;
    T* tv = Va;
    Va = Vb;
    Vb = tv;
    // the words of the sweep before this one, which every wavefront has read,
    // are cleared for the sweep after the next
    const int old = slot == 0 ? 2 : slot - 1;
    if (threadIdx.x == 0) {
      up[old] = 0;
      bad[old] = 0;
    }
    slot = slot == 2 ? 0 : slot + 1;
    if (!more) {
      stop = true;
      break;
    }
  }
  dmax = wave_max(dmax);
  if (lane == 0) part[threadIdx.x / kWave] = dmax;
  T* Vo = static_cast<T*>((it & 1) ? W.V[1] : W.V[0]);
  double* Ao = (it & 1) ? W.A[1] : W.A[0];
  for (uint32_t i = threadIdx.x; i < n * L; i += blockDim.x) Vo[i] = Va[i];
  for (uint32_t i = threadIdx.x; i < n; i += blockDim.x) Ao[i] = Aa[i];
  __syncthreads();
  if (threadIdx.x == 0) {
    double m = part[0];
    for (uint32_t w = 1; w < blockDim.x / kWave; ++w) m = (part[w] > m || part[w] != part[w]) ? part[w] : m;
    ended(it0 + it, m, stop);
  }
}

}  // namespace mdpvi
