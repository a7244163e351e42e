// orbit.hip -- kernels of the orbit form of value iteration (orbit.hpp): the
// rank table, the check that a starting iterate is invariant under host
// permutations, sweeps over the orbits (one launch each, or all of them in
// one workgroup's LDS) and the expansion to the full state space.
//
// Measured against the full sweeps of the same solve (to ||dV|| < 1e-6, wall
// time): K = 6, C = 10, J = 3 47.5 -> 5.7 ms (31 -> 3.6 us per sweep); K = 7
// 565 -> 7.2 ms (408 -> 4.5 us); K = 4, C = 12, J = 3 2.7 -> 1.7 ms; in LDS
// K = 3, C = 8, J = 2 1.80 -> 0.17 ms (0.63 us per sweep).
#include "kernels.hpp"
#include "orbit.hpp"

namespace mdpvi {

// ------------------------------------------------------------------ table

// One thread per orbit: unranks it and ranks the orbits its backup reads.
template <int KX, typename Idx>
__global__ __launch_bounds__(256) void orbit_table_kernel(OrbitShape S, const Model M, uint64_t* __restrict__ dig,
                                                          uint32_t* __restrict__ rep, Idx* __restrict__ tab) {
  __shared__ uint32_t B[kOrbitBinom];
  for (int i = threadIdx.x; i < S.K * S.R; i += blockDim.x) B[i] = S.binom[i];
  __syncthreads();
  const uint32_t r = blockIdx.x * blockDim.x + threadIdx.x;
  if (r >= S.n) return;
  const int K = S.K, R = S.R;
  int n[KX];
  uint32_t left = r;
  int v = S.C;
  uint64_t packed = 0;
  uint64_t o = 0;
#pragma unroll
  for (int i = KX - 1; i >= 0; --i) {
    n[i] = 0;
    if (i < K) {
      while (B[i * R + v] > left) --v;   // B[i R] = 0: ends at v = 0
      left -= B[i * R + v];
      n[i] = v;
      packed |= static_cast<uint64_t>(v) << (S.dig_bits * i);
      o += static_cast<uint64_t>(v) * static_cast<uint64_t>(M.stride[i]);
    }
  }
  dig[r] = packed;
  rep[r] = static_cast<uint32_t>(o);
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
        const int w = n[k] + M.size[e];
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

// ------------------------------------------------------------ start and end

// The orbits' values and arrival terms from the representatives of V, the
// -inf entries and the control words.
__global__ __launch_bounds__(256) void orbit_begin_kernel(OrbitShape S, OrbitParams P, const float* __restrict__ V,
                                                          float* __restrict__ Vr, double* __restrict__ A0,
                                                          double* __restrict__ A1, OrbitCtl* ctl, double* res,
                                                          double tol) {
  const uint32_t r = blockIdx.x * blockDim.x + threadIdx.x;
  // the slot before the first sweep's holds one word that passes no test
  if (blockIdx.x == 0)
    for (uint32_t w = threadIdx.x; w < kResSlots * kOrbitGrid; w += blockDim.x)
      res[w] = w == (kResSlots - 1) * kOrbitGrid ? INFINITY : 0.0;
  if (r == 0) {
    ctl->done = -1;
    ctl->flag = 0;
    ctl->base = 0;
    ctl->tol = tol;
    A0[S.n] = -INFINITY;
    A1[S.n] = -INFINITY;
  }
  if (r >= S.n) return;
  const uint32_t o = S.rep[r];
  double a = 0.0;
  for (int e = 0; e < S.L; ++e) {
    const float v = e < S.J ? V[o + static_cast<uint64_t>(e) * S.n_occ] : 0.0f;
    Vr[r * static_cast<uint32_t>(S.L) + e] = v;
    if (e < S.J) a = fma(P.p[e], static_cast<double>(v), a);
  }
  A0[r] = a;
}

// Compares every state with its orbit's representative, bit for bit; raises
// ctl->flag where one differs.
template <int KX>
__global__ __launch_bounds__(256) void orbit_check_kernel(OrbitShape S, FastDiv divR, const float* __restrict__ V,
                                                          const float* __restrict__ Vr, OrbitCtl* ctl,
                                                          OrbitCtl* mirror) {
  __shared__ uint32_t B[kOrbitBinom];
  for (int i = threadIdx.x; i < S.K * S.R; i += blockDim.x) B[i] = S.binom[i];
  __syncthreads();
  bool bad = false;
  const uint64_t step = static_cast<uint64_t>(gridDim.x) * blockDim.x;
  for (uint64_t o = static_cast<uint64_t>(blockIdx.x) * blockDim.x + threadIdx.x; o < S.n_occ; o += step) {
    const uint32_t r = orbit_rank<KX>(S.K, S.R, divR, B, static_cast<uint32_t>(o));
    for (int e = 0; e < S.J; ++e)
      bad = bad || __float_as_uint(V[o + static_cast<uint64_t>(e) * S.n_occ]) !=
                       __float_as_uint(Vr[r * static_cast<uint32_t>(S.L) + e]);
  }
  if (__ballot(bad) != 0 && threadIdx.x % kWave == 0) {
    volatile long long* f = &ctl->flag;
    if (*f == 0) {
      *f = 1;
      ctl->tol = NAN;   // no residual is >= NaN: every sweep stops
      mirror->flag = 1;
    }
  }
}

// V := the final iterate (ctl->done, or `issued` sweeps when none stopped the
// loop) at every state; nothing when the form was refused.  Workgroup 0
// records the index and the residual.
template <int KX>
__global__ __launch_bounds__(256) void orbit_expand_kernel(OrbitShape S, FastDiv divR, float* __restrict__ V,
                                                           const float* __restrict__ V0,
                                                           const float* __restrict__ V1, const OrbitCtl* ctl,
                                                           long long issued) {
  if (ctl->flag) return;
  const long long done = ctl->done;
  const float* __restrict__ Vr = ((done >= 0 ? done : issued) & 1) ? V1 : V0;
  __shared__ uint32_t B[kOrbitBinom];
  for (int i = threadIdx.x; i < S.K * S.R; i += blockDim.x) B[i] = S.binom[i];
  __syncthreads();
  const uint64_t step = static_cast<uint64_t>(gridDim.x) * blockDim.x;
  for (uint64_t o = static_cast<uint64_t>(blockIdx.x) * blockDim.x + threadIdx.x; o < S.n_occ; o += step) {
    const uint32_t r = orbit_rank<KX>(S.K, S.R, divR, B, static_cast<uint32_t>(o));
    for (int e = 0; e < S.J; ++e)
      V[o + static_cast<uint64_t>(e) * S.n_occ] = Vr[r * static_cast<uint32_t>(S.L) + e];
  }
}

// ----------------------------------------------------------------- sweeps

// One sweep over the orbits, L lanes per orbit (one per class), each
// workgroup the orbits of its lanes and every grid-th such group after them.
// A sweep of a few thousand orbits is bound by latency (8,008 orbits at
// K = 6, C = 10 are two wavefronts per CU), so its loads form two dependent
// steps only, table rows and then values, and nothing waits for the stop
// test: the tolerance and the previous sweep's residual words are loaded
// first, the backup runs, and only the stores wait for the verdict.  Every
// workgroup leaves its largest |V' - V| in its own word of slot i mod 4; the
// next sweep's workgroups each read all of them (at most kOrbitGrid).  A
// stopped sweep passes the residual on, so that every later one stops too.
//
// i: the sweep's place in its chunk, known when the chunk is built; the chunk
// starts after ctl->base sweeps, a multiple of kOrbitChunk, so that i alone
// decides the buffers and the residual slot.  A small kernel after the chunk
// moves base on.  A chunk is a recorded graph: issued one by one, the launches
// are bound by the host (5.3 us each at 360 bytes of arguments); a graph node
// with no work takes 2.0 us, the table rows 0.85, values and backup 0.7, the
// verdict and the residual 0.2.
template <int K, int L, typename Idx>
__global__ __launch_bounds__(kOrbitBlock) void orbit_sweep_kernel(OrbitShape S, OrbitParams P, const float* Vin,
                                                                  float* Vout, const double* Ain, double* Aout,
                                                                  OrbitCtl* ctl, OrbitCtl* mirror, double* res,
                                                                  uint32_t grid, int i) {
  __shared__ double part[kOrbitBlock / kWave];
  __shared__ int go[kOrbitBlock / kWave], bad[kOrbitBlock / kWave];
  constexpr uint32_t kWords = kOrbitGrid / kOrbitBlock;
  const BufView prev = make_view(res + static_cast<size_t>((i + kResSlots - 1) % kResSlots) * kOrbitGrid,
                                 kOrbitGrid * 8u);
  const double tol = load_agent(&ctl->tol);
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
  const F32View vin{make_view(Vin, S.n * L * 4u)};
  const F64View ain{make_view(Ain, (S.n + 1) * 8u)};
  const BufView dig{make_view(S.dig, S.n * 8u)};
  const BufView vout = make_view(Vout, S.n * L * 4u), aout = make_view(Aout, S.n * 8u);
  constexpr uint32_t per = kOrbitBlock / L;
  double dmax = 0.0;
  bool nan = false;
  bool tested = false;
  for (uint32_t base = blockIdx.x * per; base < S.n; base += grid * per) {
    const uint32_t r = base + threadIdx.x / L;
    const uint32_t rc = r < S.n ? r : S.n - 1;
    OrbitIdx<K> x;
    orbit_load_idx<K>(S, tab, rc, ec, x);
    const uint64_t dg = __builtin_bit_cast(uint64_t, ld_f64(dig, rc * 8u, 0));
    float own;
    const float vn = orbit_backup<K, L>(S, x, dg, vin, ain, rc, ec, r_place, r_reject, P, own);
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
          res[static_cast<size_t>(i % kResSlots) * kOrbitGrid + blockIdx.x] = pm;
          if (blockIdx.x == 0 && ctl->flag == 0 && ctl->done < 0) {
            ctl->done = ctl->base + i;
            mirror->residual = pm;
            mirror->done = ctl->base + i;
          }
        }
        return;
      }
    }
    if (r < S.n && e < static_cast<uint32_t>(S.J)) {
      st_f32(vout, vn, (r * L + e) * 4u, 0);
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
    res[static_cast<size_t>(i % kResSlots) * kOrbitGrid + blockIdx.x] = m;
  }
}

// The residual of the last of `issued` sweeps when none stopped the loop.
__global__ __launch_bounds__(256) void orbit_last_residual_kernel(const double* res, uint32_t grid, long long issued,
                                                                  const OrbitCtl* ctl, OrbitCtl* mirror) {
  __shared__ double part[256 / kWave];
  const double* w = res + static_cast<size_t>((issued - 1) % kResSlots) * kOrbitGrid;
  double m = 0.0;
  for (uint32_t b = threadIdx.x; b < grid; b += 256) {
    const double v = w[b];
    m = (v > m || v != v) ? v : m;
  }
  m = wave_max(m);
  if (threadIdx.x % kWave == 0) part[threadIdx.x / kWave] = m;
  __syncthreads();
  if (threadIdx.x == 0 && ctl->done < 0) {
    for (int i = 1; i < 256 / kWave; ++i) m = (part[i] > m || part[i] != part[i]) ? part[i] : m;
    mirror->residual = m;
  }
}

// ------------------------------------------------------------- LDS solve

// Up to `most` sweeps by one workgroup with both iterates and both arrays of
// arrival terms in LDS: one barrier per sweep, no launch.  Lane t owns the
// classes of orbits t / L, t / L + threads / L, ..; with HOIST the table
// rows of its (at most HOIST) orbits stay in registers, else they are read
// from the caches every sweep.  it0: sweeps done before this launch.
template <int K, int L, int HOIST>
__global__ __launch_bounds__(kOrbitLdsBlock) void orbit_lds_kernel(OrbitShape S, OrbitParams P, float* __restrict__ V0,
                                                                   float* __restrict__ V1, double* __restrict__ A0,
                                                                   double* __restrict__ A1, OrbitCtl* ctl,
                                                                   OrbitCtl* mirror, long long it0, long long most, double tol) {
  if (ctl->flag || ctl->done >= 0) return;
  extern __shared__ double orbit_lds[];
  __shared__ int up[3], bad[3];
  __shared__ double part[kOrbitLdsBlock / kWave];
  const TabView<uint16_t> tab = tab_view<uint16_t>(S);
  const uint32_t n = S.n, na = n + 1;
  double* Aa = orbit_lds;
  double* Ab = Aa + na;
  float* Va = reinterpret_cast<float*>(Ab + na);
  float* Vb = Va + n * L;
  const float* Vg = (it0 & 1) ? V1 : V0;
  const double* Ag = (it0 & 1) ? A1 : A0;
  for (uint32_t i = threadIdx.x; i < n * L; i += blockDim.x) {
    Va[i] = Vg[i];
    Vb[i] = 0.0f;
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
  OrbitIdx<K> hx[H];
  uint64_t hd[H];
  if constexpr (HOIST > 0) {
#pragma unroll
    for (int h = 0; h < HOIST; ++h) {
      const uint32_t r = first + h * per;
      const uint32_t rc = r < n ? r : n - 1;
      orbit_load_idx<K>(S, tab, rc, ec, hx[h]);
      hd[h] = S.dig[rc];
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
    auto one = [&](uint32_t r, uint32_t rc, const OrbitIdx<K>& x, uint64_t dig) {
      float own;
      const float vn = orbit_backup<K, L>(S, x, dig, LdsView<float>{Va}, LdsView<double>{Aa}, rc, ec, r_place, r_reject, P, own);
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
      for (int h = 0; h < HOIST; ++h) {
        const uint32_t r = first + h * per;
        one(r, r < n ? r : n - 1, hx[h], hd[h]);
      }
    } else {
      for (uint32_t base = 0; base < n; base += per) {
        const uint32_t r = base + first;
        const uint32_t rc = r < n ? r : n - 1;
        OrbitIdx<K> x;
        orbit_load_idx<K>(S, tab, rc, ec, x);
        one(r, rc, x, S.dig[rc]);
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
    float* tv = Va;
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
  float* Vo = ((it0 + it) & 1) ? V1 : V0;
  double* Ao = ((it0 + it) & 1) ? A1 : A0;
  for (uint32_t i = threadIdx.x; i < n * L; i += blockDim.x) Vo[i] = Va[i];
  for (uint32_t i = threadIdx.x; i < n; i += blockDim.x) Ao[i] = Aa[i];
  __syncthreads();
  if (threadIdx.x == 0) {
    double m = part[0];
    for (uint32_t w = 1; w < blockDim.x / kWave; ++w) m = (part[w] > m || part[w] != part[w]) ? part[w] : m;
    mirror->residual = m;
    if (stop) {
      ctl->done = it0 + it;
      mirror->done = it0 + it;
    }
  }
}

// --------------------------------------------------------------- launchers

#define MDPVI_ORBIT_K(K_, CALL) \
  switch (K_) {                 \
    case 1: CALL(1); break;     \
    case 2: CALL(2); break;     \
    case 3: CALL(3); break;     \
    case 4: CALL(4); break;     \
    case 5: CALL(5); break;     \
    case 6: CALL(6); break;     \
    case 7: CALL(7); break;     \
    case 8: CALL(8); break;     \
    default: CALL(16);          \
  }

hipError_t launch_orbit_table(const OrbitShape& S, const Model& M, uint64_t* dig, uint32_t* rep, void* tab,
                              hipStream_t s) {
  const uint32_t grid = (S.n + 255) / 256;
#define MDPVI_CALL(KX_, T_)                                                                              \
  hipLaunchKernelGGL((orbit_table_kernel<KX_, T_>), dim3(grid), dim3(256), 0, s, S, M, dig, rep, \
                     static_cast<T_*>(tab))
  if (S.wide) {
    if (S.K <= 4) MDPVI_CALL(4, uint32_t);
    else if (S.K <= 8) MDPVI_CALL(8, uint32_t);
    else MDPVI_CALL(16, uint32_t);
  } else {
    if (S.K <= 4) MDPVI_CALL(4, uint16_t);
    else if (S.K <= 8) MDPVI_CALL(8, uint16_t);
    else MDPVI_CALL(16, uint16_t);
  }
#undef MDPVI_CALL
  return hipGetLastError();
}

// Workgroups of a pass over the full state space: enough to fill the chip a
// few times over, several occupancies per thread beyond that (each workgroup
// reads the rank table once).
static uint32_t full_grid(const OrbitShape& S) {
  const uint64_t g = (S.n_occ + 255) / 256;
  return static_cast<uint32_t>(g < 8192 ? g : 8192);
}

hipError_t launch_orbit_begin(const OrbitShape& S, const OrbitParams& P, const Model& M, const float* V, float* Vr,
                              double* A0, double* A1, OrbitCtl* ctl, OrbitCtl* mirror, double* res, double tol,
                              hipStream_t s) {
  hipLaunchKernelGGL(orbit_begin_kernel, dim3((S.n + 255) / 256), dim3(256), 0, s, S, P, V, Vr, A0, A1, ctl, res,
                     tol);
#define MDPVI_CALL(KX_)                                                                                            \
  hipLaunchKernelGGL((orbit_check_kernel<KX_>), dim3(full_grid(S)), dim3(256), 0, s, S, M.divR, V, \
                     static_cast<const float*>(Vr), ctl, mirror)
  MDPVI_ORBIT_K(S.K, MDPVI_CALL)
#undef MDPVI_CALL
  return hipGetLastError();
}

hipError_t launch_orbit_expand(const OrbitShape& S, const Model& M, float* V, const float* V0, const float* V1,
                               const OrbitCtl* ctl, long long issued, hipStream_t s) {
#define MDPVI_CALL(KX_) \
  hipLaunchKernelGGL((orbit_expand_kernel<KX_>), dim3(full_grid(S)), dim3(256), 0, s, S, M.divR, V, V0, V1, ctl, issued)
  MDPVI_ORBIT_K(S.K, MDPVI_CALL)
#undef MDPVI_CALL
  return hipGetLastError();
}

uint32_t orbit_grid(const OrbitShape& S) {
  const uint64_t lanes = static_cast<uint64_t>(S.n) * S.L;
  const uint64_t g = (lanes + kOrbitBlock - 1) / kOrbitBlock;
  return static_cast<uint32_t>(g < kOrbitGrid ? g : kOrbitGrid);
}

template <int K, typename Idx>
static const void* sweep_l(int L) {
  switch (L) {
    case 1: return reinterpret_cast<const void*>(&orbit_sweep_kernel<K, 1, Idx>);
    case 2: return reinterpret_cast<const void*>(&orbit_sweep_kernel<K, 2, Idx>);
    case 4: return reinterpret_cast<const void*>(&orbit_sweep_kernel<K, 4, Idx>);
    default: return reinterpret_cast<const void*>(&orbit_sweep_kernel<K, 8, Idx>);
  }
}

static const void* sweep_fn(const OrbitShape& S) {
  const void* f = nullptr;
#define MDPVI_CALL(K_) f = S.wide ? sweep_l<K_, uint32_t>(S.L) : sweep_l<K_, uint16_t>(S.L)
  MDPVI_ORBIT_K(S.K, MDPVI_CALL)
#undef MDPVI_CALL
  return f;
}

hipError_t launch_orbit_sweep(const OrbitShape& S, const OrbitParams& P, float* const V[2], double* const A[2],
                              OrbitCtl* ctl, OrbitCtl* mirror, double* res, int i, hipStream_t s) {
  OrbitShape sh = S;
  OrbitParams pr = P;
  const float* vin = V[i & 1];
  float* vout = V[(i + 1) & 1];
  const double* ain = A[i & 1];
  double* aout = A[(i + 1) & 1];
  uint32_t grid = orbit_grid(S);
  void* args[] = {&sh, &pr, &vin, &vout, &ain, &aout, &ctl, &mirror, &res, &grid, &i};
  return hipLaunchKernel(sweep_fn(S), dim3(grid), dim3(kOrbitBlock), args, 0, s);
}

// Moves the chunk's base on by n sweeps (after the sweeps of the chunk).
__global__ void orbit_next_kernel(OrbitCtl* ctl, int n) { ctl->base += n; }

hipError_t launch_orbit_next(OrbitCtl* ctl, int n, hipStream_t s) {
  hipLaunchKernelGGL(orbit_next_kernel, dim3(1), dim3(1), 0, s, ctl, n);
  return hipGetLastError();
}

hipError_t build_orbit_chunk(const OrbitShape& S, const OrbitParams& P, float* const V[2], double* const A[2],
                             OrbitCtl* ctl, OrbitCtl* mirror, double* res, hipGraphExec_t* out) {
  *out = nullptr;
  hipGraph_t g = nullptr;
  hipError_t e = hipGraphCreate(&g, 0);
  if (e != hipSuccess) return e;
  OrbitShape sh = S;
  OrbitParams pr = P;
  uint32_t grid = orbit_grid(S);
  hipGraphNode_t node = nullptr;
  for (int i = 0; i <= kOrbitChunk && e == hipSuccess; ++i) {
    const float* vin = V[i & 1];
    float* vout = V[(i + 1) & 1];
    const double* ain = A[i & 1];
    double* aout = A[(i + 1) & 1];
    void* args[] = {&sh, &pr, &vin, &vout, &ain, &aout, &ctl, &mirror, &res, &grid, &i};
    int n = kOrbitChunk;
    void* last[] = {&ctl, &n};
    hipKernelNodeParams p{};
    p.func = const_cast<void*>(i < kOrbitChunk ? sweep_fn(S) : reinterpret_cast<const void*>(&orbit_next_kernel));
    p.gridDim = i < kOrbitChunk ? dim3(grid) : dim3(1);
    p.blockDim = i < kOrbitChunk ? dim3(kOrbitBlock) : dim3(1);
    p.kernelParams = i < kOrbitChunk ? args : last;
    const hipGraphNode_t before = node;
    e = hipGraphAddKernelNode(&node, g, before ? &before : nullptr, before ? 1 : 0, &p);
  }
  if (e == hipSuccess) e = hipGraphInstantiate(out, g, nullptr, nullptr, 0);
  (void)hipGraphDestroy(g);
  return e;
}

hipError_t launch_orbit_last_residual(const OrbitShape& S, const double* res, long long issued, const OrbitCtl* ctl,
                                      OrbitCtl* mirror, hipStream_t s) {
  hipLaunchKernelGGL(orbit_last_residual_kernel, dim3(1), dim3(256), 0, s, res, orbit_grid(S), issued, ctl,
                     mirror);
  return hipGetLastError();
}

size_t orbit_lds_bytes(const OrbitShape& S) {
  return 2 * (static_cast<size_t>(S.n) + 1) * 8 + 2 * static_cast<size_t>(S.n) * S.L * 4;
}

template <int K, int L>
static void lds_h(const OrbitShape& S, const OrbitParams& P, float* V0, float* V1, double* A0, double* A1,
                  OrbitCtl* ctl, OrbitCtl* mirror, long long it0, long long most, double tol, hipStream_t s) {
  const uint32_t lanes = S.n * L;
  const uint32_t threads = lanes < kOrbitLdsBlock ? (lanes + kWave - 1) / kWave * kWave : kOrbitLdsBlock;
  const size_t lds = orbit_lds_bytes(S);
#define MDPVI_CALL(H_)                                                                                             \
  hipLaunchKernelGGL((orbit_lds_kernel<K, L, H_>), dim3(1), dim3(threads), lds, s, S, P, V0, V1, A0, A1, ctl, mirror, \
                     it0, most, tol)
  // the table rows of more orbits, or of more hosts, would not fit the 128
  // registers that 16 wavefronts leave a lane
  if (K <= 8 && lanes <= threads) MDPVI_CALL((K <= 8 ? 1 : 0));
  else if (K <= 6 && lanes <= 2 * threads) MDPVI_CALL((K <= 6 ? 2 : 0));
  else MDPVI_CALL(0);
#undef MDPVI_CALL
}

template <int K>
static void lds_l(const OrbitShape& S, const OrbitParams& P, float* V0, float* V1, double* A0, double* A1,
                  OrbitCtl* ctl, OrbitCtl* mirror, long long it0, long long most, double tol, hipStream_t s) {
  switch (S.L) {
    case 1: lds_h<K, 1>(S, P, V0, V1, A0, A1, ctl, mirror, it0, most, tol, s); break;
    case 2: lds_h<K, 2>(S, P, V0, V1, A0, A1, ctl, mirror, it0, most, tol, s); break;
    case 4: lds_h<K, 4>(S, P, V0, V1, A0, A1, ctl, mirror, it0, most, tol, s); break;
    default: lds_h<K, 8>(S, P, V0, V1, A0, A1, ctl, mirror, it0, most, tol, s);
  }
}

hipError_t launch_orbit_lds(const OrbitShape& S, const OrbitParams& P, float* V0, float* V1, double* A0, double* A1,
                            OrbitCtl* ctl, OrbitCtl* mirror, long long it0, long long most, double tol, hipStream_t s) {
#define MDPVI_CALL(K_) lds_l<K_>(S, P, V0, V1, A0, A1, ctl, mirror, it0, most, tol, s)
  MDPVI_ORBIT_K(S.K, MDPVI_CALL)
#undef MDPVI_CALL
  return hipGetLastError();
}

}  // namespace mdpvi
