// orbit.hip -- kernels of the orbit form (orbit.hpp) of one instance: the
// rank table, the check that a start (and a policy) is invariant under host
// permutations, sweeps over the orbits (one launch each, or all of them in
// one workgroup's LDS) and the expansion to the full state space.
//
// Measured against the full sweeps of the same solve.  Value iteration to
// ||dV|| < 1e-6, wall time: K = 6, C = 10, J = 3 43 -> 5.4 ms (31 -> 3.4 us per
// sweep); K = 7 530 -> 7.6 ms (392 -> 4.8 us); K = 4, C = 12, J = 3 2.75 -> 1.86
// ms; in LDS K = 3, C = 8, J = 2 2.28 -> 0.17 ms (0.42 us per sweep in the
// kernel's own time).
// Evaluation of the least-loaded heuristic to 1e-10: K = 6, C = 10, J = 3 94 ->
// 8.3 ms (42 -> 3.5 us per sweep); in LDS K = 3, C = 8, J = 2 2.35 -> 0.20 ms.
#include "kernels.hpp"
#include "orbit.hpp"
#include "orbit_impl.hpp"

namespace mdpvi {

// ------------------------------------------------------------------ table

template <int KX, typename Idx>
__global__ __launch_bounds__(256) void orbit_table_kernel(OrbitShape S, OrbitParams P, uint64_t* __restrict__ dig,
                                                          uint32_t* __restrict__ rep, Idx* __restrict__ tab) {
  __shared__ uint32_t B[kOrbitBinom];
  orbit_stage_binom(S, B);
  const uint32_t r = blockIdx.x * blockDim.x + threadIdx.x;
  if (r < S.n) orbit_table<KX, Idx>(S, P, B, r, dig, rep, tab);
}

// ------------------------------------------------------------ start and end

// The start of a solve from V after it0 sweeps: control words, the orbits'
// values, and the check that V (and pi) is invariant.  Each workgroup leaves
// what it found in a word of its own (raising one shared word, even only after
// a look at it, took 40 us more for a refused policy of a million states).
template <class Op, int KX>
__global__ __launch_bounds__(256) void orbit_check_kernel(OrbitShape S, OrbitParams P, OrbitWork W,
                                                          const typename Op::T* __restrict__ V,
                                                          const uint8_t* __restrict__ pi, double tol, long long it0) {
  const uint64_t step = static_cast<uint64_t>(gridDim.x) * blockDim.x;
  const uint64_t first = static_cast<uint64_t>(blockIdx.x) * blockDim.x + threadIdx.x;
  // the slot before the first sweep's holds one word that passes no test
  if (blockIdx.x == 0)
    for (uint32_t w = threadIdx.x; w < kResSlots * kOrbitGrid; w += blockDim.x)
      W.res[w] = w == (kResSlots - 1) * kOrbitGrid ? INFINITY : 0.0;
  if (first == 0) {
    W.ctl->done = -1;
    W.ctl->base = it0;
    W.ctl->tol = tol;
    W.A[0][S.n] = -INFINITY;
    W.A[1][S.n] = -INFINITY;
  }
  uint32_t bits = 0;
  for (uint64_t o = first; o < S.n_occ; o += step) {
    if (o < S.n) orbit_begin<Op>(S, P, W, V, pi, static_cast<uint32_t>(o));
    bits |= orbit_check<Op, KX>(S, P, V, pi, static_cast<uint32_t>(o));
  }
  bits = orbit_found(bits);
  if (threadIdx.x == 0) W.found[blockIdx.x] = bits;
}

// The check's verdict from the words of its `grid` workgroups (a whole
// workgroup calls it): true where it refuses.
__device__ __forceinline__ bool orbit_refused(const OrbitWork& W, uint32_t grid, OrbitCtl* mirror) {
  const uint32_t bits = orbit_found(W.found, grid);
  if (threadIdx.x == 0) {
    W.ctl->refused = bits;
    if (bits) mirror->done = bits & kOrbitNoRoom ? kOrbitDoneInfeasible : kOrbitDoneRefused;
  }
  return bits != 0;
}
__global__ __launch_bounds__(1024) void orbit_verdict_kernel(OrbitWork W, uint32_t grid, OrbitCtl* mirror) {
  orbit_refused(W, grid, mirror);
}

// V := the final iterate (ctl->done, or `issued` sweeps when none stopped the
// loop) at every state; nothing when the form was refused.
template <class Op, int KX>
__global__ __launch_bounds__(256) void orbit_expand_kernel(OrbitShape S, OrbitWork W,
                                                           typename Op::T* __restrict__ V, long long issued) {
  using T = typename Op::T;
  if (W.ctl->refused) return;
  const long long done = W.ctl->done;
  const T* Vr = static_cast<const T*>(W.V[(done >= 0 ? done : issued) & 1]);
  __shared__ uint32_t B[kOrbitBinom];
  orbit_stage_binom(S, B);
  const uint64_t step = static_cast<uint64_t>(gridDim.x) * blockDim.x;
  for (uint64_t o = static_cast<uint64_t>(blockIdx.x) * blockDim.x + threadIdx.x; o < S.n_occ; o += step)
    orbit_expand<T, KX>(S, B, Vr, V, static_cast<uint32_t>(o));
}

// ----------------------------------------------------------------- sweeps

// Sweep i of a chunk (orbit_sweep).  The chunk starts after ctl->base sweeps,
// a multiple of kResSlots, so that i alone decides the buffers and the
// residual slot; a small kernel after the chunk moves base on.  A chunk is a
// recorded graph: issued one by one, the launches are bound by the host (5.3
// us each at 360 bytes of arguments); a graph node with no work takes 1.8 us,
// the table rows 0.85, values and backup 0.7, the verdict and the residual
// 0.2 (K = 6, C = 10, J = 3).
template <class Op, int K, int L, typename Idx>
__global__ __launch_bounds__(kOrbitBlock) void orbit_sweep_kernel(OrbitShape S, OrbitParams P, OrbitWork W,
                                                                  OrbitCtl* mirror, uint32_t grid, int i) {
  orbit_sweep<Op, K, L, Idx>(S, P, W, i, blockIdx.x, grid, [&](double residual) {
    OrbitCtl* ctl = W.ctl;
    if (ctl->done < 0) {
      ctl->done = ctl->base + i;
      mirror->residual = residual;
      mirror->done = ctl->base + i;
    }
  });
}

// Moves the chunk's base on by n sweeps.
__global__ void orbit_next_kernel(OrbitCtl* ctl, int n) { ctl->base += n; }

// The residual of the last of `issued` sweeps when none stopped the loop.
__global__ __launch_bounds__(256) void orbit_last_residual_kernel(OrbitWork W, uint32_t grid, long long issued,
                                                                  OrbitCtl* mirror) {
  __shared__ double part[256 / kWave];
  const double* w = W.res + static_cast<size_t>((issued - 1) % kResSlots) * kOrbitGrid;
  double m = 0.0;
  for (uint32_t b = threadIdx.x; b < grid; b += 256) {
    const double v = w[b];
    m = (v > m || v != v) ? v : m;
  }
  m = wave_max(m);
  if (threadIdx.x % kWave == 0) part[threadIdx.x / kWave] = m;
  __syncthreads();
  if (threadIdx.x == 0 && W.ctl->done < 0) {
    for (int i = 1; i < 256 / kWave; ++i) m = (part[i] > m || part[i] != part[i]) ? part[i] : m;
    mirror->residual = m;
  }
}

// The LDS-resident solve (orbit_lds).  HIP on this GPU takes a launch's dynamic
// LDS up to the CU's 160 KB, without the attribute that raises a limit.
template <class Op, int K, int L, int HOIST>
__global__ __launch_bounds__(kOrbitLdsBlock) void orbit_lds_kernel(OrbitShape S, OrbitParams P, OrbitWork W,
                                                                   OrbitCtl* mirror, uint32_t check_grid,
                                                                   long long it0, long long most, double tol) {
  extern __shared__ double orbit_lds_mem[];
  if (it0 == 0 ? orbit_refused(W, check_grid, mirror) : W.ctl->done >= 0) return;
  orbit_lds<Op, K, L, HOIST, kOrbitLdsBlock>(S, P, W, it0, most, tol, orbit_lds_mem,
                                             [&](long long it, double residual, bool stopped) {
                                               mirror->residual = residual;
                                               if (stopped) {
                                                 W.ctl->done = it;
                                                 mirror->done = it;
                                               }
                                             });
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

hipError_t launch_orbit_table(const OrbitShape& S, const OrbitParams& P, uint64_t* dig, uint32_t* rep, void* tab,
                              hipStream_t s) {
  const uint32_t grid = (S.n + 255) / 256;
#define MDPVI_CALL(KX_, T_)                                                                      \
  hipLaunchKernelGGL((orbit_table_kernel<KX_, T_>), dim3(grid), dim3(256), 0, s, S, P, dig, rep, \
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
// of the expansion reads the rank table once).
static uint32_t full_grid(const OrbitShape& S) {
  const uint64_t g = (S.n_occ + 255) / 256;
  return static_cast<uint32_t>(g < kOrbitCheckGrid ? g : kOrbitCheckGrid);
}

template <class Op>
hipError_t launch_orbit_check(const OrbitShape& S, const OrbitParams& P, const OrbitWork& W, const typename Op::T* V,
                              const uint8_t* pi, double tol, long long it0, hipStream_t s) {
#define MDPVI_CALL(KX_) \
  hipLaunchKernelGGL((orbit_check_kernel<Op, KX_>), dim3(full_grid(S)), dim3(256), 0, s, S, P, W, V, pi, tol, it0)
  MDPVI_ORBIT_K(S.K, MDPVI_CALL)
#undef MDPVI_CALL
  return hipGetLastError();
}

hipError_t launch_orbit_verdict(const OrbitShape& S, const OrbitWork& W, OrbitCtl* mirror, hipStream_t s) {
  hipLaunchKernelGGL(orbit_verdict_kernel, dim3(1), dim3(1024), 0, s, W, full_grid(S), mirror);
  return hipGetLastError();
}

template <class Op>
hipError_t launch_orbit_expand(const OrbitShape& S, const OrbitWork& W, typename Op::T* V, long long issued,
                               hipStream_t s) {
#define MDPVI_CALL(KX_) \
  hipLaunchKernelGGL((orbit_expand_kernel<Op, KX_>), dim3(full_grid(S)), dim3(256), 0, s, S, W, V, issued)
  MDPVI_ORBIT_K(S.K, MDPVI_CALL)
#undef MDPVI_CALL
  return hipGetLastError();
}

uint32_t orbit_grid(const OrbitShape& S) {
  const uint64_t lanes = static_cast<uint64_t>(S.n) * S.L;
  const uint64_t g = (lanes + kOrbitBlock - 1) / kOrbitBlock;
  return static_cast<uint32_t>(g < kOrbitGrid ? g : kOrbitGrid);
}

template <class Op, int K, typename Idx>
static const void* sweep_l(int L) {
  switch (L) {
    case 1: return reinterpret_cast<const void*>(&orbit_sweep_kernel<Op, K, 1, Idx>);
    case 2: return reinterpret_cast<const void*>(&orbit_sweep_kernel<Op, K, 2, Idx>);
    case 4: return reinterpret_cast<const void*>(&orbit_sweep_kernel<Op, K, 4, Idx>);
    default: return reinterpret_cast<const void*>(&orbit_sweep_kernel<Op, K, 8, Idx>);
  }
}

template <class Op>
static const void* sweep_fn(const OrbitShape& S) {
  const void* f = nullptr;
#define MDPVI_CALL(K_) f = S.wide ? sweep_l<Op, K_, uint32_t>(S.L) : sweep_l<Op, K_, uint16_t>(S.L)
  MDPVI_ORBIT_K(S.K, MDPVI_CALL)
#undef MDPVI_CALL
  return f;
}

template <class Op>
hipError_t launch_orbit_sweep(const OrbitShape& S, const OrbitParams& P, const OrbitWork& W, OrbitCtl* mirror, int i,
                              hipStream_t s) {
  OrbitShape sh = S;
  OrbitParams pr = P;
  OrbitWork w = orbit_work(W, i);
  uint32_t grid = orbit_grid(S);
  void* args[] = {&sh, &pr, &w, &mirror, &grid, &i};
  return hipLaunchKernel(sweep_fn<Op>(S), dim3(grid), dim3(kOrbitBlock), args, 0, s);
}

hipError_t launch_orbit_next(OrbitCtl* ctl, int n, hipStream_t s) {
  hipLaunchKernelGGL(orbit_next_kernel, dim3(1), dim3(1), 0, s, ctl, n);
  return hipGetLastError();
}

template <class Op>
hipError_t build_orbit_chunk(const OrbitShape& S, const OrbitParams& P, const OrbitWork& W, OrbitCtl* mirror,
                             hipGraphExec_t* out) {
  *out = nullptr;
  hipGraph_t g = nullptr;
  hipError_t e = hipGraphCreate(&g, 0);
  if (e != hipSuccess) return e;
  OrbitShape sh = S;
  OrbitParams pr = P;
  uint32_t grid = orbit_grid(S);
  hipGraphNode_t node = nullptr;
  for (int i = 0; i <= kOrbitChunk && e == hipSuccess; ++i) {
    OrbitWork w = orbit_work(W, i);
    void* args[] = {&sh, &pr, &w, &mirror, &grid, &i};
    int n = kOrbitChunk;
    void* last[] = {&w.ctl, &n};
    hipKernelNodeParams p{};
    p.func = const_cast<void*>(i < kOrbitChunk ? sweep_fn<Op>(S) : reinterpret_cast<const void*>(&orbit_next_kernel));
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

hipError_t launch_orbit_last_residual(const OrbitShape& S, const OrbitWork& W, long long issued, OrbitCtl* mirror,
                                      hipStream_t s) {
  hipLaunchKernelGGL(orbit_last_residual_kernel, dim3(1), dim3(256), 0, s, W, orbit_grid(S), issued, mirror);
  return hipGetLastError();
}

template <class Op, int K, int L>
static void lds_h(const OrbitShape& S, const OrbitParams& P, const OrbitWork& W, OrbitCtl* mirror, long long it0,
                  long long most, double tol, hipStream_t s) {
  const uint32_t lanes = S.n * L;
  const uint32_t threads = lanes < kOrbitLdsBlock ? (lanes + kWave - 1) / kWave * kWave : kOrbitLdsBlock;
  const size_t lds = orbit_lds_bytes(S, sizeof(typename Op::T));
#define MDPVI_CALL(H_)                                                                                         \
  hipLaunchKernelGGL((orbit_lds_kernel<Op, K, L, H_>), dim3(1), dim3(threads), lds, s, S, P, W, mirror, full_grid(S), \
                     it0, most, tol)
  // the table rows of more orbits, or of more hosts, would not fit the 128
  // registers that 16 wavefronts leave a lane
  if (K <= 8 && lanes <= threads) MDPVI_CALL((K <= 8 ? 1 : 0));
  else if (K <= 6 && lanes <= 2 * threads) MDPVI_CALL((K <= 6 ? 2 : 0));
  else MDPVI_CALL(0);
#undef MDPVI_CALL
}

template <class Op, int K>
static void lds_l(const OrbitShape& S, const OrbitParams& P, const OrbitWork& W, OrbitCtl* mirror, long long it0,
                  long long most, double tol, hipStream_t s) {
  switch (S.L) {
    case 1: lds_h<Op, K, 1>(S, P, W, mirror, it0, most, tol, s); break;
    case 2: lds_h<Op, K, 2>(S, P, W, mirror, it0, most, tol, s); break;
    case 4: lds_h<Op, K, 4>(S, P, W, mirror, it0, most, tol, s); break;
    default: lds_h<Op, K, 8>(S, P, W, mirror, it0, most, tol, s);
  }
}

template <class Op>
hipError_t launch_orbit_lds(const OrbitShape& S, const OrbitParams& P, const OrbitWork& W, OrbitCtl* mirror,
                            long long it0, long long most, double tol, hipStream_t s) {
#define MDPVI_CALL(K_) lds_l<Op, K_>(S, P, W, mirror, it0, most, tol, s)
  MDPVI_ORBIT_K(S.K, MDPVI_CALL)
#undef MDPVI_CALL
  return hipGetLastError();
}

#define MDPVI_ORBIT_OP(OP_)                                                                                       \
  template hipError_t launch_orbit_check<OP_>(const OrbitShape&, const OrbitParams&, const OrbitWork&,            \
                                              const OP_::T*, const uint8_t*, double, long long, hipStream_t);     \
  template hipError_t launch_orbit_expand<OP_>(const OrbitShape&, const OrbitWork&, OP_::T*, long long,           \
                                               hipStream_t);                                                      \
  template hipError_t launch_orbit_sweep<OP_>(const OrbitShape&, const OrbitParams&, const OrbitWork&, OrbitCtl*, \
                                              int, hipStream_t);                                                  \
  template hipError_t build_orbit_chunk<OP_>(const OrbitShape&, const OrbitParams&, const OrbitWork&, OrbitCtl*,  \
                                             hipGraphExec_t*);                                                    \
  template hipError_t launch_orbit_lds<OP_>(const OrbitShape&, const OrbitParams&, const OrbitWork&, OrbitCtl*,   \
                                            long long, long long, double, hipStream_t);
MDPVI_ORBIT_OP(OrbitVi)
MDPVI_ORBIT_OP(OrbitEval)

}  // namespace mdpvi
