// orbit_batch.hip -- the orbit form (orbit.hpp) of many instances at once.
//
// Each instance keeps its own start check, stopping test and outputs.  The
// smaller ones are solved LDS-resident, one workgroup each for all their
// sweeps; the larger ones advance one sweep per launch over all of them
// (rounds), concurrently on another stream.  The workgroup bodies are the
// single-instance kernels', so an instance gets the same bits either way.
// The 512-instance sweep's value iteration: 66.6 -> 8.4 ms against the full
// sweeps.
//
// Kernels carry the bodies of K <= 5 and J <= 4 (MAIN) or all the others: an
// instance's body is picked by a uniform switch, and a kernel's registers are
// its largest body's.
#include "kernels.hpp"
#include "orbit.hpp"
#include "orbit_impl.hpp"

namespace mdpvi {

#define MDPVI_OB_L(K_, BODY)             \
  switch (S.L) {                         \
    case 1: BODY(K_, 1); break;          \
    case 2: BODY(K_, 2); break;          \
    case 4: BODY(K_, 4); break;          \
    default:                             \
      if constexpr (!MAIN) BODY(K_, 8);  \
  }
#define MDPVI_OB_KL(BODY)                            \
  switch (S.K) {                                     \
    case 1: MDPVI_OB_L(1, BODY); break;              \
    case 2: MDPVI_OB_L(2, BODY); break;              \
    case 3: MDPVI_OB_L(3, BODY); break;              \
    case 4: MDPVI_OB_L(4, BODY); break;              \
    case 5: MDPVI_OB_L(5, BODY); break;              \
    default:                                         \
      if constexpr (!MAIN) {                         \
        switch (S.K) {                               \
          case 6: MDPVI_OB_L(6, BODY); break;        \
          case 7: MDPVI_OB_L(7, BODY); break;        \
          case 8: MDPVI_OB_L(8, BODY); break;        \
          default: MDPVI_OB_L(16, BODY);             \
        }                                            \
      }                                              \
  }

// The tables of the orbits [first, first + 256) of the tile's instance (the
// tiles of one instance per table).
__global__ __launch_bounds__(256) void orbit_batch_table_kernel(const OrbitInst* __restrict__ insts,
                                                                const Tile* __restrict__ tiles) {
  __shared__ uint32_t B[kOrbitBinom];
  const Tile t = tiles[blockIdx.x];
  const OrbitInst& I = insts[t.inst];
  const OrbitShape S = I.S;
  orbit_stage_binom(S, B);
  const uint32_t r = t.first + threadIdx.x;
  if (r >= S.n) return;
  uint64_t* dig = const_cast<uint64_t*>(S.dig);
  uint32_t* rep = const_cast<uint32_t*>(S.rep);
  uint16_t* tab = static_cast<uint16_t*>(const_cast<void*>(S.tab));
  if (S.K <= 4) orbit_table<4, uint16_t>(S, I.P, B, r, dig, rep, tab);
  else if (S.K <= 8) orbit_table<8, uint16_t>(S, I.P, B, r, dig, rep, tab);
  else orbit_table<16, uint16_t>(S, I.P, B, r, dig, rep, tab);
}

#define MDPVI_OB_K(BODY)        \
  switch (I.S.K) {              \
    case 1: BODY(1); break;     \
    case 2: BODY(2); break;     \
    case 3: BODY(3); break;     \
    case 4: BODY(4); break;     \
    case 5: BODY(5); break;     \
    case 6: BODY(6); break;     \
    case 7: BODY(7); break;     \
    case 8: BODY(8); break;     \
    default: BODY(16);          \
  }

template <class Op, int KX>
__device__ __forceinline__ uint32_t batch_check(const OrbitInst& I, const typename Op::T* V, const uint8_t* pi,
                                                uint32_t first) {
  uint32_t bits = 0;
  for (int k = 0; k < kOccPerThread; ++k) {
    const uint32_t o = first + threadIdx.x + static_cast<uint32_t>(k * kBlock);
    if (o >= I.S.n_occ) break;
    if (o < I.S.n) orbit_begin<Op>(I.S, I.P, I.W, V, pi, o);
    bits |= orbit_check<Op, KX>(I.S, I.P, V, pi, o);
  }
  return bits;
}

// The start of a solve of the tile's instance (orbit_check_kernel): the
// occupancies, and the orbits of the same numbers, [first, first + kBlock *
// kOccPerThread); what the tile found into its word.  slot: batch instance ->
// its entry in insts, -1 for one the form does not cover (the tiles are the
// batch's own, over every instance).  An instance that is not active counts as
// stopped before its first sweep.
template <class Op>
__global__ __launch_bounds__(kBlock) void orbit_batch_check_kernel(const OrbitInst* __restrict__ insts,
                                                                   const int32_t* __restrict__ slot,
                                                                   const Tile* __restrict__ tiles,
                                                                   const typename Op::T* __restrict__ V,
                                                                   const uint8_t* __restrict__ pi,
                                                                   const int* __restrict__ active, double tol,
                                                                   uint32_t* __restrict__ found) {
  const Tile t = tiles[blockIdx.x];
  const int at = slot[t.inst];
  if (at < 0) return;
  const OrbitInst& I = insts[at];
  const bool on = !active || active[t.inst];
  if (t.first == 0) {
    const OrbitWork W = I.W;
    if (W.res) {
      const uint32_t words = (I.grid + kOrbitBlock - 1) / kOrbitBlock * kOrbitBlock;
      for (uint32_t w = threadIdx.x; w < words; w += blockDim.x)
        for (int q = 0; q < kResSlots; ++q)
          W.res[q * kOrbitGrid + w] = q == kResSlots - 1 && w == 0 ? INFINITY : 0.0;
    }
    if (threadIdx.x == 0) {
      W.ctl->done = on ? -1 : 0;
      W.ctl->residual = 0.0;
      W.ctl->base = 0;
      W.ctl->tol = tol;
      W.A[0][I.S.n] = -INFINITY;
      W.A[1][I.S.n] = -INFINITY;
    }
  }
  uint32_t bits = 0;
  if (on) {
    const typename Op::T* Vi = V + I.offset;
    const uint8_t* p = pi ? pi + I.offset : nullptr;
#define MDPVI_BODY(KX_) bits = batch_check<Op, KX_>(I, Vi, p, t.first)
    MDPVI_OB_K(MDPVI_BODY)
#undef MDPVI_BODY
  }
  bits = orbit_found(bits);
  if (threadIdx.x == 0) found[blockIdx.x] = bits;
}

// An entry's verdict from its tiles' words.
__global__ __launch_bounds__(256) void orbit_batch_verdict_kernel(const OrbitInst* __restrict__ insts,
                                                                  const int32_t* __restrict__ tile_begin,
                                                                  const uint32_t* __restrict__ found) {
  const OrbitInst& I = insts[blockIdx.x];
  const int32_t first = tile_begin[I.inst], last = tile_begin[I.inst + 1];
  const uint32_t bits = orbit_found(found + first, static_cast<uint32_t>(last - first));
  if (threadIdx.x == 0) I.W.ctl->refused = bits;
}

template <class T, int KX>
__device__ __forceinline__ void batch_expand(const OrbitInst& I, const uint32_t* B, const T* Vr, T* V,
                                             uint32_t first) {
  for (int k = 0; k < kOccPerThread; ++k) {
    const uint32_t o = first + threadIdx.x + static_cast<uint32_t>(k * kBlock);
    if (o < I.S.n_occ) orbit_expand<T, KX>(I.S, B, Vr, V, o);
  }
}

// The final iterates to every state; nothing for an instance that was
// refused or not active.
template <class Op>
__global__ __launch_bounds__(kBlock) void orbit_batch_expand_kernel(const OrbitInst* __restrict__ insts,
                                                                    const int32_t* __restrict__ slot,
                                                                    const Tile* __restrict__ tiles,
                                                                    typename Op::T* __restrict__ V,
                                                                    long long issued) {
  using T = typename Op::T;
  __shared__ uint32_t B[kOrbitBinom];
  const Tile t = tiles[blockIdx.x];
  const int at = slot[t.inst];
  if (at < 0) return;
  const OrbitInst& I = insts[at];
  const long long done = I.W.ctl->done;
  if (I.W.ctl->refused || done == 0) return;
  orbit_stage_binom(I.S, B);
  const T* Vr = static_cast<const T*>(I.W.V[(done > 0 ? done : issued) & 1]);
  T* Vi = V + I.offset;
#define MDPVI_BODY(KX_) batch_expand<T, KX_>(I, B, Vr, Vi, t.first)
  MDPVI_OB_K(MDPVI_BODY)
#undef MDPVI_BODY
}

// One LDS-resident instance per workgroup.
template <class Op, bool MAIN, int NB>
__global__ __launch_bounds__(NB) void orbit_batch_lds_kernel(const OrbitInst* __restrict__ insts,
                                                             const int32_t* __restrict__ list, long long it0,
                                                             long long most, double tol) {
  extern __shared__ double orbit_batch_mem[];
  const OrbitInst& I = insts[__builtin_amdgcn_readfirstlane(list[blockIdx.x])];
  OrbitCtl* ctl = I.W.ctl;
  if (ctl->refused || ctl->done >= 0) return;
  const OrbitShape S = I.S;
  const OrbitParams P = I.P;
  const OrbitWork W = I.W;
  auto ended = [&](long long it, double residual, bool stopped) {
    ctl->residual = residual;
    if (stopped) ctl->done = it;
  };
#define MDPVI_BODY(K_, L_) orbit_lds<Op, K_, L_, 0, NB>(S, P, W, it0, most, tol, orbit_batch_mem, ended)
  MDPVI_OB_KL(MDPVI_BODY)
#undef MDPVI_BODY
}

// Round j over the first *n_tiles tiles {instance, workgroup of its grid}.
template <class Op, bool MAIN>
__global__ __launch_bounds__(kOrbitBlock) void orbit_round_kernel(const OrbitInst* __restrict__ insts,
                                                                  const Tile* __restrict__ tiles,
                                                                  const int* __restrict__ n_tiles, int* remaining,
                                                                  long long j) {
  if (static_cast<int>(blockIdx.x) >= *n_tiles) return;
  const Tile t = tiles[blockIdx.x];
  const OrbitInst& I = insts[t.inst];
  const OrbitShape S = I.S;
  const OrbitParams P = I.P;
  const OrbitWork W = orbit_work(I.W, j);
  const int i = static_cast<int>(j % kResSlots);
  auto stopped = [&](double residual) {
    if (W.ctl->done < 0) {
      W.ctl->done = j;
      W.ctl->residual = residual;
      atomicSub(remaining, 1);
    }
  };
#define MDPVI_BODY(K_, L_) orbit_sweep<Op, K_, L_, uint16_t>(S, P, W, i, t.first, I.grid, stopped)
  MDPVI_OB_KL(MDPVI_BODY)
#undef MDPVI_BODY
}

// The tiles whose instance was not refused and has not stopped, into out;
// their count into *n_out (cleared by the caller).
__global__ __launch_bounds__(256) void orbit_compact_kernel(const OrbitInst* __restrict__ insts,
                                                            const Tile* __restrict__ in,
                                                            const int* __restrict__ n_in, Tile* __restrict__ out,
                                                            int* n_out) {
  const int t = blockIdx.x * blockDim.x + threadIdx.x;
  Tile tile{};
  bool keep = false;
  if (t < *n_in) {
    tile = in[t];
    const OrbitCtl* ctl = insts[tile.inst].W.ctl;
    keep = ctl->done < 0 && !ctl->refused;
  }
  const unsigned long long mask = __ballot(keep);
  const int lane = threadIdx.x % kWave;
  const int before = __popcll(mask & ((1ull << lane) - 1ull));
  int base = 0;
  if (lane == 0 && mask != 0ull) base = atomicAdd(n_out, __popcll(mask));
  base = __shfl(base, 0, kWave);
  if (keep) out[base + before] = tile;
}

__global__ void orbit_set_kernel(int* p, int v) { *p = v; }

// The words of a solve's rounds: instances running, tiles of either list.
__global__ void orbit_words_kernel(int* p, int remaining, int tiles0, int tiles1) {
  p[0] = remaining;
  p[1] = tiles0;
  p[4] = tiles1;
}

// The residual of the last of `issued` sweeps of a round instance that has
// not stopped.
__global__ __launch_bounds__(256) void orbit_batch_residual_kernel(const OrbitInst* __restrict__ insts,
                                                                   const int32_t* __restrict__ list,
                                                                   long long issued) {
  const OrbitInst& I = insts[list[blockIdx.x]];
  if (I.W.ctl->done >= 0 || I.W.ctl->refused) return;
  __shared__ double part[256 / kWave];
  const double* w = I.W.res + static_cast<size_t>((issued - 1) % kResSlots) * kOrbitGrid;
  double m = 0.0;
  for (uint32_t b = threadIdx.x; b < I.grid; b += 256) {
    const double v = w[b];
    m = (v > m || v != v) ? v : m;
  }
  m = wave_max(m);
  if (threadIdx.x % kWave == 0) part[threadIdx.x / kWave] = m;
  __syncthreads();
  if (threadIdx.x == 0) {
    for (int i = 1; i < 256 / kWave; ++i) m = (part[i] > m || part[i] != part[i]) ? part[i] : m;
    I.W.ctl->residual = m;
  }
}

// --------------------------------------------------------------- launchers

hipError_t launch_orbit_batch_table(const OrbitInst* insts, const Tile* tiles, int n_tiles, hipStream_t s) {
  hipLaunchKernelGGL(orbit_batch_table_kernel, dim3(n_tiles), dim3(256), 0, s, insts, tiles);
  return hipGetLastError();
}

template <class Op>
hipError_t launch_orbit_batch_check(const OrbitInst* insts, int n_inst, const int32_t* slot, const Tile* tiles,
                                    int n_tiles, const int32_t* tile_begin, const typename Op::T* V,
                                    const uint8_t* pi, const int* active, double tol, uint32_t* found, hipStream_t s) {
  hipLaunchKernelGGL((orbit_batch_check_kernel<Op>), dim3(n_tiles), dim3(kBlock), 0, s, insts, slot, tiles, V, pi,
                     active, tol, found);
  hipLaunchKernelGGL(orbit_batch_verdict_kernel, dim3(n_inst), dim3(256), 0, s, insts, tile_begin, found);
  return hipGetLastError();
}

template <class Op>
hipError_t launch_orbit_batch_expand(const OrbitInst* insts, const int32_t* slot, const Tile* tiles, int n_tiles,
                                     typename Op::T* V, long long issued, hipStream_t s) {
  hipLaunchKernelGGL((orbit_batch_expand_kernel<Op>), dim3(n_tiles), dim3(kBlock), 0, s, insts, slot, tiles, V,
                     issued);
  return hipGetLastError();
}

template <class Op>
hipError_t launch_orbit_batch_lds(const OrbitInst* insts, const int32_t* list, int n_list, bool main_kernel,
                                  bool small, size_t lds, long long it0, long long most, double tol, hipStream_t s) {
  if (n_list == 0) return hipSuccess;
#define MDPVI_CALL(MAIN_, NB_)                                                                                    \
  hipLaunchKernelGGL((orbit_batch_lds_kernel<Op, MAIN_, NB_>), dim3(n_list), dim3(NB_), lds, s, insts, list, it0, \
                     most, tol)
  if (main_kernel) {
    if (small) MDPVI_CALL(true, kOrbitSmallBlock);
    else MDPVI_CALL(true, kOrbitBigBlock);
  } else {
    if (small) MDPVI_CALL(false, kOrbitSmallBlock);
    else MDPVI_CALL(false, kOrbitBigBlock);
  }
#undef MDPVI_CALL
  return hipGetLastError();
}

template <class Op>
hipError_t launch_orbit_round(const OrbitInst* insts, const Tile* tiles, const int* n_tiles, int most_tiles,
                              bool main_kernel, int* remaining, long long j, hipStream_t s) {
  if (most_tiles == 0) return hipSuccess;
  if (main_kernel)
    hipLaunchKernelGGL((orbit_round_kernel<Op, true>), dim3(most_tiles), dim3(kOrbitBlock), 0, s, insts, tiles,
                       n_tiles, remaining, j);
  else
    hipLaunchKernelGGL((orbit_round_kernel<Op, false>), dim3(most_tiles), dim3(kOrbitBlock), 0, s, insts, tiles,
                       n_tiles, remaining, j);
  return hipGetLastError();
}

hipError_t launch_orbit_compact(const OrbitInst* insts, const Tile* in, const int* n_in, int most_in, Tile* out,
                                int* n_out, hipStream_t s) {
  hipLaunchKernelGGL(orbit_set_kernel, dim3(1), dim3(1), 0, s, n_out, 0);
  if (most_in > 0)
    hipLaunchKernelGGL(orbit_compact_kernel, dim3((most_in + 255) / 256), dim3(256), 0, s, insts, in, n_in, out,
                       n_out);
  return hipGetLastError();
}

hipError_t launch_orbit_words(int* p, int remaining, int tiles0, int tiles1, hipStream_t s) {
  hipLaunchKernelGGL(orbit_words_kernel, dim3(1), dim3(1), 0, s, p, remaining, tiles0, tiles1);
  return hipGetLastError();
}

hipError_t launch_orbit_batch_residual(const OrbitInst* insts, const int32_t* list, int n_list, long long issued,
                                       hipStream_t s) {
  if (n_list == 0) return hipSuccess;
  hipLaunchKernelGGL(orbit_batch_residual_kernel, dim3(n_list), dim3(256), 0, s, insts, list, issued);
  return hipGetLastError();
}

#define MDPVI_ORBIT_OP(OP_)                                                                                          \
  template hipError_t launch_orbit_batch_check<OP_>(const OrbitInst*, int, const int32_t*, const Tile*, int,         \
                                                    const int32_t*, const OP_::T*, const uint8_t*, const int*,       \
                                                    double, uint32_t*, hipStream_t);                                 \
  template hipError_t launch_orbit_batch_expand<OP_>(const OrbitInst*, const int32_t*, const Tile*, int, OP_::T*,    \
                                                     long long, hipStream_t);                                        \
  template hipError_t launch_orbit_batch_lds<OP_>(const OrbitInst*, const int32_t*, int, bool, bool, size_t,         \
                                                  long long, long long, double, hipStream_t);                        \
  template hipError_t launch_orbit_round<OP_>(const OrbitInst*, const Tile*, const int*, int, bool, int*, long long, \
                                              hipStream_t);
MDPVI_ORBIT_OP(OrbitVi)
MDPVI_ORBIT_OP(OrbitEval)

}  // namespace mdpvi
