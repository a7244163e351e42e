// adjoint_group.hip -- single-instance launches of the group form of the
// transposed (adjoint) sweep (adjoint_group.hpp), with the stop test's
// control words loaded together with the weights: a workgroup per group.
#include "adjoint_group.hpp"
#include "adjoint_impl.hpp"
#include "device.hpp"
#include "kernels.hpp"
#include "tile.hpp"

namespace mdpvi {

template <int K, int J, int LMIN, int L>
__global__ __launch_bounds__(adjoint_group_threads(L, J)) void adjoint_group_kernel(
    AdjointArgs A, const uint8_t* __restrict__ pi, const float* __restrict__ win, float* __restrict__ wout, Ctl* ctl,
    double* res, long long j, double tol) {
  extern __shared__ double group_lds[];
  // Workgroup 0 alone sums the residual words of sweep j-1 and sets done_iter
  // = j where they meet the test; the launch then still computes w^{j+1}, into
  // the buffer that the answer w^j is not in, and the later ones stop.  (Every
  // wavefront of every workgroup reading the 64 words, each on a line of its
  // own, took 2 us of a large launch: 15.9 against 13.8 us at 786,432 states.)
  // A done_iter below j is older than this launch: the same for every lane.
  const long long done = load_agent(&ctl->done_iter);
  double rv = 0.0;
  if (blockIdx.x == 0 && threadIdx.x < kResLanes && j > 0) rv = load_agent(res + sum_word(j - 1, threadIdx.x));
  auto stop = [&]() -> bool {
    if (done >= 0 && done < j) return true;
    if (blockIdx.x == 0 && threadIdx.x < kResLanes) {
      double v = rv;
#pragma unroll
      for (int off = kWave / 2; off > 0; off >>= 1) v += __shfl_xor(v, off, kWave);
      if (j > 0 && !(v >= tol) && threadIdx.x == 0) store_agent(&ctl->done_iter, j);
      store_agent(res + sum_word(j + 1, threadIdx.x), 0.0);
    }
    return false;
  };
  double dsum = 0.0;
  if (!adjoint_group_block<K, J, LMIN, L>(A, pi, win, wout, xcd_block(blockIdx.x, gridDim.x), group_lds, stop, &dsum)) return;
  block_sum_to<kAnyBlock>(dsum, res, j);
}

bool adjoint_group_shape(const Model& M) {
  return M.K >= 3 && M.K <= 8 && M.J >= 1 && M.J <= 3 && M.R * M.R <= kBlock && M.C < kLineLoads &&
         M.n_states < (int64_t{1} << 29);
}

static AdjointArgs adjoint_args(const Model& M) {
  AdjointArgs A{};
  A.C = M.C;
  A.R = M.R;
  A.KC = M.KC;
  A.n_occ = static_cast<uint32_t>(M.n_occ);
  A.n_states = static_cast<uint32_t>(M.n_states);
  A.n_groups = static_cast<uint32_t>(M.n_occ / (M.R * M.R));
  A.divR = M.divR;
  for (int k = 0; k < M.K; ++k) A.stride[k] = static_cast<uint32_t>(M.stride[k]);
  for (int e = 0; e < M.J; ++e) {
    A.size[e] = M.size[e];
    A.p[e] = M.p[e];
    A.c_obj[e] = M.c_obj[e];
  }
  A.mu_L = M.mu_L;
  A.nu_L = M.nu_L;
  A.gamma = M.gamma;
  for (int x = 0; x < M.C; ++x) A.up[x] = M.mu_L * (x + 1);
  return A;
}

hipError_t launch_adjoint_group(const Model& M, const uint8_t* pi, const float* win, float* wout, Ctl* ctl,
                                double* res, long long j, double tol, hipStream_t s) {
  if (!adjoint_group_shape(M)) return hipErrorInvalidValue;
  const AdjointArgs A = adjoint_args(M);
  const dim3 grid(A.n_groups), block(adjoint_group_threads(static_cast<uint32_t>(M.R), static_cast<uint32_t>(M.J)));
  const uint32_t lds = adjoint_group_lds(static_cast<uint32_t>(M.K), static_cast<uint32_t>(M.R), static_cast<uint32_t>(M.J));
  return tile_dispatch(M.K, M.J, 2, [&](auto kc, auto jc, auto) {
    constexpr int Kc = decltype(kc)::value, Jc = decltype(jc)::value;
    auto launch = [&](auto lo, auto lc) {
      hipLaunchKernelGGL((adjoint_group_kernel<Kc, Jc, decltype(lo)::value, decltype(lc)::value>), grid, block, lds, s, A, pi, win, wout,
                         ctl, res, j, tol);
      return hipGetLastError();
    };
    // loads of a reset line: at most four more than its length
    if (M.R <= 5) return launch(IC<2>{}, IC<5>{});
    if (M.R <= 7) return launch(IC<6>{}, IC<7>{});
    if (M.R <= 9) return launch(IC<8>{}, IC<9>{});
    if (M.R <= 11) return launch(IC<10>{}, IC<11>{});
    return launch(IC<12>{}, IC<kLineLoads>{});
  });
}

}  // namespace mdpvi
