// adjoint_group.hpp -- the group form of the transposed (adjoint) backup as
// a workgroup-level device function of the single-instance group kernel
// (adjoint_group.hip).
//
// A group is the G = (C+1)^2 occupancies that share digits 2..K-1; a
// workgroup takes one, an (occupancy, class) per lane (slot l = e G + r).  The
// high digits are then the workgroup's, so the neighbours along them are loads
// at the lane's own offset plus a scalar one.  A lane loads its state's action
// and weight, its class's neighbours along the high digits and, where one is
// zero, the reset line along the first such digit, all in one round trip
// (further lines, which few groups have, later: loading them ahead too took
// 100 registers and 22 us at 786,432 states, 13 us so).  It publishes in LDS
// its weight and what it hands on as an arrival: to the paid cloud, to host 0
// or 1 of an occupancy of the group, and from the high hosts.  Then G lanes
// form the arrival inflows, 2 J (C+1) others the reset lines along digits 0
// and 1, once each instead of in every wavefront that holds a lane of n_0 = 0
// or n_1 = 0, and each lane finishes its state.  Bound by instruction issue
// (about 330 vector and 250 scalar instructions a wavefront) for large
// instances, by the round trips for small ones: a sweep of K = 5, C = 8, J = 3
// (177,147 states) 11.9 -> 6.2 us, of K = 6, C = 7, J = 3 24.6 -> 13.1 us
// against one occupancy of all classes per lane.  Two groups per lane (20 us)
// and workgroups of 512 and 1,024 lanes (22.8 and 23.3 us) were slower there.
// In the rounds of a batch, which fill the chip, a lane per occupancy with all
// its classes needs fewer instructions: the form took 94 against 63 ms.
// Terms are added in the order of adjoint_occupancy (zeros between them change
// nothing), so w is bit-identical to the other adjoint forms.
#pragma once

#include "adjoint_impl.hpp"
#include "device.hpp"

namespace mdpvi {

// What the form reads of a Model.
struct AdjointArgs {
  int32_t C, R, KC;
  uint32_t n_occ, n_states, n_groups;
  FastDiv divR;
  uint32_t stride[8];
  int32_t size[3];
  double p[3], c_obj[3];
  double mu_L, nu_L, gamma;
  double up[kLineLoads];   // mu_L (x + 1), 0 at x = C
};

// Lanes of a group's workgroup.
__host__ __device__ constexpr uint32_t adjoint_group_threads(uint32_t R, uint32_t J) {
  return (J * R * R + kWave - 1) / kWave * kWave;
}

// LDS bytes of a workgroup: the line sums along digits 0 and 1, the arrival inflows,
// the weights, K + 1 arrival terms per slot.
__host__ __device__ constexpr uint32_t adjoint_group_lds(uint32_t K, uint32_t R, uint32_t J) {
  return 8 * (2 * J * R + R * R) + 4 * J * R * R * (K + 2);
}

// stop(): called by every lane once its loads are issued; true makes the
// function return false at once (before any LDS write or barrier: the answer
// must be the same for the whole workgroup).  Otherwise the new weight is
// stored and *dsum_out receives the lane's |w' - w|; returns true.  g: the
// group; lds: adjoint_group_lds bytes.  LMIN <= C + 1 <= L: the loads of a reset
// line, those past C (of the state itself) weighted with zero.
template <int K, int J, int LMIN, int L, typename Stop>
__device__ __forceinline__ bool adjoint_group_block(const AdjointArgs& M, const uint8_t* __restrict__ pi,
                                                    const float* __restrict__ win, float* __restrict__ wout,
                                                    uint32_t g, double* lds, Stop&& stop, double* dsum_out) {
  constexpr int NH = K - 2;
  const uint32_t R = static_cast<uint32_t>(M.R), G = R * R, C = static_cast<uint32_t>(M.C);
  const uint32_t nocc = M.n_occ;
  const uint32_t slots = J * G, nl = J * R;
  double* lines = lds;                                  // [2][J][R]: digits 0 and 1
  double* Bs = lines + 2 * nl;                          // [G]
  float* ws = reinterpret_cast<float*>(Bs + G);         // [J][G] weights
  float* in = ws + slots;   // [K+1][J][G]: cloud, hosts 0 and 1 (at the source), high hosts (at the target)
  // lanes past the slots stand in for the last one and store nothing
  const uint32_t tid = threadIdx.x, threads = blockDim.x;
  const uint32_t l = tid < slots ? tid : slots - 1;
  const uint32_t q1 = fast_div(l, M.divR), e = J == 1 ? 0u : fast_div(q1, M.divR);
  const int n0 = static_cast<int>(l - q1 * R), n1 = static_cast<int>(q1 - e * R);
  // high digits, the same for the workgroup
  int nh[NH], load_high = 0;
  {
    uint32_t q = g;
#pragma unroll
    for (int x = 0; x < NH; ++x) {
      const uint32_t d = fast_div(q, M.divR);
      nh[x] = static_cast<int>(q - d * R);
      load_high += nh[x];
      q = d;
    }
  }
  auto pick = [&](auto a0, auto a1, auto a2) { return J > 2 && e == 2 ? a2 : J > 1 && e == 1 ? a1 : a0; };
  const uint32_t s = g * G + (l - e * G) + pick(0u, nocc, 2 * nocc);
  const BufView vp = make_view(pi, M.n_states);
  const BufView vw = make_view(win, M.n_states * 4u);
  const BufView vo = make_view(wout, M.n_states * 4u);
  const uint32_t s4 = 4u * s;
  const int p_own = ld_u8(vp, s, 0);
  const float w_own = ld_f32(vw, s4, 0);
  int p_k[NH];
  uint32_t d_k[NH];   // distance of the arrival predecessor; 0: none
  float w_k[NH], w_rel[NH], h[L];
#pragma unroll
  for (int x = 0; x < NH; ++x) {
    const uint32_t st = M.stride[2 + x];
    uint32_t d[3];
#pragma unroll
    for (int j = 0; j < J; ++j) d[j] = nh[x] >= M.size[j] ? static_cast<uint32_t>(M.size[j]) * st : 0u;
    d_k[x] = pick(d[0], d[J > 1 ? 1 : 0], d[J > 2 ? 2 : 0]);
    p_k[x] = ld_u8(vp, s - d_k[x], 0);
    w_k[x] = ld_f32(vw, s4 - 4u * d_k[x], 0);
    w_rel[x] = ld_f32(vw, s4, nh[x] < M.C ? 4u * st : 0u);
  }
  auto load_line = [&](uint32_t st, float (&v)[L]) {
#pragma unroll
    for (uint32_t y = 0; y < L; ++y) v[y] = ld_f32(vw, s4, y <= C ? 4u * y * st : 0u);
  };
  auto sum_line = [&](const float (&v)[L]) {
    double line = 0.0;
#pragma unroll
    for (uint32_t y = 0; y < L; ++y)
      line = y < LMIN ? line + static_cast<double>(v[y]) : fma(y <= C ? 1.0 : 0.0, static_cast<double>(v[y]), line);
    return line;
  };
  // the line along the first high digit that is zero
  int k1 = NH;
  uint32_t st1 = 0;
#pragma unroll
  for (int x = NH - 1; x >= 0; --x) {
    k1 = nh[x] == 0 ? x : k1;
    st1 = nh[x] == 0 ? M.stride[2 + x] : st1;
  }
  if (k1 < NH) load_line(st1, h);

  if (stop()) return false;

  ws[l] = w_own;
  float* il = in + l;
  il[0] = p_own == K ? w_own : 0.0f;
  il[slots] = p_own == 0 ? w_own : 0.0f;
  il[2 * slots] = p_own == 1 ? w_own : 0.0f;
#pragma unroll
  for (int x = 0; x < NH; ++x) il[(3 + x) * slots] = d_k[x] != 0 && p_k[x] == 2 + x ? w_k[x] : 0.0f;
  __syncthreads();

  // the last lanes: the reset lines along digits 0 and 1, each summed
  // from zero in the order 0..C
  if (tid >= threads - 2 * nl) {
    const uint32_t t = tid - (threads - 2 * nl);
    const bool d0 = t < nl;
    const uint32_t v = d0 ? t : t - nl;
    const uint32_t v1 = fast_div(v, M.divR);
    const uint32_t base = d0 ? v * R : v1 * G + (v - v1 * R), st = d0 ? 1u : R;
    float x[L];
#pragma unroll
    for (uint32_t y = 0; y < L; ++y) x[y] = ws[y <= C ? base + y * st : base];
    lines[t] = sum_line(x);
  }
  // the first: the arrival inflow, the paid cloud at n', then placements on
  // host k from n' - size_e 1_k, k = 0..K-1, e = 0..J-1
  if (tid < G) {
    const float* iu = in + tid;
    float c[K + 1][J];
#pragma unroll
    for (int x = 0; x < J; ++x) {
      c[0][x] = iu[x * G];
      const bool h0 = n0 >= M.size[x], h1 = n1 >= M.size[x];
      c[1][x] = iu[slots + x * G - (h0 ? static_cast<uint32_t>(M.size[x]) : 0u)];
      c[2][x] = iu[2 * slots + x * G - (h1 ? static_cast<uint32_t>(M.size[x]) * R : 0u)];
      c[1][x] = h0 ? c[1][x] : 0.0f;
      c[2][x] = h1 ? c[2][x] : 0.0f;
#pragma unroll
      for (int k = 0; k < NH; ++k) c[3 + k][x] = iu[(3 + k) * slots + x * G];
    }
    double B = 0.0;
#pragma unroll
    for (int k = 0; k <= K; ++k)
#pragma unroll
      for (int x = 0; x < J; ++x) B += static_cast<double>(c[k][x]);
    Bs[tid] = B;
  }
  const float rel0 = ws[n0 < M.C ? l + 1 : l], rel1 = ws[n1 < M.C ? l + R : l];
  __syncthreads();

  double rs = 0.0;
  if (n0 == 0) rs += lines[q1];
  if (n1 == 0) rs += lines[nl + e * R + static_cast<uint32_t>(n0)];
#pragma unroll
  for (int x = 0; x < NH; ++x) {
    if (nh[x] == 0) {
      if (x != k1) load_line(M.stride[2 + x], h);
      rs += sum_line(h);
    }
  }
  const double idle = M.mu_L * static_cast<double>(M.KC - load_high - n0 - n1);
  double acc = fma(pick(M.p[0], M.p[1], M.p[2]), Bs[l - e * G], idle * static_cast<double>(w_own));
  acc = fma(n0 < M.C ? M.mu_L * (n0 + 1) : 0.0, static_cast<double>(rel0), acc);
  acc = fma(n1 < M.C ? M.mu_L * (n1 + 1) : 0.0, static_cast<double>(rel1), acc);
#pragma unroll
  for (int x = 0; x < NH; ++x) acc = fma(M.up[nh[x]], static_cast<double>(w_rel[x]), acc);
  acc = fma(M.nu_L, rs, acc);
  const double c = g == 0 && l == e * G ? pick(M.c_obj[0], M.c_obj[1], M.c_obj[2]) : 0.0;
  const float wn = static_cast<float>(fma(M.gamma, acc, c));
  *dsum_out = 0.0;
  if (tid < slots) {
    st_f32(vo, wn, s4, 0);
    *dsum_out = fabs(static_cast<double>(wn) - static_cast<double>(w_own));
  }
  return true;
}

}  // namespace mdpvi
