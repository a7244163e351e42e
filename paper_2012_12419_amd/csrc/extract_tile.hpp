// extract_tile.hpp -- greedy extraction on tiles: the form of large exact
// shapes (K 4..8 hosts, up to 3 classes of distinct sizes).
//
// The kernel of extract_occupancy reads every neighbour of an occupancy by
// itself: at K = 6, J = 3 93 gathers per occupancy, 54 of them for the arrival
// terms of the placements.  Those gathers bound it: 121 us for the
// 5,314,683-state instance, whose values, policy and gaps are 48 MB.  Here a
// workgroup stages one tile of (C+1)^T occupancies and their arrival terms in
// LDS; neighbours along the T low digits are LDS reads, neighbours along a high
// digit are loads at the lane's own offset plus a workgroup-uniform one: 42 us
// for that instance (FP64 values 137 -> 62 us), by then the FP64 units' and
// the remaining 48 loads' time.  One occupancy per lane: 2 and 4 consecutive
// ones with 8- and 16-byte loads took 130 to 211 registers and 61 and 91 us;
// the classes in a loop, since unrolled they took 54 us; workgroups of 256
// lanes 50 us, of 704 lanes 47.  Same operations in the same order as
// extract_occupancy: the same policy and gaps.
#pragma once

#include "device.hpp"
#include "kernels.hpp"
#include "tile.hpp"

namespace mdpvi {

constexpr int kExtractBlock = 512;

template <typename TV>
__device__ __forceinline__ TV ld_value(BufView v, uint32_t lane_off, uint32_t uni_off) {
  if constexpr (sizeof(TV) == 4)
    return ld_f32(v, lane_off, uni_off);
  else
    return ld_f64(v, lane_off, uni_off);
}

template <int K, int J, int T, typename TV>
__global__ __launch_bounds__(kExtractBlock) void extract_tile_kernel(Model M, TileShape S, const TV* V, uint8_t* pi,
                                                                     float* gap) {
  constexpr int NH = K - T;
  constexpr uint32_t tv = sizeof(TV);
  extern __shared__ double extract_lds[];
  const uint32_t occ = S.occ, nocc = static_cast<uint32_t>(M.n_occ);
  double* Al = extract_lds;                        // [occ]
  TV* Vl = reinterpret_cast<TV*>(Al + occ);        // [J][occ]
  const BufView vin = make_view(V, static_cast<uint32_t>(M.n_states) * tv);
  const uint32_t cls = nocc * tv;
  const uint32_t tb = xcd_block(blockIdx.x, gridDim.x);
  int nh[NH];
  const uint32_t o0 = tile_high<K, T>(M, tb, nh);

  for (uint32_t i = threadIdx.x; i < occ; i += kExtractBlock) {
    double a = 0.0;
#pragma unroll
    for (int e = 0; e < J; ++e) {
      const TV x = ld_value<TV>(vin, i * tv, o0 * tv + e * cls);
      a = fma(M.p[e], static_cast<double>(x), a);
      Vl[e * occ + i] = x;
    }
    Al[i] = a;
  }
  __syncthreads();

  int load_high = 0;
#pragma unroll
  for (int h = 0; h < NH; ++h) load_high += nh[h];
  for (uint32_t i = threadIdx.x; i < occ; i += kExtractBlock) {
    int n[T];
    tile_low<T>(M, i, n);
    int load = load_high;
#pragma unroll
    for (int k = 0; k < T; ++k) load += n[k];
    const double fu = static_cast<double>(M.KC - load);   // free units
#pragma unroll 1
    for (int e = 0; e < J; ++e) {
      const int s = M.size[e];
      TV vd[NH], vr[NH], va[NH][J];
#pragma unroll
      for (int h = 0; h < NH; ++h) {
        const uint32_t st = static_cast<uint32_t>(M.stride[T + h]);
        vd[h] = ld_value<TV>(vin, i * tv, (nh[h] > 0 ? o0 - st : o0) * tv + e * cls);
        vr[h] = ld_value<TV>(vin, i * tv, (o0 - static_cast<uint32_t>(nh[h]) * st) * tv + e * cls);
        const uint32_t m = nh[h] + s <= M.C ? o0 + static_cast<uint32_t>(s) * st : o0;
#pragma unroll
        for (int jj = 0; jj < J; ++jj) va[h][jj] = ld_value<TV>(vin, i * tv, m * tv + jj * cls);
      }
      const TV* Ve = Vl + static_cast<uint32_t>(e) * occ;
      double D = M.mu_L * fu * static_cast<double>(Ve[i]);
      double rs = 0.0;
#pragma unroll
      for (int k = 0; k < T; ++k) {
        const uint32_t st = static_cast<uint32_t>(M.stride[k]);
        const double d = static_cast<double>(Ve[n[k] > 0 ? i - st : i]);
        D = n[k] > 0 ? fma(M.mu_L * n[k], d, D) : D;
        rs += static_cast<double>(Ve[i - static_cast<uint32_t>(n[k]) * st]);
      }
#pragma unroll
      for (int h = 0; h < NH; ++h) {
        D = nh[h] > 0 ? fma(M.mu_L * nh[h], static_cast<double>(vd[h]), D) : D;
        rs += static_cast<double>(vr[h]);
      }
      D = fma(M.nu_L, rs, D);
      double best = 0.0, second = 0.0;
      int arg = -1;
      bool have_second = false;
      // extract_occupancy's choice among the actions in order
      auto action = [&](int a, bool feasible, double q) {
        const bool first = feasible && arg < 0;
        const bool better = feasible && arg >= 0 && q > best;
        const bool next = feasible && arg >= 0 && !better && (!have_second || q > second);
        second = better ? best : next ? q : second;
        have_second = have_second || better || next;
        best = first || better ? q : best;
        arg = first || better ? a : arg;
      };
      const double base = fma(-M.hold, fu, M.r_place[e]);
#pragma unroll
      for (int k = 0; k < T; ++k) {
        const bool room = n[k] + s <= M.C;
        const double A = Al[room ? i + static_cast<uint32_t>(s) * static_cast<uint32_t>(M.stride[k]) : i];
        action(k, room, fma(M.gamma, A + D, base));
      }
#pragma unroll
      for (int h = 0; h < NH; ++h) {
        if (nh[h] + s <= M.C) {
          double A = 0.0;
#pragma unroll
          for (int jj = 0; jj < J; ++jj) A = fma(M.p[jj], static_cast<double>(va[h][jj]), A);
          action(T + h, true, fma(M.gamma, A + D, base));
        }
      }
      action(K, true, fma(M.gamma, Al[i] + D, fma(-M.hold, fu, M.r_reject[e])));
      const uint64_t out = static_cast<uint64_t>(e) * nocc + o0 + i;
      pi[out] = static_cast<uint8_t>(arg);
      if (gap) gap[out] = have_second ? static_cast<float>(best - second) : INFINITY;
    }
  }
}

// The tile of the form: the deepest within the LDS budget that leaves 1,024
// tiles (4 workgroups per CU: K = 7, C = 6 with its 343 tiles of depth 4 took
// 40 us, with the 2,401 of depth 3 33 us), else the shallowest that
// tile_worthwhile takes.  False where none is, or where the values reach
// 2 GiB.  The smallest shape it then takes is no slower than the kernel of
// extract_occupancy (196,608 states: 8.7 against 10.1 us).
template <typename TV>
bool extract_tile_shape(const Model& M, TileShape* S) {
  if (M.K < 4 || M.n_states * static_cast<int64_t>(sizeof(TV)) >= (int64_t{1} << 31)) return false;
  const uint32_t bytes = static_cast<uint32_t>(sizeof(TV)) * M.J + 8;
  bool any = false;
  TileShape t{};
  for (uint32_t limit = kTileLds; tile_shape(M, bytes, limit, &t); limit = t.occ * bytes) {
    if (!tile_worthwhile(t)) continue;
    *S = t;
    any = true;
    if (t.n >= 1024) break;
  }
  return any;
}

template <typename TV>
hipError_t launch_extract_tile_t(const Model& M, const TileShape& S, const TV* V, uint8_t* pi, float* gap,
                                 hipStream_t s) {
  const size_t lds = static_cast<size_t>(S.occ) * (8 + sizeof(TV) * M.J);
  return tile_dispatch(M.K, M.J, S.T, [&](auto kc, auto jc, auto tc) -> hipError_t {
    constexpr int K = decltype(kc)::value, J = decltype(jc)::value, T = decltype(tc)::value;
    if constexpr (K >= 4) {
      hipLaunchKernelGGL((extract_tile_kernel<K, J, T, TV>), dim3(S.n), dim3(kExtractBlock), lds, s, M, S, V, pi, gap);
      return hipGetLastError();
    } else {
      return hipErrorInvalidValue;
    }
  });
}

}  // namespace mdpvi
