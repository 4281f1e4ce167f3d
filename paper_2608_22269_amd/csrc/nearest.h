// Nearest fluid particle of a wall particle (the mirror of Sec. 2.4), by a
// team of lanes.
#pragma once

#include "common.h"

namespace wb {

// Lanes that share a wall particle: kMirrorTeam up to kMirrorTeamRows wall
// particles, where one lane each would leave most of the chip idle and take
// the latency of its 25 rows' loads in turn, else one.  One lane with a row's
// cell starts and records loaded one after the other took 67 us at 23,000 wall
// particles, 112 us at 465,000 and 277 us at 2.05M (FP64, 3D, cells of h to
// 2h); with the loads of 13 rows and of 4 records in flight 50, 65 and 234 us;
// eight lanes 17, 90 and 450 us.
constexpr int kMirrorTeam = 8;
constexpr int64_t kMirrorTeamRows = 131072;

// Index of the fluid particle with the smallest squared distance d2(j) <=
// limit (ties: lower original index fid), -1 if none.  The T lanes of a team
// take every T-th row of the walk; the result is the same in all of them.
template <int DIM, int T, class Real, class Dist>
__device__ __forceinline__ int64_t nearest_fluid(RowWalker &w, const Grid &g, const uint32_t *__restrict__ cs_f,
                                                 const uint32_t *__restrict__ fid, Real limit, Dist d2) {
  constexpr int U = T == 1 ? 13 : 4;  // rows whose cell starts are loaded together
  const int sub = (int)(threadIdx.x & (T - 1));
  uint32_t best = 0xffffffffu, best_id = 0;
  Real best_r2 = limit;
  auto take = [&](uint32_t j, Real r2) {
    if (r2 > best_r2) return;
    const uint32_t id = fid[j];
    if (best == 0xffffffffu || r2 < best_r2 || id < best_id) {
      best = j;
      best_r2 = r2;
      best_id = id;
    }
  };
  auto run = [&](uint32_t lo, uint32_t hi) {
    for (uint32_t j0 = lo; j0 < hi; j0 += 4u) {
      Real r2[4];  // four loads in flight; past the end the last record again
#pragma unroll
      for (uint32_t u = 0; u < 4u; ++u) r2[u] = d2(min(j0 + u, hi - 1u));
#pragma unroll
      for (uint32_t u = 0; u < 4u; ++u) take(min(j0 + u, hi - 1u), r2[u]);
    }
  };
  for (int r0 = sub; r0 < w.nrows; r0 += U * T) {
    uint32_t lo[U], hi[U];
#pragma unroll
    for (int u = 0; u < U; ++u) {
      uint32_t k0 = 0u, k1 = 0u;
      int iy, iz;
      const int r = r0 + u * T;
      const bool ok = r < w.nrows && walker_row<DIM>(w, g, r, k0, k1, iy, iz);
      lo[u] = ok ? cs_f[k0] : 0u;
      hi[u] = ok ? cs_f[k1] : 0u;
    }
#pragma unroll
    for (int u = 0; u < U; ++u) run(lo[u], hi[u]);
  }
#pragma unroll
  for (int o = 1; o < T; o <<= 1) {
    const uint32_t j = __shfl_xor(best, o, 64), id = __shfl_xor(best_id, o, 64);
    const Real r2 = __shfl_xor(best_r2, o, 64);
    if (j != 0xffffffffu && (best == 0xffffffffu || r2 < best_r2 || (r2 == best_r2 && id < best_id))) {
      best = j;
      best_r2 = r2;
      best_id = id;
    }
  }
  return best == 0xffffffffu ? -1 : (int64_t)best;
}

}  // namespace wb
