// Nearest fluid particle of a wall particle (the mirror of Sec. 2.4), by a
// team of lanes.
#pragma once

#include <type_traits>

#include "common.h"

namespace wb {

// Lanes that share a wall particle: kMirrorTeam up to kMirrorTeamRows wall
// particles, where one lane each would leave most of the chip idle and take
// the latency of its rows' loads in turn, else one.  One lane with a row's
// cell starts and records loaded one after the other took 67 us at 23,000 wall
// particles, 112 us at 465,000 and 277 us at 2.05M (FP64, 3D, cells of h to
// 2h); with the loads of 13 rows and of 4 records in flight 50, 65 and 234 us;
// visiting the near rows first and no farther than the particle found 53 and
// 175 us at the last two; eight lanes 17, 90 and 450 us.
constexpr int kMirrorTeam = 8;
constexpr int64_t kMirrorTeamRows = 131072;

// Index of the fluid particle with the smallest squared distance d2(j) <=
// limit (ties: lower original index fid), -1 if none.  A lane alone visits the
// rows in rings about its own and, once it has found a particle, only as far
// as that one lies (extra: what the cells may be off by, in metres): of some
// 190 particles within reach it looks at a few dozen.  The lanes of a team take
// every T-th row of the walk, all at once; the result is the same in all of
// them.
template <int DIM, int T, class Real, class Dist>
__device__ __forceinline__ int64_t nearest_fluid(RowWalker &w, const Grid &g, const uint32_t *__restrict__ cs_f,
                                                 const uint32_t *__restrict__ fid, Real limit, double extra, Dist d2) {
  constexpr int U = 4;  // rows whose cell starts a team's lane loads together
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
  if constexpr (T == 1) {
    // a particle no farther than the best one lies in no row or cell beyond
    // it, widened by extra and by 0.002 cells for positions in FP32
    auto shrink = [&]() {
      if (best == 0xffffffffu) return;
      const float r = sqrtf((float)best_r2) * (float)g.invR + (float)(extra * g.invR) + 0.002f;
      w.rr2 = fminf(w.rr2, r * r * (1.0f + 4.0f * kWalkSlack));
    };
    // N rows' cell starts in flight, the rows in the order given
    auto rows = [&](auto count, auto at) {
      constexpr int N = decltype(count)::value;
      uint32_t lo[N], hi[N];
      float dist[N];
#pragma unroll
      for (int u = 0; u < N; ++u) {
        uint32_t k0 = 0u, k1 = 0u;
        int iy, iz, dy, dz;
        at(u, dy, dz);
        dist[u] = 0.0f;
        const bool ok = walker_row_at<DIM>(w, g, dy, dz, k0, k1, iy, iz, dist[u]);
        lo[u] = ok ? cs_f[k0] : 0u;
        hi[u] = ok ? cs_f[k1] : 0u;
      }
#pragma unroll
      for (int u = 0; u < N; ++u) {
        if (dist[u] > w.rr2) continue;
        run(lo[u], hi[u]);
        shrink();
      }
    };
    // own row and the four beside it, then the corners
    auto near = [&](int first, int u, int &dy, int &dz) {
      constexpr int y[9] = {0, -1, 1, 0, 0, -1, 1, -1, 1}, z[9] = {0, 0, 0, -1, 1, -1, -1, 1, 1};
      dy = y[first + u];
      dz = z[first + u];
    };
    if constexpr (DIM == 3) {
      rows(std::integral_constant<int, 5>{}, [&](int u, int &dy, int &dz) { near(0, u, dy, dz); });
      rows(std::integral_constant<int, 4>{}, [&](int u, int &dy, int &dz) { near(5, u, dy, dz); });
    } else {
      rows(std::integral_constant<int, 3>{}, [&](int u, int &dy, int &dz) { near(0, u, dy, dz); });
    }
    for (int d = 2; d <= g.reach; ++d) {  // then ring by ring: place t on each of its four sides
      if (DIM == 2) {
        rows(std::integral_constant<int, 2>{}, [&](int u, int &dy, int &dz) {
          dy = u ? d : -d;
          dz = 0;
        });
      } else {
        for (int t = -d; t < d; ++t) {
          rows(std::integral_constant<int, 4>{}, [&](int q, int &dy, int &dz) {
            dy = q == 0 ? t : q == 1 ? d : q == 2 ? -t : -d;
            dz = q == 0 ? -d : q == 1 ? t : q == 2 ? d : -t;
          });
        }
      }
    }
    return best == 0xffffffffu ? -1 : (int64_t)best;
  }
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
