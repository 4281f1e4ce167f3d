// Nearest fluid particle of a wall particle (the mirror of Sec. 2.4), by a
// team of lanes.
#pragma once

#include <type_traits>

#include "common.h"

namespace wb {

// Lanes that share a wall particle: kMirrorTeam up to kMirrorTeamRows wall
// particles (kMirrorTeamRowsMixed with FP32 positions), where one lane each
// would leave most of the chip idle and take the latency of its rows' loads in
// turn, else one.  FP64, 3D, us, a lane / eight lanes: 29 / 22 at 55,000 wall
// particles, 32 / 37 at 121,000, 53 / 116 at 465,000; mixed 31 / 26 at 121,000,
// 34 / 38 at 200,000.  Every row's records one after the other took 67 us at
// 23,000 (eight lanes 15), 112 at 465,000 and 277 at 2.05M (a lane 175).
constexpr int kMirrorTeam = 8;
constexpr int64_t kMirrorTeamRows = 90000, kMirrorTeamRowsMixed = 150000;

// Index of the fluid particle with the smallest squared distance d2(j) <=
// limit (ties: lower original index fid), -1 if none.  The own row and those
// around it come first, then the rows ring by ring, once a particle is found
// only as far as that one lies (extra: what the cells may be off by and, where
// d2 is from FP32 positions, what those are rounded by, in metres): of some
// 190 particles within reach a few dozen are looked at.  The T lanes of a team
// get the same result.  The whole wave calls it.
template <int DIM, int T, class Real, class Dist>
__device__ __forceinline__ int64_t nearest_fluid(RowWalker &w, const Grid &g, const uint32_t *__restrict__ cs_f,
                                                 const uint32_t *__restrict__ fid, Real limit, double extra, Dist d2) {
  const int sub = (int)(threadIdx.x & (T - 1));
  uint32_t best = 0xffffffffu, best_id = 0;
  Real best_r2 = limit;
  auto take = [&](uint32_t j, Real r2) {
    if (!(r2 <= best_r2)) return;  // nor a particle at NaN
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
  // a particle no farther than the best one lies in no row or cell beyond
  // it, widened by extra and by 0.002 cells for the rounding here
  auto shrink = [&]() {
    if (best == 0xffffffffu) return;
    const float r = sqrtf((float)best_r2) * (float)g.invR + (float)(extra * g.invR) + 0.002f;
    w.rr2 = fminf(w.rr2, r * r * (1.0f + 4.0f * kWalkSlack));
  };
  if constexpr (T == 1) {
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
  // A team: a lane computes a row's window, and the team tests each row's
  // records side by side, the first eight of all rows in flight at once.
  auto team_best = [&]() {
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
    shrink();
  };
  auto window = [&](int dy, int dz, bool on, uint32_t &lo, uint32_t &hi) {
    uint32_t k0 = 0u, k1 = 0u;
    int iy, iz;
    float dist;
    const bool ok = on && walker_row_at<DIM>(w, g, dy, dz, k0, k1, iy, iz, dist);
    lo = ok ? cs_f[k0] : 0u;
    hi = ok ? cs_f[k1] : 0u;
  };
  // rows 0 .. N - 1 (N <= 9) of the windows lo, hi; row 8 is lane 0's lo8, hi8
  auto test = [&](auto count, uint32_t lo, uint32_t hi, uint32_t lo8, uint32_t hi8) {
    constexpr int N = decltype(count)::value;
    uint32_t j[N], end[N];
#pragma unroll
    for (int q = 0; q < N; ++q) {
      j[q] = __shfl(q < 8 ? lo : lo8, q < 8 ? q : 0, T) + (uint32_t)sub;
      end[q] = __shfl(q < 8 ? hi : hi8, q < 8 ? q : 0, T);
    }
    for (;;) {
      bool any = false;
#pragma unroll
      for (int q = 0; q < N; ++q) any |= j[q] < end[q];
      if (__ballot(any) == 0ull) break;
      Real r2[N];
#pragma unroll
      for (int q = 0; q < N; ++q) r2[q] = d2(j[q] < end[q] ? j[q] : 0u);
#pragma unroll
      for (int q = 0; q < N; ++q) {
        if (j[q] < end[q]) take(j[q], r2[q]);
        j[q] += T;
      }
      __builtin_amdgcn_wave_barrier();
    }
  };
  uint32_t lo, hi, lo8 = 0u, hi8 = 0u;
  {  // own row and those around it
    const int q = sub < 4 ? sub : sub + 1;  // 0 .. 8 in raster order without the middle
    if (DIM == 3) window(q % 3 - 1, q / 3 - 1, true, lo, hi);
    else window(sub - 1, 0, sub < 3, lo, hi);
    __builtin_amdgcn_wave_barrier();
    if (DIM == 3) {
      window(0, 0, sub == 0, lo8, hi8);
      __builtin_amdgcn_wave_barrier();
    }
    test(std::integral_constant<int, DIM == 3 ? 9 : 3>{}, lo, hi, lo8, hi8);
    team_best();
  }
  for (int d = 2; d <= g.reach; ++d) {  // then ring by ring, eight rows at a time
    for (int t = -d; t < d; t += DIM == 3 ? 2 : 2 * d) {
      if (DIM == 3) {
        const int side = sub / 2, at = t + sub % 2;
        window(side == 0 ? at : side == 1 ? d : side == 2 ? -at : -d,
               side == 0 ? -d : side == 1 ? at : side == 2 ? d : -at, true, lo, hi);
      } else {
        window(sub == 0 ? -d : d, 0, sub < 2, lo, hi);
      }
      __builtin_amdgcn_wave_barrier();
      if (__ballot(lo < hi) == 0ull) continue;
      test(std::integral_constant<int, DIM == 3 ? 8 : 2>{}, lo, hi, 0u, 0u);
      team_best();
    }
  }
  return best == 0xffffffffu ? -1 : (int64_t)best;
}

}  // namespace wb
