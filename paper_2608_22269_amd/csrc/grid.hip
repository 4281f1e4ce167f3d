// Neighbour-grid build (Sec. 3): cell index and HashID per particle
// (Eqs. ixyz, hashid), ordering of the particles by HashID, begin/end index
// of every cell, and the reorder of the particle arrays.
//
// The ordering is a counting sort on the dense HashID key -- a radix sort with
// a single digit of log2(ncell) bits: one histogram pass (atomic slot per
// particle), one exclusive scan over the cells (which *is* the begin/end
// table), one scatter.  The scatter order inside a cell depends on atomic
// arrival, so the reorder that follows takes each particle's place in its
// cell from its rank by original index (sorted_place): the final order is
// (HashID, original index), identical to a stable radix sort of the particles
// in original order, and deterministic.
#include <algorithm>

#include "common.h"
#include "kernels.h"
#include "sorted_place.h"

namespace wb {

// ------------------------------------------------------------------ fills

__global__ void k_fill_u32(uint32_t *p, uint32_t v, int64_t n) {
  int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (i < n) p[i] = v;
}

hipError_t launch_fill_u32(uint32_t *p, uint32_t v, int64_t n, hipStream_t s) {
  if (n <= 0) return hipSuccess;
  hipLaunchKernelGGL(k_fill_u32, dim3(grid_for(n)), dim3(kBlock), 0, s, p, v, n);
  return hipGetLastError();
}

// ------------------------------------------------------------------- scan
// Exclusive scan of u32 in three passes: per-tile sums (tile = 1024), a
// single-block scan of the tile sums, a per-tile scan that adds the offset.

static_assert(kScanTile == 1024, "256 threads x 4 items");

size_t scan_tmp_words(int64_t n) { return (size_t)((n + kScanTile - 1) / kScanTile) + 1; }

__device__ __forceinline__ uint32_t block_exclusive_scan(uint32_t v, uint32_t *sh, uint32_t &total) {
  // 256 threads, wave64: inclusive scan inside each wave, then across waves
  const int lane = threadIdx.x & 63, wid = threadIdx.x >> 6;
  uint32_t x = v;
#pragma unroll
  for (int o = 1; o < 64; o <<= 1) {
    uint32_t y = __shfl_up(x, o, 64);
    if (lane >= o) x += y;
  }
  if (lane == 63) sh[wid] = x;
  __syncthreads();
  uint32_t wbase = 0;
  for (int k = 0; k < wid; ++k) wbase += sh[k];
  total = sh[0] + sh[1] + sh[2] + sh[3];
  __syncthreads();
  return wbase + x - v;
}

__global__ void __launch_bounds__(256) k_scan_tiles(const uint32_t *__restrict__ in, uint32_t *__restrict__ sums,
                                                    int64_t n) {
  __shared__ uint32_t sh[4];
  int64_t base = (int64_t)blockIdx.x * kScanTile + threadIdx.x * 4;
  uint32_t v = 0;
#pragma unroll
  for (int k = 0; k < 4; ++k)
    if (base + k < n) v += in[base + k];
  uint32_t tot;
  block_exclusive_scan(v, sh, tot);
  if (threadIdx.x == 0) sums[blockIdx.x] = tot;
}

__global__ void __launch_bounds__(256) k_scan_sums(uint32_t *sums, int64_t m) {
  // exclusive scan of m tile sums in place by one block; sums[m] = total
  __shared__ uint32_t sh[4];
  uint32_t carry = 0;
  for (int64_t base = 0; base < m; base += 256) {
    int64_t i = base + threadIdx.x;
    uint32_t v = i < m ? sums[i] : 0;
    uint32_t tot;
    uint32_t ex = block_exclusive_scan(v, sh, tot);
    if (i < m) sums[i] = carry + ex;
    carry += tot;
  }
  if (threadIdx.x == 0) sums[m] = carry;
}

// CLEAR: the input is zeroed once read (the sort's histogram).  SUMMED: sums
// holds the plain tile sums and every block adds up those before its own
// (at most kFusedTiles: 16 loads a thread), which saves the pass over the
// counts and the one-block pass over the sums.
constexpr int64_t kFusedTiles = 4096;
// Particles up to which the hash also adds up the tiles: few tiles hold them
// all, and beyond, the atomics on those wait for one another longer than a
// pass over the counts takes (660,000 particles: hash 57 us with them, 10 us
// and a pass of 4 us without; 27,000 in raster order 21 us with, 4.6 and 2.9
// without; a step of 17,500 189 us with, 185 without; of 10,153 in 2D 82 with,
// 85 without; of 1,250 86 with, 90 without).
constexpr int64_t kTileAtomics = 12000;

template <bool CLEAR, bool SUMMED>
__global__ void __launch_bounds__(256) k_scan_apply(uint32_t *in, uint32_t *out, const uint32_t *__restrict__ sums,
                                                    int64_t n) {
  __shared__ uint32_t sh[4];
  int64_t base = (int64_t)blockIdx.x * kScanTile + threadIdx.x * 4;
  uint32_t v[4];
#pragma unroll
  for (int k = 0; k < 4; ++k) v[k] = base + k < n ? in[base + k] : 0;
  uint32_t before = 0;
  if (SUMMED) {
    uint32_t t = 0;
    for (unsigned k = threadIdx.x; k < blockIdx.x; k += 256) t += sums[k];
    block_exclusive_scan(t, sh, before);
  } else {
    before = sums[blockIdx.x];
  }
  uint32_t tot;
  uint32_t ex = block_exclusive_scan(v[0] + v[1] + v[2] + v[3], sh, tot) + before;
#pragma unroll
  for (int k = 0; k < 4; ++k) {
    if (base + k < n) {
      out[base + k] = ex;
      if (CLEAR) in[base + k] = 0u;
    }
    ex += v[k];
  }
  if (blockIdx.x == gridDim.x - 1 && threadIdx.x == 0) out[n] = before + tot;  // grand total
}

hipError_t launch_exclusive_scan(const uint32_t *in, uint32_t *out, int64_t n, uint32_t *tmp, hipStream_t s) {
  int64_t tiles = (n + kScanTile - 1) / kScanTile;
  if (tiles < 1) tiles = 1;
  hipLaunchKernelGGL(k_scan_tiles, dim3((unsigned)tiles), dim3(256), 0, s, in, tmp, n);
  hipLaunchKernelGGL(k_scan_sums, dim3(1), dim3(256), 0, s, tmp, tiles);
  hipLaunchKernelGGL((k_scan_apply<false, false>), dim3((unsigned)tiles), dim3(256), 0, s, const_cast<uint32_t *>(in),
                     out, tmp, n);
  return hipGetLastError();
}

int64_t fused_scan_tiles(int64_t nkey) {
  const int64_t tiles = (nkey + kScanTile - 1) / kScanTile;
  return tiles <= kFusedTiles ? tiles : 0;
}

// The begin/end table from the histogram (and its tile sums, if the hash has
// summed them); clears the histogram.
static hipError_t scan_counts(const SortScratch &ss, bool summed, uint32_t *start, int64_t nkey, hipStream_t s) {
  const unsigned tiles = (unsigned)((nkey + kScanTile - 1) / kScanTile);
  if (ss.tiles) {
    if (!summed) hipLaunchKernelGGL(k_scan_tiles, dim3(tiles), dim3(256), 0, s, ss.count, ss.tsum, nkey);
    hipLaunchKernelGGL((k_scan_apply<true, true>), dim3(tiles), dim3(256), 0, s, ss.count, start, ss.tsum, nkey);
  } else {
    hipLaunchKernelGGL(k_scan_tiles, dim3(tiles), dim3(256), 0, s, ss.count, ss.scan_tmp, nkey);
    hipLaunchKernelGGL(k_scan_sums, dim3(1), dim3(256), 0, s, ss.scan_tmp, (int64_t)tiles);
    hipLaunchKernelGGL((k_scan_apply<true, false>), dim3(tiles), dim3(256), 0, s, ss.count, start, ss.scan_tmp, nkey);
  }
  return hipGetLastError();
}

// --------------------------------------------------------- step bookkeeping

// dt = CFL min(dx/(C0 + |U|max), dx^2/(2 nu), sqrt(2 dx/|G|max)) at the start
// of a step (Sec. 2.3); U_max of the stage and the time of its right-hand side
// (stage 1 at t, stage 2 at t + dt); statistics counters restart.  By one wave:
// a lane folds and clears each tally, the first does the rest.
__device__ void run_prep(const Phys &P, const StepPrep &q, Scalars *sc) {
  static_assert(kTallies == 64, "one lane each");
  Tally &tl = sc->tally[threadIdx.x & 63];
  const unsigned long long own = tl.umax2_bits;
  unsigned long long u2 = own, pairs = tl.pairs, tests = tl.tests;
#pragma unroll
  for (int o = 32; o > 0; o >>= 1) {
    const unsigned long long v = __shfl_xor(u2, o, 64);
    u2 = v > u2 ? v : u2;
    pairs += __shfl_xor(pairs, o, 64);
    tests += __shfl_xor(tests, o, 64);
  }
  tl = Tally{q.reset ? 0ull : own, 0ull, 0ull, 0u, 0u, 0u, 0u};
  if (threadIdx.x != 0) return;
  const double umax = sqrt(__longlong_as_double((long long)u2));
  if (q.dt) {
    double dt = P.dx / (P.c0 + umax);
    if (P.nu > 0.0) dt = fmin(dt, P.dx * P.dx / (2.0 * P.nu));
    if (P.gmax > 0.0) dt = fmin(dt, sqrt(2.0 * P.dx / P.gmax));
    dt *= P.cfl;
    sc->dt = q.dt_override > 0.0 ? q.dt_override : dt;
  }
  if (sc->mode == (uint32_t)kPairKept) {  // statistics of the previous right-hand side by kind
    sc->pairs_k = pairs;
    sc->tests_k = tests;
  } else {
    sc->pairs_s = pairs;
    sc->tests_s = tests;
  }
  sc->mode = (uint32_t)q.mode;
  if (q.mode == kPairSearchKeep) {  // this right-hand side builds new kept lists
    sc->disp = 0.0;
    sc->vovf = 0u;
  }
  sc->umax = umax;
  sc->t_rhs = q.stage == 2 ? sc->t + sc->dt : sc->t;
  sc->n_cand = 0;
  sc->n_scan = 0;
}

__global__ void k_prep(Phys P, StepPrep q, Scalars *sc) { run_prep(P, q, sc); }

hipError_t launch_prep(const Phys &P, const StepPrep &prep, Scalars *sc, hipStream_t s) {
  hipLaunchKernelGGL(k_prep, dim3(1), dim3(64), 0, s, P, prep, sc);
  return hipGetLastError();
}

// ------------------------------------------------------------ hash + count

// Slots inside the cells: lanes of a wave with the same key in a contiguous
// run (particles arrive nearly sorted) reserve their slots with one atomic
// add by the run's first lane.  Every lane must call it (valid lanes form a
// prefix of the wave); returns this lane's slot.
__device__ __forceinline__ uint32_t reserve_slot(uint32_t *count, uint32_t k, bool valid) {
  const int lane = (int)(threadIdx.x & 63);
  const uint32_t prev = __shfl_up(k, 1, 64);
  const unsigned long long vmask = __ballot(valid);
  const unsigned long long heads = __ballot(valid && (lane == 0 || prev != k));
  const unsigned long long upto = lane == 63 ? ~0ull : ((2ull << lane) - 1ull);  // bits 0 .. lane
  const int h = 63 - __clzll((long long)(heads & upto));                      // this lane's run head
  uint32_t base = 0;
  if (valid && h == lane) {
    const unsigned long long later = heads & ~upto;
    const int end = later ? __ffsll((long long)later) - 1 : __popcll(vmask);
    base = atomicAdd(&count[k], (uint32_t)(end - lane));
  }
  base = __shfl(base, valid ? h : lane, 64);
  return base + (uint32_t)(lane - h);
}

// Adds the wave's particles to the sums of their tiles of sort keys, one
// atomic per run of lanes in the same tile (as reserve_slot).
__device__ __forceinline__ void add_tile(uint32_t *tsum, uint32_t k, bool valid) {
  const int lane = (int)(threadIdx.x & 63);
  const uint32_t t = k / kScanTile, prev = __shfl_up(t, 1, 64);
  const unsigned long long vmask = __ballot(valid);
  const unsigned long long heads = __ballot(valid && (lane == 0 || prev != t));
  if (!((heads >> lane) & 1ull)) return;
  const unsigned long long later = heads & ~(lane == 63 ? ~0ull : ((2ull << lane) - 1ull));
  const int end = later ? __ffsll((long long)later) - 1 : __popcll(vmask);
  atomicAdd(&tsum[t], (uint32_t)(end - lane));
}

// Cell of particle i, Eq. (ixyz), its sort key (the cell in the storage
// order of cell_key), plus its slot inside the cell (arrival order).
// Out-of-domain or non-finite positions set an error bit and are parked in
// cell 0 so that every later index stays valid.
template <int DIM>
__global__ void __launch_bounds__(256) k_hash_f64(Grid g, const double *__restrict__ x,
                                                  const double *__restrict__ y, const double *__restrict__ z,
                                                  int64_t n, uint32_t *__restrict__ key, uint32_t *__restrict__ slot,
                                                  uint32_t *__restrict__ count, uint32_t *__restrict__ tsum,
                                                  Scalars *sc, Phys P, StepPrep prep) {
  const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (prep.on && i < 64) run_prep(P, prep, sc);  // nothing else here touches these scalars
  const bool valid = i < n;
  double p[3] = {0.0, 0.0, 0.0};
  if (valid) {
    p[0] = x[i];
    p[1] = y[i];
    if (DIM == 3) p[2] = z[i];
  }
  int c[3] = {0, 0, 0};
  bool bad = !valid;
#pragma unroll
  for (int a = 0; a < DIM; ++a) {
    if (!valid) {
    } else if (!isfinite(p[a])) {
      atomicOr(&sc->err, kErrNonFinite);
      bad = true;
    } else if (p[a] < g.lo[a] || p[a] > g.hi[a]) {
      atomicOr(&sc->err, kErrDomain);
      bad = true;
    } else {
      c[a] = cell_coord(p[a], g.lo[a], g.R);
      if (c[a] < 0 || c[a] >= g.N[a]) {
        atomicOr(&sc->err, kErrDomain);
        bad = true;
      }
    }
  }
  uint32_t k = 0;
  if (valid && !bad) k = cell_key(g, c[0], c[1], c[2]);
  const uint32_t sl = reserve_slot(count, k, valid);
  if (tsum) add_tile(tsum, k, valid);
  if (valid) {
    key[i] = k;
    slot[i] = sl;
  }
}

// Mixed path: the cell is stored; the key is computed from it directly.
__global__ void __launch_bounds__(256) k_hash_packed(Grid g, const uint32_t *__restrict__ cell, int64_t n,
                                                     uint32_t *__restrict__ key, uint32_t *__restrict__ slot,
                                                     uint32_t *__restrict__ count, uint32_t *__restrict__ tsum,
                                                     Scalars *sc, Phys P, StepPrep prep) {
  const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (prep.on && i < 64) run_prep(P, prep, sc);
  const bool valid = i < n;
  const uint32_t c = valid ? cell[i] : 0u;
  const int cx = c & 2047u, cy = (c >> 11) & 2047u, cz = c >> 22;
  uint32_t k = 0;
  if (valid && (cx >= g.N[0] || cy >= g.N[1] || cz >= g.N[2])) {
    atomicOr(&sc->err, kErrDomain);
  } else if (valid) {
    k = cell_key(g, cx, cy, cz);
  }
  const uint32_t sl = reserve_slot(count, k, valid);
  if (tsum) add_tile(tsum, k, valid);
  if (valid) {
    key[i] = k;
    slot[i] = sl;
  }
}

// Arrival order of the sorted particles, with their original indices; clears
// the tile sums for the next sort.
__global__ void __launch_bounds__(256) k_scatter(const uint32_t *__restrict__ key, const uint32_t *__restrict__ slot,
                                                 const uint32_t *__restrict__ start, const uint32_t *__restrict__ id,
                                                 int64_t n, uint2 *__restrict__ perm, uint32_t *__restrict__ tsum,
                                                 int64_t tiles) {
  int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (i < tiles) tsum[i] = 0u;
  if (i >= n) return;
  perm[start[key[i]] + slot[i]] = make_uint2((uint32_t)i, id[i]);
}

hipError_t launch_sort_keys(const Grid &g, int dim, const double *x, const double *y, const double *z,
                            const uint32_t *packed_cell, int64_t n, const uint32_t *id, SortScratch &ss,
                            uint32_t *start, uint2 *perm, Scalars *sc, hipStream_t s, const Phys *P,
                            const StepPrep *prep) {
  const StepPrep q = prep && P ? *prep : StepPrep{};
  const Phys ph = P ? *P : Phys{};
  uint32_t *tsum = ss.tiles && n <= kTileAtomics ? ss.tsum : nullptr;
  if (n > 0) {
    if (packed_cell)
      hipLaunchKernelGGL(k_hash_packed, dim3(grid_for(n)), dim3(kBlock), 0, s, g, packed_cell, n, ss.key, ss.slot,
                         ss.count, tsum, sc, ph, q);
    else if (dim == 2)
      hipLaunchKernelGGL(k_hash_f64<2>, dim3(grid_for(n)), dim3(kBlock), 0, s, g, x, y, z, n, ss.key, ss.slot,
                         ss.count, tsum, sc, ph, q);
    else
      hipLaunchKernelGGL(k_hash_f64<3>, dim3(grid_for(n)), dim3(kBlock), 0, s, g, x, y, z, n, ss.key, ss.slot,
                         ss.count, tsum, sc, ph, q);
  }
  hipError_t e = n <= 0 && q.on ? launch_prep(ph, q, sc, s) : hipSuccess;
  if (e == hipSuccess) e = scan_counts(ss, tsum != nullptr, start, g.nkey, s);
  if (e != hipSuccess) return e;
  if (n > 0)
    hipLaunchKernelGGL(k_scatter, dim3(grid_for(std::max(n, ss.tiles))), dim3(kBlock), 0, s, ss.key, ss.slot, start, id,
                       n, perm, ss.tsum, ss.tiles);
  return hipGetLastError();
}

// ----------------------------------------------------------------- reorder

// Gathers the FP64 fluid state into sorted order (src -> dst) and writes the
// neighbour-facing records rec0 = (x, y, z, phi), rec1 = (u, v, w, V) with
// V = m / (rho0 exp(phi / C0^2)).  with_stage0 also carries the stage-0
// copies (second stage of SSP-RK2).
template <int DIM>
__global__ void __launch_bounds__(256) k_reorder_f64(Phys P, SortScratch ss, const uint32_t *__restrict__ start,
                                                     const uint2 *__restrict__ perm, int64_t n, FluidF64 src,
                                                     FluidF64 dst, double4 *__restrict__ rec0,
                                                     double4 *__restrict__ rec1, int with_stage0) {
  const int64_t t = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (t >= n) return;
  const uint2 from = perm[t];
  const uint32_t o = from.x;
  // every load before the first store (the compiler must take the arrays for
  // one another's, and waited for each axis in turn: 46.6 us before, 38.7 so,
  // at 660,000 particles)
  double xs[3] = {0.0, 0.0, 0.0}, us[3] = {0.0, 0.0, 0.0}, x0[DIM], u0[DIM], ph0 = 0.0;
#pragma unroll
  for (int a = 0; a < DIM; ++a) {
    xs[a] = src.x[a][o];
    us[a] = src.u[a][o];
  }
  const double ph = src.phi[o], m = src.m[o];
  if (with_stage0) {
#pragma unroll
    for (int a = 0; a < DIM; ++a) {
      x0[a] = src.x0[a][o];
      u0[a] = src.u0[a][o];
    }
    ph0 = src.phi0[o];
  }
  const uint32_t k = sorted_place(ss.key, start, perm, (uint32_t)t, from);
#pragma unroll
  for (int a = 0; a < DIM; ++a) {
    dst.x[a][k] = xs[a];
    dst.u[a][k] = us[a];
  }
  dst.phi[k] = ph;
  dst.m[k] = m;
  dst.id[k] = from.y;
  if (with_stage0) {
#pragma unroll
    for (int a = 0; a < DIM; ++a) {
      dst.x0[a][k] = x0[a];
      dst.u0[a][k] = u0[a];
    }
    dst.phi0[k] = ph0;
  }
  double V = m / (P.rho0 * exp(ph * P.inv_c02));
  rec0[k] = make_double4(xs[0], xs[1], xs[2], ph);
  rec1[k] = make_double4(us[0], us[1], us[2], V);
}

hipError_t launch_reorder_f64(const Phys &P, const SortScratch &ss, const uint32_t *start, const uint2 *perm,
                              int64_t n, const FluidF64 &src, const FluidF64 &dst, double4 *rec0, double4 *rec1,
                              int with_stage0, hipStream_t s) {
  if (n <= 0) return hipSuccess;
  if (P.dim == 2)
    hipLaunchKernelGGL(k_reorder_f64<2>, dim3(grid_for(n)), dim3(kBlock), 0, s, P, ss, start, perm, n, src, dst, rec0,
                       rec1, with_stage0);
  else
    hipLaunchKernelGGL(k_reorder_f64<3>, dim3(grid_for(n)), dim3(kBlock), 0, s, P, ss, start, perm, n, src, dst, rec0,
                       rec1, with_stage0);
  return hipGetLastError();
}

// Neighbour-facing records of the FP64 state in its current order, without a
// sort (second stage of a step that keeps the first stage's candidates).
template <int DIM>
__global__ void __launch_bounds__(256) k_refresh_f64(Phys P, FluidF64 f, int64_t n, double4 *__restrict__ rec0,
                                                     double4 *__restrict__ rec1) {
  int64_t k = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (k >= n) return;
  const double x = f.x[0][k], y = f.x[1][k], z = DIM == 3 ? f.x[2][k] : 0.0;
  const double u = f.u[0][k], v = f.u[1][k], w = DIM == 3 ? f.u[2][k] : 0.0;
  const double ph = f.phi[k];
  const double V = f.m[k] / (P.rho0 * exp(ph * P.inv_c02));
  rec0[k] = make_double4(x, y, z, ph);
  rec1[k] = make_double4(u, v, w, V);
}

hipError_t launch_refresh_f64(const Phys &P, const FluidF64 &f, int64_t n, double4 *rec0, double4 *rec1,
                              hipStream_t s) {
  if (n <= 0) return hipSuccess;
  if (P.dim == 2)
    hipLaunchKernelGGL(k_refresh_f64<2>, dim3(grid_for(n)), dim3(kBlock), 0, s, P, f, n, rec0, rec1);
  else
    hipLaunchKernelGGL(k_refresh_f64<3>, dim3(grid_for(n)), dim3(kBlock), 0, s, P, f, n, rec0, rec1);
  return hipGetLastError();
}

}  // namespace wb
