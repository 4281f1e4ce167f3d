// Particle interaction stage, FP64 path (Sec. 2 and Sec. 3):
//   - dummy-wall mirror (Sec. 2.4, Eq. phiBn and the slip velocity);
//   - the fused pair pass: every sum of Eq. (sph) in one neighbour pass --
//     L (Eq. renorm), the Riemann sum of Eqs. (parGrad)/(lfsover) kept on the
//     right of L^T (the correction moved out of the sum, Sec. 3), the
//     conservative sum (TIC), the velocity-gradient tensor of the continuity
//     equation, the delta-SPH sum and the shifting sum -- followed by an
//     epilogue with the closed-form eigenvalues, the small solves and the
//     free-surface pre-classification;
//   - the scan-region pass over free-surface candidates;
//   - neighbour-list export for parity checks.
//
// Work mapping.  Up to some counts a team of 8 lanes per fluid particle
// (k_pair_team_f64, by_team); beyond them one lane each, particles in storage
// (sort key) order.  The wave walks the cell rows of Algorithm 1 in lockstep; each lane
// compacts its in-range candidates into its own column of an LDS list (32
// entries), and whenever a list may overflow the wave runs the dense pair body
// over the lists.  Lanes of one wave belong to the same or neighbouring cells,
// so their candidate loads touch the same records, and the expensive body runs
// on real neighbours only instead of every candidate of the 3^d cells.
#include "common.h"
#include "kernels.h"
#include "pair_common.h"
#include "coop.h"
#include "nearest.h"

namespace wb {

// Compile-time tuning of the pair pass (values chosen by measurement on the
// 17.5M-particle sloshing tank; they change speed, never results).
#ifndef WB_PAIR_BATCH
#define WB_PAIR_BATCH 4
#endif
#ifndef WB_PAIR_UNROLL
#define WB_PAIR_UNROLL 1
#endif
// waves per SIMD the register allocation targets (4 measured fastest)
#ifndef WB_PAIR_WAVES
#define WB_PAIR_WAVES 4
#endif
// waves per SIMD of the pass from kept lists (2, 3 and 4 measured equal: its
// record gathers bound it, not latency)
#ifndef WB_KEPT_WAVES
#define WB_KEPT_WAVES 4
#endif
constexpr int kList = kPairList;       // LDS list entries per lane
constexpr int kBatch = WB_PAIR_BATCH;  // candidates fetched per search iteration
static_assert(kBatch <= kRecPad, "batched candidate loads run at most kRecPad records past a run");
#define WB_PAIR_ATTR __attribute__((amdgpu_waves_per_eu(WB_PAIR_WAVES)))

// ------------------------------------------------------------------ mirror

template <int DIM, int T>
__global__ void __launch_bounds__(256) k_mirror_f64(Phys P, Grid g, Dummies d, int64_t nd,
                                                    const double4 *__restrict__ rec0,
                                                    const double4 *__restrict__ rec1, double4 *__restrict__ drec0,
                                                    double4 *__restrict__ drec1, const uint32_t *__restrict__ cs_f,
                                                    uint32_t nf, const Scalars *__restrict__ sc,
                                                    const uint32_t *__restrict__ fid) {
  // the nearest particles by teams of lanes, then one lane per wall particle
  constexpr int kRows = kBlock / T;
  __shared__ int64_t found[kRows];
  const int64_t first = (int64_t)blockIdx.x * kRows;
  {
    const int row = (int)threadIdx.x / T;
    const int64_t k = min(first + row, nd - 1);
    const double xd = d.x[0][k], yd = d.x[1][k], zd = DIM == 3 ? d.x[2][k] : 0.0;
    RowWalker w;
    walker_init<DIM>(w, g, xd, yd, zd, P.win);
    const int64_t j = nearest_fluid<DIM, T>(w, g, cs_f, fid, P.two_h2, P.win - P.two_h, [&](uint32_t q) {
      const double4 b = rec0[q];
      return dist2_exact<DIM>(b.x - xd, b.y - yd, b.z - zd);
    });
    if ((threadIdx.x & (T - 1)) == 0) found[row] = j;
  }
  __syncthreads();
  const int64_t k = first + threadIdx.x;
  if (threadIdx.x >= kRows || k >= nd) return;
  const int64_t best = found[threadIdx.x];
  const double xd = d.x[0][k], yd = d.x[1][k], zd = DIM == 3 ? d.x[2][k] : 0.0;
  d.src[k] = (int32_t)best;
  if (best < 0) {
    drec0[k] = make_double4(xd, yd, zd, d.phi_in[k]);
    drec1[k] = make_double4(0.0, 0.0, 0.0, 0.0);  // inactive: in no fluid's support
    return;
  }
  double G[3];
  body_force(P, sc->t_rhs, G);
  double4 f0 = rec0[best], f1 = rec1[best];
  // phi_d = phi_f + G.(x_d - x_f)        (Eq. phiBn)
  double gp = G[0] * (xd - f0.x) + G[1] * (yd - f0.y);
  if (DIM == 3) gp += G[2] * (zd - f0.z);
  double phid = f0.w + gp;
  // slip: U_d = U_f - (U_f . n_d) n_d; for the moving body relative to its
  // velocity Uw, U_d = U_f - ((U_f - Uw) . n_d) n_d (the dummy keeps the
  // wall's normal velocity)
  double nx = d.n[0][k], ny = d.n[1][k], nz = DIM == 3 ? d.n[2][k] : 0.0;
  double un;
  if (d.mov != nullptr && d.mov[k]) {
    double Uw[3] = {sc->body_u[0], sc->body_u[1], sc->body_u[2]};
    if (sc->fb_on) {
      // free body: v + omega x R (x0 - c0) at this dummy
      double q[4] = {sc->fb[3], sc->fb[4], sc->fb[5], sc->fb[6]}, R[9];
      quat_rotation(q, R);
      const double d0[3] = {d.x0[0][k] - sc->fb_c0[0], d.x0[1][k] - sc->fb_c0[1],
                            DIM == 3 ? d.x0[2][k] - sc->fb_c0[2] : 0.0};
      double dr[3];
      mat3_apply(R, d0, dr);
      free_body_point_velocity(sc->fb, dr, Uw);
    }
    un = (f1.x - Uw[0]) * nx + (f1.y - Uw[1]) * ny;
    if (DIM == 3) un += (f1.z - Uw[2]) * nz;
  } else {
    un = f1.x * nx + f1.y * ny + f1.z * nz;
  }
  double V = d.m[k] / (P.rho0 * exp(phid * P.inv_c02));
  drec0[k] = make_double4(xd, yd, zd, phid);
  drec1[k] = make_double4(f1.x - un * nx, f1.y - un * ny, DIM == 3 ? f1.z - un * nz : 0.0, V);
}

// ----------------------------------------------------------- pair pass

// Dense pair body: every sum of Eq. (sph) for neighbour j (records b0, b1) of
// particle i (records a0, a1).  PST4: the shifting exponent is 4 (the paper's
// value), evaluated as two squarings; otherwise pow().
template <int DIM, bool PST4>
__device__ __forceinline__ void pair_body_f64(const Phys &P, const double4 &a0, const double4 &a1, const double4 &b0,
                                              const double4 &b1, PairSums &S) {
  const double rx = b0.x - a0.x, ry = b0.y - a0.y, rz = DIM == 3 ? b0.z - a0.z : 0.0;
  // membership was decided by the exact test; here |r| only feeds W and K
  const double r2 = DIM == 3 ? fma(rx, rx, fma(ry, ry, rz * rz)) : fma(rx, rx, ry * ry);
  S.coincident |= (r2 == 0.0);
  const double is = rsqrt_pos(r2);
  const double s = r2 * is;
  const double t = fma(s, P.m_half_inv_h, 1.0);  // 1 - q/2
  const double t2 = t * t, t3 = t2 * t;
  const double wv = P.kfac * t3 * b1.w;  // |grad W| / |r| times V_j
  const double gx = wv * rx, gy = wv * ry, gz = wv * rz;
  // S.L = sum r (x) grad W V  (symmetric for the radial kernel)
  S.L[0] += rx * gx;
  S.L[1] += ry * gy;
  S.L[3] += rx * gy;
  if (DIM == 3) {
    S.L[2] += rz * gz;
    S.L[4] += rx * gz;
    S.L[5] += ry * gz;
  }
  S.gs[0] += gx;
  S.gs[1] += gy;
  if (DIM == 3) S.gs[2] += gz;
  const double dph = b0.w - a0.w;
  const double dux = b1.x - a1.x, duy = b1.y - a1.y, duz = DIM == 3 ? b1.z - a1.z : 0.0;
  const double dun = (dux * rx + duy * ry + duz * rz) * is;
  const double c2 = dph - P.c0 * dun;  // 2 (phi*_ij - phi_i)
  const double cs = b0.w + a0.w;        // conservative form
  S.SR[0] += c2 * gx;
  S.SR[1] += c2 * gy;
  S.SC[0] += cs * gx;
  S.SC[1] += cs * gy;
  if (DIM == 3) {
    S.SR[2] += c2 * gz;
    S.SC[2] += cs * gz;
  }
  // symmetric part of N_ab = sum (U_j - U_i)_a (grad W V)_b: S.L^-1 is
  // symmetric, so tr(S.L^-1 S.N) only sees S.N + S.N^T (packed xx yy zz xy xz yz,
  // off-diagonals hold N_ab + N_ba)
  S.N[0] += dux * gx;
  S.N[1] += duy * gy;
  S.N[3] += dux * gy + duy * gx;
  if (DIM == 3) {
    S.N[2] += duz * gz;
    S.N[4] += dux * gz + duz * gx;
    S.N[5] += duy * gz + duz * gy;
  }
  S.Ds += wv * dph;  // Phi_ij . grad W V = 2 K (phi_j - phi_i) V_j (factor 2 in the epilogue)
  // shifting: sum (W / W(dx))^n grad W V; the epilogue adds sum grad W V
  // times 1 / R, i.e. P = sum [1 + R (W / W(dx))^n] grad W V
  const double u = fma(s, P.two_inv_h, 1.0);  // 2q + 1
  const double t4u = (t2 * t2) * u;
  const double wr = P.aw0 * t4u;
  const double wrn = PST4 ? (wr * wr) * (wr * wr) : pow(wr, P.pst_n);
  S.Ps[0] += wrn * gx;
  S.Ps[1] += wrn * gy;
  if (DIM == 3) S.Ps[2] += wrn * gz;
}

// The pair pass with its own candidate search (Algorithm 1).  KEEP (the
// right-hand side that builds kept lists): the search radius grows to
// 2h + skin (P.skin_max), candidates beyond 2h enter the LDS list tagged and
// are skipped by the body, and every non-empty list fill is also copied to kl
// for the later right-hand sides; a lane with more than kKeepChunks fills
// raises sc->vovf.
template <int DIM, bool PST4, bool KEEP>
__global__ void __launch_bounds__(kSearchBlock) WB_PAIR_ATTR
    k_pair_f64(Phys P, Grid g, const double4 *__restrict__ rec0, const double4 *__restrict__ rec1,
               const uint32_t *__restrict__ cs_f, const uint32_t *__restrict__ cs_d, uint32_t nf, Scalars *sc,
               Rates out, uint32_t *__restrict__ cand, KeptLists kl) {
  __shared__ uint32_t list[kList][kSearchBlock];
  const int tid = threadIdx.x;
  const uint32_t i = xcd_block(blockIdx.x, gridDim.x) * kSearchBlock + tid;
  const bool active = i < nf;

  double4 a0 = make_double4(0.0, 0.0, 0.0, 0.0), a1 = a0;
  if (active) {
    a0 = rec0[i];
    a1 = rec1[i];
  }
  PairSums S;
  sums_zero(S);
  // the kept-list work behind a run-time test (launches in this mode always
  // have a skin): compiled unconditionally it costs spilled registers
  const bool keep = KEEP && P.skin_max > 0.0;
  const double rho = keep ? P.two_h + P.skin_max : P.two_h;
  const double rho2 = keep ? rho * rho : P.two_h2;
  // this lane's kept-list bookkeeping in LDS (packed chunk counts, chunks
  // so far at bit kKeptNchShift, saturating at 15): touched once per fill,
  // it holds no registers through the search
  __shared__ unsigned long long kbook[KEEP ? kSearchBlock : 1];
  if (KEEP) kbook[tid] = 0ull;

  // consume the first cnt entries of this lane's list
  auto run_list = [&](int cnt) {
    if (keep) {  // copy the fill for the later right-hand sides
      const int kmax = wave_max_int(cnt);
      unsigned long long book = kbook[tid];
      const int chunk = (int)(book >> kKeptNchShift);
      const bool room = chunk < kKeepChunks;
      uint32_t *dst = kl.ent + kept_entry(i, min(chunk, kKeepChunks - 1), 0);
      // eight LDS reads in flight before their stores (read per entry, the
      // copy waited out the LDS latency once per entry)
      for (int k0 = 0; k0 < kmax; k0 += 8) {
        uint32_t e[8];
#pragma unroll
        for (int u = 0; u < 8; ++u) e[u] = list[min(k0 + u, kList - 1)][tid];
#pragma unroll
        for (int u = 0; u < 8; ++u)
          if (room && k0 + u < cnt) dst[(size_t)(k0 + u) * 64u] = e[u];
      }
      if (cnt > 0) {
        if (room) book |= (unsigned long long)cnt << (6 * chunk);
        else sc->vovf = 1u;
        book = (book & ((1ull << kKeptNchShift) - 1ull)) | ((unsigned long long)min(chunk + 1, 15) << kKeptNchShift);
        kbook[tid] = book;
      }
    }
    // one neighbour per iteration, the next list entry read one iteration ahead
    uint32_t en = cnt > 0 ? list[0][tid] : 0u;
    for (int k = 0; k < cnt; ++k) {
      const uint32_t e = en;
      const uint32_t j = KEEP ? e & ~kSkinTag : e;
      const double4 b0 = rec0[j], b1 = rec1[j];
      if (k + 1 < cnt) en = list[k + 1][tid];
      if (!KEEP || !(e & kSkinTag)) {
        pair_body_f64<DIM, PST4>(P, a0, a1, b0, b1, S);
        if (KEEP) S.nnb += 1;
      }
    }
    if (!KEEP) S.nnb += cnt;
  };

  // candidate search with the rows walked in lockstep by the wave
  const CellPos cp = cellpos_of<DIM>(g, a0.x, a0.y, a0.z);
  int cnt = 0;
  auto load = [&](uint32_t j) { return rec0[j]; };
  auto near = [&](const double4 &b, uint32_t j) -> uint32_t {
    const double r2 = dist2_exact<DIM>(b.x - a0.x, b.y - a0.y, DIM == 3 ? b.z - a0.z : 0.0);
    if (!KEEP) return j != i && r2 <= P.two_h2 ? 1u : 0u;
    return j != i && r2 <= rho2 ? (r2 <= P.two_h2 ? 1u : 2u) : 0u;
  };
  CoopWalk cw;
  coop_init(cw, g, active, (float)rho, DIM);
  for (;;) {
    const bool fin = coop_fill<DIM, kList, kBatch>(cw, g, cs_f, cs_d, nf, cp, &list[0][tid], kSearchBlock, cnt, S.ntest,
                                                   load, near);
    run_list(cnt);
    cnt = 0;
    if (fin) break;
  }
  if (keep) {
    const unsigned long long book = kbook[tid];
    const int nch = min((int)(book >> kKeptNchShift), kKeepChunks);
    kl.cnt[i] = (book & ((1ull << kKeptNchShift) - 1ull)) | ((unsigned long long)nch << kKeptNchShift);
  }

  pair_epilogue<DIM>(P, sc, out, cand, i, active, S);
}

// A right-hand side from kept candidates (no search): the records hold the
// current state in the order of the build, every kept candidate is tested
// exactly against 2h and the neighbours run the same body.  The caller uses
// the lists only while twice the bound on any particle's move since the build
// fits the skin: a pair within 2h now was within 2h + skin then, so the
// neighbour sets are those of a fresh search.
template <int DIM, bool PST4>
__global__ void __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(WB_KEPT_WAVES)))
    k_pair_kept_f64(Phys P, const double4 *__restrict__ rec0, const double4 *__restrict__ rec1, uint32_t nf,
                    Scalars *sc, Rates out, uint32_t *__restrict__ cand, KeptLists kl) {
  __shared__ uint32_t list[kList][kBlock];
  const int tid = threadIdx.x;
  const uint32_t i = xcd_block(blockIdx.x, gridDim.x) * kBlock + tid;
  const bool active = i < nf;
  double4 a0 = make_double4(0.0, 0.0, 0.0, 0.0), a1 = a0;
  if (active) {
    a0 = rec0[i];
    a1 = rec1[i];
  }
  PairSums S;
  sums_zero(S);
  const unsigned long long counts = active ? kl.cnt[i] : 0ull;
  const int nch = (int)(counts >> kKeptNchShift);
  const int wch = wave_max_int(nch);
  for (int c = 0; c < wch; ++c) {
    const int cnt = c < nch ? kept_count(counts, c) : 0;
    const int kmax = wave_max_int(cnt);
    // stage the chunk in this lane's LDS column, eight loads in flight at once
    const uint32_t *src = kl.ent + kept_entry(i, c, 0);
    for (int k0 = 0; k0 < kmax; k0 += 8) {
      uint32_t e[8];
#pragma unroll
      for (int u = 0; u < 8; ++u) e[u] = k0 + u < cnt ? src[(size_t)(k0 + u) * 64u] : 0u;
#pragma unroll
      for (int u = 0; u < 8; ++u) list[k0 + u][tid] = e[u];
    }
    // one neighbour per iteration, the next list entry read one iteration ahead
    uint32_t en = cnt > 0 ? list[0][tid] : 0u;
    for (int k = 0; k < cnt; ++k) {
      const uint32_t j = en & ~kSkinTag;
      const double4 b0 = rec0[j], b1 = rec1[j];
      if (k + 1 < cnt) en = list[k + 1][tid];
      if (dist2_exact<DIM>(b0.x - a0.x, b0.y - a0.y, DIM == 3 ? b0.z - a0.z : 0.0) <= P.two_h2) {
        pair_body_f64<DIM, PST4>(P, a0, a1, b0, b1, S);
        S.nnb += 1;
      }
    }
    S.ntest += (uint32_t)cnt;
  }
  pair_epilogue<DIM>(P, sc, out, cand, i, active, S);
}

// ------------------------------------------------- pair pass by teams

constexpr int kTeam = 8;                   // lanes of a particle
constexpr int kTeamRows = kBlock / kTeam;  // particles of a block

// DPP controls that exchange lanes l and l ^ O (O = 1, 2: quad_perm) or their
// mirror images in the half row of 8 lanes (4: row_half_mirror).
constexpr int dpp_swap(int o) { return o == 1 ? 0xb1 : o == 2 ? 0x4e : 0x141; }

template <int O>
__device__ __forceinline__ double lane_swap(double v) {
  const int lo = __builtin_amdgcn_update_dpp(0, __double2loint(v), dpp_swap(O), 0xf, 0xf, true);
  const int hi = __builtin_amdgcn_update_dpp(0, __double2hiint(v), dpp_swap(O), 0xf, 0xf, true);
  return __hiloint2double(hi, lo);
}

// Adds N values over the team's lanes and spreads the sums over them: each
// step halves the values a lane holds (the lanes with bit O clear keep the
// even ones) and adds the partner's.  The lane's sums are v[0 .. *n), of the
// values q[0 .. *n).
template <int O, int N>
__device__ __forceinline__ void team_reduce(double *v, int sub) {
  if constexpr (O > 0) {
    const bool odd = (sub & O) != 0;
#pragma unroll
    for (int k = 0; k < N / 2; ++k) {
      const double keep = odd ? v[2 * k + 1] : v[2 * k], send = odd ? v[2 * k] : v[2 * k + 1];
      v[k] = keep + lane_swap<O>(send);
    }
    if (N % 2) v[N / 2] = v[N - 1] + lane_swap<O>(v[N - 1]);
    team_reduce<O / 2, (N + 1) / 2>(v, sub);
  }
}
template <int O, int N>
__device__ __forceinline__ int team_slot(int sub, int s) {  // value that slot s of the lane holds
  if constexpr (O > 0) return min(2 * team_slot<O / 2, (N + 1) / 2>(sub, s) + ((sub & O) ? 1 : 0), N - 1);
  else return s;
}
template <int O, int N>
constexpr int team_left() {
  if constexpr (O > 0) return team_left<O / 2, (N + 1) / 2>();
  else return N;
}

// Inclusive prefix sum over the lanes of a team (row_shr, cut at the team).
__device__ __forceinline__ int team_scan(int v, int sub) {
  int t = __builtin_amdgcn_update_dpp(0, v, 0x111, 0xf, 0xf, true);
  v += sub >= 1 ? t : 0;
  t = __builtin_amdgcn_update_dpp(0, v, 0x112, 0xf, 0xf, true);
  v += sub >= 2 ? t : 0;
  t = __builtin_amdgcn_update_dpp(0, v, 0x114, 0xf, 0xf, true);
  return v + (sub >= 4 ? t : 0);
}

// Largest of the wave's team values (equal in a team's lanes), scalar.
__device__ __forceinline__ int team_max(int v) {
  int m = __builtin_amdgcn_readlane(v, 0);
#pragma unroll
  for (int l = kTeam; l < 64; l += kTeam) m = max(m, __builtin_amdgcn_readlane(v, l));
  return m;
}

// The sums of a particle as a list of the values that its dimension has.
template <int DIM, class F>
__device__ __forceinline__ void each_sum(PairSums &S, F f) {
  int q = 0;
#pragma unroll
  for (int k = 0; k < 6; ++k) {
    if (DIM == 2 && k != 0 && k != 1 && k != 3) continue;
    f(S.L[k], q++);
    f(S.N[k], q++);
  }
#pragma unroll
  for (int k = 0; k < DIM; ++k) {
    f(S.gs[k], q++);
    f(S.SR[k], q++);
    f(S.SC[k], q++);
    f(S.Ps[k], q++);
  }
  f(S.Ds, q++);
}

// Records below 2^27 (the launch checks it): 32-bit offsets from a scalar base.
__device__ __forceinline__ const double4 &rec_at(const double4 *rec, uint32_t j) {
  return *reinterpret_cast<const double4 *>(reinterpret_cast<const char *>(rec) + j * 32u);
}

// The 8 lanes of a team share a particle.  They compute the windows of eight
// cell rows side by side, test the windows' records, compact the neighbours
// into the team's LDS list and run the pair body over it; the sums are added
// across the team in a fixed tree, and the block's first wave runs the
// epilogue, a lane per particle.  In 3D over cells of 2h (LONG) a row holds
// several times eight records and is tested in place; else the windows' record
// indices are first listed in LDS, so that the short rows fill the lanes (the
// other way round 928 against 637 us at 651,000 particles, cells of 2h, and 710
// against 565, cells of h; in 2D both take the same).  Neighbour number n goes
// to lane n mod 8 wherever the list is emptied, so this kernel's plain search,
// the one that keeps its candidates (kPairSearchKeep: radius 2h + skin) and its
// pass from kept candidates (kPairKept, lists built by this kernel only: full
// chunks but the last) give the same sums bit for bit.  The two searches
// always come from the same kernel (by_team); above 70,000 particles in 3D
// (35,000 in 2D) its lists are read by k_pair_kept_f64, whose sums are rounded
// otherwise.
// Everything that crosses lanes sits under scalar control flow: trip counts
// come from ballots and lane reads, and stores to the team's list are
// unconditional (a lane without an entry stores to a spare slot).  A
// conditional store right before a loop that ballots let the compiler merge
// the store's branch with the loop's and run it with part of the wave.  So
// where lanes do something of their own (a kept entry, a row's window, a
// neighbour's body) a wave barrier follows: it can't be made conditional, and
// all lanes are back before the next ballot.
template <int DIM, bool PST4, int MODE, bool LONG>
__global__ void __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(PST4 ? 4 : 2)))
k_pair_team_f64(Phys P, Grid g, const double4 *__restrict__ rec0, const double4 *__restrict__ rec1,
                const uint32_t *__restrict__ cs_f, const uint32_t *__restrict__ cs_d, uint32_t nf, Scalars *sc,
                Rates out, uint32_t *__restrict__ cand, KeptLists kl) {
  constexpr bool KEEP = MODE == kPairSearchKeep, KEPT = MODE == kPairKept;
  constexpr int NS = DIM == 3 ? 25 : 15;
  constexpr int kPer = LONG ? 3 : 4;                     // records in flight per lane
  constexpr int kChunk = LONG ? kPer * kTeam : 64;                          // candidates between looks at the list
  constexpr int kList = KEPT ? kKeepChunks * kPairList : 160;               // list entries of a particle
  static_assert(kList >= 2 * kChunk, "list entries");
  __shared__ uint32_t lists[kTeamRows][kList + 1];
  __shared__ double sums[NS][kTeamRows];
  __shared__ uint32_t counts[3][kTeamRows];
  const int sub = (int)(threadIdx.x & (kTeam - 1)), team = (int)threadIdx.x / kTeam;
  const bool upper = (threadIdx.x & 32u) != 0u;
  const uint32_t shift = threadIdx.x & 31u & ~(uint32_t)(kTeam - 1), below = (1u << sub) - 1u;
  uint32_t *list = lists[team];
  const uint32_t first = xcd_block(blockIdx.x, gridDim.x) * (uint32_t)kTeamRows;
  const uint32_t i = first + (uint32_t)team;
  const bool active = i < nf;
  const double4 a0 = rec_at(rec0, active ? i : 0u), a1 = rec_at(rec1, active ? i : 0u);
  PairSums S;
  sums_zero(S);
  const double rho = KEEP ? P.two_h + P.skin_max : P.two_h;
  const double rho2 = KEEP ? rho * rho : P.two_h2;
  int cnt = 0, done = 0, kept = 0, tested = 0;  // neighbours listed and summed, candidates kept and tested
  auto ranks = [&](bool in, int &n) {  // lanes of the team below this one that have one; n: of the team
    const unsigned long long m = __ballot(in);
    const uint32_t t = ((upper ? (uint32_t)(m >> 32) : (uint32_t)m) >> shift) & ((1u << kTeam) - 1u);
    n = __popc(t);
    return __popc(t & below);
  };
  // candidates 0 .. n - 1 of the team (at most nmax in the wave): record index(k)
  auto test = [&](int n, int nmax, auto index) {
    for (int t = 0; t < nmax; t += kPer * kTeam) {
      uint32_t j[kPer];
      double4 b[kPer];
#pragma unroll
      for (int u = 0; u < kPer; ++u) {
        const int k = t + u * kTeam + sub;
        j[u] = index(k, k < n);
        if (u < 2 || t + u * kTeam < nmax) b[u] = rec_at(rec0, j[u]);
      }
      wave_lds_sync();  // the entries are read before neighbours take their places
#pragma unroll
      for (int u = 0; u < kPer; ++u) {
        if (u > 0 && t + u * kTeam >= nmax) break;
        const double r2 = dist2_exact<DIM>(b[u].x - a0.x, b[u].y - a0.y, DIM == 3 ? b[u].z - a0.z : 0.0);
        const bool other = t + u * kTeam + sub < n && j[u] != i, in = other && r2 <= P.two_h2;
        int m;
        const int at = ranks(in, m);
        list[in ? cnt + at : kList] = j[u];
        cnt += m;
        if (KEEP) {
          const bool keep = other && r2 <= rho2;
          const int k = kept + ranks(keep, m);
          kept += m;
          if (keep && k < kKeepChunks * kPairList)
            kl.ent[kept_entry(i, k / kPairList, k % kPairList)] = j[u] | (in ? 0u : kSkinTag);
          __builtin_amdgcn_wave_barrier();
        }
      }
    }
    tested += n;
  };
  // the pair body over the list where another chunk might not fit, or at the end
  auto run_list = [&](bool end) {
    const int cmax = team_max(cnt);
    if (!end && cmax <= kList - kChunk) return;
    wave_lds_sync();
    for (int t = (sub - done) & (kTeam - 1), t0 = 0; t0 < cmax; t0 += kTeam, t += kTeam) {
      if (t < cnt) {
        const uint32_t j = list[t];
        pair_body_f64<DIM, PST4>(P, a0, a1, rec_at(rec0, j), rec_at(rec1, j), S);
      }
      __builtin_amdgcn_wave_barrier();
    }
    done += cnt;
    cnt = 0;
    wave_lds_sync();
  };
  if (KEPT) {
    const unsigned long long book = active ? kl.cnt[i] : 0ull;
    const int nch = (int)(book >> kKeptNchShift);
    const int n = nch ? (nch - 1) * kPairList + kept_count(book, nch - 1) : 0;
    test(n, team_max(n), [&](int k, bool in) {
      return in ? kl.ent[kept_entry(i, k / kPairList, k % kPairList)] & ~kSkinTag : 0u;
    });
  } else {
    const CellPos cp = cellpos_of<DIM>(g, a0.x, a0.y, a0.z);
    const float rr = (float)rho * (float)g.invR;
    const float rr2 = rr * rr * (1.0f + 4.0f * kWalkSlack);
    const int nrows = DIM == 3 ? (2 * g.reach + 1) * (2 * g.reach + 1) : 2 * g.reach + 1;
    for (int r0 = 0; r0 < nrows; r0 += kTeam) {
      uint32_t fb = 0, fl = 0, db = 0, dl = 0;  // this lane's row
      if (active && r0 + sub < nrows) row_windows<DIM>(g, cp, rr2, r0 + sub, cs_f, cs_d, nf, fb, fl, db, dl);
      __builtin_amdgcn_wave_barrier();
      const bool walls = __ballot(dl > 0u) != 0ull;
      if (LONG) {
        auto row = [&](int q, uint32_t rb, uint32_t rl) {
          const uint32_t lo = __shfl(rb, q, kTeam);
          const int len = (int)__shfl(rl, q, kTeam), lmax = team_max(len);
          for (int base = 0; base < lmax; base += kChunk) {
            run_list(false);
            const uint32_t from = lo + (uint32_t)base;
            test(min(max(len - base, 0), kChunk), min(lmax - base, kChunk),
                 [&](int k, bool in) { return in ? from + (uint32_t)k : 0u; });
          }
        };
        for (int q = 0; q < kTeam && r0 + q < nrows; ++q) {
          row(q, fb, fl);
          if (walls) row(q, db, dl);
        }
      } else {
        const int len = (int)(fl + dl), pre = team_scan(len, sub) - len;
        const int total = __shfl(pre + len, kTeam - 1, kTeam), all = team_max(total);
        for (int base = 0; base < all; base += kChunk) {
          run_list(false);
          // entries [e0, e0 + n) of the set are records b, b + 1, ...
          const int from = cnt;
          auto expand = [&](int e0, int n, uint32_t b) {
            const int e1 = min(e0 + n, base + kChunk);
            int e = max(e0, base);
            b += (uint32_t)(e - e0);
            while (__ballot(e < e1)) {
              list[e < e1 ? from + e - base : kList] = b;
              ++e;
              ++b;
            }
          };
          expand(pre, (int)fl, fb);
          if (walls) expand(pre + (int)fl, (int)dl, db);
          wave_lds_sync();
          test(min(max(total - base, 0), kChunk), min(all - base, kChunk), [&](int k, bool in) {
            const uint32_t j = list[in ? from + k : kList];
            return in ? j : 0u;
          });
        }
      }
    }
  }
  run_list(true);
  if (KEEP && sub == 0 && active) {
    unsigned long long book = 0ull;
    const int nch = min((kept + kPairList - 1) / kPairList, kKeepChunks);
    for (int c = 0; c < nch; ++c) book |= (unsigned long long)min(kept - c * kPairList, kPairList) << (6 * c);
    kl.cnt[i] = book | ((unsigned long long)nch << kKeptNchShift);
    if (kept > kKeepChunks * kPairList) sc->vovf = 1u;
  }
  __builtin_amdgcn_wave_barrier();
  int same;
  ranks(S.coincident, same);
  double v[NS];
  each_sum<DIM>(S, [&](double &x, int q) { v[q] = x; });
  team_reduce<kTeam / 2, NS>(v, sub);
#pragma unroll
  for (int k = 0; k < team_left<kTeam / 2, NS>(); ++k) sums[team_slot<kTeam / 2, NS>(sub, k)][team] = v[k];
  if (sub == 0) {
    counts[0][team] = (uint32_t)done;
    counts[1][team] = (uint32_t)tested;
    counts[2][team] = (uint32_t)same;
  }
  __syncthreads();
  if (threadIdx.x >= 64) return;
  const int row = (int)threadIdx.x & (kTeamRows - 1);
  PairSums T;
  sums_zero(T);
  each_sum<DIM>(T, [&](double &x, int q) { x = sums[q][row]; });
  T.nnb = counts[0][row];
  T.ntest = counts[1][row];
  T.coincident = counts[2][row] != 0u;
  const uint32_t mine = first + threadIdx.x;
  pair_epilogue<DIM>(P, sc, out, cand, mine, threadIdx.x < kTeamRows && mine < nf, T);
}

// Whether the pass runs by teams: up to the count where one lane per particle
// (k_pair_f64, k_pair_kept_f64) catches up.  With a lane each, a wave's chain
// of loads takes 230 us in 3D (36 us in 2D) whatever the count, and the waves
// come in rounds of 4,096; the team spends more instructions per particle.
//
// The two searching passes share a line, so that one that builds lists gives
// the plain search's sums bit for bit at any count.  In 3D it depends on the
// cells: lists are built only over those with room for a skin, where the
// team's building pass falls behind early (its lanes store a particle's
// entries 256 bytes apart); without room every pass is a plain search.
//
// Measured on a sloshing tank, a dam break, a cylinder entry and a cube of
// water (3D), a tank and a dam break (2D), us, lane / team: 3D plain search,
// cells of h 529 / 423 (446,000), 1,320 to 1,350 / 1,330 to 1,415 (1.5M),
// 1,771 / 1,786 and 1,775 / 1,944 (2.1M), 2,033 / 2,228 (2.4M); cells of 2h
// 649 / 461 (446,000), 2,029 / 1,889 (1.9M), 3,080 to 3,096 / 2,984 to 3,025
// (3.0M), 4,291 / 4,304 (4.4M), 5,082 / 5,178 (5.2M).  Building lists, cells of
// 1.02 h 862 / 893 (710,000), 1,257 / 1,400 (1.12M); of 2.05 h 965 / 940
// (636,000), 1,216 / 1,261 (850,000), 2,040 / 2,325 (1.53M).  From kept lists
// (built by teams, cells of 1.02 h) 49 / 20 (15,000), 52 / 44 and 60 / 64
// (53,000), 64 / 56 (69,500), 71 / 84 (78,000), 65 / 64 (86,000), 73 / 108
// (105,000).  2D search, cells of 2h and h within 2 us: 42 / 30 (80,000), 44 /
// 40 and 42 / 40 (125,000), 47 / 47 and 44 / 46 (152,000); building lists 49 /
// 45 (125,000), 50 / 52 and 52 / 52 (152,000); from kept lists 15 / 11
// (20,000), 16 / 16 (33,000 and 36,000), 17 / 20 (41,000).
template <int DIM>
static bool by_team(const Phys &P, const Grid &g, uint32_t nf, int64_t nrec, int mode) {
  if (nrec > (int64_t)1 << 27) return false;  // rec_at's offsets
  if (mode == kPairKept) return nf <= (DIM == 3 ? 70000u : 35000u);  // within the next line: lists of this kernel
  if (DIM == 2) return nf <= 120000u;
  const bool room = (double)g.reach * g.R - P.two_h > 1e-6 * g.R;  // as for P.skin_max
  return nf <= (room ? 700000u : g.reach == 1 ? 3000000u : 2000000u);
}

template <int DIM>
void launch_pair_f64_inst(const Phys &P, const Grid &g, const double4 *rec0, const double4 *rec1,
                          const uint32_t *cs_f, const uint32_t *cs_d, uint32_t nf, int64_t nrec, Scalars *sc,
                          const Rates &out, uint32_t *cand, const KeptLists &kl, int mode, hipStream_t s) {
  const int block = mode == kPairKept ? kBlock : kSearchBlock;
  dim3 gr(grid_for(nf, block)), bl(block);
  const bool p4 = P.pst_n == 4.0;
  if (by_team<DIM>(P, g, nf, nrec, mode)) {
    const bool lng = DIM == 3 && g.reach == 1;
    gr = dim3(grid_for(nf, kTeamRows));
    bl = dim3(kBlock);
#define WB_TEAM(MODE, LONG)                                                                                       \
  do {                                                                                                            \
    if (p4)                                                                                                       \
      hipLaunchKernelGGL((k_pair_team_f64<DIM, true, MODE, LONG>), gr, bl, 0, s, P, g, rec0, rec1, cs_f, cs_d,    \
                         nf, sc, out, cand, kl);                                                                  \
    else                                                                                                          \
      hipLaunchKernelGGL((k_pair_team_f64<DIM, false, MODE, LONG>), gr, bl, 0, s, P, g, rec0, rec1, cs_f, cs_d,   \
                         nf, sc, out, cand, kl);                                                                  \
  } while (0)
    if (mode == kPairKept) WB_TEAM(kPairKept, false);
    else if (mode == kPairSearchKeep && lng) WB_TEAM(kPairSearchKeep, DIM == 3);
    else if (mode == kPairSearchKeep) WB_TEAM(kPairSearchKeep, false);
    else if (lng) WB_TEAM(kPairSearch, DIM == 3);
    else WB_TEAM(kPairSearch, false);
#undef WB_TEAM
  } else if (mode == kPairSearch) {
    if (p4)
      hipLaunchKernelGGL((k_pair_f64<DIM, true, false>), gr, bl, 0, s, P, g, rec0, rec1, cs_f, cs_d, nf, sc, out, cand,
                         kl);
    else
      hipLaunchKernelGGL((k_pair_f64<DIM, false, false>), gr, bl, 0, s, P, g, rec0, rec1, cs_f, cs_d, nf, sc, out,
                         cand, kl);
  } else if (mode == kPairSearchKeep) {
    if (p4)
      hipLaunchKernelGGL((k_pair_f64<DIM, true, true>), gr, bl, 0, s, P, g, rec0, rec1, cs_f, cs_d, nf, sc, out, cand,
                         kl);
    else
      hipLaunchKernelGGL((k_pair_f64<DIM, false, true>), gr, bl, 0, s, P, g, rec0, rec1, cs_f, cs_d, nf, sc, out,
                         cand, kl);
  } else {
    if (p4)
      hipLaunchKernelGGL((k_pair_kept_f64<DIM, true>), gr, bl, 0, s, P, rec0, rec1, nf, sc, out, cand, kl);
    else
      hipLaunchKernelGGL((k_pair_kept_f64<DIM, false>), gr, bl, 0, s, P, rec0, rec1, nf, sc, out, cand, kl);
  }
}

hipError_t launch_pair_f64(const Phys &P, const Grid &g, const double4 *rec0, const double4 *rec1,
                           const uint32_t *cs_f, const uint32_t *cs_d, uint32_t nf, int64_t nrec, Scalars *sc,
                           const Rates &out, uint32_t *cand, int mode, uint32_t *kent, unsigned long long *kcnt,
                           hipStream_t s) {
  if (nf == 0) return hipSuccess;
  if (mode != kPairSearch && (!kent || !kcnt)) return hipErrorInvalidValue;
  KeptLists kl{kent, kcnt};
  if (P.dim == 2)
    launch_pair_f64_inst<2>(P, g, rec0, rec1, cs_f, cs_d, nf, nrec, sc, out, cand, kl, mode, s);
  else
    launch_pair_f64_inst<3>(P, g, rec0, rec1, cs_f, cs_d, nf, nrec, sc, out, cand, kl, mode, s);
  return hipGetLastError();
}

// ---------------------------------------------------- classifier features

// The 16 classifier features of a particle from the raw sums the pair-pass
// epilogue left in its row (L, g = sum grad W V, the shifting sum P) and its
// eigenvalues, normal n and neighbour count: eigenvalues of L (3), det L,
// n.P h, neighbour count, |g| h, n.g h, tangential |g| h, n.L.n,
// tr L - n.L.n, |L^-T g| h, n.G / |G|, tangential |P| h, n.P / |P|, |P| h.
// Rows of the device-counted list (count != nullptr) or rows 0 .. n - 1.
template <int DIM>
__global__ void __launch_bounds__(256) k_features(Phys P, Rates out, const uint32_t *__restrict__ list,
                                                  const uint32_t *__restrict__ count, uint32_t n,
                                                  const Scalars *__restrict__ sc) {
  const uint32_t total = count ? *count : n;
  double G[3];
  body_force(P, sc->t_rhs, G);
  const double gg = sqrt(G[0] * G[0] + G[1] * G[1] + G[2] * G[2]);
  for (uint32_t k = blockIdx.x * blockDim.x + threadIdx.x; k < total; k += gridDim.x * blockDim.x) {
    const uint32_t i = list ? list[k] : k;
    float *f = out.feat + (size_t)i * kNFeat;
    float raw[12];
#pragma unroll
    for (int c = 0; c < 12; ++c) raw[c] = f[c];
    const double L[6] = {raw[0], raw[1], raw[2], raw[3], raw[4], raw[5]};
    const double g[3] = {raw[6], raw[7], raw[8]}, Pv[3] = {raw[9], raw[10], raw[11]};
    const double n[3] = {out.nrm[0][i], out.nrm[1][i], DIM == 3 ? out.nrm[2][i] : 0.0};
    const double Lm[3][3] = {{L[0], L[3], L[4]}, {L[3], L[1], L[5]}, {L[4], L[5], L[2]}};
    double ng = 0, gn2 = 0, nLn = 0, trL = 0, pn2 = 0, ngr = 0, nP = 0;
#pragma unroll
    for (int a = 0; a < DIM; ++a) {
      ng += n[a] * g[a];
      gn2 += g[a] * g[a];
      trL += Lm[a][a];
      pn2 += Pv[a] * Pv[a];
      nP += n[a] * Pv[a];
      ngr += n[a] * G[a];
#pragma unroll
      for (int b = 0; b < DIM; ++b) nLn += n[a] * Lm[a][b] * n[b];
    }
    double gt2 = 0, pt2 = 0;  // tangential parts by components (no cancellation)
#pragma unroll
    for (int a = 0; a < DIM; ++a) {
      const double t = g[a] - ng * n[a], tp = Pv[a] - nP * n[a];
      gt2 += t * t;
      pt2 += tp * tp;
    }
    const double pm = sqrt(pn2);
    // |L^-T g| (L symmetric), or |g| where L is singular (the epilogue's rule)
    double ngv[3] = {g[0], g[1], g[2]};
    if (out.lam[0][i] > P.lambda_sing) {
      double I[6];
      inv_sym<DIM>(L, I);
      sym_mul<DIM>(I, g, ngv);
    }
    const double nn = sqrt(ngv[0] * ngv[0] + ngv[1] * ngv[1] + (DIM == 3 ? ngv[2] * ngv[2] : 0.0));
    const double detL = DIM == 2 ? L[0] * L[1] - L[3] * L[3]
                                 : L[0] * (L[1] * L[2] - L[5] * L[5]) - L[3] * (L[3] * L[2] - L[5] * L[4]) +
                                       L[4] * (L[3] * L[5] - L[1] * L[4]);
    f[0] = (float)out.lam[0][i];
    f[1] = (float)out.lam[1][i];
    f[2] = (float)(DIM == 3 ? out.lam[2][i] : out.lam[1][i]);
    f[3] = (float)detL;
    f[4] = (float)(nP * P.h);
    f[5] = (float)out.nnb[i];
    f[6] = (float)(sqrt(gn2) * P.h);
    f[7] = (float)(ng * P.h);
    f[8] = (float)(sqrt(gt2) * P.h);
    f[9] = (float)nLn;
    f[10] = (float)(trL - nLn);
    f[11] = (float)(nn * P.h);
    f[12] = (float)(gg > 0.0 ? ngr / gg : 0.0);
    f[13] = (float)(sqrt(pt2) * P.h);
    f[14] = (float)(pm > 0.0 ? nP / pm : 0.0);
    f[15] = (float)(pm * P.h);
  }
}

hipError_t launch_features(const Phys &P, const Rates &out, const uint32_t *list, const uint32_t *count, uint32_t n,
                           const Scalars *sc, hipStream_t s) {
  if (n == 0) return hipSuccess;
  unsigned blocks = grid_for(n);
  if (blocks > 2048) blocks = 2048;
  if (P.dim == 2)
    hipLaunchKernelGGL(k_features<2>, dim3(blocks), dim3(kBlock), 0, s, P, out, list, count, n, sc);
  else
    hipLaunchKernelGGL(k_features<3>, dim3(blocks), dim3(kBlock), 0, s, P, out, list, count, n, sc);
  return hipGetLastError();
}

// --------------------------------------------------------- scan-region pass

// Candidates (lambda_lo < lambda <= lambda_hi) are on the free surface unless
// a neighbour lies in the umbrella-shaped region around T = x_i + h n: beyond
// sqrt(2) h from i within h of T, or closer than sqrt(2) h to i with
// |n.(x_j - T)| + |tangential part| < h.  One wave per candidate: the lanes
// take the candidate's rows (one row each) and then its neighbour candidates
// 64 at a time, until one covers it.  Grid-stride over the device-counted
// list, so the launch does not depend on the count.
template <int DIM>
__global__ void __launch_bounds__(256) k_scan_f64(Phys P, Grid g, const double4 *__restrict__ rec0,
                                                  const uint32_t *__restrict__ cs_f, const uint32_t *__restrict__ cs_d,
                                                  uint32_t nf, const uint32_t *__restrict__ list,
                                                  const uint32_t *__restrict__ count, Rates out, Scalars *sc) {
  __shared__ RowTables tab;
  const uint32_t total = *count;
  const int lane = (int)(threadIdx.x & 63);
  const uint32_t gw = (blockIdx.x * blockDim.x + threadIdx.x) >> 6, nw = (gridDim.x * blockDim.x) >> 6;
  uint32_t nfs = 0;  // surface particles found by this wave (one atomic add at the end)
  for (uint32_t k = gw; k < total; k += nw) {
    const uint32_t i = list[k];
    const double4 a = rec0[i];
    const double n[3] = {out.nrm[0][i], out.nrm[1][i], DIM == 3 ? out.nrm[2][i] : 0.0};
    const double T[3] = {a.x + P.h * n[0], a.y + P.h * n[1], DIM == 3 ? a.z + P.h * n[2] : 0.0};
    const CellPos cp = cellpos_of<DIM>(g, a.x, a.y, a.z);
    int nrows;
    const uint32_t M = rows_layout<DIM>(tab, g, cp, (float)P.win, cs_f, cs_d, nf, nrows);
    bool covered = false;
    for (uint32_t c0 = 0; c0 < M && !covered; c0 += 64u) {
      bool cov = false;
      const uint32_t idx = c0 + (uint32_t)lane;
      if (idx < M) {
        const uint32_t j = record_of(tab, nrows, idx);
        if (j != i) {
          const double4 b = rec0[j];
          const double q[3] = {b.x, b.y, DIM == 3 ? b.z : 0.0};
          const double s2 = dist2_exact<DIM>(b.x - a.x, b.y - a.y, b.z - a.z);
          cov = s2 <= P.two_h2 && scan_covers<DIM>(P, q, T, n, s2);
        }
      }
      covered = __ballot(cov) != 0ull;
    }
    wave_lds_sync();  // the tables are rewritten for the next candidate
    if (lane == 0) scan_finish<DIM>(P, out, i, n, covered);
    nfs += covered ? 0u : 1u;
  }
  if (lane == 0 && nfs) atomicAdd(&tally_of(sc).n_fs, nfs);
}

hipError_t launch_scan_f64(const Phys &P, const Grid &g, const double4 *rec0, const uint32_t *cs_f,
                           const uint32_t *cs_d, uint32_t nf, const uint32_t *list, const uint32_t *count,
                           const Rates &out, Scalars *sc, hipStream_t s) {
  if (nf == 0) return hipSuccess;
  unsigned blocks = candidate_grid(nf);
  if (P.dim == 2)
    hipLaunchKernelGGL(k_scan_f64<2>, dim3(blocks), dim3(kBlock), 0, s, P, g, rec0, cs_f, cs_d, nf, list, count, out,
                       sc);
  else
    hipLaunchKernelGGL(k_scan_f64<3>, dim3(blocks), dim3(kBlock), 0, s, P, g, rec0, cs_f, cs_d, nf, list, count, out,
                       sc);
  return hipGetLastError();
}

// ------------------------------------------------------- neighbour export

template <int DIM>
__global__ void __launch_bounds__(256) k_nb_count(Phys P, Grid g, const double4 *__restrict__ rec0,
                                                  const uint32_t *__restrict__ cs_f, const uint32_t *__restrict__ cs_d,
                                                  uint32_t nf, const uint32_t *__restrict__ fid,
                                                  uint32_t *__restrict__ cnt, uint32_t nrows) {
  uint32_t i = blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= nf) return;
  double4 a = rec0[i];
  RowWalker w;
  walker_init<DIM>(w, g, a.x, a.y, a.z, P.two_h);
  uint32_t c = 0;
  while (walker_next<DIM>(w, g, cs_f, cs_d, nf)) {
    for (uint32_t j = w.cur; j < w.end; ++j) {
      if (j == i) continue;
      double4 b = rec0[j];
      if (dist2_exact<DIM>(b.x - a.x, b.y - a.y, b.z - a.z) <= P.two_h2) ++c;
    }
  }
  if (fid[i] < nrows) cnt[fid[i]] = c;
}

template <int DIM>
__global__ void __launch_bounds__(256) k_nb_fill(Phys P, Grid g, const double4 *__restrict__ rec0,
                                                 const uint32_t *__restrict__ cs_f, const uint32_t *__restrict__ cs_d,
                                                 uint32_t nf, const uint32_t *__restrict__ fid,
                                                 const uint32_t *__restrict__ did, const uint32_t *__restrict__ off,
                                                 uint32_t r0, uint32_t r1, int32_t *__restrict__ ids) {
  uint32_t i = blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= nf) return;
  const uint32_t row = fid[i];
  if (row < r0 || row >= r1) return;
  double4 a = rec0[i];
  RowWalker w;
  walker_init<DIM>(w, g, a.x, a.y, a.z, P.two_h);
  uint32_t o = off[row];
  while (walker_next<DIM>(w, g, cs_f, cs_d, nf)) {
    for (uint32_t j = w.cur; j < w.end; ++j) {
      if (j == i) continue;
      double4 b = rec0[j];
      if (dist2_exact<DIM>(b.x - a.x, b.y - a.y, b.z - a.z) <= P.two_h2)
        ids[o++] = (int32_t)(j < nf ? fid[j] : did[j - nf]);
    }
  }
}

__global__ void __launch_bounds__(256) k_sort_rows(const uint32_t *__restrict__ off, int64_t r0, int64_t r1,
                                                   int32_t *__restrict__ ids) {
  int64_t r = r0 + (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (r >= r1) return;
  uint32_t b = off[r], e = off[r + 1];
  for (uint32_t k = b + 1; k < e; ++k) {
    int32_t v = ids[k];
    uint32_t m = k;
    while (m > b && ids[m - 1] > v) {
      ids[m] = ids[m - 1];
      --m;
    }
    ids[m] = v;
  }
}

hipError_t launch_nb_count_f64(const Phys &P, const Grid &g, const double4 *rec0, const uint32_t *cs_f,
                               const uint32_t *cs_d, uint32_t nf, const uint32_t *fid, uint32_t *cnt, hipStream_t s,
                               uint32_t nrows) {
  if (nf == 0) return hipSuccess;
  if (P.dim == 2)
    hipLaunchKernelGGL(k_nb_count<2>, dim3(grid_for(nf)), dim3(kBlock), 0, s, P, g, rec0, cs_f, cs_d, nf, fid, cnt,
                       nrows);
  else
    hipLaunchKernelGGL(k_nb_count<3>, dim3(grid_for(nf)), dim3(kBlock), 0, s, P, g, rec0, cs_f, cs_d, nf, fid, cnt,
                       nrows);
  return hipGetLastError();
}

hipError_t launch_nb_fill_f64(const Phys &P, const Grid &g, const double4 *rec0, const uint32_t *cs_f,
                              const uint32_t *cs_d, uint32_t nf, const uint32_t *fid, const uint32_t *did,
                              const uint32_t *off, uint32_t r0, uint32_t r1, int32_t *ids, hipStream_t s) {
  if (nf == 0) return hipSuccess;
  if (P.dim == 2)
    hipLaunchKernelGGL(k_nb_fill<2>, dim3(grid_for(nf)), dim3(kBlock), 0, s, P, g, rec0, cs_f, cs_d, nf, fid, did, off,
                       r0, r1, ids);
  else
    hipLaunchKernelGGL(k_nb_fill<3>, dim3(grid_for(nf)), dim3(kBlock), 0, s, P, g, rec0, cs_f, cs_d, nf, fid, did, off,
                       r0, r1, ids);
  return hipGetLastError();
}

hipError_t launch_sort_rows(const uint32_t *off, int64_t r0, int64_t r1, int32_t *ids, hipStream_t s) {
  if (r1 <= r0) return hipSuccess;
  hipLaunchKernelGGL(k_sort_rows, dim3(grid_for(r1 - r0)), dim3(kBlock), 0, s, off, r0, r1, ids);
  return hipGetLastError();
}

hipError_t launch_mirror_f64(const Phys &P, const Grid &g, const Dummies &d, int64_t nd, const double4 *rec0,
                             const double4 *rec1, double4 *drec0, double4 *drec1, const uint32_t *cs_f,
                             uint32_t nf, const Scalars *sc, hipStream_t s, const uint32_t *fid) {
  if (nd == 0) return hipSuccess;
  const bool team = nd <= kMirrorTeamRows;
#define WB_GO(D, T)                                                                                                \
  hipLaunchKernelGGL((k_mirror_f64<D, T>), dim3(grid_for(nd, kBlock / T)), dim3(kBlock), 0, s, P, g, d, nd, rec0,   \
                     rec1, drec0, drec1, cs_f, nf, sc, fid)
  if (P.dim == 2 && team) WB_GO(2, kMirrorTeam);
  else if (P.dim == 2) WB_GO(2, 1);
  else if (team) WB_GO(3, kMirrorTeam);
  else WB_GO(3, 1);
#undef WB_GO
  return hipGetLastError();
}

// ----------------------------------------------------- free body force

// Force and torque of the water on the free body: each of its dummies takes
// the conservative-form acceleration of Eq. (sph) (the branch of Sec. 2.3)
// that a dummy with mirrored potential phi_d gets from its fluid neighbours,
// a_d = -sum_i (phi_i + phi_d) grad_d W_di V_i, times its mass, and its
// moment about the body's centre.  Dummies without a mirror source (in no
// fluid particle's support) and all other rows add nothing.  Each block sums
// its rows by a fixed tree and writes one partial (6 doubles, F then the
// torque) to part[6 blockIdx.x ..]: the sums depend only on the rows' order.
template <int DIM>
__global__ void __launch_bounds__(256) k_body_force_f64(Phys P, Grid g, Dummies d, int64_t nd,
                                                        const double4 *__restrict__ rec0,
                                                        const double4 *__restrict__ rec1,
                                                        const double4 *__restrict__ drec0,
                                                        const uint32_t *__restrict__ cs_f, uint32_t nf,
                                                        const Scalars *__restrict__ sc, double *__restrict__ part) {
  __shared__ double red[6][256];
  const int64_t k = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  double f[3] = {0.0, 0.0, 0.0}, tq[3] = {0.0, 0.0, 0.0};
  if (k < nd && d.mov[k] && d.src[k] >= 0) {
    const double4 me = drec0[k];  // placed position and mirrored potential
    RowWalker w;
    walker_init<DIM>(w, g, me.x, me.y, me.z, P.win);
    double a[3] = {0.0, 0.0, 0.0};
    auto sum_run = [&](uint32_t lo, uint32_t hi) {
      for (uint32_t j = lo; j < hi; ++j) {
        const double4 b = rec0[j];
        const double rx = b.x - me.x, ry = b.y - me.y, rz = DIM == 3 ? b.z - me.z : 0.0;
        const double r2 = dist2_exact<DIM>(rx, ry, rz);
        if (r2 > P.two_h2) continue;
        const double t = fma(sqrt(r2), P.m_half_inv_h, 1.0);  // 1 - q/2
        const double c = (b.w + me.w) * (P.kfac * t * t * t) * rec1[j].w;
        a[0] -= c * rx;
        a[1] -= c * ry;
        if (DIM == 3) a[2] -= c * rz;
      }
    };
    if (g.reach == 2) {
      constexpr int NR = DIM == 3 ? 25 : 5;
      uint32_t lo[NR], hi[NR];
      walker_fluid_runs<DIM, NR>(w, g, cs_f, lo, hi);
#pragma unroll
      for (int r = 0; r < NR; ++r) sum_run(lo[r], hi[r]);
    } else {
      while (walker_next<DIM>(w, g, cs_f, cs_f, nf))
        if (w.cur < nf) sum_run(w.cur, w.end);
    }
    const double m = d.m[k];
    const double arm[3] = {me.x - sc->fb[0], me.y - sc->fb[1], DIM == 3 ? me.z - sc->fb[2] : 0.0};
    for (int c = 0; c < 3; ++c) f[c] = m * a[c];
    tq[0] = arm[1] * f[2] - arm[2] * f[1];
    tq[1] = arm[2] * f[0] - arm[0] * f[2];
    tq[2] = arm[0] * f[1] - arm[1] * f[0];
  }
  const int t = threadIdx.x;
  for (int c = 0; c < 3; ++c) {
    red[c][t] = f[c];
    red[3 + c][t] = tq[c];
  }
  __syncthreads();
  for (int w = 128; w > 0; w >>= 1) {
    if (t < w)
      for (int c = 0; c < 6; ++c) red[c][t] += red[c][t + w];
    __syncthreads();
  }
  if (t < 6) part[(size_t)6 * blockIdx.x + t] = red[t][0];
}

hipError_t launch_body_force_f64(const Phys &P, const Grid &g, const Dummies &d, int64_t nd, const double4 *rec0,
                                 const double4 *rec1, const double4 *drec0, const uint32_t *cs_f, uint32_t nf,
                                 const Scalars *sc, double *part, hipStream_t s) {
  if (nd == 0) return hipSuccess;
  if (!d.mov || !part) return hipErrorInvalidValue;
  static_assert(kBlock == 256, "the block tree of the body force assumes 256 threads");
  if (P.dim == 2)
    hipLaunchKernelGGL(k_body_force_f64<2>, dim3(grid_for(nd)), dim3(kBlock), 0, s, P, g, d, nd, rec0, rec1, drec0,
                       cs_f, nf, sc, part);
  else
    hipLaunchKernelGGL(k_body_force_f64<3>, dim3(grid_for(nd)), dim3(kBlock), 0, s, P, g, d, nd, rec0, rec1, drec0,
                       cs_f, nf, sc, part);
  return hipGetLastError();
}

}  // namespace wb
