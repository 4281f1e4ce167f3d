// Learned free-surface classifier: a per-particle MLP 16 -> 64 -> 64 -> 1
// with GELU (tanh form), trained on labels the exact scan-region criterion
// produces, used for the particles lambda_min alone cannot decide.
//
// Training (FP32, hand-written): per batch one kernel for forward, weighted
// binary cross-entropy on the logit, backward pass and the blocks' parameter
// gradients (one wave per row, one lane per hidden unit), and one that sums
// the blocks in a fixed order (deterministic) and applies Adam with bias
// correction.
//
// Inference (BF16 MFMA, FP32 accumulate): one wave handles 16 rows per
// iteration; layer 1 is a 16x16x32 bf16 MFMA per 16-unit tile with K = 16
// zero-padded to 32, layer 2 two MFMAs per tile (K = 64), biases and GELU in
// FP32 between layers, layer 3 a FP32 dot product reduced across the four
// lanes that share a row.  Weights stay in registers for the whole
// (persistent, grid-stride) kernel.
#include <algorithm>
#include <cmath>
#include <cstring>
#include <string>

#include "mlp.h"
#include "pair_common.h"
#include "wbsph.h"

namespace wb {

// flat parameter layout
constexpr int kOffW1 = 0;
constexpr int kOffB1 = kOffW1 + kMlpIn * kMlpHid;
constexpr int kOffW2 = kOffB1 + kMlpHid;
constexpr int kOffB2 = kOffW2 + kMlpHid * kMlpHid;
constexpr int kOffW3 = kOffB2 + kMlpHid;
constexpr int kOffB3 = kOffW3 + kMlpHid;
static_assert(kOffB3 + 1 == kMlpParams, "parameter layout");

__device__ __forceinline__ float gelu_f(float z) {
  const float c = 0.7978845608028654f;  // sqrt(2 / pi)
  return 0.5f * z * (1.0f + tanhf(c * (z + 0.044715f * z * z * z)));
}

// GELU (tanh form) for BF16 inference: 0.5 z (1 + tanh u) = z / (1 + e^{-2u})
// with u = sqrt(2/pi) (z + 0.044715 z^3), on the hardware exp2 and
// reciprocal (relative error ~1e-6, far below the BF16 rounding of the
// activations).  Saturates correctly: e -> inf gives 0, e -> 0 gives z.
__device__ __forceinline__ float gelu_fast(float z) {
  const float k = -2.0f * 0.7978845608028654f * 1.4426950408889634f;  // -2 sqrt(2/pi) log2(e)
  const float kc = k * 0.044715f;                                       // folded into the cubic term
  const float e = __builtin_amdgcn_exp2f(z * fmaf(kc, z * z, k));
  return z * __builtin_amdgcn_rcpf(1.0f + e);
}

// Orders the LDS writes of a wave before its later reads by other lanes.
__device__ __forceinline__ void wave_lds_order() {
  __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
  __builtin_amdgcn_wave_barrier();
  __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}

// ------------------------------------------------------------- training

// Logits of B rows of X.  blockDim = 256 = four rows, one wave per row, lane =
// hidden unit.  Nothing but the logits is stored (the gradient kernel
// recomputes the activations): 68 bytes a row instead of 900.
__global__ void __launch_bounds__(256) k_mlp_fwd(const float *__restrict__ w, const float *__restrict__ mean,
                                                 const float *__restrict__ std, const float *__restrict__ X,
                                                 int64_t B, float *__restrict__ s) {
  __shared__ float sx[4][kMlpIn];
  __shared__ float sa1[4][kMlpHid];
  const int lane = threadIdx.x & 63, r = threadIdx.x >> 6;
  const int64_t b = (int64_t)blockIdx.x * 4 + r;
  const bool on = b < B;
  if (on && lane < kMlpIn) sx[r][lane] = (X[b * kMlpIn + lane] - mean[lane]) / std[lane];
  __syncthreads();
  float z = w[kOffB1 + lane];
  for (int i = 0; i < kMlpIn; ++i) z += sx[r][i] * w[kOffW1 + i * kMlpHid + lane];
  sa1[r][lane] = gelu_f(z);
  __syncthreads();
  float y = w[kOffB2 + lane];
  for (int k = 0; k < kMlpHid; ++k) y += sa1[r][k] * w[kOffW2 + k * kMlpHid + lane];
  float p = gelu_f(y) * w[kOffW3 + lane];
#pragma unroll
  for (int o = 32; o > 0; o >>= 1) p += __shfl_xor(p, o, 64);
  if (on && lane == 0) s[b] = p + w[kOffB3];
}

hipError_t launch_mlp_fwd(const float *w, const float *mean, const float *std, const float *X, int64_t B,
                          float *logits, hipStream_t s) {
  hipLaunchKernelGGL(k_mlp_fwd, dim3((unsigned)((B + 3) / 4)), dim3(256), 0, s, w, mean, std, X, B, logits);
  return hipGetLastError();
}

// tanh form of GELU and its derivative, (1 + tanh u) / 2 as 1 / (1 + exp(-2u)).
__device__ __forceinline__ void gelu_both(float z, float &a, float &d) {
  const float c = 0.7978845608028654f;
  const float s = 1.0f / (1.0f + expf(-2.0f * c * (z + 0.044715f * z * z * z)));  // (1 + tanh) / 2
  a = z * s;
  d = s + 2.0f * z * (s * (1.0f - s)) * c * (1.0f + 3.0f * 0.044715f * z * z);
}

// Loss and parameter gradients of a batch, summed over the rows of a block:
// part[block][0 .. kMlpParams) and the block's loss at [kMlpParams].
//
// One wave per row, lane = hidden unit, rpw rows per wave.  A lane keeps its
// columns of W1 and W2 in registers (80 values) and the gradients of those (80
// sums), so a row costs 224 FMAs per lane and a few LDS broadcasts, and the
// activations never reach memory.  Bound by a row's chain of instructions (2.9
// us with one wave per SIMD): the rows of W2 come from LDS, which leaves room
// for two waves per SIMD, dot products run in four sums, and GELU's tanh is
// one exponential.  The sums of waves u and u + 4 are added, then the four in
// order, the blocks' in block order by k_mlp_reduce: the result depends only
// on the rows' order.  A batch of 4,096 rows: 19.3 us with one wave per SIMD,
// 13.8 so, and 4.2 in the reduction; an epoch of 65,536 rows in such batches
// 0.32 ms (31.9 ms with one kernel each for forward, loss and the rows'
// backward pass and one thread per parameter that walked the whole batch).
constexpr int kPart = kMlpParams + 1;
constexpr int kGradWaves = 8;

// c + a . b in four sums (one is a chain of N dependent FMAs).
template <int N>
__device__ __forceinline__ float dot(float c, const float *a, const float *b) {
  float s[4] = {c, 0.0f, 0.0f, 0.0f};
#pragma unroll
  for (int k = 0; k < N; ++k) s[k & 3] += a[k] * b[k];
  return (s[0] + s[1]) + (s[2] + s[3]);
}

__global__ void __launch_bounds__(64 * kGradWaves, 2)
    k_mlp_grad(const float *__restrict__ w, const float *__restrict__ mean, const float *__restrict__ std,
               const float *__restrict__ X, const float *__restrict__ y, const float *__restrict__ wt,
               const int32_t *__restrict__ perm, int64_t off, int64_t B, int rpw, float *__restrict__ part) {
  __shared__ __align__(16) float sx[kGradWaves][kMlpIn], sa[kGradWaves][kMlpHid], sd[kGradWaves][kMlpHid];
  __shared__ __align__(16) float w2l[kMlpHid][kMlpHid + 4];  // rows of W2 (a stride of 68: 16 lanes on all banks)
  __shared__ float sum[kGradWaves / 2][kPart];
  const int lane = threadIdx.x & 63, v = threadIdx.x >> 6;
  float w1[kMlpIn], w2c[kMlpHid];
#pragma unroll
  for (int i = 0; i < kMlpIn; ++i) w1[i] = w[kOffW1 + i * kMlpHid + lane];
#pragma unroll
  for (int k = 0; k < kMlpHid; ++k) w2c[k] = w[kOffW2 + k * kMlpHid + lane];
  for (int p = threadIdx.x; p < kMlpHid * kMlpHid; p += 64 * kGradWaves) w2l[p / kMlpHid][p % kMlpHid] = w[kOffW2 + p];
  const float b1 = w[kOffB1 + lane], b2 = w[kOffB2 + lane], w3 = w[kOffW3 + lane], b3 = w[kOffB3];
  float g1[kMlpIn], g2[kMlpHid], gb1 = 0.0f, gb2 = 0.0f, g3 = 0.0f, gb3 = 0.0f, loss = 0.0f;
#pragma unroll
  for (int i = 0; i < kMlpIn; ++i) g1[i] = 0.0f;
#pragma unroll
  for (int k = 0; k < kMlpHid; ++k) g2[k] = 0.0f;
  const int64_t b0 = ((int64_t)blockIdx.x * kGradWaves + v) * rpw;
  const int64_t b_end = b0 + rpw < B ? b0 + rpw : B;
  // the next row's inputs are requested before this one is worked on, and the
  // index of the one after
  const float mu = lane < kMlpIn ? mean[lane] : 0.0f, sg = lane < kMlpIn ? std[lane] : 1.0f;
  auto row_of = [&](int64_t b) { return b >= b_end ? (int64_t)-1 : perm ? (int64_t)perm[off + b] : off + b; };
  float xn = 0.0f, yn = 0.0f, wn = 1.0f;
  auto request = [&](int64_t row) {
    if (row < 0) return;
    if (lane < kMlpIn) xn = X[row * kMlpIn + lane];
    yn = y[row];
    if (wt) wn = wt[row];
  };
  request(row_of(b0));
  int64_t ahead = row_of(b0 + 1);
  __syncthreads();
  for (int64_t b = b0; b < b_end; ++b) {
    const float yv = yn, wv = wn;
    if (lane < kMlpIn) sx[v][lane] = (xn - mu) / sg;
    request(ahead);
    ahead = row_of(b + 2);
    wave_lds_order();
    float z = dot<kMlpIn>(b1, sx[v], w1);
    float a1, d1, a2, d2;
    gelu_both(z, a1, d1);
    sa[v][lane] = a1;
    wave_lds_order();
    const float q = dot<kMlpHid>(b2, sa[v], w2c);
    gelu_both(q, a2, d2);
    float s = a2 * w3;
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) s += __shfl_xor(s, o, 64);
    s += b3;
    // dL/ds of the weighted mean BCE and the row's loss
    const float sig = 1.0f / (1.0f + expf(-s));
    const float ds = wv * (sig - yv) / (float)B;
    loss += wv * (fmaxf(s, 0.0f) - s * yv + log1pf(expf(-fabsf(s))));
    // back through layers 3 and 2
    const float e2 = ds * w3 * d2;
    sd[v][lane] = e2;
    wave_lds_order();
    const float e1 = dot<kMlpHid>(0.0f, sd[v], w2l[lane]) * d1;
#pragma unroll
    for (int i = 0; i < kMlpIn; ++i) g1[i] += sx[v][i] * e1;
#pragma unroll
    for (int k = 0; k < kMlpHid; ++k) g2[k] += sa[v][k] * e2;
    gb1 += e1;
    gb2 += e2;
    g3 += a2 * ds;
    gb3 += ds;
    wave_lds_order();  // the row's LDS is rewritten for the next one
  }
  // wave u's and wave u + 4's sums, then the four of them in order
  for (int u = 0; u < 2; ++u) {
    if (v / (kGradWaves / 2) == u) {
      float *dst = sum[v % (kGradWaves / 2)];
      auto put = [&](int p, float x) { dst[p] = u == 0 ? x : dst[p] + x; };
#pragma unroll
      for (int i = 0; i < kMlpIn; ++i) put(kOffW1 + i * kMlpHid + lane, g1[i]);
      put(kOffB1 + lane, gb1);
#pragma unroll
      for (int k = 0; k < kMlpHid; ++k) put(kOffW2 + k * kMlpHid + lane, g2[k]);
      put(kOffB2 + lane, gb2);
      put(kOffW3 + lane, g3);
      if (lane == 0) {
        put(kOffB3, gb3);
        put(kMlpParams, loss);
      }
    }
    __syncthreads();
  }
  for (int p = threadIdx.x; p < kPart; p += 64 * kGradWaves) {
    float t = sum[0][p];
#pragma unroll
    for (int u = 1; u < kGradWaves / 2; ++u) t += sum[u][p];
    part[(size_t)blockIdx.x * kPart + p] = t;
  }
}

// Sums the blocks' partial gradients (and the losses: *loss the batch mean,
// acc += or = it) and, with adam, updates the parameters.  kRedParams
// parameters per block, each summed by kRedSlices threads over a contiguous
// share of the blocks, eight loads in flight (6.8 us one at a time, 4.2 so,
// 4,096 rows): one thread per parameter waited out a serial chain of loads on
// 21 of 256 CUs.
constexpr int kRedParams = 64, kRedSlices = 16;

struct AdamArgs {
  float *w, *m, *v;
  float lr, b1, b2, eps, c1, c2;
};

__device__ __forceinline__ void adam_update(const AdamArgs &A, int p, float gp) {
  const float mp = A.b1 * A.m[p] + (1.0f - A.b1) * gp;
  const float vp = A.b2 * A.v[p] + (1.0f - A.b2) * gp * gp;
  A.m[p] = mp;
  A.v[p] = vp;
  A.w[p] -= A.lr * (mp / A.c1) / (sqrtf(vp / A.c2) + A.eps);
}

__global__ void __launch_bounds__(kRedParams *kRedSlices)
    k_mlp_reduce(const float *__restrict__ part, int nblk, int64_t B, float *__restrict__ g, float *__restrict__ loss,
                 float *acc, int acc_reset, int adam, AdamArgs A) {
  __shared__ float sh[kRedSlices][kRedParams];
  const int c = threadIdx.x & (kRedParams - 1), sl = threadIdx.x / kRedParams;
  const int p = blockIdx.x * kRedParams + c;
  const int per = (nblk + kRedSlices - 1) / kRedSlices;
  const int k0 = sl * per, k1 = k0 + per < nblk ? k0 + per : nblk;
  float t = 0.0f;
  if (p < kPart)
    for (int k = k0; k < k1; k += 8) {  // eight loads in flight, added in block order
      float x[8];
#pragma unroll
      for (int u = 0; u < 8; ++u) x[u] = part[(size_t)min(k + u, k1 - 1) * kPart + p];
#pragma unroll
      for (int u = 0; u < 8; ++u) t += k + u < k1 ? x[u] : 0.0f;
    }
  sh[sl][c] = t;
  __syncthreads();
  if (sl != 0 || p >= kPart) return;
#pragma unroll
  for (int k = 1; k < kRedSlices; ++k) t += sh[k][c];
  if (p == kMlpParams) {
    t /= (float)B;
    *loss = t;
    if (acc) *acc = (acc_reset ? 0.0f : *acc) + t;
    return;
  }
  g[p] = t;
  if (adam) adam_update(A, p, t);
}

__global__ void k_mlp_adam(const float *__restrict__ g, AdamArgs A) {
  const int p = blockIdx.x * blockDim.x + threadIdx.x;
  if (p < kMlpParams) adam_update(A, p, g[p]);
}

// --------------------------------------------------------- BF16 inference

typedef __attribute__((__vector_size__(8 * sizeof(__bf16)))) __bf16 bf16x8;
typedef __attribute__((__vector_size__(4 * sizeof(float)))) float f32x4;

__device__ __forceinline__ __bf16 to_bf16(float x) { return (__bf16)x; }

// One wave per 16-row tile (grid-stride over tiles).  rows: optional index
// list (feature row r of output k is rows[k]); nrows_dev: optional device
// count overriding n.
//
// Bound by the vector ALU: the 128 GELUs per row.  The products are taken
// transposed, units x rows: a lane then holds 16 units of one row, which are
// the K slots of its own operand of the next layer once the weights' rows are
// loaded in that order -- slot (grp, e) of K block q is unit 16 (2 q + e / 4)
// + 4 grp + e % 4.  So the activations stay in registers (rows x units needed
// an exchange through LDS and 16 cross-lane sums per tile where this needs
// 2).  17,500,000 rows, whole calls one after another, the weights uploaded by
// three transfers each: 1.41 ms before, 1.28 ms transposed, 0.91 ms with the
// next tile's features requested a tile ahead, at three waves per SIMD (two:
// 1.05 ms); with one transfer 0.88 ms, and the kernel alone 0.99 ms under
// rocprofv3, at its lower clock.  The GELUs' instructions alone (96 of 160
// cycles of exp2 and reciprocal at a quarter rate among them) take about
// 0.85 ms.
__global__ void __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(3)))
    k_mlp_infer_bf16(const float *__restrict__ w, const float *__restrict__ mean, const float *__restrict__ std,
                     const float *__restrict__ X, const uint32_t *__restrict__ rows,
                     const uint32_t *__restrict__ nrows_dev, int64_t n, float *__restrict__ logits) {
  // biases and output weights per wave (in 48 registers they spill at three
  // waves per SIMD)
  __shared__ __align__(16) float vec[4][3][kMlpHid];
  const int lane = threadIdx.x & 63, wv = threadIdx.x >> 6;
  const int col = lane & 15, grp = lane >> 4;  // MFMA lane coordinates
  const int64_t total = nrows_dev ? (int64_t)(*nrows_dev) : n;
  const int64_t ntiles = (total + 15) / 16;
  const int64_t wave_id = (int64_t)blockIdx.x * 4 + wv;
  const int64_t nwaves = (int64_t)gridDim.x * 4;
  // waves without a tile leave before loading the weights (the grid is sized
  // for the largest possible count; the device count may be far smaller)
  if (wave_id >= ntiles) return;

  // A operands (weights) in registers: A[m][k] for unit m = col + 16 t.
  // Layer 1 has K = 16: groups 2, 3 hold zeros.
  bf16x8 w1b[4], w2b[4][2];
#pragma unroll
  for (int t = 0; t < 4; ++t) {
    const int nn = col + 16 * t;
#pragma unroll
    for (int e = 0; e < 8; ++e) {
      const int k = 8 * grp + e;
      w1b[t][e] = to_bf16(k < kMlpIn ? w[kOffW1 + k * kMlpHid + nn] : 0.0f);
#pragma unroll
      for (int q = 0; q < 2; ++q) {
        const int u = 16 * (2 * q + e / 4) + 4 * grp + e % 4;
        w2b[t][q][e] = to_bf16(w[kOffW2 + u * kMlpHid + nn]);
      }
    }
  }
  vec[wv][0][lane] = w[kOffB1 + lane];
  vec[wv][1][lane] = w[kOffB2 + lane];
  vec[wv][2][lane] = w[kOffW3 + lane];
  wave_lds_order();
  // unit 16 t + 4 grp + j is register j of tile t's result
  auto units = [&](int which, int t) { return *reinterpret_cast<const f32x4 *>(&vec[wv][which][16 * t + 4 * grp]); };
  const float b3 = w[kOffB3];
  float mu[8], isd[8];
#pragma unroll
  for (int e = 0; e < 8; ++e) {
    const int k = 8 * grp + e;
    mu[e] = k < kMlpIn ? mean[k] : 0.0f;
    isd[e] = k < kMlpIn ? 1.0f / std[k] : 0.0f;
  }

  // the next tile's features are requested before this tile is computed
  // (waiting for them left the ALU idle)
  float xn[8];
  auto request = [&](int64_t tile) {
    const int64_t rr = tile * 16 + col;
    const bool on = rr < total && grp < kMlpIn / 8;  // B operand of layer 1: row = col, k = 8 grp + e
    const int64_t src = on ? (rows ? (int64_t)rows[rr] : rr) * kMlpIn + 8 * grp : 0;
#pragma unroll
    for (int e = 0; e < 8; ++e) xn[e] = on ? X[src + e] : mu[e];  // mu: zero after the standardisation
  };
  request(wave_id);
  for (int64_t tile = wave_id; tile < ntiles; tile += nwaves) {
    const int64_t rr = tile * 16 + col;
    bf16x8 xa;
#pragma unroll
    for (int e = 0; e < 8; ++e) xa[e] = to_bf16((xn[e] - mu[e]) * isd[e]);
    if (tile + nwaves < ntiles) request(tile + nwaves);
    // layer 1 -> GELU -> this lane's operand of layer 2
    bf16x8 h[2];
#pragma unroll
    for (int t = 0; t < 4; ++t) {
      f32x4 acc = {0.f, 0.f, 0.f, 0.f};
      acc = __builtin_amdgcn_mfma_f32_16x16x32_bf16(w1b[t], xa, acc, 0, 0, 0);
      const f32x4 b1 = units(0, t);
#pragma unroll
      for (int j = 0; j < 4; ++j) h[t / 2][4 * (t & 1) + j] = to_bf16(gelu_fast(acc[j] + b1[j]));
    }
    float part = 0.0f;
#pragma unroll
    for (int t = 0; t < 4; ++t) {
      f32x4 acc = units(1, t);
      const f32x4 w3 = units(2, t);
      acc = __builtin_amdgcn_mfma_f32_16x16x32_bf16(w2b[t][0], h[0], acc, 0, 0, 0);
      acc = __builtin_amdgcn_mfma_f32_16x16x32_bf16(w2b[t][1], h[1], acc, 0, 0, 0);
#pragma unroll
      for (int j = 0; j < 4; ++j) part += gelu_fast(acc[j]) * w3[j];
    }
    // layer 3: the four lanes that hold the row's units
    part += __shfl_xor(part, 16, 64);
    part += __shfl_xor(part, 32, 64);
    if (grp == 0 && rr < total) logits[rr] = part + b3;
  }
}

hipError_t launch_mlp_infer(const float *w, const float *mean, const float *std, const float *X, const uint32_t *rows,
                            const uint32_t *nrows_dev, int64_t n, float *logits, hipStream_t s) {
  int64_t tiles = (n + 15) / 16;
  int64_t blocks = (tiles + 3) / 4;
  if (blocks > 4096) blocks = 4096;
  if (blocks < 1) blocks = 1;
  hipLaunchKernelGGL(k_mlp_infer_bf16, dim3((unsigned)blocks), dim3(256), 0, s, w, mean, std, X, rows, nrows_dev, n,
                     logits);
  return hipGetLastError();
}

// ---------------------------------------------------- classify candidates

// Candidates' features are the rows feat[cand[k] * 16]; logit k belongs to
// particle cand[k].  Decide: logit >= margin -> surface, <= -margin ->
// interior, otherwise append to the fallback list for the scan pass.
template <int DIM>
__global__ void __launch_bounds__(256) k_decide(Phys P, Rates out, const uint32_t *__restrict__ cand,
                                                const uint32_t *__restrict__ n_cand, const float *__restrict__ lg,
                                                float margin, uint32_t *__restrict__ fallback, Scalars *sc) {
  const uint32_t total = *n_cand;
  const uint32_t stride = gridDim.x * blockDim.x;
  // every lane runs the same number of iterations (wave-level atomics inside)
  const uint32_t iters = (total + stride - 1) / stride;
  for (uint32_t it = 0; it < iters; ++it) {
    const uint32_t k = it * stride + blockIdx.x * blockDim.x + threadIdx.x;
    const bool on = k < total;
    uint32_t i = 0;
    float l = 0.0f;
    bool fb = false, fs = false;
    if (on) {
      i = cand[k];
      l = lg[k];
      out.logit[i] = l;
      fb = fabsf(l) < margin;
      fs = !fb && l > 0.0f;
    }
    const uint32_t slot = wave_append(&sc->n_scan, on && fb);
    if (on && fb) fallback[slot] = i;
    wave_count(&tally_of(sc).n_mlp, on && !fb);
    if (on && !fb) {
      uint32_t fl = out.flags[i] | kFlagByMLP;
      if (fs) {
        fl |= kFlagFS;
        if ((P.flags & SPH_F_FS_PROJECT) && (P.flags & SPH_F_PST)) {
          const double n0 = out.nrm[0][i], n1 = out.nrm[1][i], n2 = DIM == 3 ? out.nrm[2][i] : 0.0;
          double u0 = out.dus[0][i], u1 = out.dus[1][i], u2 = DIM == 3 ? out.dus[2][i] : 0.0;
          double d = u0 * n0 + u1 * n1 + u2 * n2;
          out.dus[0][i] = u0 - d * n0;
          out.dus[1][i] = u1 - d * n1;
          if (DIM == 3) out.dus[2][i] = u2 - d * n2;
        }
      }
      out.flags[i] = fl;
    }
    wave_count(&tally_of(sc).n_fs, on && fs);
  }
}

hipError_t launch_classify(const Classifier &c, const Rates &r, const uint32_t *cand, const uint32_t *n_cand,
                           uint32_t *fallback, Scalars *sc, const Phys &P, uint32_t nf, float *lgbuf, hipStream_t s) {
  if (nf == 0) return hipSuccess;
  hipError_t e = launch_mlp_infer(c.w, c.mean, c.std, r.feat, cand, n_cand, nf, lgbuf, s);
  if (e != hipSuccess) return e;
  unsigned db = grid_for(nf);
  if (db > 1024) db = 1024;
  if (P.dim == 2)
    hipLaunchKernelGGL(k_decide<2>, dim3(db), dim3(256), 0, s, P, r, cand, n_cand, lgbuf, c.margin, fallback, sc);
  else
    hipLaunchKernelGGL(k_decide<3>, dim3(db), dim3(256), 0, s, P, r, cand, n_cand, lgbuf, c.margin, fallback, sc);
  return hipGetLastError();
}

}  // namespace wb

// ====================================================================== ABI

using namespace wb;

struct sph_mlp {
  int64_t max_batch;
  hipStream_t s;
  float *w, *g, *m, *v, *mean, *std;
  float *part;               // the gradient kernel's block sums
  float *loss, *loss_acc;
  int64_t step;
};

namespace {

// Rows per wave and blocks of the gradient kernel for a batch: one wave per
// row up to 2,048 rows (two waves per SIMD), then more rows per wave, so that
// there are at most kGradBlocks block sums (21 KB each).
constexpr int64_t kGradBlocks = 256;

void grad_split(int64_t B, int &rpw, int &nblk) {
  constexpr int64_t waves = kGradWaves * kGradBlocks;
  rpw = (int)((B + waves - 1) / waves);
  nblk = (int)((B + kGradWaves * (int64_t)rpw - 1) / (kGradWaves * (int64_t)rpw));
}

size_t mlp_carve(sph_mlp *m, uintptr_t base, int64_t B) {
  uintptr_t off = 0;
  auto take = [&](int64_t count) {
    off = (off + 255) & ~(uintptr_t)255;
    float *p = base ? reinterpret_cast<float *>(base + off) : nullptr;
    off += (uintptr_t)(count > 0 ? count : 1) * sizeof(float);
    return p;
  };
  m->w = take(kMlpParams);
  m->g = take(kMlpParams);
  m->m = take(kMlpParams);
  m->v = take(kMlpParams);
  m->mean = take(kMlpIn);
  m->std = take(kMlpIn);
  m->part = take(std::min<int64_t>(kGradBlocks, (B + kGradWaves - 1) / kGradWaves) * kPart);  // any batch up to B
  m->loss = take(1);
  m->loss_acc = take(1);
  return off + 256;
}

// Gradient of rows off .. off + B - 1 (of perm, or of X) into m->g and the
// mean loss into m->loss; acc != null: also added to (reset: written to) *acc;
// adam != null: also the parameter update.
hipError_t mlp_loss_grad(sph_mlp *m, const float *X, const float *y, const float *w, const int32_t *perm, int64_t off,
                         int64_t B, float *acc, int acc_reset, const AdamArgs *adam) {
  int rpw, nblk;
  grad_split(B, rpw, nblk);
  hipLaunchKernelGGL(k_mlp_grad, dim3((unsigned)nblk), dim3(64 * kGradWaves), 0, m->s, m->w, m->mean, m->std, X, y, w,
                     perm, off, B, rpw, m->part);
  hipLaunchKernelGGL(k_mlp_reduce, dim3((kPart + kRedParams - 1) / kRedParams), dim3(kRedParams * kRedSlices), 0, m->s,
                     m->part, nblk, B, m->g, m->loss, acc, acc_reset, adam ? 1 : 0, adam ? *adam : AdamArgs{});
  return hipGetLastError();
}

// The next Adam update's constants (counts the step).
AdamArgs adam_next(sph_mlp *m, float lr, float b1, float b2, float eps) {
  m->step += 1;
  const float c1 = 1.0f - std::pow(b1, (float)m->step);
  const float c2 = 1.0f - std::pow(b2, (float)m->step);
  return AdamArgs{m->w, m->m, m->v, lr, b1, b2, eps, c1, c2};
}

}  // namespace

extern "C" {

size_t sph_mlp_workspace_bytes(int64_t max_batch) {
  if (max_batch <= 0 || max_batch > (1 << 24)) return 0;
  sph_mlp m;
  return mlp_carve(&m, 0, max_batch);
}

sph_status sph_mlp_create(int64_t max_batch, const float *params0, const float *mean, const float *std, void *workspace,
                          size_t ws_bytes, void *hip_stream, sph_mlp **out) {
  if (!out || !params0 || !mean || !std) return SPH_EINVAL;
  *out = nullptr;
  size_t need = sph_mlp_workspace_bytes(max_batch);
  if (need == 0) return SPH_EINVAL;
  if (!workspace || ((uintptr_t)workspace % 256) != 0 || ws_bytes < need) return SPH_EWORKSPACE;
  for (int k = 0; k < kMlpIn; ++k)
    if (!(std[k] > 0.0f) || !std::isfinite(mean[k])) return SPH_EINVAL;
  sph_mlp *m = new sph_mlp();
  m->max_batch = max_batch;
  m->s = (hipStream_t)hip_stream;
  m->step = 0;
  mlp_carve(m, (uintptr_t)workspace, max_batch);
  hipError_t e = hipMemcpyAsync(m->w, params0, sizeof(float) * kMlpParams, hipMemcpyHostToDevice, m->s);
  if (e == hipSuccess) e = hipMemcpyAsync(m->mean, mean, sizeof(float) * kMlpIn, hipMemcpyHostToDevice, m->s);
  if (e == hipSuccess) e = hipMemcpyAsync(m->std, std, sizeof(float) * kMlpIn, hipMemcpyHostToDevice, m->s);
  if (e == hipSuccess) e = hipMemsetAsync(m->m, 0, sizeof(float) * kMlpParams, m->s);
  if (e == hipSuccess) e = hipMemsetAsync(m->v, 0, sizeof(float) * kMlpParams, m->s);
  if (e == hipSuccess) e = hipStreamSynchronize(m->s);
  if (e != hipSuccess) {
    delete m;
    return SPH_EHIP;
  }
  *out = m;
  return SPH_OK;
}

void sph_mlp_destroy(sph_mlp *m) { delete m; }

sph_status sph_mlp_forward(sph_mlp *m, const float *X, int64_t B, float *logits) {
  if (!m || !X || !logits || B < 0 || B > m->max_batch) return SPH_EINVAL;
  if (B == 0) return SPH_OK;
  return launch_mlp_fwd(m->w, m->mean, m->std, X, B, logits, m->s) == hipSuccess ? SPH_OK : SPH_EHIP;
}

sph_status sph_mlp_loss_grad(sph_mlp *m, const float *X, const float *y, const float *w, int64_t B, float *loss,
                             float *grad) {
  if (!m || !X || !y || B <= 0 || B > m->max_batch) return SPH_EINVAL;
  hipError_t e = mlp_loss_grad(m, X, y, w, nullptr, 0, B, nullptr, 0, nullptr);
  if (e == hipSuccess && loss) e = hipMemcpyAsync(loss, m->loss, sizeof(float), hipMemcpyDeviceToDevice, m->s);
  if (e == hipSuccess && grad)
    e = hipMemcpyAsync(grad, m->g, sizeof(float) * kMlpParams, hipMemcpyDeviceToDevice, m->s);
  return e == hipSuccess ? SPH_OK : SPH_EHIP;
}

sph_status sph_mlp_adam(sph_mlp *m, float lr, float beta1, float beta2, float eps) {
  if (!m || !(lr > 0) || !(beta1 >= 0 && beta1 < 1) || !(beta2 >= 0 && beta2 < 1) || !(eps > 0)) return SPH_EINVAL;
  const AdamArgs A = adam_next(m, lr, beta1, beta2, eps);
  hipLaunchKernelGGL(k_mlp_adam, dim3(grid_for(kMlpParams)), dim3(256), 0, m->s, m->g, A);
  return hipGetLastError() == hipSuccess ? SPH_OK : SPH_EHIP;
}

sph_status sph_mlp_train_epoch(sph_mlp *m, const float *X, const float *y, const float *w, const int32_t *perm,
                               int64_t n, int64_t batch, float lr, float *mean_loss) {
  if (!m || !X || !y || !perm || n <= 0 || batch <= 0 || batch > m->max_batch || !(lr > 0)) return SPH_EINVAL;
  // the batch losses accumulate on the device; one synchronisation at the end
  int64_t nb = 0;
  for (int64_t off = 0; off < n; off += batch) {
    const int64_t B = std::min(batch, n - off);
    const AdamArgs A = adam_next(m, lr, 0.9f, 0.999f, 1e-8f);
    if (mlp_loss_grad(m, X, y, w, perm, off, B, m->loss_acc, nb == 0 ? 1 : 0, &A) != hipSuccess) return SPH_EHIP;
    ++nb;
  }
  if (mean_loss) {
    float l = 0.0f;
    if (hipMemcpyAsync(&l, m->loss_acc, sizeof(float), hipMemcpyDeviceToHost, m->s) != hipSuccess ||
        hipStreamSynchronize(m->s) != hipSuccess)
      return SPH_EHIP;
    *mean_loss = l / (float)nb;
  }
  return SPH_OK;
}

sph_status sph_mlp_get_params(sph_mlp *m, float *out, int32_t out_on_device) {
  if (!m || !out) return SPH_EINVAL;
  hipError_t e = hipMemcpyAsync(out, m->w, sizeof(float) * kMlpParams,
                                out_on_device ? hipMemcpyDeviceToDevice : hipMemcpyDeviceToHost, m->s);
  if (e == hipSuccess && !out_on_device) e = hipStreamSynchronize(m->s);
  return e == hipSuccess ? SPH_OK : SPH_EHIP;
}

sph_status sph_mlp_forward_noalloc(const float *params, const float *mean, const float *std, const float *X,
                                   int64_t B, float *logits, void *hip_stream) {
  if (!params || !mean || !std || !X || !logits || B < 0 || B > SPH_MLP_NOALLOC_MAX_ROWS) return SPH_EINVAL;
  if (B == 0) return SPH_OK;
  return launch_mlp_fwd(params, mean, std, X, B, logits, (hipStream_t)hip_stream) == hipSuccess ? SPH_OK : SPH_EHIP;
}

sph_status sph_mlp_infer_bf16(const float *params, const float *mean, const float *std, const float *X, int64_t n,
                              float *logits, void *hip_stream) {
  if (!params || !mean || !std || !X || !logits || n < 0) return SPH_EINVAL;
  if (n == 0) return SPH_OK;
  return launch_mlp_infer(params, mean, std, X, nullptr, nullptr, n, logits, (hipStream_t)hip_stream) == hipSuccess
             ? SPH_OK
             : SPH_EHIP;
}

}  // extern "C"
