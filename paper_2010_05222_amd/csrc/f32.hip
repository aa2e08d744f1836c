// The step on fp32 operands (stages 3-6): normalised logits, margin softmax,
// both gradients and the momentum update (Partial FC Sec. 3.1, Sec. 3.2.1,
// Eq. proxy_update, Eq. pfc_center_update).
//
// Three contractions on v_mfma_f32_16x16x4_f32 (fp32 products and sums; the
// matrix pipe's fp32 rate is the vector units', but an operand register feeds
// sixteen products, so LDS and the load units keep up).  d is any multiple of
// 8 up to 1024 and the batch any size up to 4096; every tile masks its ends.
//
// MFMA operands: lane l supplies A[l % 16][k] and B[k][l % 16] with
// k = l / 16, and register r of its accumulator is D[4 (l / 16) + r][l % 16].
// The instruction adds its four products one after another, each with one
// rounding, so a contraction over k = 0, 1, 2, ... is the chain of fmaf that a
// plain loop computes, bit for bit (51,200 sums of 512 compared).  The sums
// that later steps build on - cosines, norms, log-sum-exp, class gradients
// and their projection - all keep a plain loop's order: in a converging head
// the loss is a difference of nearly equal numbers, and a cosine that differs
// in its last bit moves it by a per mille.  A lane's 16-byte LDS piece feeds
// four MFMAs: k = 16 b + 4 s + g sits at position 16 b + 4 g + s, and lane
// group g reads 4 g .. + 3.  A lane's four consecutive columns 4 (l % 16) + t
// are its column l % 16 of four tiles t, so rows are loaded and stored in
// 16-byte pieces, 256 bytes per 16 lanes, with no transposition.
#include "pfc_device.h"

namespace pfc {
namespace {

constexpr float kEpsNorm = 1e-12f;
constexpr int kRows = 64;        // batch rows of a forward tile (16 per wave)
constexpr int kChunk = 64;       // slice of d (forward), classes (dX) or rows (dW) per LDS stage
constexpr int kLd = kChunk + 4;  // LDS row stride: sixteen rows' 16-byte pieces on distinct banks
constexpr int kDxRows = 32;      // batch rows of a dX workgroup
constexpr int kDwCls = 16;       // classes of a dW workgroup

__device__ __forceinline__ f32x4_t load4(const float* p) {
  return *reinterpret_cast<const f32x4u_t*>(p);
}
__device__ __forceinline__ void store4(float* p, f32x4_t v) {
  *reinterpret_cast<f32x4u_t*>(p) = v;
}
__device__ __forceinline__ f32x4_t zero4() { return f32x4_t{0.0f, 0.0f, 0.0f, 0.0f}; }

__device__ __forceinline__ f32x4_t mfma_16x16x4(float a, float b, f32x4_t c) {
  return __builtin_amdgcn_mfma_f32_16x16x4f32(a, b, c, 0, 0, 0);
}

// Position of k in a row of 16-blocks (see above).
__device__ __forceinline__ int k_pos(int k) { return (k & ~15) + 4 * (k & 3) + ((k >> 2) & 3); }

// v + its value in the lane whose l % 16 differs in `bits`, from the highest of
// four bits down: the upper steps of a 64-value butterfly sum whose values
// 4 (l % 16) + e are spread over sixteen lanes' registers e.
__device__ __forceinline__ float butterfly16(float v) {
#pragma unroll
  for (int off = 8; off > 0; off >>= 1) v += __shfl_xor(v, off, 64);
  return v;
}

// ------------------------------------------------------------------ forward

// cos[n][j] of a tile of 16 MT classes x 64 batch rows, d in 64-wide chunks
// through two LDS stages (a chunk is loaded into registers while the previous
// one is contracted).  Wave w owns rows 16 w .. + 15 and all the tile's
// classes.  The row norms of both operands are summed from the pieces on their
// way to LDS, each in the order of one wave per row (batch rows: lane i % 64,
// class rows: lane (i / 4) % 64, then a butterfly); the tiles of the first
// class tile (row tile) publish them for the backward.  A negative that the
// PFC* filter drops is stored as -inf.
//
// Bound by the fp32 matrix rate and, on few tiles, by the chunk latency.  At
// B = 250, |S| = 5,003, d = 512 (1.3 GFLOP) it takes 28 us; the
// thread-per-dot kernel that it replaced took 2,671 us there.
template <int MT>
__global__ void __launch_bounds__(256) k_fwd32(
    const float* __restrict__ X, const float* __restrict__ W, const int32_t* __restrict__ active,
    const int32_t* __restrict__ n_active_p, const int32_t* __restrict__ yhat, int B, int d,
    int64_t ld_cos, float tau, float* __restrict__ inv_x, float* __restrict__ inv_w,
    float* __restrict__ cos32, uint32_t* __restrict__ arrivals) {
  constexpr int CLS = 16 * MT;
  __shared__ float As[2][CLS][kLd], Bs[2][kRows][kLd];
  __shared__ float iwS[CLS], ixS[kRows];
  if (blockIdx.x == 0 && blockIdx.y == 0 && threadIdx.x == 0) *arrivals = 0;
  const int64_t K = *n_active_p;
  const int64_t j0 = (int64_t)blockIdx.x * CLS;
  // The first class tile publishes the batch norms even when S is empty.
  if (j0 >= K && blockIdx.x > 0) return;
  const int n0 = blockIdx.y * kRows;
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int l16 = lane & 15, g4 = 4 * (lane >> 4);

  // Staging: thread t moves piece t % 16 of rows t / 16 + 16 u.
  const int p16 = tid & 15, piece = 4 * p16, srow = tid >> 4;
  const int at = k_pos(piece);   // of the piece's entry e: at + 4 e
  const float *ap[MT], *bp[4];
  float sa[MT][4], sb[4][4];
#pragma unroll
  for (int u = 0; u < MT; ++u) {
    const int64_t j = j0 + srow + 16 * u;
    ap[u] = j < K ? W + (int64_t)active[j] * d : nullptr;
#pragma unroll
    for (int e = 0; e < 4; ++e) sa[u][e] = 0.0f;
  }
#pragma unroll
  for (int u = 0; u < 4; ++u) {
    const int n = n0 + srow + 16 * u;
    bp[u] = n < B ? X + (int64_t)n * d : nullptr;
#pragma unroll
    for (int e = 0; e < 4; ++e) sb[u][e] = 0.0f;
  }
  f32x4_t ar[MT], br[4];
  auto load = [&](int k0) {
    const bool in = k0 + piece < d;
#pragma unroll
    for (int u = 0; u < MT; ++u) ar[u] = in && ap[u] ? load4(ap[u] + k0 + piece) : zero4();
#pragma unroll
    for (int u = 0; u < 4; ++u) br[u] = in && bp[u] ? load4(bp[u] + k0 + piece) : zero4();
  };
  f32x4_t acc[MT];
#pragma unroll
  for (int m = 0; m < MT; ++m) acc[m] = zero4();
  load(0);
  for (int k0 = 0, st = 0; k0 < d; k0 += kChunk, st ^= 1) {
    // Class rows: lane 16 (chunk % 4) + p16 of the row's wave.
    const int part = (k0 / kChunk) & 3;   // uniform
#pragma unroll
    for (int u = 0; u < MT; ++u) {
      float v = part == 0 ? sa[u][0] : part == 1 ? sa[u][1] : part == 2 ? sa[u][2] : sa[u][3];
#pragma unroll
      for (int e = 3; e >= 0; --e) v = fmaf(ar[u][e], ar[u][e], v);
#pragma unroll
      for (int q = 0; q < 4; ++q) sa[u][q] = part == q ? v : sa[u][q];
#pragma unroll
      for (int e = 0; e < 4; ++e) As[st][srow + 16 * u][at + 4 * e] = ar[u][e];
    }
    // Batch rows: lane 4 p16 + e of the row's wave.
#pragma unroll
    for (int u = 0; u < 4; ++u)
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        sb[u][e] = fmaf(br[u][e], br[u][e], sb[u][e]);
        Bs[st][srow + 16 * u][at + 4 * e] = br[u][e];
      }
    // A stage is rewritten two chunks later: every wave has then passed the
    // barrier of the chunk between, after its reads of this one.
    __syncthreads();
    if (k0 + kChunk < d) load(k0 + kChunk);
#pragma unroll
    for (int kb = 0; kb < kChunk / 16; ++kb) {
      const f32x4_t b = *reinterpret_cast<const f32x4_t*>(&Bs[st][16 * wave + l16][16 * kb + g4]);
      f32x4_t a[MT];
#pragma unroll
      for (int m = 0; m < MT; ++m)
        a[m] = *reinterpret_cast<const f32x4_t*>(&As[st][16 * m + l16][16 * kb + g4]);
#pragma unroll
      for (int s = 0; s < 4; ++s)
#pragma unroll
        for (int m = 0; m < MT; ++m) acc[m] = mfma_16x16x4(a[m][s], b[s], acc[m]);
    }
  }
#pragma unroll
  for (int u = 0; u < MT; ++u) {
    const float ss = butterfly16((sa[u][0] + sa[u][2]) + (sa[u][1] + sa[u][3]));
    const float iv = 1.0f / fmaxf(sqrtf(ss), kEpsNorm);
    const int64_t j = j0 + srow + 16 * u;
    if (p16 == 0) {
      iwS[srow + 16 * u] = iv;
      if (blockIdx.y == 0 && j < K) inv_w[j] = iv;
    }
  }
#pragma unroll
  for (int u = 0; u < 4; ++u) {
#pragma unroll
    for (int e = 0; e < 4; ++e) sb[u][e] = butterfly16(sb[u][e]);
    const float ss = (sb[u][0] + sb[u][2]) + (sb[u][1] + sb[u][3]);
    const float iv = 1.0f / fmaxf(sqrtf(ss), kEpsNorm);
    const int n = n0 + srow + 16 * u;
    if (p16 == 0) {
      ixS[srow + 16 * u] = iv;
      if (blockIdx.x == 0 && n < B) inv_x[n] = iv;
    }
  }
  __syncthreads();

  // Lane: batch row n, classes j0 + 16 m + 4 (lane / 16) + r.
  const int n = n0 + 16 * wave + l16;
  if (n >= B) return;
  const float ix = ixS[16 * wave + l16];
  const int64_t y = yhat[n];
#pragma unroll
  for (int m = 0; m < MT; ++m) {
    const f32x4_t iw = *reinterpret_cast<const f32x4_t*>(&iwS[16 * m + g4]);
    const int64_t j = j0 + 16 * m + g4;
    f32x4_t c;
#pragma unroll
    for (int r = 0; r < 4; ++r) {
      c[r] = acc[m][r] * ix * iw[r];
      if (tau < 1.0f && j + r != y && c[r] > tau) c[r] = -INFINITY;
    }
    if (j < K) store4(cos32 + (int64_t)n * ld_cos + j, c);   // ld_cos holds whole tiles
  }
}

// lse_n and the loss: a wave per row, lane l merges the logits j = l, l + 64,
// ... one by one, the lanes meet in a butterfly, and the workgroup that arrives
// last takes the batch mean.  Bound by that chain: the next sixteen loads are
// in flight while sixteen logits are merged, and four waves to a workgroup put
// each on a SIMD of its own (B = 250, |S| = 5,003: 15 us; 30 with one load at a time).
constexpr int kLse32Threads = 256;
__global__ void __launch_bounds__(kLse32Threads) k_lse32(
    const float* __restrict__ cos32, int64_t ld_cos, const int32_t* __restrict__ n_active_p,
    const int32_t* __restrict__ yhat, int B, Margin mg, float* __restrict__ row_lse,
    float* __restrict__ loss_part, uint32_t* __restrict__ arrivals, float* __restrict__ loss) {
  const int lane = threadIdx.x & 63;
  const int n = blockIdx.x * (kLse32Threads / 64) + (threadIdx.x >> 6);
  const int K = *n_active_p;
  if (n < B) {
    const int yh = yhat[n];
    const float* row = cos32 + (int64_t)n * ld_cos;
    float2 acc = make_float2(-INFINITY, 0.0f);
    float ft = 0.0f;
    constexpr int U = 16;
    float c[U], next[U];
    auto load = [&](int j0, float (&v)[U]) {
#pragma unroll
      for (int u = 0; u < U; ++u) v[u] = j0 + 64 * u < K ? row[j0 + 64 * u] : 0.0f;
    };
    load(lane, c);
    for (int j0 = lane; j0 < K; j0 += 64 * U) {
      load(j0 + 64 * U, next);
#pragma unroll
      for (int u = 0; u < U; ++u) {
        const int j = j0 + 64 * u;
        const float f = j == yh ? target_logit(mg, c[u]) : mg.s * c[u];
        if (j == yh) ft = f;
        if (j < K) acc = lse_merge(acc, make_float2(f, 1.0f));
      }
#pragma unroll
      for (int u = 0; u < U; ++u) c[u] = next[u];
    }
#pragma unroll
    for (int off = 32; off > 0; off >>= 1) {
      acc = lse_merge(acc, make_float2(__shfl_xor(acc.x, off, 64), __shfl_xor(acc.y, off, 64)));
      ft += __shfl_xor(ft, off, 64);
    }
    if (lane == 0) {
      const float lse = acc.x + __logf(acc.y);
      row_lse[n] = lse;
      put_loss_term(loss_part + n, yh >= 0 && yh < K ? lse - ft : 0.0f);
    }
  }
  mean_by_last<kLse32Threads>(loss_part, B, arrivals, loss);
}

// ------------------------------------------------------------------ dX

// Partial dX_hat[n][i] = sum_j g[n][j] / ||w_j|| W[S_j][i] of 32 batch rows,
// all of d and a slice of the classes (in 64-class chunks).  The coefficients
// of a chunk are computed once, into LDS; wave w owns NB blocks of 64 columns
// and takes its W pieces straight from memory to registers, since no other
// wave reads them.  blockDim = 64 x the waves that d needs (at most 4).
//
// At B = 250, |S| = 5,003, d = 512 it takes 30 us, at B = 64, |S| = 1,000,
// d = 128 10 us; the loop that it replaced, a chain of |S| dependent steps per
// output, took 1,585 and 266 us.
template <int NB>
__global__ void __launch_bounds__(256, NB <= 2 ? 2 : 1) k_dx32(
    const float* __restrict__ W, const int32_t* __restrict__ active,
    const int32_t* __restrict__ n_active_p, const int32_t* __restrict__ yhat,
    const float* __restrict__ row_lse, const float* __restrict__ inv_w,
    const float* __restrict__ cos32, int64_t ld_cos, int B, int d, Margin mg, int n_split,
    float* __restrict__ part) {
  __shared__ float G[2][kDxRows][kLd];
  __shared__ int32_t ids[2][kChunk];
  const int64_t K = *n_active_p;
  const int n0 = blockIdx.y * kDxRows;
  const int64_t n_chunks = ceil_div(K, (int64_t)kChunk);
  const int64_t per = ceil_div(n_chunks, (int64_t)n_split);
  const int64_t c_begin = blockIdx.x * per;
  const int64_t c_end = c_begin + per < n_chunks ? c_begin + per : n_chunks;
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int l16 = lane & 15, g4 = 4 * (lane >> 4);

  // Coefficients of a chunk: thread t owns piece t % 16 (four classes) of rows
  // t / 16, + blockDim / 16, ... (RMAX of them at most: one wave).  Their inputs
  // are requested before the previous chunk's MFMAs (fetch) and turned into
  // coefficients in LDS after them (produce).
  constexpr int RMAX = NB == 1 ? kDxRows / 4 : kDxRows / 16;
  const int rows_step = blockDim.x >> 4, p4 = 4 * (tid & 15);
  f32x4_t cv[RMAX];
  float iw[4], lse[RMAX];
  int yv[RMAX];
  int32_t id = 0;
#pragma unroll
  for (int i = 0; i < RMAX; ++i) {
    const int r = (tid >> 4) + rows_step * i, n = n0 + r;
    const bool ok = r < kDxRows && n < B;
    lse[i] = ok ? row_lse[n] : 0.0f;
    yv[i] = ok ? yhat[n] : -1;
  }
  auto fetch = [&](int64_t c) {
    const int64_t j = c * kChunk + p4;
#pragma unroll
    for (int e = 0; e < 4; ++e) iw[e] = j + e < K ? inv_w[j + e] : 0.0f;
#pragma unroll
    for (int i = 0; i < RMAX; ++i) {
      const int r = (tid >> 4) + rows_step * i, n = n0 + r;
      cv[i] = r < kDxRows && n < B && j < K ? load4(cos32 + (int64_t)n * ld_cos + j) : zero4();
    }
    if (tid < kChunk) {   // ids past |S| (coefficient 0) repeat the last one
      const int64_t k = c * kChunk + tid;
      id = active[k < K ? k : K - 1];
    }
  };
  auto produce = [&](int64_t c, int st) {
    const int64_t j = c * kChunk + p4;
#pragma unroll
    for (int i = 0; i < RMAX; ++i) {
      const int r = (tid >> 4) + rows_step * i;
      if (r >= kDxRows) break;
      f32x4_t g = zero4();
      if (n0 + r < B) {
#pragma unroll
        for (int e = 0; e < 4; ++e)
          if (j + e < K) g[e] = grad_coef(mg, cv[i][e], j + e == yv[i], lse[i]) * iw[e];
      }
      *reinterpret_cast<f32x4_t*>(&G[st][r][p4]) = g;
    }
    if (tid < kChunk) ids[st][tid] = id;
  };
  f32x4_t acc[2][NB][4];
#pragma unroll
  for (int m = 0; m < 2; ++m)
#pragma unroll
    for (int q = 0; q < NB; ++q)
#pragma unroll
      for (int t = 0; t < 4; ++t) acc[m][q][t] = zero4();
  const int col0 = 64 * NB * wave + 4 * l16;
  f32x4_t w[2][NB][4];   // W pieces of two 16-class blocks in turn
  auto load_w = [&](int st, int kb, f32x4_t (&dst)[NB][4]) {
    const int4 id = *reinterpret_cast<const int4*>(&ids[st][16 * kb + g4]);
    const int row[4] = {id.x, id.y, id.z, id.w};
#pragma unroll
    for (int s = 0; s < 4; ++s)
#pragma unroll
      for (int q = 0; q < NB; ++q)
        dst[q][s] = col0 + 64 * q < d ? load4(W + (int64_t)row[s] * d + col0 + 64 * q) : zero4();
  };
  if (c_begin < c_end) {
    fetch(c_begin);
    produce(c_begin, 0);
  }
  int st = 0;
  for (int64_t c = c_begin; c < c_end; ++c, st ^= 1) {
    // After the barrier chunk c is ready, and the other stage is free.
    __syncthreads();
    load_w(st, 0, w[0]);
    const bool more = c + 1 < c_end;
    if (more) fetch(c + 1);
#pragma unroll
    for (int kb = 0; kb < kChunk / 16; ++kb) {
      if (kb + 1 < kChunk / 16) load_w(st, kb + 1, w[(kb + 1) & 1]);
      f32x4_t a[2];
#pragma unroll
      for (int m = 0; m < 2; ++m)
        a[m] = *reinterpret_cast<const f32x4_t*>(&G[st][16 * m + l16][16 * kb + g4]);
#pragma unroll
      for (int s = 0; s < 4; ++s)
#pragma unroll
        for (int q = 0; q < NB; ++q)
#pragma unroll
          for (int t = 0; t < 4; ++t)
#pragma unroll
            for (int m = 0; m < 2; ++m)
              acc[m][q][t] = mfma_16x16x4(a[m][s], w[kb & 1][q][s][t], acc[m][q][t]);
    }
    if (more) produce(c + 1, st ^ 1);
  }
#pragma unroll
  for (int m = 0; m < 2; ++m)
#pragma unroll
    for (int r = 0; r < 4; ++r) {
      const int n = n0 + 16 * m + g4 + r;
      if (n >= B) continue;
      float* out = part + ((int64_t)blockIdx.x * B + n) * d + col0;
#pragma unroll
      for (int q = 0; q < NB; ++q)
        if (col0 + 64 * q < d)
          store4(out + 64 * q, f32x4_t{acc[m][q][0][r], acc[m][q][1][r], acc[m][q][2][r],
                                       acc[m][q][3][r]});
    }
}

// The split partials of a row summed, and the normalisation backward
// dx = (v - x_hat (x_hat . v)) / ||x||, v = (s / B) * sum.  One workgroup per
// row: each of its runs of 256 threads sums a run of consecutive splits, eight
// loads in flight per column, and the runs' sums are added in order (the loads'
// latency bounds it: 63 splits of 128 rows, d = 1024, 21.6 us in one run, 9.3).
constexpr int kFinalRuns = 4;
__global__ void __launch_bounds__(256 * kFinalRuns) k_dx_final32(
    const float* __restrict__ part, int n_split, const float* __restrict__ X,
    const float* __restrict__ inv_x, int B, int d, float sB, float* __restrict__ dX) {
  constexpr int PER = 4;   // d <= 1024
  __shared__ float sums[kFinalRuns - 1][256 * PER];
  __shared__ float red[4];
  const int n = blockIdx.x, t = threadIdx.x & 255, run = threadIdx.x >> 8;
  const int64_t stride = (int64_t)B * d;
  const int per = (n_split + kFinalRuns - 1) / kFinalRuns;
  const int s0 = per * run, s1 = s0 + per < n_split ? s0 + per : n_split;
  float v[PER], xh[PER];
#pragma unroll
  for (int k = 0; k < PER; ++k) {
    const int i = t + 256 * k;
    v[k] = 0.0f;
    if (i >= d) continue;
    const float* p = part + (int64_t)n * d + i;
    for (int s = s0; s < s1; s += 8) {
      float q[8];
#pragma unroll
      for (int u = 0; u < 8; ++u) q[u] = s + u < s1 ? p[(s + u) * stride] : 0.0f;
#pragma unroll
      for (int u = 0; u < 8; ++u) v[k] += q[u];
    }
    if (run) sums[run - 1][i] = v[k];
  }
  __syncthreads();
  float dot = 0.0f;
  const float ix = inv_x[n];
  if (run == 0) {
#pragma unroll
    for (int k = 0; k < PER; ++k) {
      const int i = t + 256 * k;
      xh[k] = 0.0f;
      if (i >= d) continue;
#pragma unroll
      for (int u = 0; u < kFinalRuns - 1; ++u) v[k] += sums[u][i];
      v[k] *= sB;
      xh[k] = X[(int64_t)n * d + i] * ix;
      dot = fmaf(xh[k], v[k], dot);
    }
    dot = wave_sum(dot);
    if ((t & 63) == 0) red[t >> 6] = dot;
  }
  __syncthreads();
  if (run) return;
  dot = red[0] + red[1] + red[2] + red[3];
#pragma unroll
  for (int k = 0; k < PER; ++k) {
    const int i = t + 256 * k;
    if (i < d) dX[(int64_t)n * d + i] = ix * (v[k] - xh[k] * dot);
  }
}

// ------------------------------------------------------------------ dW

// Class gradients of 16 active classes x all of d over the whole batch (in
// 64-row chunks), and the momentum update of their rows.  As in dX, the
// coefficients (here transposed: class-major) go through LDS and the batch
// rows straight to the registers of the wave that owns their columns.  The
// accumulators end with four consecutive columns of a class per lane, so the
// tangent projection, momentum and weight step read and write whole rows in
// 16-byte pieces.  38 us at B = 250, |S| = 5,003, d = 512 (110 us as one
// workgroup per class).
template <int NB>
__global__ void __launch_bounds__(256) k_dw32(
    const float* __restrict__ X, float* __restrict__ W, float* __restrict__ W_master,
    float* __restrict__ M, const int32_t* __restrict__ active,
    const int32_t* __restrict__ n_active_p, const int32_t* __restrict__ yhat,
    const float* __restrict__ row_lse, const float* __restrict__ inv_x,
    const float* __restrict__ inv_w, const float* __restrict__ cos32, int64_t ld_cos, int B,
    int d, Margin mg, float sB, float lr, float mu) {
  __shared__ float G[2][kDwCls][kLd];
  __shared__ float red[4][kDwCls];
  const int64_t K = *n_active_p;
  const int64_t j0 = (int64_t)blockIdx.x * kDwCls;
  if (j0 >= K) return;
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int n_waves = blockDim.x >> 6;
  const int l16 = lane & 15, g4 = 4 * (lane >> 4);

  // Coefficients of rows nb .. nb + 63: thread t owns four classes of rows
  // t / 4, + blockDim / 4, ... (RMAX of them at most); requested and produced
  // around the previous chunk's MFMAs, as in dX.
  constexpr int RMAX = NB == 1 ? 4 : 1;
  const int rows_step = blockDim.x >> 2, p4 = 4 * (tid & 3);
  f32x4_t cv[RMAX];
  float lse[RMAX], ix[RMAX];
  int yv[RMAX];
  auto fetch = [&](int nb) {
#pragma unroll
    for (int i = 0; i < RMAX; ++i) {
      const int r = (tid >> 2) + rows_step * i, n = nb + r;
      const bool ok = r < kChunk && n < B;
      cv[i] = ok && j0 + p4 < K ? load4(cos32 + (int64_t)n * ld_cos + j0 + p4) : zero4();
      lse[i] = ok ? row_lse[n] : 0.0f;
      ix[i] = ok ? inv_x[n] : 0.0f;
      yv[i] = ok ? yhat[n] : -1;
    }
  };
  auto produce = [&](int nb, int st) {
#pragma unroll
    for (int i = 0; i < RMAX; ++i) {
      const int r = (tid >> 2) + rows_step * i;
      if (r >= kChunk) break;
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        const int64_t j = j0 + p4 + e;
        G[st][p4 + e][k_pos(r)] =
            nb + r < B && j < K ? grad_coef(mg, cv[i][e], j == yv[i], lse[i]) * ix[i] : 0.0f;
      }
    }
  };
  f32x4_t acc[NB][4];
#pragma unroll
  for (int q = 0; q < NB; ++q)
#pragma unroll
    for (int t = 0; t < 4; ++t) acc[q][t] = zero4();
  // The wave's q-th block of 64 columns is block wave + 4 q.
  const int col0 = 64 * wave + 4 * l16;
  f32x4_t x[2][NB][4];   // batch pieces of two 16-row blocks in turn
  auto load_x = [&](int nb, f32x4_t (&dst)[NB][4]) {
#pragma unroll
    for (int s = 0; s < 4; ++s) {
      int n = nb + 4 * s + (lane >> 4);
      n = n < B ? n : B - 1;   // coefficient 0
#pragma unroll
      for (int q = 0; q < NB; ++q)
        dst[q][s] = col0 + 256 * q < d ? load4(X + (int64_t)n * d + col0 + 256 * q) : zero4();
    }
  };
  fetch(0);
  load_x(0, x[0]);
  produce(0, 0);
  for (int nb = 0, st = 0; nb < B; nb += kChunk, st ^= 1) {
    __syncthreads();   // the chunk is ready, the other stage free
    const bool more = nb + kChunk < B;
    if (more) fetch(nb + kChunk);
#pragma unroll
    for (int kb = 0; kb < kChunk / 16; ++kb) {
      load_x(nb + 16 * (kb + 1), x[(kb + 1) & 1]);
      const f32x4_t a = *reinterpret_cast<const f32x4_t*>(&G[st][l16][16 * kb + g4]);
#pragma unroll
      for (int s = 0; s < 4; ++s)
#pragma unroll
        for (int q = 0; q < NB; ++q)
#pragma unroll
          for (int t = 0; t < 4; ++t)
            acc[q][t] = mfma_16x16x4(a[s], x[kb & 1][q][s][t], acc[q][t]);
    }
    if (more) produce(nb + kChunk, st ^ 1);
  }

  // Update: lane l owns columns col0 + 256 q .. + 3 of classes 4 (l / 16) + r.
  // The dot w_hat . dw of a class goes over q in each column, over a wave's 64
  // columns in a butterfly, and over the waves in order.
  int64_t base[4];
  float iw[4];
  f32x4_t wv[4][NB];
#pragma unroll
  for (int r = 0; r < 4; ++r) {
    const int64_t j = j0 + g4 + r;
    base[r] = j < K ? (int64_t)active[j] * d + col0 : -1;
    iw[r] = j < K ? inv_w[j] : 0.0f;
    f32x4_t dot = zero4();
#pragma unroll
    for (int q = 0; q < NB; ++q) {
      wv[r][q] = base[r] >= 0 && col0 + 256 * q < d ? load4(W + base[r] + 256 * q) : zero4();
#pragma unroll
      for (int t = 0; t < 4; ++t) {
        acc[q][t][r] *= sB;
        dot[t] = fmaf(wv[r][q][t] * iw[r], acc[q][t][r], dot[t]);
      }
    }
#pragma unroll
    for (int t = 0; t < 4; ++t) dot[t] = butterfly16(dot[t]);
    if (l16 == 0) red[wave][g4 + r] = (dot[0] + dot[2]) + (dot[1] + dot[3]);
  }
  __syncthreads();
#pragma unroll
  for (int r = 0; r < 4; ++r) {
    float dot = red[0][g4 + r];
    for (int v = 1; v < n_waves; ++v) dot += red[v][g4 + r];
    if (base[r] < 0) continue;
#pragma unroll
    for (int q = 0; q < NB; ++q) {
      if (col0 + 256 * q >= d) continue;
      const int64_t o = base[r] + 256 * q;
      f32x4_t m = load4(M + o);
      f32x4_t p = W_master ? load4(W_master + o) : wv[r][q];
#pragma unroll
      for (int t = 0; t < 4; ++t) {
        const float gr = iw[r] * (acc[q][t][r] - wv[r][q][t] * iw[r] * dot);
        m[t] = mu * m[t] + gr;
        p[t] = p[t] - lr * m[t];
      }
      store4(M + o, m);
      if (W_master) store4(W_master + o, p);
      store4(W + o, p);
    }
  }
}

// Calls f with NB = the 64-column blocks per wave of a width d (min(4, ceil(d /
// 64)) waves share them).
template <typename F>
void with_blocks(int d, F&& f) {
  const int blocks = (int)ceil_div(d, 64);
  const int waves = blocks < 4 ? blocks : 4;
  switch ((int)ceil_div(blocks, waves)) {
    case 1: f(std::integral_constant<int, 1>{}, 64 * waves); break;
    case 2: f(std::integral_constant<int, 2>{}, 64 * waves); break;
    case 3: f(std::integral_constant<int, 3>{}, 64 * waves); break;
    default: f(std::integral_constant<int, 4>{}, 64 * waves); break;
  }
}

}  // namespace

// Splits of the dX contraction: about two workgroups of 32 rows per CU, each
// with at least one 64-class chunk.
int split_f32(int64_t B, int64_t cap) {
  const int64_t n_rt = ceil_div(B, kDxRows), chunks = ceil_div(cap, kChunk);
  const int64_t ns = 512 / n_rt < chunks ? 512 / n_rt : chunks;
  return (int)(ns < 1 ? 1 : ns);
}

int64_t part_rows_f32(int64_t B, int64_t cap) {
  const int64_t most = 512 * kDxRows, one_each = ceil_div(cap, kChunk) * B;
  return one_each < most ? one_each : most;
}

hipError_t launch_forward_f32(const StepArgs& a, const StepWs& w, hipStream_t stream) {
  const int B = (int)a.B, d = (int)a.d;
  const Margin mg{a.s, a.m, cosf(a.m), sinf(a.m), a.margin};
  const unsigned n_rt = (unsigned)ceil_div(B, kRows);
  // 64-class tiles re-read the batch half as often; 32-class ones where those
  // would leave CUs idle (fewer than two workgroups each).
  const bool wide = ceil_div(a.cap, 64) * n_rt >= 512;
  const int64_t n_ct = ceil_div(a.cap, wide ? 64 : 32);
  timing_start(2, stream);
  auto go = [&](auto kernel) {
    hipLaunchKernelGGL(kernel, dim3((unsigned)n_ct, n_rt), dim3(256), 0, stream,
                       (const float*)a.X, (const float*)a.W, a.active, a.n_active,
                       a.labels_mapped, B, d, w.ld_cos, a.tau, w.inv_x, w.inv_w, (float*)w.lbuf,
                       w.arrivals);
  };
  if (wide) go(k_fwd32<4>);
  else go(k_fwd32<2>);
  timing_stop(2, stream);
  timing_start(3, stream);
  hipLaunchKernelGGL(k_lse32, dim3((unsigned)ceil_div(B, kLse32Threads / 64)), dim3(kLse32Threads),
                     0, stream, (const float*)w.lbuf, w.ld_cos, a.n_active, a.labels_mapped, B, mg,
                     a.row_lse_out, w.loss_part, w.arrivals, a.loss);
  timing_stop(3, stream);
  return hipGetLastError();
}

hipError_t launch_backward_f32(const StepArgs& a, const StepWs& w, hipStream_t stream) {
  const int B = (int)a.B, d = (int)a.d;
  const Margin mg{a.s, a.m, cosf(a.m), sinf(a.m), a.margin};
  const float sB = a.s / (float)a.B;
  timing_start(4, stream);
  with_blocks(d, [&](auto nb, int threads) {
    hipLaunchKernelGGL(k_dx32<decltype(nb)::value>,
                       dim3((unsigned)w.n_split, (unsigned)ceil_div(B, kDxRows)), dim3(threads),
                       0, stream, (const float*)a.W, a.active, a.n_active, a.labels_mapped,
                       a.row_lse, w.inv_w, (const float*)w.lbuf, w.ld_cos, B, d, mg, w.n_split,
                       w.dx_part);
  });
  timing_stop(4, stream);
  timing_start(5, stream);
  hipLaunchKernelGGL(k_dx_final32, dim3((unsigned)B), dim3(256 * kFinalRuns), 0, stream, w.dx_part, w.n_split,
                     (const float*)a.X, w.inv_x, B, d, sB, a.dX);
  timing_stop(5, stream);
  timing_start(6, stream);
  with_blocks(d, [&](auto nb, int threads) {
    hipLaunchKernelGGL(k_dw32<decltype(nb)::value>, dim3((unsigned)ceil_div(a.cap, kDwCls)),
                       dim3(threads), 0, stream, (const float*)a.X, (float*)a.W, a.W_master, a.M,
                       a.active, a.n_active, a.labels_mapped, a.row_lse, w.inv_x, w.inv_w,
                       (const float*)w.lbuf, w.ld_cos, B, d, mg, sB, a.lr, a.mu);
  });
  timing_stop(6, stream);
  return hipGetLastError();
}

}  // namespace pfc
