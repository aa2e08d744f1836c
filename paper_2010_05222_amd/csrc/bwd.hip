// Stage 6: backward through the sampled margin softmax and both
// normalisations, and lazy momentum SGD on the active rows
// (Partial FC Eq. proxy_update, Eq. pfc_center_update, Sec. 3.2.1 matrix form:
// G = (P - Y)/B, dW = X^T G, dX = G W^T, restricted to the active set S).
//
// With dcos = (s/B) g and g_{nj} = (p_{nj} - [j = y_n]) * slope_{nj}, the
// contractions run over the non-target part p_{nj} only (p <= 1, which keeps
// the 16-bit operands in range), rebuilt on the fly from the forward's logit
// store as p = E * gscale (E = 2^(f - m) per row and 128-class group, zero at
// targets and past |S|; gscale = 2^(m - lse log2 e) per row and group).  The
// single target term of each row, (p_t - 1) * slope_t, is added exactly in
// fp32 outside the MFMA loops.
//
// dX (k_dx16): split-K MFMA contraction over classes, dX_hat^T[i][n] =
//   sum_j W[S_j][i] * p_{nj} / ||w_j||.  A workgroup owns 128 batch rows x all
//   of d and a slice of the classes.  The gathered W rows go straight from
//   HBM into a three-stage LDS ring (direct-to-LDS loads) and are read as MFMA
//   operands with transposing LDS reads, so they are never staged in
//   registers.  k_dx_final sums the split partials in a fixed order, adds the
//   target terms and applies the normalisation backward of x.
// dW + update (k_dw16): a workgroup (eight waves, two per SIMD) owns 128
//   active classes x all of d and reduces over the whole batch, so its
//   epilogue has complete rows: target terms, tangent projection, momentum,
//   weight step and the scatter into the persistent W / momentum rows (unique
//   rows, no atomics).  It runs after the dX kernels, which read the old W.
#include <math.h>

#include <atomic>

#include "pfc_gemm.h"

namespace pfc {
namespace {

constexpr float kLog2e = 1.4426950408889634f;
constexpr int kBwKC = 32;          // reduction chunk: classes (dX) or batch rows (dW)
constexpr int kRowLd = 528;        // LDS row stride of a DMA'd row of up to 512 (1 KB + 32 B)
constexpr int kRowStage = kBwKC * kRowLd;
constexpr int kDxRows = 128;       // batch rows of a dX workgroup
constexpr int kDwCls = 128;        // classes of a dW workgroup
constexpr int kTLd = 260;         // LDS row stride (floats) of the update's staged gradient rows
constexpr int kHitCap = 256;      // target rows listed per wave of a dW workgroup
constexpr int kGateSpins = 512;   // polls of a dW start gate before the workgroup goes ahead anyway

// Every operand reaches LDS through direct-to-LDS loads into three-stage
// rings (one array per stage, so the compiler can keep later stages in
// flight while a stage is read); the coefficient producer reads the raw
// logit-store values from LDS and writes the 16-bit MFMA operand back to LDS.
//
// dX: W rows, raw logit-store values [128 rows x 32 classes], 1/||w|| of the
// chunk, the rows' scales, and the coefficient tile (K-major, 64-byte rows).
__shared__ __attribute__((aligned(1024))) uint16_t xW0[kRowStage], xW1[kRowStage], xW2[kRowStage];
__shared__ __attribute__((aligned(1024))) int16_t xR0[kDxRows * kBwKC], xR1[kDxRows * kBwKC],
    xR2[kDxRows * kBwKC];
__shared__ __attribute__((aligned(16))) float xI0[kBwKC], xI1[kBwKC], xI2[kBwKC];
__shared__ __attribute__((aligned(16))) float xS0[kDxRows], xS1[kDxRows], xS2[kDxRows];
__shared__ __attribute__((aligned(1024))) uint16_t xG0[kDxRows * kBwKC], xG1[kDxRows * kBwKC],
    xG2[kDxRows * kBwKC];
// dX: active row ids of four chunks (a ring: chunk c in slot c % 4).
__shared__ __attribute__((aligned(16))) int32_t xIds[4][kBwKC];
// dW: X^T rows (K-major: d rows of 32 batch rows, bf16), raw logit-store
// values [32 rows x 128 classes] (16-byte pieces swizzled per row), the rows'
// scales, and the coefficient tile G^T (K-major: 128 class rows of 32 batch
// rows).  After the loop the X^T stages (33 KB each) hold the update's staged
// gradient rows, a coefficient stage the target-row lists.
__shared__ __attribute__((aligned(1024))) uint16_t wX0[kRowStage], wX1[kRowStage], wX2[kRowStage];
__shared__ __attribute__((aligned(1024))) int16_t wR0[kBwKC * kDwCls], wR1[kBwKC * kDwCls],
    wR2[kBwKC * kDwCls];
__shared__ __attribute__((aligned(16))) float wQ0[kBwKC], wQ1[kBwKC], wQ2[kBwKC];
__shared__ __attribute__((aligned(1024))) uint16_t wG0[kDwCls * kBwKC], wG1[kDwCls * kBwKC],
    wG2[kDwCls * kBwKC];

// The same at d = 128, where a stage is a quarter as large, so that two
// workgroups share a CU (why: at k_dx16).
constexpr int kRowLd128 = 144;   // 256 B + 32 B
__shared__ __attribute__((aligned(1024))) uint16_t xV0[kBwKC * kRowLd128],
    xV1[kBwKC * kRowLd128], xV2[kBwKC * kRowLd128];
// dW: the three stages together also hold the update's 32 staged rows of 132 floats.
constexpr int kTLd128 = 132;
__shared__ __attribute__((aligned(1024))) uint16_t wV[3][128 * kBwKC];

#define PFC_STAGE3(name, T, a0, a1, a2)          \
  template <int S>                               \
  __device__ __forceinline__ T* name() {         \
    if constexpr (S == 0) return a0;             \
    else if constexpr (S == 1) return a1;        \
    else return a2;                              \
  }
PFC_STAGE3(dx_r, int16_t, xR0, xR1, xR2)
PFC_STAGE3(dx_i, float, xI0, xI1, xI2)
PFC_STAGE3(dx_s, float, xS0, xS1, xS2)
PFC_STAGE3(dx_g, uint16_t, xG0, xG1, xG2)
PFC_STAGE3(dw_r, int16_t, wR0, wR1, wR2)
PFC_STAGE3(dw_q, float, wQ0, wQ1, wQ2)
PFC_STAGE3(dw_g, uint16_t, wG0, wG1, wG2)
#undef PFC_STAGE3
template <int S, int WI>
__device__ __forceinline__ uint16_t* dx_w() {
  if constexpr (WI == 1) return S == 0 ? xV0 : S == 1 ? xV1 : xV2;
  else if constexpr (S == 0) return xW0;
  else if constexpr (S == 1) return xW1;
  else return xW2;
}
template <int S, int WI>
__device__ __forceinline__ uint16_t* dw_x() {
  if constexpr (WI == 1) return wV[S];
  else if constexpr (S == 0) return wX0;
  else if constexpr (S == 1) return wX1;
  else return wX2;
}

// Target term of a row, (p_t - 1) * slope_t, from its unmargined target cosine.
__device__ __forceinline__ float target_coef(const Margin& mg, float c, float lse) {
  const float p = __expf(target_logit(mg, c) - lse);
  return (p - 1.0f) * target_slope(mg, c);
}

// Scale of the fp16 coefficient operand of dX: a power of two that keeps
// p / ||w_j|| * scale inside the fp16 range for every active class (p <= 1).
__device__ __forceinline__ float dx_operand_scale(F16Tag, float inv_w_max) {
  return exp2f(floorf(log2f(60000.0f / fmaxf(inv_w_max, 1e-30f))));
}
__device__ __forceinline__ float dx_operand_scale(Bf16Tag, float) { return 1.0f; }

// Two floats to a packed pair of 16-bit values, round to nearest even
// (v_cvt_pk_bf16_f32 / v_cvt_f16_f32 on gfx950).
typedef __bf16 bf16x2_t __attribute__((ext_vector_type(2)));
typedef _Float16 f16x2_t __attribute__((ext_vector_type(2)));
template <typename Tag>
__device__ __forceinline__ uint32_t pack2(float a, float b);
template <>
__device__ __forceinline__ uint32_t pack2<Bf16Tag>(float a, float b) {
  const bf16x2_t v = {(__bf16)a, (__bf16)b};
  return __builtin_bit_cast(uint32_t, v);
}
template <>
__device__ __forceinline__ uint32_t pack2<F16Tag>(float a, float b) {
  const f16x2_t v = {(_Float16)a, (_Float16)b};
  return __builtin_bit_cast(uint32_t, v);
}

template <typename Tag>
__device__ __forceinline__ uint4 pack8(const float (&v)[8]) {
  uint4 o;
  o.x = pack2<Tag>(v[0], v[1]);
  o.y = pack2<Tag>(v[2], v[3]);
  o.z = pack2<Tag>(v[4], v[5]);
  o.w = pack2<Tag>(v[6], v[7]);
  return o;
}

// An MFMA operand from the two halves of a transposing read pair.
__device__ __forceinline__ uint4 frag_of(const u32x2_t& lo, const u32x2_t& hi) {
  return make_uint4(lo.x, lo.y, hi.x, hi.y);
}
__device__ __forceinline__ uint4 as_uint4(const u32x4_t& v) { return make_uint4(v.x, v.y, v.z, v.w); }

template <typename T, int NB>
__device__ __forceinline__ void zero_acc(T (&acc)[4][NB]) {
#pragma unroll
  for (int mb = 0; mb < 4; ++mb)
#pragma unroll
    for (int nb = 0; nb < NB; ++nb)
#pragma unroll
      for (int r = 0; r < 16; ++r) acc[mb][nb][r] = 0.0f;
}

// ------------------------------------------------------------------ dX

// D = 128 * WI; 2 * WI waves: wave (wi, wn) owns d entries [128 wi, +128) and
// batch rows [64 wn, +64) of the workgroup's 128 (4 x 2 MFMA blocks).
// Pipeline per chunk c (32 classes): the raw cosines and 1/||w|| of chunk
// c + 3 and the W rows of chunk c + 2 are requested, the coefficients of
// chunk c + 1 are produced, and chunk c is contracted.
//
// At d = 128 four waves own [0, 128) and 32 rows each (4 x 1 blocks), and two
// workgroups share a CU: two waves of 64 rows left half of the SIMDs idle (B =
// 1024, |S| = 400,000: 445 -> 342 us; the class gradient, whose eight waves now
// come twice to a CU as well, 478 -> 398).
constexpr int dx_threads(int wi) { return wi == 1 ? 256 : 128 * wi; }
template <typename Tag, int WI>
__global__ void __launch_bounds__(dx_threads(WI)) k_dx16(
    const uint16_t* __restrict__ W, const int32_t* __restrict__ act_pad,
    const int32_t* __restrict__ n_active_p, const float* __restrict__ inv_w,
    const float* __restrict__ inv_w_max, const uint16_t* __restrict__ lbuf, int64_t ld_cos,
    const float* __restrict__ gscale, int64_t ld_g, int B, int n_rt, int n_split,
    int64_t n_tiles, int64_t per_xcd, float* __restrict__ dx_part) {
  constexpr int D = 128 * WI;
  constexpr int NT = dx_threads(WI);        // threads
  constexpr int NW = NT / 64;               // waves
  constexpr int NBD = WI == 1 ? 1 : 2;      // 32-row blocks of a wave
  constexpr int WROWS = kBwKC / NW;         // W rows DMA'd by each wave per chunk
  constexpr int RDMA = 8 / NW;              // 1-KB logit-store blocks DMA'd by each wave
  constexpr int GROUPS = 512 / NT;          // 8-coefficient groups per thread per chunk
  constexpr int LD = WI == 1 ? kRowLd128 : kRowLd;   // LDS row stride of the W rows
  constexpr int PER_ITER = WROWS + RDMA + 3;  // DMAs a wave issues per chunk
  const int64_t t = (int64_t)(blockIdx.x % 8) * per_xcd + blockIdx.x / 8;
  if (t >= n_tiles) return;
  // The batch-row tiles of one split share its class range: they run on one
  // XCD so the split's W rows are fetched from HBM once.
  const int split = (int)(t / n_rt);
  const int n0 = (int)(t % n_rt) * kDxRows;
  const int K = *n_active_p;
  const int64_t n_chunks = ceil_div((int64_t)K, (int64_t)kBwKC);
  const int64_t per = ceil_div(n_chunks, (int64_t)n_split);
  const int64_t c_begin = split * per;
  const int64_t c_end = c_begin + per < n_chunks ? c_begin + per : n_chunks;
  const int64_t c_stop =
      c_begin + ceil_div(c_end > c_begin ? c_end - c_begin : 0, (int64_t)3) * 3;

  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int wi = WI == 1 ? 0 : wave >> 1, wn = WI == 1 ? wave : wave & 1;
  const float scale = dx_operand_scale(Tag{}, *inv_w_max);

  // Coefficient-producer slots of this thread (fixed for the whole kernel):
  // row prow, classes 8 pchunk .. + 7 of each chunk.
  int prow[GROUPS], pchunk[GROUPS];
#pragma unroll
  for (int u = 0; u < GROUPS; ++u) {
    const int q = tid + NT * u;
    prow[u] = q >> 2;
    pchunk[u] = q & 3;
  }
  // Logit-store DMA of this lane: block b holds rows 16 b .. 16 b + 15.
  int64_t rsrc[RDMA];
#pragma unroll
  for (int v = 0; v < RDMA; ++v) {
    const int r = 16 * (wave * RDMA + v) + (lane >> 2);
    const int n = n0 + r < B ? n0 + r : B - 1;
    rsrc[v] = (int64_t)n * ld_cos + 8 * (lane & 3);
  }

  auto dma_raw = [&](auto st, int64_t c) {
    constexpr int S = decltype(st)::value;
    const int64_t jb = (c < n_chunks ? c : n_chunks - 1) * kBwKC;
#pragma unroll
    for (int v = 0; v < RDMA; ++v)
      dma16(lbuf + rsrc[v] + jb, dx_r<S>() + 512 * (wave * RDMA + v));
    // 1/||w|| of the chunk's 32 classes: 8 / NW 16-byte pieces per wave.
    if (lane < 8 / NW) dma16(inv_w + jb + 4 * (wave * (8 / NW) + lane), dx_i<S>() + 4 * wave * (8 / NW));
    // Row scales of the chunk's 128-class group for the 128 rows: 32 / NW pieces per wave.
    const float* gs = gscale + (jb / kLogitGroup) * ld_g + n0;
    if (lane < 32 / NW) dma16(gs + 4 * (wave * (32 / NW) + lane), dx_s<S>() + 4 * wave * (32 / NW));
  };
  // Active-set indices of the W rows this wave DMAs for a chunk.  The first
  // two chunks' come from scalar loads; later chunks' travel with the loads,
  // four chunks ahead, into the index ring (their wait is then the chunk's
  // load wait, not a scalar-load round trip inside the loop).  The padded copy
  // holds a valid row id at every index of a chunk.
  int32_t rows_pf[WROWS];
  auto load_rows = [&](int64_t c) {
    const int64_t jb = (c < n_chunks ? c : n_chunks - 1) * kBwKC;
#pragma unroll
    for (int v = 0; v < WROWS; ++v)
      rows_pf[v] = act_pad[__builtin_amdgcn_readfirstlane((int)(jb + wave * WROWS + v))];
  };
  auto dma_ids = [&](int64_t c) {
    const int64_t jb = (c < n_chunks ? c : n_chunks - 1) * kBwKC;
    if (lane < WROWS / 4) dma16(act_pad + jb + wave * WROWS + 4 * lane, &xIds[c & 3][wave * WROWS]);
  };
  auto read_ids = [&](int64_t c, u32x4_t (&iv)[WROWS / 4]) {
#pragma unroll
    for (int q = 0; q < WROWS / 4; ++q)
      ds_read_128<0>(iv[q], lds_addr(&xIds[c & 3][wave * WROWS + 4 * q]));
  };
  auto rows_of = [&](u32x4_t (&iv)[WROWS / 4]) {
#pragma unroll
    for (int q = 0; q < WROWS / 4; ++q) {
      rows_pf[4 * q + 0] = __builtin_amdgcn_readfirstlane((int)iv[q].x);
      rows_pf[4 * q + 1] = __builtin_amdgcn_readfirstlane((int)iv[q].y);
      rows_pf[4 * q + 2] = __builtin_amdgcn_readfirstlane((int)iv[q].z);
      rows_pf[4 * q + 3] = __builtin_amdgcn_readfirstlane((int)iv[q].w);
    }
  };
  auto dma_w = [&](auto st) {
    constexpr int S = decltype(st)::value;
#pragma unroll
    for (int v = 0; v < WROWS; ++v) {
      const int r = wave * WROWS + v;
      if (lane < D / 8) dma16(W + (int64_t)rows_pf[v] * D + 8 * lane, dx_w<S, WI>() + r * LD);
    }
  };
  // Coefficients of chunk c (K-major, rows of 32 classes): the LDS reads are
  // issued first (produce_load) and consumed later (produce_store), after an
  // lgkm wait that covers them.
  // Coefficient of (row, class): p / ||w_j|| * scale = E * gscale_row * scale * (1/||w_j||);
  // E is 0 at the row's target and past |S|, gscale 0 past the batch, so only
  // chunks past the split's end need masking.
  struct ProdIn {
    u32x4_t qv[GROUPS], i0v[GROUPS], i1v[GROUPS];
    uint32_t sv[GROUPS];
  };
  auto produce_load = [&](auto st, ProdIn& in) {
    constexpr int S = decltype(st)::value;
#pragma unroll
    for (int u = 0; u < GROUPS; ++u) {
      ds_read_128<0>(in.qv[u], lds_addr(dx_r<S>()) + (prow[u] * kBwKC + 8 * pchunk[u]) * 2);
      ds_read_128<0>(in.i0v[u], lds_addr(dx_i<S>()) + 32 * pchunk[u]);
      ds_read_128<16>(in.i1v[u], lds_addr(dx_i<S>()) + 32 * pchunk[u]);
      ds_read_32<0>(in.sv[u], lds_addr(dx_s<S>()) + 4 * prow[u]);
    }
  };
  auto produce_store = [&](auto st, int64_t c, ProdIn& in) {
    constexpr int S = decltype(st)::value;
    const bool cvalid = c < c_end;   // wave-uniform
#pragma unroll
    for (int u = 0; u < GROUPS; ++u) {
      pin_reg(in.qv[u]);
      pin_reg(in.i0v[u]);
      pin_reg(in.i1v[u]);
      pin_reg(in.sv[u]);
      const uint4 q = as_uint4(in.qv[u]);
      const uint32_t qw[4] = {q.x, q.y, q.z, q.w};
      const float iw[8] = {__uint_as_float(in.i0v[u].x), __uint_as_float(in.i0v[u].y),
                           __uint_as_float(in.i0v[u].z), __uint_as_float(in.i0v[u].w),
                           __uint_as_float(in.i1v[u].x), __uint_as_float(in.i1v[u].y),
                           __uint_as_float(in.i1v[u].z), __uint_as_float(in.i1v[u].w)};
      const float sc = cvalid ? __uint_as_float(in.sv[u]) * scale : 0.0f;
      float v[8];
#pragma unroll
      for (int e = 0; e < 8; ++e) {
        const float ev = (e & 1) ? f16_hi(qw[e >> 1]) : f16_lo(qw[e >> 1]);
        v[e] = ev * (sc * iw[e]);
      }
      const uint4 o = pack8<Tag>(v);
      ds_write_128<0>(lds_addr(dx_g<S>()) + k_major32_offset(prow[u], pchunk[u]) * 2,
                      u32x4_t{o.x, o.y, o.z, o.w});
    }
  };

  // Per-lane byte offsets of the fragment reads (see frag_mn_major and
  // frag_k_major32): W rows MN-major, coefficients K-major.
  const int fg = lane >> 4, fsrc = lane & 15;
  const uint32_t a_lane =
      ((8 * (fg >> 1) + (fsrc >> 2)) * LD + 16 * (fg & 1) + 4 * (fsrc & 3) + 128 * wi) * 2;
  const uint32_t b_lane0 = k_major32_offset(32 * NBD * wn + (lane & 31), lane >> 5) * 2;
  const uint32_t b_lane1 = k_major32_offset(32 * NBD * wn + (lane & 31), 2 + (lane >> 5)) * 2;

  f32x16_t acc[4][NBD];
  zero_acc(acc);

  if (c_begin < c_stop) {
    using S0 = std::integral_constant<int, 0>;
    using S1 = std::integral_constant<int, 1>;
    using S2 = std::integral_constant<int, 2>;
    // Prologue: raw data of chunks 0..2, W rows of chunks 0, 1; coefficients of chunk 0.
    load_rows(c_begin);
    dma_raw(S0{}, c_begin);
    dma_w(S0{});
    load_rows(c_begin + 1);
    dma_raw(S1{}, c_begin + 1);
    dma_ids(c_begin + 2);
    dma_ids(c_begin + 3);
    dma_w(S1{});
    dma_raw(S2{}, c_begin + 2);
    wait_vmcnt_lgkm0<2 * (RDMA + 1) + WROWS + 2>();
    stage_barrier();
    ProdIn in0;
    produce_load(S0{}, in0);
    lgkm_wait<0>();
    produce_store(S0{}, c_begin, in0);
    for (int64_t c = c_begin; c < c_stop; c += 3) {
      static_for<0, 3>([&](auto uu) {
        constexpr int u = decltype(uu)::value;
        const int64_t cu = c + u;
        // Landed: W rows of chunk cu, raw data of chunk cu + 1; this wave's
        // coefficient writes of the previous iteration are complete.
        wait_vmcnt_lgkm0<PER_ITER>();
        stage_barrier();
        // The row ids of chunk cu + 2 (landed: requested before the W rows of
        // chunk cu) and the producer's reads of chunk cu + 1 go first
        // (consumed while the first k-step's MFMAs run), then the fragments of
        // chunk cu...
        u32x4_t idv[WROWS / 4];
        read_ids(cu + 2, idv);
        ProdIn pin;
        produce_load(std::integral_constant<int, (u + 1) % 3>{}, pin);
        const uint32_t wb = lds_addr(dx_w<u, WI>()) + a_lane;
        const uint32_t gb0 = lds_addr(dx_g<u>()) + b_lane0;
        const uint32_t gb1 = lds_addr(dx_g<u>()) + b_lane1;
        u32x2_t alo[2][4], ahi[2][4];
        u32x4_t bq[2][NBD];
        static_for<0, 4>([&](auto mm) {
          constexpr int mb = decltype(mm)::value;
          ds_read_tr_b64<(0 * LD + 32 * mb) * 2>(alo[0][mb], wb);
          ds_read_tr_b64<(4 * LD + 32 * mb) * 2>(ahi[0][mb], wb);
        });
        ds_read_128<0>(bq[0][0], gb0);
        if constexpr (NBD > 1) ds_read_128<32 * 64>(bq[0][1], gb0);
        static_for<0, 4>([&](auto mm) {
          constexpr int mb = decltype(mm)::value;
          ds_read_tr_b64<(16 * LD + 32 * mb) * 2>(alo[1][mb], wb);
          ds_read_tr_b64<(20 * LD + 32 * mb) * 2>(ahi[1][mb], wb);
        });
        ds_read_128<0>(bq[1][0], gb1);
        if constexpr (NBD > 1) ds_read_128<32 * 64>(bq[1][1], gb1);
        // ... then later chunks' loads; the next coefficients are produced
        // while the first k-step's MFMAs run.
        dma_raw(std::integral_constant<int, u>{}, cu + 3);
        dma_ids(cu + 4);
        static_for<0, 2>([&](auto kq) {
          constexpr int kk = decltype(kq)::value;
          if constexpr (kk == 0) {
            lgkm_wait<8 + NBD>(alo[0][0], alo[0][1], alo[0][2], alo[0][3], ahi[0][0], ahi[0][1],
                          ahi[0][2], ahi[0][3], bq[0], idv);
            // W rows of chunk cu + 2, from the ids read above.
            rows_of(idv);
            dma_w(std::integral_constant<int, (u + 2) % 3>{});
          } else {
            produce_store(std::integral_constant<int, (u + 1) % 3>{}, cu + 1, pin);
            lgkm_wait<0>(alo[1][0], alo[1][1], alo[1][2], alo[1][3], ahi[1][0], ahi[1][1],
                         ahi[1][2], ahi[1][3], bq[1]);
          }
#pragma unroll
          for (int mb = 0; mb < 4; ++mb)
#pragma unroll
            for (int nb = 0; nb < NBD; ++nb)
              acc[mb][nb] = mfma_32x32x16(frag_of(alo[kk][mb], ahi[kk][mb]), as_uint4(bq[kk][nb]),
                                          acc[mb][nb], Tag{});
        });
      });
    }
    wait_vmcnt<0>();
  }

  const float inv_scale = 1.0f / scale;
  const int half = lane >> 5, l32 = lane & 31;
#pragma unroll
  for (int nb = 0; nb < NBD; ++nb) {
    const int n = n0 + 32 * (NBD * wn + nb) + l32;
    if (n >= B) continue;
    float* out = dx_part + ((int64_t)split * B + n) * D;
#pragma unroll
    for (int mb = 0; mb < 4; ++mb)
#pragma unroll
      for (int g = 0; g < 4; ++g) {
        const int i = 128 * wi + 32 * mb + 8 * g + 4 * half;
        *reinterpret_cast<float4*>(out + i) =
            make_float4(acc[mb][nb][4 * g] * inv_scale, acc[mb][nb][4 * g + 1] * inv_scale,
                        acc[mb][nb][4 * g + 2] * inv_scale, acc[mb][nb][4 * g + 3] * inv_scale);
      }
  }
}

// Row scales of the logit store: gscale[g][n] = 2^(m_gn - lse_n log2 e), so that
// E * gscale is the softmax probability (0 for rows past the batch).  A row
// with an empty denominator (lse = -inf: its label is outside the shard and the
// PFC* filter dropped every logit, so all its E are 0) gets scale 0, and with
// it no gradient.  Groups past |S| are never read and are skipped.
__global__ void __launch_bounds__(256) k_scales(const float* __restrict__ gmax,
                                                const float* __restrict__ row_lse, int B,
                                                int64_t ld_g, int64_t n_groups,
                                                const int32_t* __restrict__ n_active_p,
                                                float* __restrict__ gscale) {
  // Four consecutive entries per thread (ld_g is a multiple of 4, so the four
  // rows share one group and the 16-byte accesses are aligned).
  const int64_t i = 4 * ((int64_t)blockIdx.x * blockDim.x + threadIdx.x);
  const int64_t K = *n_active_p;
  if (i >= n_groups * ld_g) return;
  const int64_t g = i / ld_g;
  const int n = (int)(i - g * ld_g);
  if (g * kLogitGroup >= K) return;
  const float4 m4 = *reinterpret_cast<const float4*>(gmax + i);
  const float mv[4] = {m4.x, m4.y, m4.z, m4.w};
  float v[4];
#pragma unroll
  for (int e = 0; e < 4; ++e) {
    const float lse = n + e < B ? row_lse[n + e] : -INFINITY;
    v[e] = lse > -INFINITY ? __builtin_amdgcn_exp2f(mv[e] - lse * kLog2e) : 0.0f;
  }
  *reinterpret_cast<float4*>(gscale + i) = make_float4(v[0], v[1], v[2], v[3]);
}

// Sum the split partials of a row, add the row's target term
// g_t * W[S_t] / ||w_t||, and apply the normalisation backward:
// dx = (dX_hat - x_hat (x_hat . dX_hat)) / ||x||, dX_hat = (s/B) * sum.  A
// mapped label outside [0, |S|) counts as unowned: no target term, and no
// row of W or of the id list is read for it.
//
// One workgroup per batch row: d / 4 threads of four entries each sum one of
// its runs of consecutive splits (independent loads, eight in flight), and the
// runs' sums are added in order.  Bound by the partials' bytes on a large
// batch (B = 1024, 32 splits, d = 512, 67 MB: 13.9 us, 15.7 with one run), by the
// loads' latency on a small one, which the runs divide.  Few splits (a large
// batch) take fewer threads: B = 4096, 8 splits: 15.0 us, 18.5 with 512.
template <typename Tag, int D, int THREADS>
__global__ void __launch_bounds__(THREADS) k_dx_final(
    const float* __restrict__ dx_part, int n_split, const uint16_t* __restrict__ X,
    const uint16_t* __restrict__ W, const int32_t* __restrict__ active,
    const int32_t* __restrict__ n_active_p,
    const int32_t* __restrict__ yhat, const float* __restrict__ row_lse,
    const float* __restrict__ inv_x, const float* __restrict__ inv_w,
    const float* __restrict__ tgtc, int B, Margin mg, float sB, float* __restrict__ dX) {
  constexpr int TPR = D / 4;                     // threads of a run
  constexpr int RUNS = THREADS / TPR;
  constexpr int NW = TPR > 64 ? TPR / 64 : 1;    // waves that hold the row
  __shared__ f32x4_t sums[RUNS][TPR];
  __shared__ float red[NW];
  const int n = blockIdx.x;
  const int t = threadIdx.x % TPR, run = threadIdx.x / TPR;
  const int per = (n_split + RUNS - 1) / RUNS;
  const int s1 = per * (run + 1) < n_split ? per * (run + 1) : n_split;
  const float* p = dx_part + (int64_t)n * D + 4 * t;
  const int64_t stride = (int64_t)B * D;
  f32x4_t sum = {0.0f, 0.0f, 0.0f, 0.0f};
  for (int s = per * run; s < s1; s += 8) {
    f32x4_t q[8];
#pragma unroll
    for (int u = 0; u < 8; ++u)
      q[u] = s + u < s1 ? *reinterpret_cast<const f32x4_t*>(p + (s + u) * stride)
                        : f32x4_t{0.0f, 0.0f, 0.0f, 0.0f};
#pragma unroll
    for (int u = 0; u < 8; ++u) sum += q[u];
  }
  sums[run][t] = sum;
  // The first run's threads go on with the row.
  const bool mine = run == 0;
  const float ix = inv_x[n];
  f32x4_t v = {0.0f, 0.0f, 0.0f, 0.0f}, xh = v;
  float gt = 0.0f;
  uint2 w4 = make_uint2(0, 0), x4 = make_uint2(0, 0);
  if (mine) {
    const int yt = yhat[n];
    if (yt >= 0 && yt < *n_active_p) {
      gt = target_coef(mg, tgtc[n], row_lse[n]) * inv_w[yt];
      w4 = *reinterpret_cast<const uint2*>(W + (int64_t)active[yt] * D + 4 * t);
    }
    x4 = *reinterpret_cast<const uint2*>(X + (int64_t)n * D + 4 * t);
  }
  __syncthreads();
  float dot = 0.0f;
  if (mine) {
    const uint32_t wq[2] = {w4.x, w4.y}, xq[2] = {x4.x, x4.y};
#pragma unroll
    for (int u = 1; u < RUNS; ++u) sum += sums[u][t];
#pragma unroll
    for (int e = 0; e < 4; ++e) {
      const int sh = 16 * (e & 1);
      v[e] = sB * fmaf(gt, to_float<Tag>((uint16_t)(wq[e >> 1] >> sh)), sum[e]);
      xh[e] = to_float<Tag>((uint16_t)(xq[e >> 1] >> sh)) * ix;
      dot = fmaf(xh[e], v[e], dot);
    }
    if constexpr (TPR < 64) {   // the row's half of its wave
#pragma unroll
      for (int off = TPR / 2; off > 0; off >>= 1) dot += __shfl_xor(dot, off, 64);
    } else {
      dot = wave_sum(dot);
      if ((t & 63) == 0) red[t >> 6] = dot;
    }
  }
  if constexpr (NW > 1) {
    __syncthreads();
    dot = 0.0f;
#pragma unroll
    for (int w = 0; w < NW; ++w) dot += red[w];
  }
  if (mine) {
    f32x4_t o;
#pragma unroll
    for (int e = 0; e < 4; ++e) o[e] = ix * (v[e] - xh[e] * dot);
    *reinterpret_cast<f32x4u_t*>(dX + (int64_t)n * D + 4 * t) = o;
  }
}

// ------------------------------------------------------------------ dW

// D = 128 * WI; eight waves, two per SIMD: wave w owns d entries
// [D/4 (w % 4), +D/4) and classes [64 (w / 4), +64) of the workgroup (MB x 2
// accumulator tiles of 32 x 32), so that a SIMD's second wave issues while
// the first waits at a barrier or on its loads.  Both MFMA operands are
// K-major in LDS, so every fragment is one 16-byte read: X^T from the
// transposed bf16 copy of the batch, and G^T written by the producer.
// Pipeline per chunk c (32 batch rows): raw logit-store values and row
// scales of chunk c + 3 and X^T of chunk c + 2 requested, coefficients of
// chunk c + 1 produced, chunk c contracted.  The second k-step of chunk c is
// contracted at the start of the next chunk, from fragments read in this
// one, so that the matrix pipe is busy while the next fragments arrive.
//
// That is a tile of CLS = 128 classes, and a tile of 64 classes is the same with
// half the classes per wave; one of 32 gives each wave an eighth of d (a
// quarter at D = 128, which two waves then share the work of, with the same
// results).  Where a tile has fewer pieces to load or coefficients to produce
// than the waves have slots, several waves load and write the same bytes, so
// that all waves' load counts stay alike.
template <typename Tag, int WI, bool MASTER, int CLS>
__global__ void __launch_bounds__(512, WI == 1 ? 4 : 2) k_dw16(
    const uint16_t* __restrict__ xbT, const void* __restrict__ X,
    uint16_t* __restrict__ W, float* __restrict__ W_master, float* __restrict__ M,
    const int32_t* __restrict__ active, const int32_t* __restrict__ n_active_p,
    const int32_t* __restrict__ yhat, const float* __restrict__ row_lse,
    const float* __restrict__ inv_x, const float* __restrict__ inv_w,
    const float* __restrict__ tgtc, const uint16_t* __restrict__ lbuf, int64_t ld_cos,
    const float* __restrict__ gscale, int64_t ld_g, int B, Margin mg, float sB, float lr,
    float mu, int32_t* __restrict__ gate, int n_gate, int epoch) {
  constexpr int D = 128 * WI;
  constexpr int NW = 8;
  constexpr int WD = CLS == 32 && D > 128 ? 8 : 4;   // waves that share d
  constexpr int DW = D / WD;            // d entries of a wave
  constexpr int CW = CLS == 128 ? 64 : 32;   // classes of a wave
  constexpr int MB = DW / 32;           // 32-entry d blocks of a wave
  constexpr int NB = CW / 32;           // 32-class blocks of a wave
  constexpr int PIECES = CLS / 8;       // 16-byte pieces of a logit-store row
  constexpr int RROWS = 64 / PIECES;    // rows of one load
  constexpr int XDMA = D / 16 / NW;     // X^T loads (16 d rows each) per wave per chunk
  constexpr int RDMA = 8 / NW;          // logit-store loads (4 rows each) per wave
  constexpr int QL = 8 / NW;            // row-scale pieces (4 rows each) per wave
  constexpr int GROUPS = 1;             // producer slots per thread (512 / 512)
  constexpr int PER_ITER = XDMA + RDMA + 1;
  constexpr int NF = MB + NB;           // fragment reads per k-step
  static_assert(PER_ITER + 2 * (RDMA + 1) < 64, "vmcnt range");
  const int K = *n_active_p;
  const int64_t j0 = (int64_t)blockIdx.x * CLS;
  if (j0 >= K) return;
  // Start gates (n_gate > 0 on a long grid of one workgroup per CU, d >= 256): workgroup
  // 2 i + 1 of the first wave starts once workgroup 2 i has finished its
  // contraction, which it signals by writing this launch's number to gate[i].
  // Otherwise all CUs run the contraction and then the memory-bound update in
  // step for the first few hundred microseconds, and the updates, all at
  // once, saturate HBM; with the gates about half of the CUs update at any
  // time from the start.  The wait is bounded (kGateSpins polls), and the
  // results never depend on it: a gate that is never opened, or holds the
  // number by chance, only changes when the workgroup starts.
  const bool gated = WI > 1 && (int)blockIdx.x < 2 * n_gate;
  if (gated && (blockIdx.x & 1)) {
    if (threadIdx.x == 0) {
      const int32_t* g = gate + blockIdx.x / 2;
      for (int it = 0; it < kGateSpins; ++it) {
        if (__hip_atomic_load(g, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) == epoch) break;
        __builtin_amdgcn_s_sleep(8);
      }
    }
    __syncthreads();
  }
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  // The wave's part of d and of the classes.
  const int wd = wave & (WD - 1), wc = CLS == 128 ? wave >> 2 : wave / WD % (CLS / CW);
  const int half = lane >> 5, l32 = lane & 31;
  const int n_chunks = (int)ceil_div(B, kBwKC);
  const int c_stop = (int)ceil_div(n_chunks, 3) * 3;
  // The tile is one 128-class group of the logit store: its row scales.
  const float* gsc = gscale + (j0 / kLogitGroup) * ld_g;
  // Row ids and 1/||w|| of the tile's classes for the update, requested now
  // so that they have long arrived when the update forms its row addresses:
  // lane l holds classes l (u = 0) and 64 + l (u = 1).
  int act_l[2];
  float iw_l[2];
#pragma unroll
  for (int u = 0; u < 2; ++u) {
    const int64_t j = j0 + 64 * u + lane;
    const bool in = 64 * u + lane < CLS && j < K;
    act_l[u] = in ? active[j] : 0;
    iw_l[u] = in ? inv_w[j] : 0.0f;
  }

  // Swizzle of a logit-store row's pieces: the rows of a transposing read on
  // distinct banks.
  auto swz = [](int r) { return 2 * (r & (PIECES < 8 ? 1 : 3)); };
  // Producer slots: a 16-lane group owns 16 classes x 8 batch rows of a chunk;
  // lane gi of the group owns class 16 cb + gi.
  const int grp = lane >> 4, gi = lane & 15;
  int pcls[GROUPS], prg[GROUPS];
  uint32_t ptr_off[GROUPS];   // byte offset of the lane's transposing raw read
#pragma unroll
  for (int u = 0; u < GROUPS; ++u) {
    const int s = 4 * wave + grp + 16 * u;
    const int cb = CLS == 128 ? s >> 2 : (s >> 2) % (CLS / 16);
    pcls[u] = 16 * cb + gi;
    prg[u] = s & 3;
    // Lane 4 e + q of the group points at row 8 rg + e, classes 16 cb + 4 q .. + 3
    // (16-byte piece 2 cb + q / 2, stored at piece ^ swz(row)), half q & 1.
    const int e = gi >> 2, q = gi & 3;
    const int r = 8 * prg[u] + e;
    ptr_off[u] = (uint32_t)(r * CLS * 2 + 16 * ((2 * cb + (q >> 1)) ^ swz(r)) + 8 * (q & 1));
  }

  // Raw logit-store values: load v of this wave covers rows RROWS b .. + RROWS - 1
  // (b = wave RDMA + v, modulo the tile's 32 / RROWS); lane l fills piece
  // l % PIECES of row RROWS b + l / PIECES with source piece (l % PIECES) ^ swz(row).
  auto dma_raw_piece = [&](auto st, int c, int v) __attribute__((always_inline)) {
    constexpr int S = decltype(st)::value;
    const int cc = c < n_chunks ? c : n_chunks - 1;
    constexpr int BLKS = kBwKC / RROWS;
    const int blk = BLKS == NW * RDMA ? wave * RDMA + v : (wave * RDMA + v) % BLKS;
    const int r = RROWS * blk + lane / PIECES;
    int n = cc * kBwKC + r;
    n = n < B ? n : B - 1;
    const int piece = lane % PIECES ^ swz(r);
    dma16(lbuf + (int64_t)n * ld_cos + j0 + 8 * piece, dw_r<S>() + 512 * blk);
  };
  // Row scales of the chunk: QL 16-byte pieces (4 rows each) per wave; rows < ld_g always.
  auto dma_scale = [&](auto st, int c) __attribute__((always_inline)) {
    constexpr int S = decltype(st)::value;
    const int cc = c < n_chunks ? c : n_chunks - 1;
    if (lane < QL) dma16(gsc + cc * kBwKC + 4 * (QL * wave + lane), dw_q<S>() + 4 * QL * wave);
  };
  auto dma_raw = [&](auto st, int c) __attribute__((always_inline)) {
#pragma unroll
    for (int v = 0; v < RDMA; ++v) dma_raw_piece(st, c, v);
    dma_scale(st, c);
  };
  // X^T: block cc of the transposed batch ([d][32], contiguous); load v of this
  // wave covers d rows 16 m .. 16 m + 15 (m = wave XDMA + v), 4 pieces each;
  // lane l fills piece l & 3 of row 16 m + l / 4 with source piece
  // (l & 3) ^ ((row >> 2) & 3).
  auto dma_x_piece = [&](auto st, int c, int v) __attribute__((always_inline)) {
    constexpr int S = decltype(st)::value;
    const int cc = c < n_chunks ? c : n_chunks - 1;
    const int m = wave * XDMA + v;
    const int i = 16 * m + (lane >> 2);
    const int piece = (lane & 3) ^ ((i >> 2) & 3);
    dma16(xbT + ((int64_t)cc * D + i) * kBwKC + 8 * piece, dw_x<S, WI>() + 512 * m);
  };
  auto dma_x = [&](auto st, int c) __attribute__((always_inline)) {
#pragma unroll
    for (int v = 0; v < XDMA; ++v) dma_x_piece(st, c, v);
  };
  // Coefficients of chunk c: G^T[class][row] = p = E * gscale_row (the operand
  // X^T holds x_hat, so no 1/||x|| here).  E is 0 at targets and past |S|,
  // gscale 0 past the batch.  The LDS reads are issued first (produce_load)
  // and consumed later (produce_store), after an lgkm wait that covers them.
  struct ProdIn {
    u32x2_t qlo[GROUPS], qhi[GROUPS];
    u32x4_t sq[GROUPS][2];
  };
  auto produce_load = [&](auto st, ProdIn& in) {
    constexpr int S = decltype(st)::value;
#pragma unroll
    for (int u = 0; u < GROUPS; ++u) {
      const uint32_t ra = lds_addr(dw_r<S>()) + ptr_off[u];
      ds_read_tr_b64<0>(in.qlo[u], ra);
      ds_read_tr_b64<4 * CLS * 2>(in.qhi[u], ra);
      const uint32_t qa = lds_addr(dw_q<S>()) + 32 * prg[u];
      ds_read_128<0>(in.sq[u][0], qa);
      ds_read_128<16>(in.sq[u][1], qa);
    }
  };
  auto pin_group = [&](ProdIn& in, int u) __attribute__((always_inline)) {
    pin_reg(in.qlo[u]);
    pin_reg(in.qhi[u]);
    pin_reg(in.sq[u][0]);
    pin_reg(in.sq[u][1]);
  };
  // Group u's coefficients into stage S; gmask 0 writes zeros (a chunk past
  // the batch, whose MFMAs then add nothing).
  auto produce_group = [&](auto st, ProdIn& in, int u, uint32_t gmask) __attribute__((always_inline)) {
    constexpr int S = decltype(st)::value;
    const uint32_t qw[4] = {in.qlo[u].x, in.qlo[u].y, in.qhi[u].x, in.qhi[u].y};
    const float sc[8] = {__uint_as_float(in.sq[u][0].x), __uint_as_float(in.sq[u][0].y),
                         __uint_as_float(in.sq[u][0].z), __uint_as_float(in.sq[u][0].w),
                         __uint_as_float(in.sq[u][1].x), __uint_as_float(in.sq[u][1].y),
                         __uint_as_float(in.sq[u][1].z), __uint_as_float(in.sq[u][1].w)};
    float v[8];
#pragma unroll
    for (int e = 0; e < 8; ++e) {
      const float ev = (e & 1) ? f16_hi(qw[e >> 1]) : f16_lo(qw[e >> 1]);
      v[e] = ev * sc[e];
    }
    const uint4 o = pack8<Bf16Tag>(v);
    const int cl = pcls[u];
    ds_write_128<0>(lds_addr(dw_g<S>()) + cl * kBwKC * 2 + 16 * (prg[u] ^ ((cl >> 2) & 3)),
                    u32x4_t{o.x & gmask, o.y & gmask, o.z & gmask, o.w & gmask});
  };

  // Fragment byte offsets: operand row (d entry or class) 32 q + l32 of the
  // wave's block, chunk 2 kk + half stored at chunk ^ ((row >> 2) & 3).
  const int sw = (l32 >> 2) & 3;
  const uint32_t a_lane0 = (uint32_t)((DW * wd + l32) * kBwKC * 2 + 16 * ((0 + half) ^ sw));
  const uint32_t a_lane1 = (uint32_t)((DW * wd + l32) * kBwKC * 2 + 16 * ((2 + half) ^ sw));
  const uint32_t b_lane0 = (uint32_t)((CW * wc + l32) * kBwKC * 2 + 16 * ((0 + half) ^ sw));
  const uint32_t b_lane1 = (uint32_t)((CW * wc + l32) * kBwKC * 2 + 16 * ((2 + half) ^ sw));

  f32x16_t acc[MB][NB];
#pragma unroll
  for (int mb = 0; mb < MB; ++mb)
#pragma unroll
    for (int nb = 0; nb < NB; ++nb)
#pragma unroll
      for (int r = 0; r < 16; ++r) acc[mb][nb][r] = 0.0f;
  // Second k-step fragments, carried from one chunk to the next.
  u32x4_t a1[MB], b1[NB];
#pragma unroll
  for (int mb = 0; mb < MB; ++mb) a1[mb] = u32x4_t{0, 0, 0, 0};
#pragma unroll
  for (int nb = 0; nb < NB; ++nb) b1[nb] = u32x4_t{0, 0, 0, 0};

  {
    using S0 = std::integral_constant<int, 0>;
    using S1 = std::integral_constant<int, 1>;
    using S2 = std::integral_constant<int, 2>;
    dma_raw(S0{}, 0);
    dma_x(S0{}, 0);
    dma_raw(S1{}, 1);
    dma_x(S1{}, 1);
    dma_raw(S2{}, 2);
    wait_vmcnt_lgkm0<2 * (RDMA + 1) + XDMA>();
    stage_barrier();
    ProdIn in0;
    produce_load(S0{}, in0);
    lgkm_wait<0>();
#pragma unroll
    for (int u = 0; u < GROUPS; ++u) {
      pin_group(in0, u);
      produce_group(S0{}, in0, u, 0xFFFFFFFFu);
    }
  }
  // Instruction slots of a chunk: NMF MFMAs per k-step, each followed by
  // the work placed after it, so that the wave issues its other instructions
  // while the matrix pipe works through the MFMAs already issued.
  constexpr int NMF = MB * NB;
  constexpr int W_AT = NMF >= 16 ? 3 : NMF / 4;      // wait for the chunk's fragment and producer reads
  constexpr int G0_AT = NMF / 2 - 1 > W_AT ? NMF / 2 - 1 : W_AT;   // coefficients written
  constexpr int NITEM = RDMA + 1 + XDMA + NF;        // loads and reads spread over the second k-step
  static_assert(GROUPS == 1, "one producer slot per thread");
  for (int c = 0; c < c_stop; c += 3) {
    static_for<0, 3>([&](auto uu) {
      constexpr int u = decltype(uu)::value;
      using SU = std::integral_constant<int, u>;
      using SN = std::integral_constant<int, (u + 1) % 3>;
      using SX = std::integral_constant<int, (u + 2) % 3>;
      const int cu = c + u;
      // Landed: X^T of chunk cu, raw data of chunk cu + 1; this wave's
      // coefficient writes and second k-step reads of the previous chunk are
      // complete.
      wait_vmcnt_lgkm0<PER_ITER>();
      stage_barrier();
      const uint32_t xs = lds_addr(dw_x<u, WI>());
      const uint32_t gs = lds_addr(dw_g<u>());
      u32x4_t a0[MB], b0[NB];
      static_for<0, MB>([&](auto mm) {
        constexpr int mb = decltype(mm)::value;
        ds_read_128<32 * mb * kBwKC * 2>(a0[mb], xs + a_lane0);
      });
      static_for<0, NB>([&](auto nn) {
        constexpr int nb = decltype(nn)::value;
        ds_read_128<32 * nb * kBwKC * 2>(b0[nb], gs + b_lane0);
      });
      ProdIn pin;
      produce_load(SN{}, pin);
      const uint32_t gmask = cu + 1 < n_chunks ? 0xFFFFFFFFu : 0u;
      // Second k-step of the previous chunk (fragments landed before the
      // barrier), with the next chunk's coefficients produced alongside.
      pin_reg(a1);
      pin_reg(b1);
      static_for<0, NMF>([&](auto ii) {
        constexpr int i = decltype(ii)::value;
        acc[i / NB][i % NB] = mfma_32x32x16(as_uint4(a1[i / NB]), as_uint4(b1[i % NB]), acc[i / NB][i % NB], Bf16Tag{});
        if constexpr (i == W_AT) {
          lgkm_wait<0>(a0, b0);
          pin_group(pin, 0);
        }
        if constexpr (i == G0_AT) produce_group(SN{}, pin, 0, gmask);
      });
      // First k-step of this chunk, with the loads of later chunks and this
      // chunk's second k-step reads spread over its slots.
      static_for<0, NMF>([&](auto ii) {
        constexpr int i = decltype(ii)::value;
        acc[i / NB][i % NB] = mfma_32x32x16(as_uint4(a0[i / NB]), as_uint4(b0[i % NB]), acc[i / NB][i % NB], Bf16Tag{});
        static_for<(i * NITEM + NMF - 1) / NMF, ((i + 1) * NITEM + NMF - 1) / NMF>([&](auto kk) {
          constexpr int k = decltype(kk)::value;
          if constexpr (k < RDMA) {
            dma_raw_piece(SU{}, cu + 3, k);
          } else if constexpr (k == RDMA) {
            dma_scale(SU{}, cu + 3);
          } else if constexpr (k < RDMA + 1 + XDMA) {
            dma_x_piece(SX{}, cu + 2, k - RDMA - 1);
          } else if constexpr (k < RDMA + 1 + XDMA + MB) {
            constexpr int mb = k - RDMA - 1 - XDMA;
            ds_read_128<32 * mb * kBwKC * 2>(a1[mb], xs + a_lane1);
          } else {
            constexpr int nb = k - RDMA - 1 - XDMA - MB;
            ds_read_128<32 * nb * kBwKC * 2>(b1[nb], gs + b_lane1);
          }
        });
      });
    });
  }
  wait_vmcnt<0>();
  wait_lgkm0();
  // Second k-step of the last chunk (zero coefficients past the batch).
  pin_reg(a1);
  pin_reg(b1);
#pragma unroll
  for (int mb = 0; mb < MB; ++mb)
#pragma unroll
    for (int nb = 0; nb < NB; ++nb)
      acc[mb][nb] = mfma_32x32x16(as_uint4(a1[mb]), as_uint4(b1[nb]), acc[mb][nb], Bf16Tag{});
  if (gated && !(blockIdx.x & 1) && threadIdx.x == 0)
    __hip_atomic_store(gate + blockIdx.x / 2, epoch, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);

  // ---- update: the tile goes through LDS in passes of 32 classes so
  // that each wave then owns whole rows: W, momentum and master rows are read
  // and written in full contiguous segments.  Pass p holds the classes
  // 32 p + r (r < 32); entry d of row r sits in stage array d / 256 at
  // r * kTLd + d % 256.  Wave w owns rows 4 w .. 4 w + 3 of each pass; lane l
  // owns d = 256 h + 4 l .. + 3.  A wave's rows of a pass are loaded while
  // the previous pass is updated, one row after each row written.
  constexpr int NH = D > 256 ? 2 : 1;         // 256-entry halves of a row
  constexpr int LPH = (D > 256 ? 256 : D) / 4;  // lanes that own entries
  constexpr int RPW = 32 / NW;                // rows of a pass per wave
  constexpr int TLD = WI == 1 ? kTLd128 : kTLd;
  float* const tlo = reinterpret_cast<float*>(dw_x<0, WI>());
  float* const thi = reinterpret_cast<float*>(dw_x<1, WI>());
  const bool lane_on = LPH == 64 || lane < LPH;
  const int kt = (int)(K - j0);               // classes from the tile's first on that exist (>= 1)
  int* const hits = reinterpret_cast<int*>(wG0);   // NW lists of kHitCap entries
  int* const hit_n = reinterpret_cast<int*>(wQ0);  // their lengths
  static_assert(NW * kHitCap * 4 <= kDwCls * kBwKC * 2, "hit lists fit a coefficient stage");

  // A wave's rows of one pass.  Row ids, 1/||w|| and the count of rows that
  // exist are wave-uniform; a row past |S| reads row 0 and is not updated.
  struct Rows {
    uint2 wv[RPW][NH];   // four 16-bit weights
    float4 mv[RPW][NH], pv[MASTER ? RPW : 1][NH];
    int row[RPW];
    float iwr[RPW];
    int nv;              // rows k < nv exist
  };
  auto set_rows = [&](Rows& bt, int p) __attribute__((always_inline)) {
    const int cb = 32 * p + RPW * wave;   // tile offset of the wave's first class of the pass
    bt.nv = kt - cb < 0 ? 0 : (kt - cb > RPW ? RPW : kt - cb);
  };
  auto load_row = [&](Rows& bt, int p, int k) __attribute__((always_inline)) {
    const int src = 32 * (p & 1) + RPW * wave + k;   // lane that holds class 32 p + RPW wave + k
    bt.row[k] = __builtin_amdgcn_readlane(act_l[p >> 1], src);
    bt.iwr[k] = __int_as_float(__builtin_amdgcn_readlane(__float_as_int(iw_l[p >> 1]), src));
    const int64_t rb = (int64_t)bt.row[k] * D;   // uniform row base
#pragma unroll
    for (int h = 0; h < NH; ++h) {
      const uint32_t o = 256u * h + 4u * (uint32_t)lane;
      bt.wv[k][h] = make_uint2(0, 0);
      bt.mv[k][h] = make_float4(0.0f, 0.0f, 0.0f, 0.0f);
      if constexpr (MASTER) bt.pv[k][h] = make_float4(0.0f, 0.0f, 0.0f, 0.0f);
      if (lane_on) {
        // Non-temporal: each row is read once here and written back once.
        const u32x2_t w2 = __builtin_nontemporal_load(
            reinterpret_cast<const u32x2_t*>(reinterpret_cast<const char*>(W + rb) + 2 * o));
        const f32x4_t m4 = __builtin_nontemporal_load(
            reinterpret_cast<const f32x4_t*>(reinterpret_cast<const char*>(M + rb) + 4 * o));
        bt.wv[k][h] = make_uint2(w2.x, w2.y);
        bt.mv[k][h] = make_float4(m4.x, m4.y, m4.z, m4.w);
        if constexpr (MASTER) {
          const f32x4_t p4 = __builtin_nontemporal_load(reinterpret_cast<const f32x4_t*>(
              reinterpret_cast<const char*>(W_master + rb) + 4 * o));
          bt.pv[k][h] = make_float4(p4.x, p4.y, p4.z, p4.w);
        }
      }
    }
  };
  auto load_rows = [&](Rows& bt, int p) __attribute__((always_inline)) {
    set_rows(bt, p);
#pragma unroll
    for (int k = 0; k < RPW; ++k) load_row(bt, p, k);
  };
  constexpr int PASSES = CLS / 32;
  // Pass p's classes are block p % NB of the waves of class part p / NB.
  auto park = [&](auto pp) __attribute__((always_inline)) {
    constexpr int p = decltype(pp)::value;
    if (wc != p / NB) return;
#pragma unroll
    for (int mb = 0; mb < MB; ++mb)
#pragma unroll
      for (int g = 0; g < 4; ++g) {
        const int d0 = DW * wd + 32 * mb + 8 * g + 4 * half;
        *reinterpret_cast<float4*>((d0 >= 256 ? thi : tlo) + l32 * TLD + (d0 & 255)) =
            make_float4(acc[mb][p % NB][4 * g], acc[mb][p % NB][4 * g + 1],
                        acc[mb][p % NB][4 * g + 2], acc[mb][p % NB][4 * g + 3]);
      }
  };
  // Target term of batch row nn added to staged row r (this wave's own row).
  auto add_target = [&](int nn, int r) {
    const float gt = target_coef(mg, tgtc[nn], row_lse[nn]) * inv_x[nn];
    if (!lane_on) return;
#pragma unroll
    for (int h = 0; h < NH; ++h) {
      const uint2 x4 = *reinterpret_cast<const uint2*>(
          reinterpret_cast<const uint16_t*>(X) + (int64_t)nn * D + 256 * h + 4 * lane);
      float4* t = reinterpret_cast<float4*>((h ? thi : tlo) + r * TLD + 4 * lane);
      float4 a = *t;
      a.x = fmaf(gt, to_float<Tag>((uint16_t)(x4.x & 0xFFFF)), a.x);
      a.y = fmaf(gt, to_float<Tag>((uint16_t)(x4.x >> 16)), a.y);
      a.z = fmaf(gt, to_float<Tag>((uint16_t)(x4.y & 0xFFFF)), a.z);
      a.w = fmaf(gt, to_float<Tag>((uint16_t)(x4.y >> 16)), a.w);
      *t = a;
    }
  };
  auto wf_of = [&](uint2 w4) __attribute__((always_inline)) {
    return make_float4(to_float<Tag>((uint16_t)(w4.x & 0xFFFF)), to_float<Tag>((uint16_t)(w4.x >> 16)),
                       to_float<Tag>((uint16_t)(w4.y & 0xFFFF)), to_float<Tag>((uint16_t)(w4.y >> 16)));
  };
  // Row update, with a = the staged row (dL/dw_hat = sB a), w_hat = w / ||w||:
  // g_w = (sB a - w_hat (w_hat . sB a)) / ||w|| = ga a - gb w,
  // ga = sB / ||w||, gb = ga (w . a) / ||w||^2; then momentum and the step.
  // With PN < PASSES each row's registers are refilled, right after the row is
  // written, with the same row of pass PN: the next pass's loads spread over
  // this pass's arithmetic and stores instead of queueing behind them.
  auto update_rows = [&](Rows& bt, auto pn_c) __attribute__((always_inline)) {
    constexpr int PN = decltype(pn_c)::value;
    // The dots w . a of all of this wave's rows first, then their reductions.
    float dots[RPW];
#pragma unroll
    for (int k = 0; k < RPW; ++k) {
      const int r = RPW * wave + k;
      float dot = 0.0f;
#pragma unroll
      for (int h = 0; h < NH; ++h) {
        if (!lane_on) continue;
        const float4 wf = wf_of(bt.wv[k][h]);
        const float4 a4 = *reinterpret_cast<const float4*>((h ? thi : tlo) + r * TLD + 4 * lane);
        dot = fmaf(wf.x, a4.x, dot);
        dot = fmaf(wf.y, a4.y, dot);
        dot = fmaf(wf.z, a4.z, dot);
        dot = fmaf(wf.w, a4.w, dot);
      }
      dots[k] = dot;
    }
#pragma unroll
    for (int k = 0; k < RPW; ++k) dots[k] = wave_total(dots[k]);
    const int nv = bt.nv;
    if constexpr (PN < PASSES) set_rows(bt, PN);
#pragma unroll
    for (int k = 0; k < RPW; ++k) {
      const int r = RPW * wave + k;
      if (k < nv) {
        const float ga = sB * bt.iwr[k];
        const float gb = ga * bt.iwr[k] * bt.iwr[k] * dots[k];
        // Uniform row base, made opaque so that the stores below address it as
        // base + lane offset instead of sharing the loads' 64-bit addresses.
        int rw = bt.row[k];
        asm volatile("" : "+s"(rw));
        const int64_t rb = (int64_t)rw * D;
#pragma unroll
        for (int h = 0; h < NH; ++h) {
          if (!lane_on) continue;
          const uint32_t o = 256u * h + 4u * (uint32_t)lane;
          const float4 wf = wf_of(bt.wv[k][h]);
          const float4 a4 = *reinterpret_cast<const float4*>((h ? thi : tlo) + r * TLD + 4 * lane);
          const float wo[4] = {wf.x, wf.y, wf.z, wf.w};
          const float ao[4] = {a4.x, a4.y, a4.z, a4.w};
          float mo[4] = {bt.mv[k][h].x, bt.mv[k][h].y, bt.mv[k][h].z, bt.mv[k][h].w};
          float po[4] = {0.0f, 0.0f, 0.0f, 0.0f};
          if constexpr (MASTER) {
            po[0] = bt.pv[k][h].x;
            po[1] = bt.pv[k][h].y;
            po[2] = bt.pv[k][h].z;
            po[3] = bt.pv[k][h].w;
          }
          float wn[4];
#pragma unroll
          for (int e = 0; e < 4; ++e) {
            const float gr = fmaf(-gb, wo[e], ga * ao[e]);
            mo[e] = fmaf(mu, mo[e], gr);
            if constexpr (MASTER) {
              po[e] = fmaf(-lr, mo[e], po[e]);
              wn[e] = po[e];
            } else {
              wn[e] = fmaf(-lr, mo[e], wo[e]);
            }
          }
          *reinterpret_cast<float4*>(reinterpret_cast<char*>(M + rb) + 4 * o) =
              make_float4(mo[0], mo[1], mo[2], mo[3]);
          if constexpr (MASTER)
            *reinterpret_cast<float4*>(reinterpret_cast<char*>(W_master + rb) + 4 * o) =
                make_float4(po[0], po[1], po[2], po[3]);
          uint2 ov;
          ov.x = pack2<Tag>(wn[0], wn[1]);
          ov.y = pack2<Tag>(wn[2], wn[3]);
          *reinterpret_cast<uint2*>(reinterpret_cast<char*>(W + rb) + 2 * o) = ov;
        }
      }
      if constexpr (PN < PASSES) load_row(bt, PN, k);
    }
  };

  // One row set in registers: pass p's rows, refilled row by row with pass
  // p + 1 (requesting two passes ahead measured no faster: the update's
  // loads and stores are bound by the HBM read-modify-write rate).
  Rows bat;
  load_rows(bat, 0);
  stage_barrier();  // every wave's fragment reads of the stage arrays are done
  // Target terms: wave w lists, in row order, the rows n of its quarter of the
  // batch whose label is one of the tile's classes (entry n * 128 + class
  // offset).  A quarter with more than kHitCap such rows makes each wave scan
  // all labels instead.  Either way the terms are added to the staged
  // gradient rows by the wave that owns the row, in increasing n.
  {
    const int q0 = (int)((int64_t)B * wave / NW), q1 = (int)((int64_t)B * (wave + 1) / NW);
    int cnt = 0;
    for (int nbase = q0; nbase < q1; nbase += 64) {
      const int n = nbase + lane;
      const int yv = n < q1 ? yhat[n] : -1;
      const bool hit = yv >= j0 && yv < j0 + CLS;
      const uint64_t mask = __ballot(hit);
      const int pos = cnt + __builtin_amdgcn_mbcnt_hi((uint32_t)(mask >> 32),
                                                      __builtin_amdgcn_mbcnt_lo((uint32_t)mask, 0));
      if (hit && pos < kHitCap) hits[kHitCap * wave + pos] = n * kDwCls + (int)(yv - j0);
      cnt += __popcll(mask);
    }
    if (lane == 0) hit_n[wave] = cnt;
  }
  park(std::integral_constant<int, 0>{});
  wait_lgkm0();
  stage_barrier();
  int hn[NW];
  bool hit_scan = false;
#pragma unroll
  for (int w = 0; w < NW; ++w) {
    hn[w] = __builtin_amdgcn_readfirstlane(hit_n[w]);
    hit_scan |= hn[w] > kHitCap;
  }
  static_for<0, PASSES>([&](auto pp) {
    constexpr int p = decltype(pp)::value;
    if constexpr (p > 0) {
      wait_lgkm0();
      stage_barrier();  // the stage arrays are rewritten by this pass
      park(pp);
      wait_lgkm0();
      stage_barrier();
    }
    // This wave's rows of the pass: class offsets c0 .. c0 + RPW - 1.
    const int c0 = 32 * p + RPW * wave;
    if (!hit_scan) {
      for (int w = 0; w < NW; ++w)
        for (int i = 0; i < hn[w]; ++i) {
          const int ent = hits[kHitCap * w + i];
          const int ct = ent & (kDwCls - 1);
          if (ct >= c0 && ct < c0 + RPW) add_target(ent / kDwCls, ct & 31);
        }
    } else {
      for (int nbase = 0; nbase < B; nbase += 64) {
        const int n = nbase + lane;
        const int yv = n < B ? yhat[n] : -1;
        uint64_t mask = __ballot(yv >= j0 + c0 && yv < j0 + c0 + RPW);
        while (mask) {
          const int bit = __ffsll((unsigned long long)mask) - 1;
          mask &= mask - 1;
          const int yt = __shfl(yv, bit, 64);
          add_target(nbase + bit, (int)(yt - j0) & 31);
        }
      }
    }
    update_rows(bat, std::integral_constant<int, p + 1>{});
  });
}

}  // namespace

// Class splits of the feature gradient: workgroups of 128 batch rows, one per
// CU, in one round (one more would be a second round, as ceil(256 / n_rt) gave
// at B = 777: 90 us for 45).  At d = 128 two share a CU once 24 chunks are left
// to one of 256 (B = 1024, |S| = 32,768, 32 chunks, 47 -> 41 us; with 8 chunks,
// B = 128, |S| = 65,536, 20 -> 25).  On few classes fewer
// splits: a split costs its partial sums, written and read again (8 B d bytes
// at the copy rate, 4.7 MB/us), and saves its share of the 1.2 us that a
// chunk of 32 classes takes, so their sum is least at
// sqrt(1.2 chunks 4.7e6 / (8 B d)).
// At B = 128, |S| = 10,000, d = 512 that is 59 splits instead of 256: the sum
// of the partials takes 5.7 instead of 26.8 us, dX 21.6 instead of 21.0.  The 1.2
// us are a chunk's at d = 512.  With half or twice that, dX and its sum together
// change by at most 7 % either way at any d (B = 32 to 1024, |S| = 1,000 to 120,000;
// d = 128, B = 128, |S| = 50,000 32.5 us, 30.9 with 0.6; B = 1024, |S| = 4,096 29.0, 30.8).
// The counts are those of 256 CUs whatever the device has, since the layout of the
// workspace follows from them.
namespace {
// Workgroups of one round; and how many elements of a partial sum cost a chunk's time.
int64_t dx_round(int64_t n_rt, int64_t d, double chunks) {
  return d == 128 && chunks * (double)n_rt >= 24.0 * 256.0 ? 512 : 256;
}
constexpr double kChunkElements = 1.2 * 4.7e6 / 8.0;
}  // namespace

int split_16(int64_t B, int64_t d, int64_t cap) {
  const int64_t n_rt = ceil_div(B, kDxRows);
  const double chunks = (double)ceil_div(cap, kBwKC);
  const int64_t most = dx_round(n_rt, d, chunks) / n_rt;   // B <= 8192: at least 4
  const int64_t best = (int64_t)ceil(sqrt(kChunkElements * chunks / ((double)B * (double)d)));
  const int64_t ns = best < most ? best : most;
  return (int)(ns < (int64_t)chunks ? ns : (int64_t)chunks);
}

// splits x B is at most each of the three: a round's rows, ceil(x) B <= x B + B, and
// chunks x B; none of them falls when B grows.
int64_t part_rows_16(int64_t B, int64_t d, int64_t cap) {
  const double chunks = (double)ceil_div(cap, kBwKC);
  const int64_t round = dx_round(ceil_div(B, kDxRows), d, chunks) * kDxRows;
  const int64_t best = (int64_t)ceil(sqrt(kChunkElements * chunks * (double)B / (double)d)) + B;
  const int64_t one_each = (int64_t)chunks * B;
  const int64_t rows = best < round ? best : round;
  return rows < one_each ? rows : one_each;
}

namespace {

// Compute units of the current device (0 if the query fails).
int device_cu_count() {
  int dev = 0, n = 0;
  if (hipGetDevice(&dev) != hipSuccess) return 0;
  if (hipDeviceGetAttribute(&n, hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess) return 0;
  return n;
}

template <typename Tag, int WI>
void launch_bwd16(const StepArgs& a, const StepWs& w, const Margin& mg, float sB,
                  hipStream_t stream) {
  const int B = (int)a.B;
  // Start gates on grids of at least four waves of one workgroup per CU; each
  // launch writes a number of its own to the gates it opens.  Not at d = 128,
  // where two workgroups share a CU, so that one already updates while the other
  // contracts: B = 1024, |S| = 131,072 107 us with gates, 101 without; B = 4096 310,
  // 286; |S| = 262,144, B = 1024 204, 198 (219 with gates for all resident pairs).
  static std::atomic<int> launches{0};
  const int n_cu = device_cu_count();
  // A shard whose 128-class tiles leave half of the CUs without a workgroup goes
  // in tiles of 64 or 32 classes (d = 512, us with 128 -> now:
  // |S| = 8,192, B = 128 28 -> 17, B = 1024 52 -> 34, B = 4096 140 -> 102; |S| =
  // 16,384 34 -> 26, 56 -> 46, 149 -> 134).  Also at d = 128, whose two workgroups
  // per CU share its matrix cores: up to half of 512 workgroups is worse there
  // (|S| = 16,384, B = 1024 29 -> 36, B = 4096 74 -> 104; |S| = 32,768, B = 1024 37 ->
  // 39, but B = 128 21.8 -> 20.6).  The last round of a longer grid
  // does not: cut that way in the same kernel it made the full tiles 2 % slower,
  // in a launch of its own it cost what it saved (|S| = 100,000 with a master
  // 311 -> 304 us, |S| = 45,000, d = 256 66 -> 68).
  const int64_t tiles = ceil_div(a.cap, kDwCls);
  const int n_slots = n_cu > 0 ? n_cu : 256;
  const int cls = tiles * 4 <= n_slots ? 32 : tiles * 2 <= n_slots ? 64 : kDwCls;
  const int n_gate =
      (WI > 1 && n_cu > 0 && tiles >= 4LL * n_cu) ? (n_cu / 2 < kDwGates ? n_cu / 2 : kDwGates) : 0;
  const int epoch = 1 + (launches.fetch_add(1, std::memory_order_relaxed) & 0x3FFFFFFF);
  const int n_rt = (int)ceil_div(B, kDxRows);
  const int64_t n_tiles = (int64_t)n_rt * w.n_split;
  const int64_t per_xcd = ceil_div(n_tiles, 8);
  timing_start(4, stream);
  // Row scales of the logit store from the lse the gradient is normalised with.
  hipLaunchKernelGGL(k_scales, dim3((unsigned)ceil_div(w.n_groups * w.ld_g, 4 * 256)), dim3(256), 0,
                     stream, w.gmax, a.row_lse, B, w.ld_g, w.n_groups, a.n_active, w.gscale);
  hipLaunchKernelGGL((k_dx16<Tag, WI>), dim3((unsigned)(8 * per_xcd)), dim3(dx_threads(WI)), 0, stream,
                     (const uint16_t*)a.W, w.act_pad, a.n_active, w.inv_w, w.inv_w_max,
                     (const uint16_t*)w.lbuf, w.ld_cos, w.gscale, w.ld_g, B, n_rt, w.n_split,
                     n_tiles, per_xcd, w.dx_part);
  timing_stop(4, stream);
  timing_start(5, stream);
  auto final = [&](auto kernel, int threads) {
    hipLaunchKernelGGL(kernel, dim3((unsigned)B), dim3(threads), 0, stream, w.dx_part, w.n_split,
                       (const uint16_t*)a.X, (const uint16_t*)a.W, a.active, a.n_active,
                       a.labels_mapped, a.row_lse, w.inv_x, w.inv_w, w.tgtc, B, mg, sB, a.dX);
  };
  if (w.n_split <= 8) final(k_dx_final<Tag, 128 * WI, 128>, 128);
  else final(k_dx_final<Tag, 128 * WI, 512>, 512);
  timing_stop(5, stream);
  timing_start(6, stream);
  auto update = [&](auto kernel) {
    hipLaunchKernelGGL(kernel, dim3((unsigned)ceil_div(a.cap, cls)), dim3(512), 0, stream,
                       (const uint16_t*)w.xbT, a.X, (uint16_t*)a.W, a.W_master, a.M, a.active,
                       a.n_active, a.labels_mapped, a.row_lse, w.inv_x, w.inv_w, w.tgtc,
                       (const uint16_t*)w.lbuf, w.ld_cos, w.gscale, w.ld_g, B, mg, sB, a.lr, a.mu,
                       w.dw_gate, n_gate, epoch);
  };
  auto update_in = [&](auto c) {
    constexpr int CLS = decltype(c)::value;
    if (a.W_master) update(k_dw16<Tag, WI, true, CLS>);
    else update(k_dw16<Tag, WI, false, CLS>);
  };
  if (cls == 32) update_in(std::integral_constant<int, 32>{});
  else if (cls == 64) update_in(std::integral_constant<int, 64>{});
  else update_in(std::integral_constant<int, 128>{});
  timing_stop(6, stream);
}

template <typename Tag>
void launch_bwd16_d(const StepArgs& a, const StepWs& w, const Margin& mg, float sB,
                    hipStream_t stream) {
  switch (a.d) {
    case 128: launch_bwd16<Tag, 1>(a, w, mg, sB, stream); break;
    case 256: launch_bwd16<Tag, 2>(a, w, mg, sB, stream); break;
    default: launch_bwd16<Tag, 4>(a, w, mg, sB, stream); break;
  }
}

}  // namespace

hipError_t launch_backward(const StepArgs& a, const StepWs& w, hipStream_t stream) {
  if (a.dtype == 0) return launch_backward_f32(a, w, stream);
  Margin mg{a.s, a.m, cosf(a.m), sinf(a.m), a.margin};
  const float sB = a.s / (float)a.B;
  if (a.dtype == 1)
    launch_bwd16_d<Bf16Tag>(a, w, mg, sB, stream);
  else
    launch_bwd16_d<F16Tag>(a, w, mg, sB, stream);
  return hipGetLastError();
}

}  // namespace pfc
