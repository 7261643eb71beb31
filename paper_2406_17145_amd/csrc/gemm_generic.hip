// Branch-grouped GEMM, generic variant: fp32 FMA on LDS-staged tiles, 64x64x16 for large launches and
// 32x32x64 with the contraction split over the waves for small ones.
// It serves the fp32 numeric mode and any bf16 problem whose pointers or
// leading dimensions do not meet the MFMA kernels' alignment rules.  One
// launch covers every independent branch of a topological level; a workgroup
// locates its problem through the records' workgroup prefix sums.
#include "device_utils.h"

namespace gpp {

constexpr int GT = 64;   // tile edge
constexpr int GK = 16;   // contraction step
constexpr int GS = 32, GSK = 64;   // the same of the kernel for small launches

int gemm_generic_tiles(int tile, int M, int N, int *tiles_n) {
  int tm = (M + tile - 1) / tile, tn = (N + tile - 1) / tile;
  if (tiles_n) *tiles_n = tn;
  return tm * tn;
}
// Tile of a launch with this many 64 x 64 tiles: up to two workgroups per compute unit the launch is one chain of memory
// round trips, which the small tiles shorten, and they spread it over four times the compute units.  Forward, small / large tiles:
// 1 to 255 tiles of 64 x 64 behind K 8 .. 16 0.8 - 0.9 of the time, 64 0.65, 256 0.4, 1000 0.25; 256 to 511 behind K 8 0.95,
// 64 0.77, 256 0.6, 1000 0.4; from 512 on, where the small tiles take several rounds, between 0.6 and 1.7 (2048 tiles: 2.1).
int gemm_generic_tile(int tiles64) { return tiles64 < 512 ? GS : GT; }

// element strides of the logical operands A(i, kk) [M x K] and B(kk, j) [K x N]
struct GenericStrides {
  int64_t ai, ak, bk, bj;
};
__device__ __forceinline__ GenericStrides generic_strides(const GemmProb &p) {
  if (p.form == FORM_FWD) return {p.lda, 1, 1, p.ldb};
  if (p.form == FORM_DX) return {p.lda, 1, p.ldb, 1};
  return {1, p.lda, p.ldb, 1};
}

// Small launches (the fp32 perceptron: 8 rows, layers of 64 .. 256).  What bounds them is latency, so: 64 contraction
// elements per step, all sixteen loads of a thread out together (unconditional, clamped addresses; a branch in front
// of a load would make each a round trip of its own) and the next step's on the way while one is multiplied; what the
// epilogue reads is requested in front of everything; the four waves take a quarter of every step each, over the whole
// tile, and meet in LDS once.  A launch of [8 x 256] = [8 x 128] x [128 x 256] and its two gradients: 10 .. 18 us on
// the 64 x 64 tiles, whose every 16 elements cost two barriers and a memory round trip.
template <typename T>
__global__ __launch_bounds__(256, 2) void k_gemm_generic_small(const GemmProb *__restrict__ probs, int n, int accumulate_dw) {
  constexpr int ST = GS + 4;
  __shared__ __attribute__((aligned(16))) float As[GSK * ST], Bs[GSK * ST], bias_part[4][GS];
  const int pi = find_prob(probs, n, blockIdx.x);
  const GemmProb p = probs[pi];
  const int tile = blockIdx.x - p.blk_begin;
  const int m0 = (tile / p.tiles_n) * GS, n0 = (tile % p.tiles_n) * GS;
  const int t = threadIdx.x, wave = t >> 6, lane = t & 63;
  const GenericStrides sd = generic_strides(p);
  const T *A = (const T *)p.A, *B = (const T *)p.B;

  // ---- epilogue operands of this thread's four outputs: row er, columns ec ..
  const int er = m0 + (t >> 3), ec = n0 + (t & 7) * 4;
  const int lr = min(er, p.M - 1);
  float old[4] = {}, res[4] = {}, aux[4] = {}, bias[4] = {};
  if (p.form == FORM_DW) {
    if (accumulate_dw) {
#pragma unroll
      for (int e = 0; e < 4; ++e) old[e] = ((const float *)p.C)[(int64_t)lr * p.ldc + min(ec + e, p.N - 1)];
    }
  } else {
    if (p.form == FORM_FWD && p.bias) {
#pragma unroll
      for (int e = 0; e < 4; ++e) bias[e] = p.bias[min(ec + e, p.N - 1)];
    }
    if (p.res) {
#pragma unroll
      for (int e = 0; e < 4; ++e) res[e] = load_as_f32(p.res, p.res_dtype, (int64_t)lr * p.ldres + min(ec + e, p.N - 1));
    }
    if (p.form == FORM_DX && p.act != ACT_NONE) {
#pragma unroll
      for (int e = 0; e < 4; ++e) aux[e] = load_as_f32(p.aux, p.aux_dtype, (int64_t)lr * p.ldaux + min(ec + e, p.N - 1));
    }
  }

  // element q of a thread: along the operand's contiguous direction from lane to lane
  const bool a_k = sd.ak == 1, b_k = sd.bk == 1;
  auto place = [&](bool k_contiguous, int q, int &x, int &kk) {
    const int e = t + 256 * q;
    if (k_contiguous) { kk = e & (GSK - 1); x = e / GSK; } else { x = e & (GS - 1); kk = e / GS; }
  };
  float ra[8], rb[8];
  auto fetch = [&](int k0) {
#pragma unroll
    for (int q = 0; q < 8; ++q) {
      int x, kk;
      place(a_k, q, x, kk);
      ra[q] = to_f32<T>(A[(int64_t)min(m0 + x, p.M - 1) * sd.ai + (int64_t)min(k0 + kk, p.K - 1) * sd.ak]);
      place(b_k, q, x, kk);
      rb[q] = to_f32<T>(B[(int64_t)min(k0 + kk, p.K - 1) * sd.bk + (int64_t)min(n0 + x, p.N - 1) * sd.bj]);
    }
  };
  const bool do_bias = p.form == FORM_DW && p.bias != nullptr && n0 == 0;
  float bsum = 0.0f;
  float acc[4][4];
#pragma unroll
  for (int i = 0; i < 4; ++i)
#pragma unroll
    for (int j = 0; j < 4; ++j) acc[i][j] = 0.0f;
  const int ti = (lane >> 3) * 4, tj = (lane & 7) * 4;
  fetch(0);
  for (int k0 = 0; k0 < p.K; k0 += GSK) {
#pragma unroll
    for (int q = 0; q < 8; ++q) {          // (a clamped row or column only feeds outputs that are not stored)
      int x, kk;
      place(a_k, q, x, kk);
      As[kk * ST + x] = k0 + kk < p.K ? ra[q] : 0.0f;
      place(b_k, q, x, kk);
      Bs[kk * ST + x] = k0 + kk < p.K ? rb[q] : 0.0f;
    }
    __syncthreads();
    if (k0 + GSK < p.K) fetch(k0 + GSK);
#pragma unroll 4        // (all sixteen at once take 256 registers and spill 53: twice the time at any size)
    for (int u = 0; u < GSK / 4; ++u) {
      const int kk = wave * (GSK / 4) + u;
      const float4 a = *(const float4 *)(As + kk * ST + ti), b = *(const float4 *)(Bs + kk * ST + tj);
      const float av[4] = {a.x, a.y, a.z, a.w}, bv[4] = {b.x, b.y, b.z, b.w};
#pragma unroll
      for (int i = 0; i < 4; ++i)
#pragma unroll
        for (int j = 0; j < 4; ++j) acc[i][j] = fmaf(av[i], bv[j], acc[i][j]);
    }
    if (do_bias && lane < GS) {
#pragma unroll
      for (int u = 0; u < GSK / 4; ++u) bsum += As[(wave * (GSK / 4) + u) * ST + lane];
    }
    __syncthreads();
  }

  // ---- the waves' partial tiles meet: two in each operand's block, added in wave order
  static_assert(GSK * ST >= 2 * GS * GS, "two partial tiles fit an operand block");
  float *part = (wave & 2 ? Bs : As) + (wave & 1) * GS * GS;
#pragma unroll
  for (int i = 0; i < 4; ++i) *(float4 *)(part + (ti + i) * GS + tj) = make_float4(acc[i][0], acc[i][1], acc[i][2], acc[i][3]);
  if (lane < GS) bias_part[wave][lane] = bsum;
  __syncthreads();
  if (do_bias && t < GS && m0 + t < p.M) {
    const float total = (bias_part[0][t] + bias_part[1][t]) + (bias_part[2][t] + bias_part[3][t]);
    GPP_G float *db = (GPP_G float *)p.bias + m0 + t;
    *db = accumulate_dw ? *db + total : total;
  }
  if (er >= p.M) return;
  const int at = (t >> 3) * GS + (t & 7) * 4;
#pragma unroll
  for (int e = 0; e < 4; ++e) {
    if (ec + e >= p.N) continue;
    float v = (As[at + e] + As[GS * GS + at + e]) + (Bs[at + e] + Bs[GS * GS + at + e]);
    const int64_t ci = (int64_t)er * p.ldc + ec + e;
    if (p.form == FORM_FWD) {
      v += bias[e];
      if (p.aux) store_from_f32(p.aux, p.aux_dtype, (int64_t)er * p.ldaux + ec + e, act_stash(v, p.act));
      v = act_apply(v, p.act) + res[e];
      store_from_f32(p.C, p.c_dtype, ci, v);
    } else if (p.form == FORM_DX) {
      v += res[e];
      if (p.act != ACT_NONE) v = grad_times(v, aux[e], p.act);
      store_from_f32(p.C, p.c_dtype, ci, v);
    } else {
      ((float *)p.C)[ci] = old[e] + v;
    }
  }
}

// BIAS: the launch holds weight gradients with a bias gradient (without them, eight waves per SIMD need no bound and a
// forward launch of [8192 x 1000 x 1000] takes 383 us instead of 391)
template <typename T, bool BIAS>
__global__ __launch_bounds__(256, BIAS ? 8 : 1) void k_gemm_generic(const GemmProb *__restrict__ probs, int n,
                                                       int accumulate_dw) {
  __shared__ float As[GK][GT + 4];
  __shared__ float Bs[GK][GT + 4];
  const int pi = find_prob(probs, n, blockIdx.x);
  const GemmProb p = probs[pi];
  const int tile = blockIdx.x - p.blk_begin;
  const int m0 = (tile / p.tiles_n) * GT, n0 = (tile % p.tiles_n) * GT;
  const int t = threadIdx.x, tx = t & 15, ty = t >> 4;

  const GenericStrides sd = generic_strides(p);
  const int64_t sai = sd.ai, sak = sd.ak, sbk = sd.bk, sbj = sd.bj;
  const T *A = (const T *)p.A;
  const T *B = (const T *)p.B;

  // backward-weight tiles of the first column block also sum the columns of dZ, the bias gradient: four row groups, in
  // a loop of its own (a test for it inside the contraction loop doubled the time of every launch) and in front of that
  // loop (behind it, next to the sixteen sums, it takes two registers more than eight waves per SIMD leave: forward of
  // [8192 x 1000 x 1000] 375 -> 467 us with seven)
  if (BIAS && p.form == FORM_DW && p.bias != nullptr && n0 == 0) {
    float bsum = 0.0f;
    const int bi = min(m0 + (t & (GT - 1)), p.M - 1);
#pragma unroll 4
    for (int k = t / GT; k < p.K; k += 256 / GT) bsum += to_f32<T>(A[(int64_t)k * sak + bi]);
    float *red = &As[0][0];
    red[t] = bsum;
    __syncthreads();
    if (t < GT && m0 + t < p.M) {
      const float total = (red[t] + red[GT + t]) + (red[2 * GT + t] + red[3 * GT + t]);
      GPP_G float *db = (GPP_G float *)p.bias + m0 + t;
      *db = accumulate_dw ? *db + total : total;
    }
    __syncthreads();
  }

  float acc[4][4];
#pragma unroll
  for (int i = 0; i < 4; ++i)
#pragma unroll
    for (int j = 0; j < 4; ++j) acc[i][j] = 0.0f;

  for (int k0 = 0; k0 < p.K; k0 += GK) {
#pragma unroll
    for (int r = 0; r < 4; ++r) {
      int e = t + 256 * r, ii, kk;
      if (sak == 1) { kk = e & 15; ii = e >> 4; } else { ii = e & 63; kk = e >> 6; }
      float v = 0.0f;
      if (m0 + ii < p.M && k0 + kk < p.K) v = to_f32<T>(A[(int64_t)(m0 + ii) * sai + (int64_t)(k0 + kk) * sak]);
      As[kk][ii] = v;
      int jj;
      if (sbk == 1) { kk = e & 15; jj = e >> 4; } else { jj = e & 63; kk = e >> 6; }
      v = 0.0f;
      if (n0 + jj < p.N && k0 + kk < p.K) v = to_f32<T>(B[(int64_t)(k0 + kk) * sbk + (int64_t)(n0 + jj) * sbj]);
      Bs[kk][jj] = v;
    }
    __syncthreads();
#pragma unroll
    for (int kk = 0; kk < GK; ++kk) {
      float a[4], b[4];
#pragma unroll
      for (int i = 0; i < 4; ++i) a[i] = As[kk][ty + 16 * i];
#pragma unroll
      for (int j = 0; j < 4; ++j) b[j] = Bs[kk][tx + 16 * j];
#pragma unroll
      for (int i = 0; i < 4; ++i)
#pragma unroll
        for (int j = 0; j < 4; ++j) acc[i][j] = fmaf(a[i], b[j], acc[i][j]);
    }
    __syncthreads();
  }
#pragma unroll
  for (int i = 0; i < 4; ++i) {
    const int row = m0 + ty + 16 * i;
    if (row >= p.M) continue;
#pragma unroll
    for (int j = 0; j < 4; ++j) {
      const int col = n0 + tx + 16 * j;
      if (col >= p.N) continue;
      float v = acc[i][j];
      const int64_t ci = (int64_t)row * p.ldc + col;
      if (p.form == FORM_FWD) {
        if (p.bias) v += p.bias[col];
        if (p.aux) store_from_f32(p.aux, p.aux_dtype, (int64_t)row * p.ldaux + col, act_stash(v, p.act));
        v = act_apply(v, p.act);
        if (p.res) v += load_as_f32(p.res, p.res_dtype, (int64_t)row * p.ldres + col);
        store_from_f32(p.C, p.c_dtype, ci, v);
      } else if (p.form == FORM_DX) {
        if (p.res) v += load_as_f32(p.res, p.res_dtype, (int64_t)row * p.ldres + col);
        if (p.act != ACT_NONE) v = grad_times(v, load_as_f32(p.aux, p.aux_dtype, (int64_t)row * p.ldaux + col), p.act);
        store_from_f32(p.C, p.c_dtype, ci, v);
      } else {
        float *c = (float *)p.C;
        c[ci] = accumulate_dw ? c[ci] + v : v;
      }
    }
  }
}

template <typename T>
static void launch_generic_type(const GemmProb *probs, int n, int blocks, int accumulate_dw, int tile, bool bias, hipStream_t s) {
  const dim3 g(blocks), b(256);
  if (tile == GS) hipLaunchKernelGGL(k_gemm_generic_small<T>, g, b, 0, s, probs, n, accumulate_dw);
  else if (bias) hipLaunchKernelGGL((k_gemm_generic<T, true>), g, b, 0, s, probs, n, accumulate_dw);
  else hipLaunchKernelGGL((k_gemm_generic<T, false>), g, b, 0, s, probs, n, accumulate_dw);
}
// bias: some weight-gradient record has a bias gradient
void launch_gemm_generic(const GemmProb *probs, int n, int total_blocks, int accumulate_dw, int in_dtype, int tile, bool bias,
                         hipStream_t s) {
  if (total_blocks <= 0) return;
  if (in_dtype == DT_BF16) launch_generic_type<uint16_t>(probs, n, total_blocks, accumulate_dw, tile, bias, s);
  else launch_generic_type<float>(probs, n, total_blocks, accumulate_dw, tile, bias, s);
}

}  // namespace gpp
