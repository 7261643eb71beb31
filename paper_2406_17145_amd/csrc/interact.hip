// Pairwise-dot feature interaction of a DLRM-shaped stage (forward and backward),
// grouped over operators; a workgroup per sample with the F vectors in LDS, or a wave per
// sample on the matrix cores.
#include <algorithm>

#include "gemm_direct.h"

namespace gpp {

// ------------------------------------------------------------------ pairwise-dot interaction
// one workgroup per sample; the F vectors sit in LDS
__device__ __forceinline__ void term_to_pair(int t, int &i, int &j) {
  i = (int)((1.0f + sqrtf(1.0f + 8.0f * (float)t)) * 0.5f);
  while (i * (i - 1) / 2 > t) --i;
  while ((i + 1) * i / 2 <= t) ++i;
  j = t - i * (i - 1) / 2;
}

// ---- vector bodies: rows of whole, aligned 16-byte chunks, one storage type for x / y / dy.  The type
// is a template parameter, so that the loads of a phase are requested together (a run-time type test in
// front of every load is a branch, and a wave waits for its earlier loads at a branch).
template <int DT>
__device__ __forceinline__ void ld8(const void *base, int64_t i, float (&v)[8]) {
  if (DT == DT_BF16) {
    const uint4 u = *(const uint4 *)((const uint16_t *)base + i);
    const uint32_t w[4] = {u.x, u.y, u.z, u.w};
#pragma unroll
    for (int e = 0; e < 4; ++e) {
      v[2 * e] = __uint_as_float(w[e] << 16);
      v[2 * e + 1] = __uint_as_float(w[e] & 0xffff0000u);
    }
  } else {
    const float4 a = *(const float4 *)((const float *)base + i), b = *(const float4 *)((const float *)base + i + 4);
    v[0] = a.x; v[1] = a.y; v[2] = a.z; v[3] = a.w; v[4] = b.x; v[5] = b.y; v[6] = b.z; v[7] = b.w;
  }
}
template <int DT>
__device__ __forceinline__ void st8(void *base, int64_t i, const float (&v)[8]) {
  if (DT == DT_BF16) {
    uint4 u;
    u.x = (uint32_t)f32_to_bf16_bits(v[0]) | ((uint32_t)f32_to_bf16_bits(v[1]) << 16);
    u.y = (uint32_t)f32_to_bf16_bits(v[2]) | ((uint32_t)f32_to_bf16_bits(v[3]) << 16);
    u.z = (uint32_t)f32_to_bf16_bits(v[4]) | ((uint32_t)f32_to_bf16_bits(v[5]) << 16);
    u.w = (uint32_t)f32_to_bf16_bits(v[6]) | ((uint32_t)f32_to_bf16_bits(v[7]) << 16);
    *(uint4 *)((uint16_t *)base + i) = u;
  } else {
    *(float4 *)((float *)base + i) = make_float4(v[0], v[1], v[2], v[3]);
    *(float4 *)((float *)base + i + 4) = make_float4(v[4], v[5], v[6], v[7]);
  }
}
constexpr int INT_GP = 32;          // row stride of the F x F gradient matrix in the vector backward body
constexpr int INT_MAX_CHUNKS = 4;   // 8-element chunks of the F x d block per thread: F * d <= 8192
__device__ __forceinline__ bool interact_vec_ok(const InteractProb &p, bool bwd) {
  if ((p.d & 7) || p.F * p.d > 256 * 8 * INT_MAX_CHUNKS) return false;
  if ((p.ld_x & 7) || ((uintptr_t)p.x & 15)) return false;
  if (bwd && ((p.ld_y & 7) || ((uintptr_t)p.y & 15) || p.F > INT_GP)) return false;   // G in rows of INT_GP
  return true;
}
// the F x d block of sample s into LDS rows of stride d + 4 floats: rows stay 16-byte aligned, and sixteen
// consecutive rows read with 16-byte reads fall into sixteen different groups of four banks
__device__ __forceinline__ int interact_stride(int d) { return d + 4; }
template <int DT>
__device__ __forceinline__ void interact_stage_x(const InteractProb &p, int s, float *T, int st) {
  const int chunks = (p.F * p.d) >> 3;
  float v[INT_MAX_CHUNKS][8];
#pragma unroll
  for (int u = 0; u < INT_MAX_CHUNKS; ++u) {
    const int q = threadIdx.x + 256 * u;
    ld8<DT>(p.x, (int64_t)s * p.ld_x + 8 * (q < chunks ? q : 0), v[u]);
  }
#pragma unroll
  for (int u = 0; u < INT_MAX_CHUNKS; ++u) {
    const int q = threadIdx.x + 256 * u;
    if (q < chunks) {
      const int row = (8 * q) / p.d, col = 8 * q - row * p.d;
      float4 *dst = (float4 *)(T + row * st + col);
      dst[0] = make_float4(v[u][0], v[u][1], v[u][2], v[u][3]);
      dst[1] = make_float4(v[u][4], v[u][5], v[u][6], v[u][7]);
    }
  }
}
// A thread per dot product, four columns per pair of 16-byte LDS reads, summed in column order.  (One 4-byte
// read per operand and column was two LDS instructions per multiply-add: 18 us for 2048 samples of 27 x 128.)
template <int DT>
__device__ __forceinline__ void interact_fwd_vec(const InteractProb &p, int s, float *lds) {
  const int st = interact_stride(p.d);
  interact_stage_x<DT>(p, s, lds, st);
  __syncthreads();
  for (int c = threadIdx.x; c < p.d; c += 256) store_from_f32(p.y, DT, (int64_t)s * p.ld_y + c, lds[c]);
  const int terms = p.F * (p.F - 1) / 2;
  for (int t = threadIdx.x; t < terms; t += 256) {
    int i, j;
    term_to_pair(t, i, j);
    const float4 *xi = (const float4 *)(lds + i * st), *xj = (const float4 *)(lds + j * st);
    float a = 0.0f;
    for (int c = 0; c < (p.d >> 2); ++c) {
      const float4 u = xi[c], v = xj[c];
      a += u.x * v.x;
      a += u.y * v.y;
      a += u.z * v.z;
      a += u.w * v.w;
    }
    store_from_f32(p.y, DT, (int64_t)s * p.ld_y + p.d + t, a);
  }
}
// Backward: dT[i][c] = sum_j G[i][j] T[j][c] (+ the pass-through of vector 0), G the symmetric matrix of the
// dot-product gradients with a zero diagonal.  COLS: the vector width d when it divides 256 (64, 128, 256), else 0.
// With COLS a thread owns one column c and the rows i = g, g + 256 / d, ...: it keeps its column of T in
// registers (F <= 32 values) and reads G four entries at a time; a wave covers 64 columns of ONE row, so those
// reads are the same address for all its lanes.  About one LDS instruction per six multiply-adds instead of two
// per multiply-add (34 -> ~12 us for 2048 samples of 27 x 128).  Sums run over j in ascending order either way.
template <int DT, int COLS>
__device__ __forceinline__ void interact_bwd_vec(const InteractProb &p, int s, float *lds) {
  const int st = interact_stride(p.d);
  float *T = lds;
  float *G = lds + p.F * st;  // symmetric F x F in rows of INT_GP, zero diagonal
  const int terms = p.F * (p.F - 1) / 2;
  // the gradients of the dot products (their offset d + t is not chunk-aligned: element loads), all
  // of a thread's requested before the block of x is staged
  constexpr int GT = 4;
  float g[GT];
#pragma unroll
  for (int u = 0; u < GT; ++u) {
    const int t = threadIdx.x + 256 * u;
    g[u] = load_as_f32(p.dy, DT, (int64_t)s * p.ld_dy + p.d + (t < terms ? t : 0));
  }
  interact_stage_x<DT>(p, s, T, st);
  for (int e = threadIdx.x; e < p.F; e += 256) G[e * INT_GP + e] = 0.0f;
#pragma unroll
  for (int u = 0; u < GT; ++u) {
    const int t = threadIdx.x + 256 * u;
    if (t < terms) {
      int i, j;
      term_to_pair(t, i, j);
      G[i * INT_GP + j] = g[u];
      G[j * INT_GP + i] = g[u];
    }
  }
  for (int t = threadIdx.x + 256 * GT; t < terms; t += 256) {   // more than 1024 terms (F > 45)
    int i, j;
    term_to_pair(t, i, j);
    const float gv = load_as_f32(p.dy, DT, (int64_t)s * p.ld_dy + p.d + t);
    G[i * INT_GP + j] = gv;
    G[j * INT_GP + i] = gv;
  }
  __syncthreads();
  if (COLS > 0) {
    const int c = threadIdx.x % COLS, g0 = threadIdx.x / COLS;
    float tc[INT_GP];
#pragma unroll
    for (int j = 0; j < INT_GP; ++j) tc[j] = j < p.F ? T[j * st + c] : 0.0f;
    const float pass = load_as_f32(p.dy, DT, (int64_t)s * p.ld_dy + c);
    for (int i = g0; i < p.F; i += 256 / COLS) {
      float a = i == 0 ? pass : 0.0f;
      const float4 *gr = (const float4 *)(G + i * INT_GP);
#pragma unroll
      for (int q = 0; q < INT_GP / 4; ++q) {
        const float4 gv = gr[q];
        if (4 * q + 0 < p.F) a += gv.x * tc[4 * q + 0];
        if (4 * q + 1 < p.F) a += gv.y * tc[4 * q + 1];
        if (4 * q + 2 < p.F) a += gv.z * tc[4 * q + 2];
        if (4 * q + 3 < p.F) a += gv.w * tc[4 * q + 3];
      }
      store_from_f32(p.y, DT, (int64_t)s * p.ld_y + (int64_t)i * p.d + c, a);
    }
    return;
  }
  // a thread per element, consecutive columns in consecutive lanes (LDS reads without bank conflicts)
  for (int e = threadIdx.x; e < p.F * p.d; e += 256) {
    const int i = e / p.d, c = e - i * p.d;
    float a = i == 0 ? load_as_f32(p.dy, DT, (int64_t)s * p.ld_dy + c) : 0.0f;
    for (int j = 0; j < p.F; ++j) a += G[i * INT_GP + j] * T[j * st + c];
    store_from_f32(p.y, DT, (int64_t)s * p.ld_y + e, a);
  }
}
template <int DT>
__device__ __forceinline__ void interact_bwd_pick(const InteractProb &p, int s, float *lds) {
  if (p.F <= INT_GP && p.d == 64) return interact_bwd_vec<DT, 64>(p, s, lds);
  if (p.F <= INT_GP && p.d == 128) return interact_bwd_vec<DT, 128>(p, s, lds);
  if (p.F <= INT_GP && p.d == 256) return interact_bwd_vec<DT, 256>(p, s, lds);
  return interact_bwd_vec<DT, 0>(p, s, lds);
}

__global__ __launch_bounds__(256) void k_interact_fwd(const InteractProb *__restrict__ probs, int n) {
  extern __shared__ float lds[];
  const int pi = find_prob(probs, n, blockIdx.x);
  const InteractProb p = probs[pi];
  const int s = blockIdx.x - p.blk_begin;
  if (interact_vec_ok(p, false) && p.x_dtype == p.y_dtype) {
    if (p.x_dtype == DT_BF16) return interact_fwd_vec<DT_BF16>(p, s, lds);
    if (p.x_dtype == DT_F32) return interact_fwd_vec<DT_F32>(p, s, lds);
  }
  const int st = p.d + 1;
  for (int e = threadIdx.x; e < p.F * p.d; e += 256)
    lds[(e / p.d) * st + (e % p.d)] = load_as_f32(p.x, p.x_dtype, (int64_t)s * p.ld_x + e);
  __syncthreads();
  for (int c = threadIdx.x; c < p.d; c += 256) store_from_f32(p.y, p.y_dtype, (int64_t)s * p.ld_y + c, lds[c]);
  const int terms = p.F * (p.F - 1) / 2;
  for (int t = threadIdx.x; t < terms; t += 256) {
    int i, j;
    term_to_pair(t, i, j);
    float a = 0.0f;
    for (int c = 0; c < p.d; ++c) a += lds[i * st + c] * lds[j * st + c];
    store_from_f32(p.y, p.y_dtype, (int64_t)s * p.ld_y + p.d + t, a);
  }
}

__global__ __launch_bounds__(256) void k_interact_bwd(const InteractProb *__restrict__ probs, int n) {
  extern __shared__ float lds[];
  const int pi = find_prob(probs, n, blockIdx.x);
  const InteractProb p = probs[pi];
  const int s = blockIdx.x - p.blk_begin;
  if (interact_vec_ok(p, true) && p.x_dtype == p.y_dtype && p.x_dtype == p.dy_dtype && (p.ld_dy & 7) == 0 &&
      ((uintptr_t)p.dy & 15) == 0) {
    if (p.x_dtype == DT_BF16) return interact_bwd_pick<DT_BF16>(p, s, lds);
    if (p.x_dtype == DT_F32) return interact_bwd_pick<DT_F32>(p, s, lds);
  }
  const int st = p.d + 1;
  float *T = lds;
  float *G = lds + p.F * st;  // symmetric F x F, zero diagonal
  for (int e = threadIdx.x; e < p.F * p.d; e += 256)
    T[(e / p.d) * st + (e % p.d)] = load_as_f32(p.x, p.x_dtype, (int64_t)s * p.ld_x + e);
  for (int e = threadIdx.x; e < p.F; e += 256) G[e * p.F + e] = 0.0f;
  const int terms = p.F * (p.F - 1) / 2;
  for (int t = threadIdx.x; t < terms; t += 256) {
    int i, j;
    term_to_pair(t, i, j);
    float g = load_as_f32(p.dy, p.dy_dtype, (int64_t)s * p.ld_dy + p.d + t);
    G[i * p.F + j] = g;
    G[j * p.F + i] = g;
  }
  __syncthreads();
  for (int e = threadIdx.x; e < p.F * p.d; e += 256) {
    const int i = e / p.d, c = e % p.d;
    float a = i == 0 ? load_as_f32(p.dy, p.dy_dtype, (int64_t)s * p.ld_dy + c) : 0.0f;
    for (int j = 0; j < p.F; ++j) a += G[i * p.F + j] * T[j * st + c];
    store_from_f32(p.y, p.y_dtype, (int64_t)s * p.ld_y + e, a);
  }
}

// ---- on the matrix cores: bf16 storage everywhere, up to 32 vectors of 64, 128 or 256 columns.  A WAVE per sample, four to a
// workgroup, no barrier: the dot products are one 32 x 32 product of the vectors with themselves, whose two operand fragments
// are the same registers, loaded straight from memory.  Bound by latency (a sample is 7 KB).  The products of bf16 values are exact in
// fp32 and summed in fp32, as on the vector path.  2048 samples of 27 x 128: forward 12.3 us there, 6.1 here; backward 26.1 and
// 10.5 (17.5 while the lanes stored their four columns straight to memory, 32 rows to a store).
template <int D>
__global__ __launch_bounds__(256) void k_interact_fwd_mfma(const InteractProb *__restrict__ probs, int n) {
  const int pi = find_prob(probs, n, blockIdx.x);
  const InteractProb p = probs[pi];
  const int s = (blockIdx.x - p.blk_begin) * 4 + (threadIdx.x >> 6), l = threadIdx.x & 63;
  if (s >= p.batch) return;
  const GPP_G uint16_t *x = (const GPP_G uint16_t *)p.x + (int64_t)s * p.ld_x;
  GPP_G uint16_t *y = (GPP_G uint16_t *)p.y + (int64_t)s * p.ld_y;
  const GPP_G uint16_t *row = x + min(l & 31, p.F - 1) * D + 8 * (l >> 5);      // (rows beyond F feed products that are not stored)
  bf16x8 a[D / 16];
#pragma unroll
  for (int c = 0; c < D / 16; ++c) a[c] = *(const GPP_G bf16x8 *)(row + 16 * c);
  uint16_t first[D / 64];
#pragma unroll
  for (int u = 0; u < D / 64; ++u) first[u] = x[l + 64 * u];
  f32x16 acc;
#pragma unroll
  for (int r = 0; r < 16; ++r) acc[r] = 0.0f;
#pragma unroll
  for (int c = 0; c < D / 16; ++c) acc = __builtin_amdgcn_mfma_f32_32x32x16_bf16(a[c], a[c], acc, 0, 0, 0);
#pragma unroll
  for (int u = 0; u < D / 64; ++u) y[l + 64 * u] = first[u];
  const int j = l & 31;
#pragma unroll
  for (int r = 0; r < 16; ++r) {
    const int i = epi_row(r) + 4 * (l >> 5);
    if (i < p.F && j < i) y[D + i * (i - 1) / 2 + j] = f32_to_bf16_bits(acc[r]);
  }
}
// Backward: dT^T [column][i] = sum_j T^T [column][j] G[j][i].  T goes through a wave-private LDS tile for the transposing read (rows
// beyond F as zeros: they meet zeros of G), G is symmetric, a lane gathers its eight entries of a row; a lane's four consecutive
// accumulators are four consecutive columns of one vector and go back into the tile, in place of the columns just read, so that the
// result leaves in whole rows.
template <int D>
__global__ __launch_bounds__(256) void k_interact_bwd_mfma(const InteractProb *__restrict__ probs, int n) {
  __shared__ __attribute__((aligned(16))) uint16_t lds[4 * 32 * D];
  const int pi = find_prob(probs, n, blockIdx.x);
  const InteractProb p = probs[pi];
  const int wave = threadIdx.x >> 6, s = (blockIdx.x - p.blk_begin) * 4 + wave, l = threadIdx.x & 63;
  if (s >= p.batch) return;
  const GPP_G uint16_t *x = (const GPP_G uint16_t *)p.x + (int64_t)s * p.ld_x, *dy = (const GPP_G uint16_t *)p.dy + (int64_t)s * p.ld_dy;
  GPP_G uint16_t *dx = (GPP_G uint16_t *)p.y + (int64_t)s * p.ld_y;
  uint16_t *tile = lds + wave * 32 * D;
  constexpr int CPR = D / 8, LOADS = 32 * CPR / 64;
  u32x4 v[LOADS];
#pragma unroll
  for (int u = 0; u < LOADS; ++u) {
    const int q = l + 64 * u;
    v[u] = *(const GPP_G u32x4 *)(x + min(q / CPR, p.F - 1) * D + (q % CPR) * 8);
  }
  const int i = l & 31;
  uint32_t g[2][4];
#pragma unroll
  for (int kk = 0; kk < 2; ++kk)
#pragma unroll
    for (int e = 0; e < 8; ++e) {
      const int j = 16 * kk + 8 * (l >> 5) + e, hi = max(i, j), lo = min(i, j);
      const bool ok = hi < p.F && i != j;
      const uint32_t w = dy[D + (ok ? hi * (hi - 1) / 2 + lo : 0)];
      g[kk][e / 2] = (e & 1) ? g[kk][e / 2] | (ok ? w << 16 : 0u) : (ok ? w : 0u);
    }
#pragma unroll
  for (int u = 0; u < LOADS; ++u) {
    const int q = l + 64 * u, row = q / CPR;
    const u32x4 zero = {0u, 0u, 0u, 0u};
    *(u32x4 *)(tile + row * D + (((q % CPR) ^ direct_tr_swizzle<D>(row)) << 3)) = row < p.F ? v[u] : zero;
  }
  typedef uint32_t u32x2 __attribute__((ext_vector_type(2)));
  u32x2 pass[D / 8];
#pragma unroll
  for (int u = 0; u < D / 8; ++u) pass[u] = *(const GPP_G u32x2 *)(dy + 8 * u + 4 * (l >> 5));
  __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
  __builtin_amdgcn_wave_barrier();
#pragma unroll
  for (int ct = 0; ct < D / 32; ++ct) {
    f32x16 acc;
#pragma unroll
    for (int r = 0; r < 16; ++r)
      acc[r] = i == 0 ? bf16_bits_to_f32((uint16_t)(pass[4 * ct + r / 4][(r & 3) / 2] >> (16 * (r & 1)))) : 0.0f;
#pragma unroll
    for (int kk = 0; kk < 2; ++kk) {
      const u32x4 gv = {g[kk][0], g[kk][1], g[kk][2], g[kk][3]};
      acc = __builtin_amdgcn_mfma_f32_32x32x16_bf16(direct_frag_tr<D>(tile, 32 * ct, 16 * kk), __builtin_bit_cast(bf16x8, gv), acc, 0, 0, 0);
    }
    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
    // (the columns just read: nothing reads them again)
#pragma unroll
    for (int q = 0; q < 4; ++q) {
      const u32x2 w = {(uint32_t)f32_to_bf16_bits(acc[4 * q]) | ((uint32_t)f32_to_bf16_bits(acc[4 * q + 1]) << 16),
                       (uint32_t)f32_to_bf16_bits(acc[4 * q + 2]) | ((uint32_t)f32_to_bf16_bits(acc[4 * q + 3]) << 16)};
      *(u32x2 *)(tile + i * D + (((4 * ct + q) ^ direct_tr_swizzle<D>(i)) << 3) + 4 * (l >> 5)) = w;
    }
  }
  __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
  __builtin_amdgcn_wave_barrier();
#pragma unroll
  for (int u = 0; u < LOADS; ++u) {
    const int q = l + 64 * u, row = q / CPR;
    if (row < p.F) *(GPP_G u32x4 *)(dx + row * D + (q % CPR) * 8) = *(const u32x4 *)(tile + row * D + (((q % CPR) ^ direct_tr_swizzle<D>(row)) << 3));
  }
}
bool interact_mfma_ok(const InteractProb &p, bool backward) {
  if (p.x_dtype != DT_BF16 || p.y_dtype != DT_BF16 || (backward && p.dy_dtype != DT_BF16)) return false;
  if (p.F < 2 || p.F > 32 || (p.d != 64 && p.d != 128 && p.d != 256)) return false;
  if ((p.ld_x & 7) || ((uintptr_t)p.x & 15)) return false;
  return !backward || ((p.ld_y & 7) == 0 && ((uintptr_t)p.y & 15) == 0 && (p.ld_dy & 3) == 0 && ((uintptr_t)p.dy & 7) == 0);
}
int interact_mfma_blocks(int batch) { return (batch + 3) / 4; }

// rows of d + 4 (vector bodies; the scalar bodies use d + 1) and a gradient matrix of max(F, 32) x max(F, 32)
static size_t interact_lds(int F, int d) { return ((size_t)F * (d + 4) + (size_t)std::max(F, 32) * std::max(F, 32)) * sizeof(float); }
// mfma: the width that all records share where they run on the matrix cores, else 0
void launch_interact_fwd(const InteractProb *probs, int n, int total_blocks, int maxF, int maxd, int mfma, hipStream_t s) {
  if (total_blocks <= 0) return;
  const dim3 g(total_blocks), b(256);
  if (mfma == 64) hipLaunchKernelGGL(k_interact_fwd_mfma<64>, g, b, 0, s, probs, n);
  if (mfma == 128) hipLaunchKernelGGL(k_interact_fwd_mfma<128>, g, b, 0, s, probs, n);
  if (mfma == 256) hipLaunchKernelGGL(k_interact_fwd_mfma<256>, g, b, 0, s, probs, n);
  if (mfma == 0) hipLaunchKernelGGL(k_interact_fwd, g, b, interact_lds(maxF, maxd), s, probs, n);
}
void launch_interact_bwd(const InteractProb *probs, int n, int total_blocks, int maxF, int maxd, int mfma, hipStream_t s) {
  if (total_blocks <= 0) return;
  const dim3 g(total_blocks), b(256);
  if (mfma == 64) hipLaunchKernelGGL(k_interact_bwd_mfma<64>, g, b, 0, s, probs, n);
  if (mfma == 128) hipLaunchKernelGGL(k_interact_bwd_mfma<128>, g, b, 0, s, probs, n);
  if (mfma == 256) hipLaunchKernelGGL(k_interact_bwd_mfma<256>, g, b, 0, s, probs, n);
  if (mfma == 0) hipLaunchKernelGGL(k_interact_bwd, g, b, interact_lds(maxF, maxd), s, probs, n);
}
size_t interact_lds_bytes(int F, int d) { return interact_lds(F, d); }

}  // namespace gpp
