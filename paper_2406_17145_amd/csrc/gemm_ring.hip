// Branch-grouped bf16 GEMM out of a ring of LDS buffers: the operand tiles of the next BUFS - 1 k-steps are on their way from
// memory into LDS (gemm_direct.h) while one is multiplied, one barrier per k-step, nothing staged in registers.  Small
// workgroups, two or three to a compute unit:
//
// k_gemm_ring   forward and backward-data of launches that the large tiles would leave compute units idle with: 128 x 64
//               (eight waves, a wave tile of 32 x 32) and 64 x 64 (four waves) outputs, k-steps of 64, three buffers
//               (72 / 48 KB of LDS: two / three workgroups per compute unit).  What bounds such a launch is the chain of a
//               tile's k-steps, which the copies in flight shorten, and the launch itself.
// k_gemm_ring_dw   weight gradients over the stash slots of a group of backward passes (or one pass's): 256 x 128 outputs, four
//               waves with a wave tile of 128 x 64, k-steps of 32, three buffers, two workgroups per compute unit whose
//               stores hide behind each other's products.  Both operands run along the contraction, so a k-step of any
//               length reads whole cache lines.  Bound by the matrix cores and, at 512 rows, by the stores.
#include <algorithm>

#include "gemm_direct.h"

namespace gpp {

// BK: contraction elements per k-step (64 where a k-contiguous operand's row should be a cache line)
template <int FORM, int WGM, int WGN, int TM, int TN, int BUFS, int BK>
struct RingCfg {
  static constexpr int NW = WGM * WGN, THREADS = 64 * NW, BM = 32 * TM * WGM, BN = 32 * TN * WGN;
  static constexpr int A_ELEMS = BK * BM, B_ELEMS = BK * BN, EPI = NW * epi_lds_floats<TN>() * 2;
  static constexpr int ELEMS = BUFS * (A_ELEMS + B_ELEMS) > EPI ? BUFS * (A_ELEMS + B_ELEMS) : EPI;
  static constexpr int COPIES = (BM + BN) * BK / 8 / 64 / NW;      // copy instructions of a wave per k-step
  static_assert(BK == GB_BK || FORM == FORM_DW, "k-contiguous tiles are 64 elements wide");
  static_assert((BUFS - 1) * COPIES < 64, "vmcnt is a 6-bit counter");
  static_assert(ELEMS * 2 <= 160 * 1024, "the buffers do not fit the LDS");
};

// Order of the sums: the large tiles' one chain per output over the whole contraction, the small tiles' two, added at the end.
template <int FORM, int WGM, int WGN, int TM, int TN, int BUFS, int BK, bool STREAM = false>
__device__ __forceinline__ void ring_body(const GemmProb &p, int m0, int n0, uint16_t *lds, int accumulate_dw, const ExtPtrs &ext,
                                          const SlotGroup &grp) {
  typedef RingCfg<FORM, WGM, WGN, TM, TN, BUFS, BK> C;
  constexpr int BM = C::BM, BN = C::BN, NW = C::NW;
  constexpr bool A_TR = FORM == FORM_DW, B_TR = FORM != FORM_FWD;
  const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int wi0 = (wave / WGN) * (32 * TM), wj0 = (wave % WGN) * (32 * TN);
  rsrc4 rs_a = matrix_rsrc4(p.A, A_TR ? p.K : p.M, p.lda, A_TR ? p.M : p.K);
  rsrc4 rs_b = matrix_rsrc4(p.B, B_TR ? p.K : p.N, p.ldb, B_TR ? p.N : p.K);
  settle(rs_a, rs_b);
  // (a wave with one MFMA tile sums even and odd 16-wide chunks apart: its MFMAs are two chains instead of one)
  constexpr int CHAINS = TM * TN == 1 ? 2 : 1;
  f32x16 acc_of[CHAINS][TM][TN];
  f32x16 (&acc)[TM][TN] = acc_of[0];
#pragma unroll
  for (int q = 0; q < CHAINS; ++q)
#pragma unroll
    for (int i = 0; i < TM; ++i)
#pragma unroll
      for (int j = 0; j < TN; ++j)
#pragma unroll
        for (int r = 0; r < 16; ++r) acc_of[q][i][j][r] = 0.0f;
  auto da = [&](int b) { return lds + b * C::A_ELEMS; };
  auto db = [&](int b) { return lds + BUFS * C::A_ELEMS + b * C::B_ELEMS; };
  const uint32_t lds0 = lds_address(lds);
  const int nk_slot = cdiv(p.K, BK), nk = FORM == FORM_DW ? nk_slot * grp.n : nk_slot;

  // The k-steps are copied in order.  Weight gradients: contraction elements of the group's slots one after the other; a
  // k-step behind the last one copies zeros from descriptors of no bytes (no address outside the slots is formed).
  int copy_k = 0, copy_slot = grp.first, copy_left = nk;
  const uint32_t bytes_a = rs_a[2], bytes_b = rs_b[2];
  auto point_at_slot = [&]() {
    const uint64_t a = (uint64_t)p.A + (uint64_t)copy_slot * (uint64_t)grp.stride, b = (uint64_t)p.B + (uint64_t)copy_slot * (uint64_t)grp.stride;
    rs_a[0] = (uint32_t)__builtin_amdgcn_readfirstlane((int)(uint32_t)a);
    rs_a[1] = (uint32_t)__builtin_amdgcn_readfirstlane((int)((uint32_t)(a >> 32) & 0xffffu));
    rs_b[0] = (uint32_t)__builtin_amdgcn_readfirstlane((int)(uint32_t)b);
    rs_b[1] = (uint32_t)__builtin_amdgcn_readfirstlane((int)((uint32_t)(b >> 32) & 0xffffu));
    settle(rs_a, rs_b);
  };
  if constexpr (FORM == FORM_DW) point_at_slot();
  auto copy_next = [&](int buf) {
    const uint32_t to_a = lds0 + buf * C::A_ELEMS * 2, to_b = lds0 + (BUFS * C::A_ELEMS + buf * C::B_ELEMS) * 2;
    if constexpr (FORM == FORM_DW) {
      rs_a[2] = copy_left > 0 ? bytes_a : 0u;
      rs_b[2] = copy_left > 0 ? bytes_b : 0u;
      direct_tr<BM, NW, BK>(rs_a, p.lda, copy_k, m0, to_a, wave, lane);
      direct_tr<BN, NW, BK>(rs_b, p.ldb, copy_k, n0, to_b, wave, lane);
      copy_k += BK;
      --copy_left;
      if (copy_k >= p.K && copy_left > 0) {
        copy_k = 0;
        copy_slot = copy_slot + 1 == grp.total ? 0 : copy_slot + 1;
        point_at_slot();
      }
    } else {
      direct_kmajor<BM, NW>(rs_a, p.lda, m0, copy_k, p.K, to_a, wave, lane);
      if constexpr (B_TR) direct_tr<BN, NW, BK>(rs_b, p.ldb, copy_k, n0, to_b, wave, lane);
      else direct_kmajor<BN, NW>(rs_b, p.ldb, n0, copy_k, p.K, to_b, wave, lane);
      copy_k += BK;
    }
  };

  // weight gradients: tiles of the first column block also sum the rows of dZ^T they stream, the bias gradient.  A k-step
  // holds its columns in BM / 8 chunks per row; a thread sums one column over a group of rows
  constexpr int BGROUPS = A_TR ? C::THREADS / BM : 1, BROWS = BK / BGROUPS;
  const bool do_bias = FORM == FORM_DW && p.bias != nullptr && n0 == 0;
  float bsum = 0.0f;
  auto bias_rows = [&](const uint16_t *tile) {
    const int col = tid % BM, r0 = (tid / BM) * BROWS;
#pragma unroll
    for (int r = 0; r < BROWS; ++r)
      bsum += bf16_bits_to_f32(tile[(r0 + r) * BM + ((((col >> 3) ^ direct_tr_swizzle<BM>(r0 + r)) << 3) | (col & 7))]);
  };

  // one k-step out of buffer `cur`; TAIL: the contraction ends inside it, and what lies beyond it in a chunk of a
  // k-contiguous row (row padding) is cleared -- both operands' in forward; in backward-data the other operand's rows
  // beyond the contraction have read zero, but zero times what padding holds need not be
  auto multiply = [&](int cur, int k0, auto tail) {
    constexpr bool TAIL = decltype(tail)::value;
    constexpr int NC = BK / 16;
    bf16x8 a[2][TM], b[2][TN];
    auto clear = [&](bf16x8 v, int c) {
      return __builtin_bit_cast(bf16x8, chunk_clear_tail(__builtin_bit_cast(u32x4, v), k0 + 16 * c + 8 * (lane >> 5), p.K));
    };
    auto frags = [&](int set, int c) {
#pragma unroll
      for (int j = 0; j < TN; ++j) {
        b[set][j] = B_TR ? direct_frag_tr<BN>(db(cur), wj0 + 32 * j, 16 * c) : direct_frag_kmajor(db(cur), wj0 + 32 * j, 16 * c);
        if (TAIL && !B_TR) b[set][j] = clear(b[set][j], c);
      }
#pragma unroll
      for (int i = 0; i < TM; ++i) {
        a[set][i] = A_TR ? direct_frag_tr<BM>(da(cur), wi0 + 32 * i, 16 * c) : direct_frag_kmajor(da(cur), wi0 + 32 * i, 16 * c);
        if (TAIL && !A_TR) a[set][i] = clear(a[set][i], c);
      }
    };
    frags(0, 0);
#pragma unroll
    for (int c = 0; c < NC; ++c) {
      if (c + 1 < NC) frags((c + 1) & 1, c + 1);
#pragma unroll
      for (int i = 0; i < TM; ++i)
#pragma unroll
        for (int j = 0; j < TN; ++j) {
          f32x16 &sum = acc_of[c % CHAINS][i][j];
          sum = __builtin_amdgcn_mfma_f32_32x32x16_bf16(a[c & 1][i], b[c & 1][j], sum, 0, 0, 0);
        }
      if (!TAIL && TM * TN > 1) big_mix<TM * TN, (A_TR ? 2 : 1) * TM + (B_TR ? 2 : 1) * TN>();
    }
  };

  const int whole = FORM != FORM_DW && (p.K & 7) != 0 ? nk - 1 : nk;      // k-steps without a ragged chunk
#pragma unroll
  for (int u = 0; u < BUFS - 1; ++u) copy_next(u);
  int cur = 0;
  for (int kt = 0; kt < whole; ++kt) {
    // k-step kt has landed, and every wave has read k-step kt - 1, whose buffer is refilled
    copies_landed_barrier<(BUFS - 2) * C::COPIES>();
    copy_next(cur == 0 ? BUFS - 1 : cur - 1);
    multiply(cur, 0, std::false_type());
    if (FORM == FORM_DW && do_bias) bias_rows(da(cur));
    cur = cur + 1 == BUFS ? 0 : cur + 1;
  }
  if (FORM != FORM_DW && whole < nk) {
    copies_landed_barrier<(BUFS - 2) * C::COPIES>();
    multiply(cur, whole * BK, std::true_type());
  }
  if constexpr (CHAINS == 2) acc[0][0] += acc_of[1][0][0];
  asm volatile("s_waitcnt vmcnt(0)" ::: "memory");   // the copies of the k-steps beyond the end
  __syncthreads();                                   // the epilogue reuses the operand LDS

  if constexpr (FORM == FORM_DW) {
    if (do_bias) {        // fold the row groups in a fixed order
      float *red = (float *)lds;
      red[tid] = bsum;
      __syncthreads();
      if (tid < BM && m0 + tid < p.M) {
        float total = 0.0f;
#pragma unroll
        for (int g = 0; g < BGROUPS; ++g) total += red[g * BM + tid];
        GPP_G float *out = (GPP_G float *)p.bias + m0 + tid;
        *out = accumulate_dw ? *out + total : total;
      }
      __syncthreads();
    }
  }
  void *Cout = FORM == FORM_DW ? (void *)p.C : result_ptr(p, ext);
  if (Cout == nullptr) return;
  const bool inside = m0 + BM <= p.M && n0 + BN <= p.N;
  if (FORM == FORM_DW || epi_lds_ok(p, Cout, FORM)) {
    float *stage = (float *)lds + wave * epi_lds_floats<TN>();
    if (inside) epilogue_wave_lds<FORM, false, TM, TN, STREAM>(p, Cout, acc, m0 + wi0, n0 + wj0, lane, accumulate_dw, stage);
    else epilogue_wave_lds<FORM, true, TM, TN, STREAM>(p, Cout, acc, m0 + wi0, n0 + wj0, lane, accumulate_dw, stage);
  } else {
    epilogue_wave<FORM, true, TM, TN>(p, Cout, acc, m0 + wi0, n0 + wj0, lane, accumulate_dw);
  }
}

// A group launch covers the same problems for several micro-batches: the records are member 0's, the members are further row blocks
// of every column block (whose weight tile they then share in one L2), and everything of a member that lives in a stash slot
// lies `stride` bytes, its per-call pointers `ext_stride` entries behind the previous member's.
template <int FORM, int WGM, int WGN>
__global__ __launch_bounds__(64 * WGM * WGN, WGM == 4 ? 4 : 3) void k_gemm_ring(const GemmProb *__restrict__ probs, int n, int total_blocks,
                                                                               ExtPtrs ext, MemberGroup group) {
  typedef RingCfg<FORM, WGM, WGN, 1, 1, 3, GB_BK> C;
  __shared__ __attribute__((aligned(16))) uint16_t lds[C::ELEMS];
  const int bid = big_spread(total_blocks);
  int lo = 0, hi = n - 1;         // (every record's workgroup range is `members` times the one in its table)
  while (lo < hi) {
    const int mid = (lo + hi + 1) >> 1;
    if (probs[mid].blk_begin * group.members <= bid) lo = mid;
    else hi = mid - 1;
  }
  GemmProb p = probs[lo];
  const int tile = bid - p.blk_begin * group.members, tiles_m = cdiv(p.M, C::BM), row_blocks = tiles_m * group.members;
  int mt = tile % row_blocks;
  if (group.members > 1) {
    const int member = mt / tiles_m;
    mt -= member * tiles_m;
    const int64_t off = (int64_t)member * group.stride;
    p.A = (const GPP_G char *)p.A + off;
    if (p.C) p.C = (GPP_G char *)p.C + off;
    if (p.aux) p.aux = (GPP_G char *)p.aux + off;
    if (p.res) p.res = (const GPP_G char *)p.res + off;
    if (p.c_ext > 0) p.c_ext += member * group.ext_stride;
  }
  ring_body<FORM, WGM, WGN, 1, 1, 3, GB_BK>(p, mt * C::BM, (tile / row_blocks) * C::BN, lds, 0, ext, SlotGroup());
}

// (ADD, gradients are added to, at compile time: the other epilogue is not in the kernel)
template <int WGM, int WGN, int TM, int TN, int BK, int OCC, bool STREAM, bool ADD>
__global__ __launch_bounds__(64 * WGM * WGN, OCC) void k_gemm_ring_dw(const GemmProb *__restrict__ probs, int n, int total_blocks,
                                                                     SlotGroup grp) {
  typedef RingCfg<FORM_DW, WGM, WGN, TM, TN, 3, BK> C;
  __shared__ __attribute__((aligned(16))) uint16_t lds[C::ELEMS];
  const BigTile t = big_locate<C::BM, C::BN, (C::BM == 256 ? 4 : 8)>(probs, n, total_blocks);
  const GemmProb p = probs[t.pi];
  ExtPtrs none;
  ring_body<FORM_DW, WGM, WGN, TM, TN, 3, BK, STREAM>(p, t.m0, t.n0, lds, ADD ? 1 : 0, none, grp);
}

// ---- host side -------------------------------------------------------------------------
// (k-steps that stick out of the matrices, and the ones copied beyond the end, keep their 32-bit offsets)
bool gemm_ring_supported(const GemmProb &p) {
  if (!gemm_mfma_supported(p)) return false;
  const int64_t a_rows = p.form == FORM_DW ? p.K : p.M, b_rows = p.form == FORM_FWD ? p.N : p.K;
  return (a_rows + 512) * p.lda * 2 < 0xffffff00ll && (b_rows + 512) * p.ldb * 2 < 0xffffff00ll;
}
int gemm_ring_blocks(int tile_rows, int M, int N) { return cdiv(M, tile_rows) * cdiv(N, 64); }
void launch_gemm_ring(const GemmProb *probs, int n, int total_blocks, int form, int tile_rows, const ExtPtrs &ext, hipStream_t s,
                      const MemberGroup &group) {
  total_blocks *= group.members;
  if (total_blocks <= 0) return;
  const dim3 g(total_blocks), b(tile_rows == 128 ? 512 : 256);
  if (form == FORM_FWD) {
    if (tile_rows == 128) hipLaunchKernelGGL((k_gemm_ring<FORM_FWD, 4, 2>), g, b, 0, s, probs, n, total_blocks, ext, group);
    else hipLaunchKernelGGL((k_gemm_ring<FORM_FWD, 2, 2>), g, b, 0, s, probs, n, total_blocks, ext, group);
  } else {
    if (tile_rows == 128) hipLaunchKernelGGL((k_gemm_ring<FORM_DX, 4, 2>), g, b, 0, s, probs, n, total_blocks, ext, group);
    else hipLaunchKernelGGL((k_gemm_ring<FORM_DX, 2, 2>), g, b, 0, s, probs, n, total_blocks, ext, group);
  }
}
template <bool STREAM, bool ADD>
static void launch_ring_dw(const GemmProb *probs, int n, int blocks, int tile_rows, const SlotGroup &grp, hipStream_t s) {
  const dim3 g(blocks), b4(256), b8(512);
  if (tile_rows == 256) hipLaunchKernelGGL((k_gemm_ring_dw<2, 2, 4, 2, 32, 2, STREAM, ADD>), g, b4, 0, s, probs, n, blocks, grp);
  else if (tile_rows == 128) hipLaunchKernelGGL((k_gemm_ring_dw<4, 2, 1, 1, 64, 4, STREAM, ADD>), g, b8, 0, s, probs, n, blocks, grp);
  else hipLaunchKernelGGL((k_gemm_ring_dw<2, 2, 1, 1, 64, 3, STREAM, ADD>), g, b4, 0, s, probs, n, blocks, grp);
}
void launch_gemm_ring_dw(const GemmProb *probs, int n, int total_blocks, int accumulate_dw, int tile_rows, bool stream,
                         const SlotGroup &grp, hipStream_t s) {
  if (total_blocks <= 0 || grp.n <= 0) return;
  if (accumulate_dw) launch_ring_dw<false, true>(probs, n, total_blocks, tile_rows, grp, s);
  else if (stream) launch_ring_dw<true, false>(probs, n, total_blocks, tile_rows, grp, s);
  else launch_ring_dw<false, false>(probs, n, total_blocks, tile_rows, grp, s);
}

}  // namespace gpp
