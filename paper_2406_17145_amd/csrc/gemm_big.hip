// Branch-grouped bf16 GEMM for problems with many rows AND many columns (the transformer and MLP
// stacks at full micro-batch), on v_mfma_f32_32x32x16_bf16 with fp32 accumulation.  Two kernels:
//
// k_gemm_big   eight waves (512 threads) share a 256 x 256 or 128 x 256 output tile as a 2 x 4 grid
//              of wave tiles of 128 x 64 (64 x 64) elements.  Per 16-wide contraction chunk a wave reads
//              6 KB (4 KB) of operand fragments from LDS for 8 (4) MFMAs.  One workgroup per compute
//              unit (the double-buffered tiles fill the LDS), so prologue and epilogue of a tile are
//              exposed: best when the launch has a whole number of tiles per compute unit.
// k_gemm_mid   four waves (256 threads), 128 x 128 tile, ONE LDS buffer (37 KB) and a register
//              budget of three waves per SIMD, so three workgroups share a compute unit and one
//              workgroup's loads, barriers and epilogue hide behind the others' MFMAs.  Best when the
//              large tiles would leave compute units idle (few tiles) or quantise badly.
//
// A k-step is 64 contraction elements, so a k-contiguous operand row contributes one whole 128-byte
// cache line per step.  Operands come from memory through buffer loads (out-of-range rows read as
// zero without a branch; a chunk beyond the contraction length is steered out of range).  Two kinds of loop:
// staged (operands wait in registers and are stored to padded LDS tiles) and direct (copied straight into
// swizzled LDS tiles, with the LDS reads software-pipelined under the MFMAs).  The three forms and the two
// LDS layouts (k-contiguous rows read with b128, contraction-major rows read with the transposing read) are
// those of the smaller tile kernel.
#include <algorithm>

#include "gemm_direct.h"

namespace gpp {

constexpr int GB_KST = GB_BK + 8;   // LDS row stride of k-contiguous tiles: 144-byte rows, conflict-free b128 reads

// tile geometry: WGM x WGN waves, each WTM x WTN MFMA tiles of 32 x 32; LDS buffers (1 or 2)
// DIRECT: the operand tiles go from memory straight into LDS (buffer loads with the LDS destination,
// no staging registers), unpadded and XOR-swizzled instead of padded (see the direct loaders below).
template <int FORM, int WGM, int WGN, int WTM, int WTN, int BUFS, bool DIRECT = false>
struct BigCfg {
  static constexpr int NW = WGM * WGN, THREADS = 64 * NW;
  static constexpr int BM = 32 * WTM * WGM, BN = 32 * WTN * WGN;
  static constexpr bool A_TR = FORM == FORM_DW, B_TR = FORM != FORM_FWD;
  static constexpr int A_ELEMS = DIRECT ? GB_BK * BM : (A_TR ? GB_BK * (BM + PAD_TR) : BM * GB_KST);
  static constexpr int B_ELEMS = DIRECT ? GB_BK * BN : (B_TR ? GB_BK * (BN + PAD_TR) : BN * GB_KST);
  static constexpr int LDS_ELEMS = BUFS * (A_ELEMS + B_ELEMS);
  static_assert(LDS_ELEMS * 2 <= 160 * 1024, "tile does not fit the LDS");
};

// one k-step of one operand in registers: EXT rows/columns of the tile, 16-byte chunks, THREADS threads
template <int EXT, int THREADS>
struct BigRegs {
  static constexpr int PER_THREAD = EXT * GB_BK / 8 / THREADS;
  u32x4 v[PER_THREAD];
};

// k-contiguous operand: tile rows [r0, r0 + EXT) x k [k0, k0 + 64); eight lanes read one 128-byte row
// segment.  Rows beyond the buffer read zero, chunks at k >= k_lim are steered out of range (k_lim
// is a multiple of 8).
template <int EXT, int THREADS>
__device__ __forceinline__ void big_fetch_kmajor(BigRegs<EXT, THREADS> &t, __amdgpu_buffer_rsrc_t rs, int64_t ld, int r0, int k0,
                                                 int k_lim, int tid) {
#pragma unroll
  for (int q = 0; q < BigRegs<EXT, THREADS>::PER_THREAD; ++q) {
    const int row = r0 + (tid >> 3) + (THREADS / 8) * q, k = k0 + (tid & 7) * 8;
    // branch-free (a branch here makes the compiler wait for earlier loads between the loads)
    const uint32_t oob = (uint32_t)-(int32_t)(k >= k_lim) & OOB_OFFSET;
    const uint32_t off = (uint32_t)(((int64_t)row * ld + k) * 2) | oob;
    t.v[q] = __builtin_amdgcn_raw_buffer_load_b128(rs, off, 0, 0);
  }
}
template <int EXT, int THREADS>
__device__ __forceinline__ void big_store_kmajor(const BigRegs<EXT, THREADS> &t, uint16_t *lds, int tid) {
#pragma unroll
  for (int q = 0; q < BigRegs<EXT, THREADS>::PER_THREAD; ++q)
    *(u32x4 *)(lds + ((tid >> 3) + (THREADS / 8) * q) * GB_KST + (tid & 7) * 8) = t.v[q];
}
// contraction-major operand: rows k [k0, k0 + 64) x columns [c0, c0 + EXT); rows beyond the buffer
// (k >= contraction length) read zero; columns beyond the matrix only feed outputs that are never stored
template <int EXT, int THREADS>
__device__ __forceinline__ void big_fetch_tr(BigRegs<EXT, THREADS> &t, __amdgpu_buffer_rsrc_t rs, int64_t ld, int k0, int c0,
                                             int tid) {
  constexpr int CPR = EXT / 8, RPP = THREADS / CPR;   // chunks per row, rows per pass
#pragma unroll
  for (int q = 0; q < BigRegs<EXT, THREADS>::PER_THREAD; ++q) {
    const int row = k0 + tid / CPR + RPP * q, col = c0 + (tid % CPR) * 8;
    t.v[q] = __builtin_amdgcn_raw_buffer_load_b128(rs, (uint32_t)(((int64_t)row * ld + col) * 2), 0, 0);
  }
}
template <int EXT, int THREADS>
__device__ __forceinline__ void big_store_tr(const BigRegs<EXT, THREADS> &t, uint16_t *lds, int tid) {
  constexpr int CPR = EXT / 8, RPP = THREADS / CPR;
#pragma unroll
  for (int q = 0; q < BigRegs<EXT, THREADS>::PER_THREAD; ++q)
    *(u32x4 *)(lds + (tid / CPR + RPP * q) * (EXT + PAD_TR) + (tid % CPR) * 8) = t.v[q];
}

// LDS -> MFMA operand.  k-contiguous tile [rows][64 + 8]: lane l takes row (l % 32), 8 k-values at 8 * (l / 32)
__device__ __forceinline__ bf16x8 big_frag_kmajor(const uint16_t *lds, int row0, int k0) {
  const int l = threadIdx.x & 63;
  return *(const bf16x8 *)(lds + (row0 + (l & 31)) * GB_KST + k0 + 8 * (l >> 5));
}

// k-loop + bias gradient + epilogue of one output tile.  PIPE: operands copied straight into BUFS LDS buffers (forward and
// backward-data; whole chunks of k-contiguous rows).  Otherwise staged through registers: one LDS buffer, the next k-step waits
// in registers while the current one is multiplied (two barriers per step; other workgroups on the compute unit fill the gaps).
//
// GROUP (backward-weight only): the contraction runs over the rows of SEVERAL stash slots, one after
// the other -- the weight gradient of a group of backward passes in one pass over the accumulator.
// Both operands live in the slots at the same offsets: slot g of the group is `grp.stride` bytes times
// its slot number behind slot 0, whose addresses the record holds.
//
// STREAM (backward-weight): stored gradients go past the caches, see epilogue_wave_lds.
// PARTIAL (forward): the record covers a slice of a contraction; its result is that slice's sum, stored as plain fp32.
template <int FORM, int WGM, int WGN, int WTM, int WTN, int BUFS, bool GROUP = false, int PIPE = 0, bool PARTIAL = false, bool STREAM = false>
__device__ __forceinline__ void big_tile_body(const GemmProb &p, int m0, int n0, uint16_t *lds, int accumulate_dw,
                                              const ExtPtrs &ext, const SlotGroup grp = SlotGroup(), int total_blocks = 1 << 30) {
  static_assert(!GROUP || FORM == FORM_DW, "only the weight gradient contracts over a group of slots");
  constexpr bool DIRECT = PIPE != 0;     // operands copied straight into LDS, software-pipelined loop 1 or 2 (below)
  static_assert(!DIRECT || BUFS >= 2, "direct loads fill the other LDS buffers while one is multiplied");
  typedef BigCfg<FORM, WGM, WGN, WTM, WTN, BUFS, DIRECT> C;
  constexpr int BM = C::BM, BN = C::BN, THREADS = C::THREADS;
  constexpr bool A_TR = C::A_TR, B_TR = C::B_TR;
  static_assert(DIRECT || BUFS == 1, "the staged path has one LDS buffer");
  uint16_t *lds_a = lds, *lds_b = lds + C::A_ELEMS;      // staged path
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = DIRECT ? __builtin_amdgcn_readfirstlane(tid >> 6) : tid >> 6;      // (copy destinations are scalar)
  const int wi0 = (wave / WGN) * (32 * WTM), wj0 = (wave % WGN) * (32 * WTN);

  // operand buffers: rows beyond the matrix read as zero
  //   FWD: A = X [M x K],  B = W [N x K]      DX: A = dZ [M x K],  B = W [K x N]
  //   DW:  A = dZ [K x M], B = X [K x N]      (K = contraction length in every form)
  const __amdgpu_buffer_rsrc_t rs_a = matrix_rsrc(p.A, A_TR ? p.K : p.M, p.lda, A_TR ? p.M : p.K);
  const __amdgpu_buffer_rsrc_t rs_b = matrix_rsrc(p.B, B_TR ? p.K : p.N, p.ldb, B_TR ? p.N : p.K);
  rsrc4 ra4 = matrix_rsrc4(p.A, A_TR ? p.K : p.M, p.lda, A_TR ? p.M : p.K);           // (the same for the copies)
  rsrc4 rb4 = matrix_rsrc4(p.B, B_TR ? p.K : p.N, p.ldb, B_TR ? p.N : p.K);
  if (DIRECT) settle(ra4, rb4);

  f32x16 acc[WTM][WTN];
#pragma unroll
  for (int i = 0; i < WTM; ++i)
#pragma unroll
    for (int j = 0; j < WTN; ++j)
#pragma unroll
      for (int r = 0; r < 16; ++r) acc[i][j][r] = 0.0f;

  typedef BigRegs<BM, THREADS> RegsA;
  typedef BigRegs<BN, THREADS> RegsB;
  RegsA ra;       // unused (and removed by the compiler) with direct loads
  RegsB rb;
  const int nk_slot = cdiv(p.K, GB_BK);              // k-steps of one slot (of the whole contraction without a group)
  const int nk = GROUP ? nk_slot * grp.n : nk_slot;
  // k-step `kt` of the tile: without a group, contraction elements [64 kt, 64 kt + 64)
  auto fetch = [&](RegsA &xa, RegsB &xb, int kt) {
    if (GROUP) {
      const int g = kt / nk_slot, k0 = (kt - g * nk_slot) * GB_BK;    // wave-uniform
      int slot = grp.first + g;
      slot = slot >= grp.total ? slot - grp.total : slot;
      const int64_t off = (int64_t)slot * grp.stride;
      const __amdgpu_buffer_rsrc_t ga = matrix_rsrc((const char *)p.A + off, p.K, p.lda, p.M);
      const __amdgpu_buffer_rsrc_t gb = matrix_rsrc((const char *)p.B + off, p.K, p.ldb, p.N);
      big_fetch_tr<BM, THREADS>(xa, ga, p.lda, k0, m0, tid);
      big_fetch_tr<BN, THREADS>(xb, gb, p.ldb, k0, n0, tid);
      return;
    }
    const int k0 = kt * GB_BK;
    if (A_TR) big_fetch_tr<BM, THREADS>(xa, rs_a, p.lda, k0, m0, tid);
    else      big_fetch_kmajor<BM, THREADS>(xa, rs_a, p.lda, m0, k0, p.K, tid);
    if (B_TR) big_fetch_tr<BN, THREADS>(xb, rs_b, p.ldb, k0, n0, tid);
    else      big_fetch_kmajor<BN, THREADS>(xb, rs_b, p.ldb, n0, k0, p.K, tid);
  };
  // LDS buffers of the direct path as offsets from the array itself: a pointer picked out of a small array
  // of pointers loses its address space, and the operand reads then turn into generic (flat) loads
  auto da = [&](int b) { return lds + b * C::A_ELEMS; };
  auto db = [&](int b) { return lds + BUFS * C::A_ELEMS + b * C::B_ELEMS; };
  const uint32_t lds0 = lds_address(lds);
  auto to_a = [&](int b) { return lds0 + b * C::A_ELEMS * 2; };                       // copy destinations
  auto to_b = [&](int b) { return lds0 + (BUFS * C::A_ELEMS + b * C::B_ELEMS) * 2; };
  // the same k-step straight into LDS buffer `buf` (a k-step beyond the contraction copies zeros: its rows or
  // chunks lie outside the buffer range)
  auto fetch_direct = [&](int kt, int buf) {
    const int k0 = kt * GB_BK;
    if (A_TR) direct_tr<BM, C::NW>(ra4, p.lda, k0, m0, to_a(buf), wave, lane);
    else      direct_kmajor<BM, C::NW>(ra4, p.lda, m0, k0, p.K, to_a(buf), wave, lane);
    if (B_TR) direct_tr<BN, C::NW>(rb4, p.ldb, k0, n0, to_b(buf), wave, lane);
    else      direct_kmajor<BN, C::NW>(rb4, p.ldb, n0, k0, p.K, to_b(buf), wave, lane);
  };
  auto to_lds = [&](const RegsA &xa, const RegsB &xb) {
    if (A_TR) big_store_tr<BM, THREADS>(xa, lds_a, tid);
    else      big_store_kmajor<BM, THREADS>(xa, lds_a, tid);
    if (B_TR) big_store_tr<BN, THREADS>(xb, lds_b, tid);
    else      big_store_kmajor<BN, THREADS>(xb, lds_b, tid);
  };
  auto multiply = [&]() {       // staged loop
#pragma unroll
    for (int kc = 0; kc < GB_BK; kc += 16) {
      bf16x8 a[WTM], b[WTN];
#pragma unroll
      for (int i = 0; i < WTM; ++i) a[i] = A_TR ? frag_tr<BM>(lds_a, wi0 + 32 * i, kc) : big_frag_kmajor(lds_a, wi0 + 32 * i, kc);
#pragma unroll
      for (int j = 0; j < WTN; ++j) b[j] = B_TR ? frag_tr<BN>(lds_b, wj0 + 32 * j, kc) : big_frag_kmajor(lds_b, wj0 + 32 * j, kc);
#pragma unroll
      for (int i = 0; i < WTM; ++i)
#pragma unroll
        for (int j = 0; j < WTN; ++j) acc[i][j] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(a[i], b[j], acc[i][j], 0, 0, 0);
    }
  };

  // backward-weight tiles of the first column block also sum the rows of dZ^T they stream: the bias
  // gradient db[n] = sum_m dZ[m,n] comes out of the same launch
  constexpr int BGROUPS = THREADS / BM, BROWS = GB_BK / BGROUPS;
  const bool do_bias = FORM == FORM_DW && p.bias != nullptr && n0 == 0;
  float bsum = 0.0f;
  auto bias_rows = [&]() {
    if (FORM == FORM_DW && do_bias) {
      const uint16_t *la = lds_a + (tid / BM) * BROWS * (BM + PAD_TR) + (tid % BM);
#pragma unroll
      for (int rr = 0; rr < BROWS; ++rr) bsum += bf16_bits_to_f32(la[rr * (BM + PAD_TR)]);
    }
  };
  static_assert(!DIRECT || (FORM != FORM_DW && !GROUP), "backward-weight stages its operands through registers");

  if constexpr (PIPE == 1) {
    // Software-pipelined form: the operand fragments of 16-wide chunk c + 1 are read from LDS while the MFMAs
    // of chunk c run (two register sets), also across the k-step boundary.  One barrier per k-step, in front of
    // its LAST chunk: by then every wave has all fragments of the k-step in registers, so the buffer is free
    // and is refilled at once with k-step kt + BUFS; behind the barrier the first fragments of k-step kt + 1
    // (landed: at most BUFS - 2 later k-steps are outstanding) are read under the last chunk's MFMAs.
    constexpr int LPF = (A_TR ? GB_BK * (BM / 8) / 64 / C::NW : BM / C::NW / 8) + (B_TR ? GB_BK * (BN / 8) / 64 / C::NW : BN / C::NW / 8);
    bf16x8 fa[2][WTM], fb[2][WTN];
    // read in the order of first use: the MFMAs run a-major, so the first of them needs every b and a[0]
    auto frags = [&](int set, int buf, int kc) {
#pragma unroll
      for (int j = 0; j < WTN; ++j)
        fb[set][j] = B_TR ? direct_frag_tr<BN>(db(buf), wj0 + 32 * j, kc) : direct_frag_kmajor(db(buf), wj0 + 32 * j, kc);
#pragma unroll
      for (int i = 0; i < WTM; ++i)
        fa[set][i] = A_TR ? direct_frag_tr<BM>(da(buf), wi0 + 32 * i, kc) : direct_frag_kmajor(da(buf), wi0 + 32 * i, kc);
    };
    auto mfmas = [&](int set) {
#pragma unroll
      for (int i = 0; i < WTM; ++i)
#pragma unroll
        for (int j = 0; j < WTN; ++j) acc[i][j] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(fa[set][i], fb[set][j], acc[i][j], 0, 0, 0);
    };
    constexpr int READS = (A_TR ? 2 : 1) * WTM + (B_TR ? 2 : 1) * WTN, MFMAS = WTM * WTN;
    static_assert((BUFS - 1) * LPF < 64, "vmcnt is a 6-bit counter");
    auto interleave = [&]() { big_mix<MFMAS, READS>(); };
    // No branch inside the loop (a branch would end the scheduling region and the interleaving with it): k-steps
    // beyond the contraction are copied like the others -- their rows lie outside the operand's buffer range and
    // read zero -- into buffers nobody multiplies any more, and the fragments read for a k-step that does not
    // exist are dropped.  The number of outstanding copies is then the same in every iteration.
#pragma unroll
    for (int u = 0; u < BUFS; ++u) fetch_direct(u, u);
    copies_landed_barrier<(BUFS - 1) * LPF>();
    frags(0, 0, 0);
    int cur = 0;
    for (int kt = 0; kt < nk; ++kt) {
      const int nxt = cur + 1 == BUFS ? 0 : cur + 1;
      frags(1, cur, 16); mfmas(0); interleave();
      frags(0, cur, 32); mfmas(1); interleave();
      frags(1, cur, 48); mfmas(0); interleave();
      copies_landed_barrier<(BUFS - 2) * LPF>();
      fetch_direct(kt + BUFS, cur);
      frags(0, nxt, 0); mfmas(1); interleave();
      cur = nxt;
    }
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");   // the copies of the k-steps beyond the end
    __syncthreads();      // the epilogue reuses the operand LDS
  } else if constexpr (PIPE == 2) {
    // As above, and the copies of a k-step are issued in TWO batches so that the copy path never runs empty (with
    // one batch per k-step and two buffers, a batch can only be issued when the batch before it has landed: one
    // memory round trip per k-step in which nothing moves).  A wave multiplies the TOP half of its rows for all
    // four 16-wide chunks first (keeping the b fragments of the four chunks), then the BOTTOM half: after the
    // first phase the b tile and the top halves of the a tile are free and are refilled with k-step kt + 2 (batch
    // 1) while the second phase runs; after the second phase the bottom halves follow (batch 2).  Every batch has
    // one and a half k-steps to land, and two batches are in flight at any time.  Each accumulator still adds
    // its chunks in the order 0..3, so the result is the same as in the other loops, bit by bit.
    static_assert(!A_TR && BUFS == 2 && WTM % 2 == 0, "rows of a k-contiguous A split into halves");
    constexpr int HM = WTM / 2, RB = 16 * WTM;                    // MFMA row tiles and rows of a half of a wave's rows
    constexpr int A_HALF = BM / 2 / 8 / C::NW;                    // copy instructions per wave and half of the a tile
    static_assert(A_HALF * C::NW * 8 * 2 == BM, "whole copy instructions");
    constexpr int B_ALL = B_TR ? GB_BK * (BN / 8) / 64 / C::NW : BN / C::NW / 8;
    constexpr int N1 = A_HALF + B_ALL, N2 = A_HALF;
    static_assert(2 * (N1 + N2) < 64, "vmcnt is a 6-bit counter");
    auto copy_a = [&](int kt, int buf, int h) {                   // rows [h RB, h RB + RB) of every wave row block
      const int k0 = kt * GB_BK;
#pragma unroll
      for (int q = 0; q < A_HALF; ++q) {
        const int idx = q * C::NW + wave, wr = idx / (RB / 8), sub = idx % (RB / 8);
        const int base = wr * 32 * WTM + h * RB + sub * 8, row = base + (lane >> 3);
        const int k = k0 + (((lane & 7) ^ ((row >> 1) & 7)) << 3);
        const uint32_t oob = (uint32_t)-(int32_t)(k >= p.K) & OOB_OFFSET;
        lds_copy16(ra4, to_a(buf) + base * GB_BK * 2, (uint32_t)(((int64_t)(m0 + row) * p.lda + k) * 2) | oob);
      }
    };
    auto copy_b = [&](int kt, int buf) {
      if (B_TR) direct_tr<BN, C::NW>(rb4, p.ldb, kt * GB_BK, n0, to_b(buf), wave, lane);
      else direct_kmajor<BN, C::NW>(rb4, p.ldb, n0, kt * GB_BK, p.K, to_b(buf), wave, lane);
    };
    bf16x8 fa[2][HM], fb[4][WTN];
    auto read_b = [&](int buf, int c) {
#pragma unroll
      for (int j = 0; j < WTN; ++j)
        fb[c][j] = B_TR ? direct_frag_tr<BN>(db(buf), wj0 + 32 * j, 16 * c) : direct_frag_kmajor(db(buf), wj0 + 32 * j, 16 * c);
    };
    auto read_a = [&](int set, int buf, int h, int c) {
#pragma unroll
      for (int i = 0; i < HM; ++i) fa[set][i] = direct_frag_kmajor(da(buf), wi0 + 32 * (h * HM + i), 16 * c);
    };
    auto mf = [&](int set, int h, int c) {
#pragma unroll
      for (int i = 0; i < HM; ++i)
#pragma unroll
        for (int j = 0; j < WTN; ++j)
          acc[h * HM + i][j] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(fa[set][i], fb[c][j], acc[h * HM + i][j], 0, 0, 0);
    };
    constexpr int MF = HM * WTN, R1 = (B_TR ? 2 : 1) * WTN + HM, R2 = HM;
    copy_a(0, 0, 0); copy_b(0, 0); copy_a(0, 0, 1);
    copy_a(1, 1, 0); copy_b(1, 1); copy_a(1, 1, 1);
    copies_landed_barrier<N2 + N1 + N2>();
    read_b(0, 0); read_a(0, 0, 0, 0);
    for (int kt = 0; kt < nk; ++kt) {
      const int cur = kt & 1, nxt = cur ^ 1;
      read_b(cur, 1); read_a(1, cur, 0, 1); mf(0, 0, 0); big_mix<MF, R1>();
      read_b(cur, 2); read_a(0, cur, 0, 2); mf(1, 0, 1); big_mix<MF, R1>();
      read_b(cur, 3); read_a(1, cur, 0, 3); mf(0, 0, 2); big_mix<MF, R1>();
      copies_landed_barrier<N1 + N2>();        // the bottom halves of this k-step have landed; top halves and b are free
      copy_a(kt + 2, cur, 0); copy_b(kt + 2, cur);
      read_a(0, cur, 1, 0); mf(1, 0, 3);
      big_mix<MF, R2>();
      read_a(1, cur, 1, 1); mf(0, 1, 0); big_mix<MF, R2>();
      read_a(0, cur, 1, 2); mf(1, 1, 1); big_mix<MF, R2>();
      read_a(1, cur, 1, 3); mf(0, 1, 2); big_mix<MF, R2>();
      copies_landed_barrier<N1 + N2>();        // top halves and b of the next k-step have landed; bottom halves are free
      copy_a(kt + 2, cur, 1);
      read_b(nxt, 0); read_a(0, nxt, 0, 0); mf(1, 1, 3);
      big_mix<MF, R1>();
    }
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");   // the copies of the k-steps beyond the end
    __syncthreads();      // the epilogue reuses the operand LDS
  } else {
    fetch(ra, rb, 0);
    const bool ragged = FORM != FORM_DW && (p.K & 7) != 0;     // the contraction ends inside a chunk of k-contiguous rows
    for (int kt = 0; kt < nk; ++kt) {
      if (ragged && kt + 1 == nk) {                            // clear what lies beyond it (row padding)
        const int k = kt * GB_BK + (tid & 7) * 8;
#pragma unroll
        for (int q = 0; q < RegsA::PER_THREAD; ++q) ra.v[q] = chunk_clear_tail(ra.v[q], k, p.K);
        if (!B_TR) {
#pragma unroll
          for (int q = 0; q < RegsB::PER_THREAD; ++q) rb.v[q] = chunk_clear_tail(rb.v[q], k, p.K);
        }
      }
      to_lds(ra, rb);
      __syncthreads();
      if (kt + 1 < nk) fetch(ra, rb, kt + 1);
      multiply();
      bias_rows();
      __syncthreads();
    }
  }

  if (FORM == FORM_DW && do_bias) {   // fold the row groups in a fixed order (the k-loop ended with a barrier)
    float *red = (float *)lds;
    red[tid] = bsum;
    __syncthreads();
    if (tid < BM && m0 + tid < p.M) {
      float total = 0.0f;
#pragma unroll
      for (int g = 0; g < BGROUPS; ++g) total += red[g * BM + tid];
      GPP_G float *db = (GPP_G float *)p.bias + m0 + tid;
      *db = accumulate_dw ? *db + total : total;
    }
  }

  void *Cout = FORM == FORM_DW ? p.C : result_ptr(p, ext);
  if (Cout == nullptr) return;
  // ---- epilogue.  Where all rows are 16-byte aligned it goes through LDS and touches memory in whole 16-byte
  // pieces of rows (each wave has a private block; the operand tiles are dead: the k-loop and the bias sums ended
  // with a barrier); other results (fp32 outputs among them) keep the accumulator layout, and so do weight-gradient
  // tiles that stick out of their matrix where nothing is read and the launch is small: their predicated stores wait for
  // nothing, while the row-wise ones each wait for their LDS read (grouped gradients, backward pass of [425 x 85] 17.8 against
  // 19.4 us, 4 x [299 x 26] over 466 rows 39.0 against 41.4; added to, the row-wise form is ahead: 19.5 against 24.5, 36.7
  // against 37.3, and so it is in launches of more tiles than run at once, whose stores pile up: 4 x [999 x 1001] 27.2, 26.5).
  static_assert(C::NW * epi_lds_floats<WTN>() * 4 <= C::LDS_ELEMS * 2, "epilogue blocks do not fit the operand LDS");
  const bool inside = m0 + BM <= p.M && n0 + BN <= p.N;
  if constexpr (PARTIAL) {      // fp32 rows as a gradient's (the planner's buffer has whole, aligned rows)
    float *stage = (float *)lds + wave * epi_lds_floats<WTN>();
    if (inside) epilogue_wave_lds<FORM_DW, false, WTM, WTN>(p, Cout, acc, m0 + wi0, n0 + wj0, lane, 0, stage);
    else epilogue_wave_lds<FORM_DW, true, WTM, WTN>(p, Cout, acc, m0 + wi0, n0 + wj0, lane, 0, stage);
    return;
  }
  // (also for a plain bias / cast epilogue: rows in 16-byte pieces beat the accumulator layout's 2-byte pieces
  // sixteen rows apart -- 4 x [2048 x 4096 x 1024] forward 78 -> 75.5 us, a one-k-step launch of the same output
  // 29 -> 26 us.  While the stores were flat instructions, which count on the LDS wait counter as well, it
  // was the other way round: 87 against 95 us)
  if (FORM == FORM_DW ? inside || accumulate_dw || total_blocks > 256 : epi_lds_ok(p, Cout, FORM)) {      // (gradients have aligned rows)
    if (FORM == FORM_DW && do_bias) __syncthreads();   // the bias sums were read from LDS after the last barrier
    float *stage = (float *)lds + wave * epi_lds_floats<WTN>();
    if (inside) epilogue_wave_lds<FORM, false, WTM, WTN, STREAM>(p, Cout, acc, m0 + wi0, n0 + wj0, lane, accumulate_dw, stage);
    else epilogue_wave_lds<FORM, true, WTM, WTN, STREAM>(p, Cout, acc, m0 + wi0, n0 + wj0, lane, accumulate_dw, stage);
  } else {
    epilogue_wave<FORM, true, WTM, WTN>(p, Cout, acc, m0 + wi0, n0 + wj0, lane, accumulate_dw);
  }
}

template <int FORM, int WTM, int WTN, int PIPE, int BUFS>
__global__ __launch_bounds__(512) void k_gemm_big(const GemmProb *__restrict__ probs, int n, int total_blocks,
                                                  ExtPtrs ext) {
  typedef BigCfg<FORM, 2, 4, WTM, WTN, BUFS, true> C;
  __shared__ __attribute__((aligned(16))) uint16_t lds[C::LDS_ELEMS];
  const BigTile t = big_locate<C::BM, C::BN>(probs, n, total_blocks);
  const GemmProb p = probs[t.pi];
  big_tile_body<FORM, 2, 4, WTM, WTN, BUFS, false, PIPE>(p, t.m0, t.n0, lds, 0, ext);
}

// Forward with a long contraction and few output tiles (the layer behind a merge of many branches): `split_k` workgroups
// share an output tile of 128 x 256, each sums a slice of the contraction into its own fp32 matrix, and the launch behind
// this one adds the slices in order and finishes the result.  The workgroups of one slice follow each other, so an XCD
// works on few slices and its L2 sees a tile row of that slice's operands once.  [512 x 4096 x 28672]: 211 us on
// the 64 x 64 blocks, 124 + 12 here; [256 x 4096 x 73472]: 292 and 176 + 10.
__global__ __launch_bounds__(512) void k_gemm_big_split(const GemmProb *__restrict__ probs, int total_blocks) {
  typedef BigCfg<FORM_FWD, 2, 4, 2, 2, 3, true> C;
  __shared__ __attribute__((aligned(16))) uint16_t lds[C::LDS_ELEMS];
  const int w = big_spread(total_blocks);
  GemmProb p = probs[0];
  const int tiles = total_blocks / p.split_k, split = w / tiles, tile = w - split * tiles, tiles_m = cdiv(p.M, C::BM);
  const int slice = cdiv(cdiv(p.K, GB_BK), p.split_k) * GB_BK, k0 = split * slice;     // (every slice holds some of the contraction)
  p.A = (const GPP_G uint16_t *)p.A + k0;
  p.B = (const GPP_G uint16_t *)p.B + k0;
  p.K = min(slice, p.K - k0);
  p.ldc = split_sum_ld(p.N);
  p.C = p.partial + (int64_t)split * p.M * p.ldc;
  ExtPtrs none;
  big_tile_body<FORM_FWD, 2, 4, 2, 2, 3, false, 1, true>(p, (tile % tiles_m) * C::BM, (tile / tiles_m) * C::BN, lds, 0, none);
}
// sum of the slices in order, then what the forward epilogue does; a thread takes four columns of a row
__global__ __launch_bounds__(256) void k_split_sum(const GemmProb *__restrict__ probs) {
  typedef float f32x4 __attribute__((ext_vector_type(4)));
  const GemmProb p = probs[0];
  const int ld = (int)split_sum_ld(p.N), quads = ld / 4;
  const int64_t at = (int64_t)blockIdx.x * 256 + threadIdx.x;
  const int row = (int)(at / quads), col = (int)(at - (int64_t)row * quads) * 4;
  if (row >= p.M || col >= p.N) return;
  const GPP_G float *src = p.partial + (int64_t)row * ld + col;
  const int64_t step = (int64_t)p.M * ld;
  float v[4] = {0.0f, 0.0f, 0.0f, 0.0f}, d[4];
  for (int q = 0; q < p.split_k; q += 4) {
    f32x4 x[4];
#pragma unroll
    for (int u = 0; u < 4; ++u) x[u] = *(const GPP_G f32x4 *)(src + (int64_t)min(q + u, p.split_k - 1) * step);   // (loads without a branch)
#pragma unroll
    for (int u = 0; u < 4; ++u)
#pragma unroll
      for (int e = 0; e < 4; ++e) v[e] += q + u < p.split_k ? x[u][e] : 0.0f;
  }
#pragma unroll
  for (int e = 0; e < 4; ++e) {
    const int c = min(col + e, p.N - 1);
    if (p.bias) v[e] += p.bias[c];
    d[e] = act_stash(v[e], p.act);
    v[e] = act_apply(v[e], p.act);
    if (p.res) v[e] += load_as_f32(p.res, p.res_dtype, (int64_t)row * p.ldres + c);
  }
  auto put = [&](void *dst, int dtype, int64_t ldd, const float (&o)[4]) {
    const int64_t i = (int64_t)row * ldd + col;
    if (dtype == DT_BF16 && col + 4 <= p.N && (ldd & 3) == 0 && ((uintptr_t)dst & 7) == 0) {
      typedef uint32_t u32x2 __attribute__((ext_vector_type(2)));
      *(u32x2 *)((uint16_t *)dst + i) = (u32x2){(uint32_t)f32_to_bf16_bits(o[0]) | ((uint32_t)f32_to_bf16_bits(o[1]) << 16),
                                                (uint32_t)f32_to_bf16_bits(o[2]) | ((uint32_t)f32_to_bf16_bits(o[3]) << 16)};
      return;
    }
#pragma unroll
    for (int e = 0; e < 4; ++e)
      if (col + e < p.N) store_from_f32(dst, dtype, i + e, o[e]);
  };
  if (p.act == ACT_GELU && p.aux) put((void *)p.aux, p.aux_dtype, p.ldaux, d);
  put((void *)p.C, p.c_dtype, p.ldc, v);
}

// 128 x 128 tile, 2 x 2 waves of 64 x 64, one LDS buffer, three waves per SIMD
template <int FORM>
__global__ __launch_bounds__(256, 3) void k_gemm_mid(const GemmProb *__restrict__ probs, int n, int total_blocks,
                                                     int accumulate_dw, ExtPtrs ext) {
  typedef BigCfg<FORM, 2, 2, 2, 2, 1> C;
  __shared__ __attribute__((aligned(16))) uint16_t lds[C::LDS_ELEMS];
  const BigTile t = big_locate<C::BM, C::BN>(probs, n, total_blocks);
  const GemmProb p = probs[t.pi];
  big_tile_body<FORM, 2, 2, 2, 2, 1>(p, t.m0, t.n0, lds, accumulate_dw, ext, SlotGroup(), total_blocks);
}

// backward-weight over a group of stash slots (see big_tile_body).
// Tile order of the grouped weight gradient: bands of eight tile rows.  Its launch holds thousands of 128 x 128 tiles,
// 128 of them in flight per XCD; numbered column by column these are 32 rows x 4 columns of a [4096 x 1024] gradient
// (36 operand panels of 512 KB through a 4 MB L2), in bands 8 x 16 (24 panels).  Measured on the transformer stage's
// launch of all layers: 497-505 -> 483 us (bands of 4: 497, of 16: 487 scaled to the same box).
constexpr int DW_BAND = 8;
// (four workgroups per compute unit: 40 KB of LDS and 128 registers each; with three the transformer stage's launch
// is 6 % slower)
// (ADD, gradients are added to, at compile time: with both epilogues in one kernel three registers are spilled)
template <bool STREAM, bool ADD>
__global__ __launch_bounds__(256, 4) void k_gemm_mid_dw_group(const GemmProb *__restrict__ probs, int n, int total_blocks,
                                                              SlotGroup grp) {
  typedef BigCfg<FORM_DW, 2, 2, 2, 2, 1> C;
  __shared__ __attribute__((aligned(16))) uint16_t lds[C::LDS_ELEMS];
  const BigTile t = big_locate<C::BM, C::BN, DW_BAND>(probs, n, total_blocks);
  const GemmProb p = probs[t.pi];
  ExtPtrs none;
  big_tile_body<FORM_DW, 2, 2, 2, 2, 1, true, 0, false, STREAM>(p, t.m0, t.n0, lds, ADD ? 1 : 0, none, grp, total_blocks);
}

// ---- host side -------------------------------------------------------------------------
// The kernels take a problem when its matrices fit the 32-bit buffer offsets; the eight-wave ones also need whole chunks
// of k-contiguous operands (contraction length a multiple of 8).  Rows and base pointers on 16 bytes are gemm_mfma_supported's
// condition, so the eight-wave forward and backward-data kernels can always copy operands straight into LDS.
// Of an operand whose rows run along the contraction whole k-steps are fetched, and rows beyond
// the matrix read zero by lying beyond its bytes: those of the last k-step must not wrap around to the first rows
bool gemm_big_supported(const GemmProb &p) {
  if (!gemm_mfma_supported(p)) return false;
  const int64_t k_rows = (int64_t)cdiv(p.K, GB_BK) * GB_BK;
  const int64_t a_rows = p.form == FORM_DW ? k_rows : p.M, b_rows = p.form == FORM_FWD ? p.N : k_rows;
  return a_rows * p.lda * 2 < 0xffffff00ll && b_rows * p.ldb * 2 < 0xffffff00ll;
}
// Kernel of a forward / backward-data launch: tiles of 256 x 256 or 128 x 256 (256, 128: eight waves), of 128 x 128 (64: four waves,
// three workgroups per compute unit), of 128 x 64 or 64 x 64 out of a ring of LDS buffers (GEMM_RING + 128, + 64: two and three
// workgroups per compute unit), or the kernel whose waves split the contraction (0).  Whatever takes least by the estimates below,
// which are microseconds fitted to launches with operands from memory: 1 to 7 records of M 64 .. 4096, N 64 .. 4096 and K 64 ..
// 4096, K / 64 k-steps, workgroups as counted in `c`.
//   256 x 256: one workgroup per compute unit, rounds of 256.       4 x [2048 x 4096 x 1024] 87 forward, 84 backward-data
//   128 x 256: the same with half the work in a workgroup.          7 x [256 x 4096 x 4096] forward 81 (256: 104, 64: 92, 0: 151)
//                                                                   the same backward-data 76 (256: 91, 64: 89, 0: 159)
//   128 x 128: 1, 2 or 3 per compute unit; a partial round is partly hidden under the full ones.
//                                                                   2 x [2000 x 2056 x 136] backward-data 16.0 (256: 19.6, ring 18.1)
//   ring: a chain of k-steps and a share of the chip's rate.        4 x [512 x 1000 x 1000] forward 13.6, backward-data 12.5 with
//                                                                   128 x 64 (0: 22.5, 20.5; 64: 25.3, 20.9); 7 x [129 x 1500 x 1000]
//                                                                   forward 14.4 with 64 x 64 (128 x 64: 18.2, 0: 22.4)
//   0:         few tiles and a long contraction, whose chain it cuts to an eighth.     [300 x 1000 x 4096] 15.1 (ring 19.5)
// 384 rows (7 x [384 x 4096 x 4096]): 256 106, 128 135, 64 116, 0 218.
// `whole_chunks`: every contraction length is a multiple of 8; `large_tiles`, `ring`: those kernels are choices.
// Behind a short contraction the estimate of the 256 x 256 tiles is too low (their prologue and epilogue are all that such a
// launch is), so there they are left out unless the launch is whole rounds of them, or in forward from K 768 on at least half
// of its last one.  us with 256 / 64, forward from K 1024 down, backward-data from K 256 down:
//   4 x [9679 x 1000 x K], 608 tiles: K 16 117 / 82, 128 124 / 95, 512 170 / 144, 768 195 / 175, 1024 219 / 208, 1536 the same
//   [3000 x 4096 x K], 192 tiles:     K 512 56 / 50, 768 60 / 52, 1024 66 / 60;     4 x [2048 x 4096 x 512], 512 tiles: 105 / 110
//   4 x [9679 x 4096 x K], 2432 tiles: K 512 481 / 465, 768 430 / 453
//   backward-data, 4 x [9679 x 1000 x K], 608 tiles: K 256 64 / 57, 1000 112 / 127;   4 x [2048 x 4096 x K], 512 tiles: K 64 44 / 41,
//     256 47 / 48, 512 58 / 62.  The 128 x 256 tiles from K 768: 4 x [2048 x 1024 x K], 256 tiles, with 128 / 64: K 256 15.7 / 15.3,
//     512 18.8 / 19.4, 1024 24.0 / 27.5;   4 x [2048 x 4096 x 512], 1024 tiles: 70 / 62
// The estimates are within 20 % of what was measured, so a ring kernel has to be ahead of the large tiles by 8 %, behind ragged
// contractions, which the fit has none of, by 20 %; the few-row kernel is credited 5 %, and 15 % where it has fewer tiles than
// compute units behind at least 30 k-steps (over 1342 launches: 17 % faster than with the large tiles and the few-row kernel
// alone, 1.1 % of them more than 3 % slower).
// Both rules meet in 4 x [512 x 1000] over contractions of 942, 3820, 2048 and 1, operands from memory: few-row 33.1, which it takes, ring 128 x 64
// 36.4, 64 x 64 43.2, 128 x 128 69.3.  Ragged ones of one length on ring 128 x 64, which they take / the next best: 942 16.1 / 17.7,
// 2042 25.2 / 29.0, 3820 41.5 / 48.4;  7 x [512 x 4096 x 2042] stays on 128 x 128: 108 / 121.
int gemm_tile_choice(int form, int max_k, const GemmTileCounts &c, bool ring, bool large_tiles, bool whole_chunks, float *us) {
  constexpr float CUS = 256.0f;
  const float nk = (float)cdiv(max_k, GB_BK);
  const bool fwd = form == FORM_FWD;
  auto rounds = [&](float tiles, auto cost) {          // rounds of one workgroup per compute unit
    const float full = floorf(tiles / CUS), part = tiles / CUS - full;
    return full * cost(1.0f) + (full == 0.0f || part > 0.01f ? cost(part) : 0.0f);
  };
  auto t256 = [&](float fill) { return fwd ? 10.0f + 8.0f * fill + (1.35f + 0.2f * fill) * nk : 9.0f + 8.0f * fill + (0.85f + 0.65f * fill) * nk; };
  auto t128 = [&](float fill) { return fwd ? 9.8f + 4.2f * fill + (0.62f + 0.31f * fill) * nk : 6.2f + 5.3f * fill + (0.67f + 0.21f * fill) * nk; };
  auto mid = [&](float tiles) {
    auto level = [&](float per_cu) {                   // workgroups that share a compute unit
      const float fixed = per_cu <= 1.0f ? 9.0f : (per_cu <= 2.0f ? 13.5f : 16.0f);
      const float step = per_cu <= 1.0f ? 1.06f : (per_cu <= 2.0f ? 1.13f : 1.55f);
      return fixed - (fwd ? 0.0f : 3.0f) + step * nk;
    };
    const float full = floorf(tiles / (3.0f * CUS)), rest = tiles / CUS - 3.0f * full;
    if (full == 0.0f) return level(rest);
    return full * level(3.0f) + (rest > 0.01f ? 0.6f * level(rest) : 0.0f);
  };
  // workgroups that share compute units: fixed part and chain of k-steps, what every workgroup adds, and what each beyond one per
  // compute unit adds
  auto shared = [&](float blocks, float a, float ak, float b, float bk, float d, float dk) {
    const float w = blocks / CUS;
    return a + ak * nk + w * (b + bk * nk) + fmaxf(1.0f, w) * (d + dk * nk);
  };
  // The ring's workgroups all run at once up to two (128 x 64) or three (64 x 64) on a compute unit.  In forward the first ones behind that
  // cost as much as half a round of them, which the fit, with no launch there, does not show; a handful of them hides behind the others.
  // n x [250 x 2056 x 520], 66 n workgroups, ring 128 x 64 / large tiles: n 7 17.8 / 19.8, 8 22.4 / 21.4, 9 23.8 / 22.1, 11 25.3 / 22.6;
  // 9 x [512 x 1000 x 512], 576: 21.0 / 19.8;  3 x [590 x 2304 x 576] with GELU in a transformer stage, 540: 1.5 us the other way.  64 x 64:
  // 12 x [130 x 1500 x 1000], 864: 28.0 / 26.5;  4 x [288 x 2688 x 896], 840: 4 us over the 504 of 128 x 64.
  // (Backward-data of the first six: 13.2 / 15.1, 17.0 / 16.8, 17.4 / 17.2, 17.8 / 17.7;  16.4 / 16.4;  19.3 / 23.0)
  auto ring_blocks = [&](float blocks, float per_cu) {
    const float rounds_of = blocks / (per_cu * CUS);
    return fwd && rounds_of > 1.07f && rounds_of < 1.5f ? 1.5f * per_cu * CUS : blocks;
  };
  float best = 1e30f;
  int rows = 64;
  auto take = [&](int r, float t, float handicap) {
    if (t * handicap < best) {
      best = t * handicap;
      rows = r;
    }
  };
  if (large_tiles) take(64, mid(c.t128), 1.0f);
  const float rest256 = c.t256 / CUS - floorf(c.t256 / CUS);
  const bool whole_rounds = c.t256 >= CUS && (rest256 < 0.01f || (fwd && max_k >= 768 && rest256 >= 0.5f));
  if (large_tiles && whole_chunks && (max_k > (fwd ? 1024 : 256) || whole_rounds)) take(256, rounds(c.t256, t256), 1.0f);
  if (large_tiles && whole_chunks && (fwd || max_k >= 768)) take(128, rounds(c.t128x256, t128), 1.0f);
  const float n128x64 = ring_blocks(c.t128x64, 2.0f), n64 = ring_blocks(c.t64, 3.0f);
  const float large = best, r128 = fwd ? shared(n128x64, 2.14f, 0.18f, 1.36f, 0.181f, 2.0f, 0.138f) : shared(n128x64, 2.04f, 0.179f, 1.27f, 0.219f, 1.16f, 0.104f);
  const float r64 = fwd ? shared(n64, 2.51f, 0.153f, 0.64f, 0.122f, 0.95f, 0.092f) : shared(n64, 2.35f, 0.134f, 0.63f, 0.155f, 0.62f, 0.074f);
  if (ring && fminf(r128, r64) < (whole_chunks ? 0.92f : 0.8f) * large) {
    take(GEMM_RING + 128, r128, 1.0f);
    take(GEMM_RING + 64, r64, 1.0f);
  }
  *us = best;
  if (c.few > 0.0f) {
    // (for slices of a contraction, of 64 k-steps and more, which the fit does not reach: the few-row kernel's own line there)
    *us = fminf(*us, 0.9f * (3.0f + fmaxf(1.0f, c.t64 / CUS) * (3.2f + 0.30f * nk)));
    const float t = fwd ? shared(c.few, 1.06f, 0.028f, 2.06f, 0.184f, 3.45f, 0.109f) : shared(c.few, 1.18f, 0.032f, 1.63f, 0.179f, 2.55f, 0.134f);
    // (against the ring alone, for launches that share the GPU with another stream's, the other way round: [4 x 64 x 1000 x 4000] is
    // 15 us on 128 workgroups and 19 on 64 of the ring, but a step of two such streams 190 and 179)
    take(0, t, !large_tiles ? 1.15f : nk >= 30.0f && c.t64 <= CUS ? 0.85f : 0.95f);
  }
  return rows;
}
// Backward-weight: 64 (128 x 128 tiles staged through registers, three or four workgroups per compute unit) or 256 (256 x 128 tiles
// out of LDS buffers filled by copies, two).  The larger tile moves a quarter less through the LDS for a product and keeps its copies
// in flight across k-steps, but has fewer workgroups to hide its prologue and its stores.  us with 64 / 256, gradients stored and
// added to:
//   four [4096 x 4096], rows 256: 61 / 64, 116 / 120     512: 88 / 87, 130 / 137     1024: 136 / 132, 180 / 178
//                       2048: 242 / 222, 288 / 263       4096: 465 / 399, 525 / 439  8192: 1514 / 768, 1554 / 810
//   the sixteen gradients of four transformer layers (768 x 2 tiles), rows 512: 78 / 76, 109 / 107    2048: 196 / 182, 221 / 204
//   four [2048 x 2048] (512 tiles), rows 512: 26 / 23, 42 / 40;   six [1536 x 3000] (864), rows 1024: 70 / 70, 87 / 91
//   four [1000 x 1000] (128 tiles), rows 2048: 38 / 42, 43 / 50
// (a grouped launch mostly stores, a launch per backward pass mostly adds; ragged matrices that leave the larger tiles more than a
// tenth emptier stay)
int gemm_big_dw_tile(bool grouped, int k, int tiles256x128, int tiles128) {
  return k >= (grouped ? 512 : 1024) && tiles256x128 >= 512 && 20 * tiles256x128 <= 11 * tiles128 ? 256 : 64;
}
// The launch that holds the weight gradients of all layers, where 256 x 128 tiles are not for it: 128 x 128 (64), or 128 x 64 or
// 64 x 64 out of a ring of LDS buffers (GEMM_RING + 128, + 64), by estimates fitted to 1298 launches of 1 to 40 gradients of 64 ..
// 4096 rows and columns over 64 .. 4096 rows, stored and added to (48 % faster than 128 x 128 alone, the ring kernels mostly ahead
// below a few hundred tiles: [504 x 256] over 4096 rows 55 us with 64, 26 with 128 x 64, 19 with 64 x 64; 12 x [64 x 256] 72, 30,
// 28; 4 x [2048 x 2048] over 512 rows 32, 43, 43).
int gemm_dw_small_tile(int k, const GemmTileCounts &c) {
  const float nk = (float)cdiv(k, GB_BK);
  auto est = [&](float blocks, float a, float ak, float b, float bk, float d, float dk) {
    const float w = blocks / 256.0f;
    return a + ak * nk + w * (b + bk * nk) + fmaxf(1.0f, w) * (d + dk * nk);
  };
  const float mid = est(c.t128, 3.8f, 0.834f, 4.3f, 0.319f, -0.21f, -0.012f), r128 = est(c.t128x64, 2.5f, 0.172f, 2.34f, 0.136f, 0.67f, 0.187f);
  const float r64 = est(c.t64, 2.46f, 0.189f, 1.36f, 0.129f, 0.17f, 0.073f);
  if (fminf(r128, r64) >= 0.97f * mid) return 64;
  return GEMM_RING + (r64 <= r128 ? 64 : 128);
}
// Slices of a lone forward record's contraction (0: not split): as many workgroups as compute units, slices of at least 16
// k-steps, where one round of them and the pass over the slices (written and read once, 4 TB/s, and a launch) take 15 %
// less than the kernel chosen otherwise, by the estimates above.
int gemm_big_split(int M, int N, int K, int64_t most, float us) {
  const int tiles = cdiv(M, 128) * cdiv(N, 256), nk = cdiv(K, GB_BK);
  int s = (int)std::min<int64_t>(std::min(std::min(16, 256 / tiles), nk / 16), most);
  if (s < 2) return 0;
  s = cdiv(nk, cdiv(nk, s));                            // no slice without k-steps
  const float t = 13.0f + 0.95f * (float)cdiv(nk, s) + 8.0f + (float)M * (float)N * 8.0f * (float)s / 4e6f;
  return s >= 2 && t < 0.85f * us ? s : 0;
}
// (backward-weight: the columns of a tile are always 128)
int gemm_big_dw_tiles(int tile_rows, int M, int N, int *tiles_n) {
  if (tiles_n) *tiles_n = cdiv(N, 128);
  return cdiv(M, tile_rows == 64 ? 128 : tile_rows) * cdiv(N, 128);
}
int gemm_big_tiles_for(int tile_rows, int M, int N, int *tiles_n) {
  const int bn = tile_rows == 64 ? 128 : 256, bm = tile_rows == 64 ? 128 : tile_rows;
  if (tiles_n) *tiles_n = cdiv(N, bn);
  return cdiv(M, bm) * cdiv(N, bn);
}

void launch_gemm_big(const GemmProb *probs, int n, int total_blocks, int accumulate_dw, int form, int tile_rows, const ExtPtrs &ext,
                     hipStream_t s) {
  if (total_blocks <= 0) return;
  const dim3 g(total_blocks), b8(512), b4(256);
  // operands straight into LDS on the eight-wave tiles (4 x [2048 x 4096 x 1024] forward cold: 83 us staged, 78 direct; the eight
  // backward-data launches of a transformer stage of four branches, 1024 rows each: 643 us staged on 128 x 128, 486)
  if (form == FORM_FWD) {
    if (tile_rows == 256) hipLaunchKernelGGL((k_gemm_big<FORM_FWD, 4, 2, 2, 2>), g, b8, 0, s, probs, n, total_blocks, ext);
    else if (tile_rows == 128) hipLaunchKernelGGL((k_gemm_big<FORM_FWD, 2, 2, 1, 3>), g, b8, 0, s, probs, n, total_blocks, ext);
    else hipLaunchKernelGGL((k_gemm_mid<FORM_FWD>), g, b4, 0, s, probs, n, total_blocks, 0, ext);
  } else if (form == FORM_DX) {
    if (tile_rows == 256) hipLaunchKernelGGL((k_gemm_big<FORM_DX, 4, 2, 2, 2>), g, b8, 0, s, probs, n, total_blocks, ext);
    else if (tile_rows == 128) hipLaunchKernelGGL((k_gemm_big<FORM_DX, 2, 2, 1, 3>), g, b8, 0, s, probs, n, total_blocks, ext);
    else hipLaunchKernelGGL((k_gemm_mid<FORM_DX>), g, b4, 0, s, probs, n, total_blocks, 0, ext);
  } else {
    if (tile_rows == 256) launch_gemm_ring_dw(probs, n, total_blocks, accumulate_dw, 256, false, SlotGroup(), s);
    else hipLaunchKernelGGL((k_gemm_mid<FORM_DW>), g, b4, 0, s, probs, n, total_blocks, accumulate_dw, ext);
  }
}

void launch_gemm_split(const GemmProb *probs, int total_blocks, int M, int N, hipStream_t s) {
  if (total_blocks <= 0) return;
  hipLaunchKernelGGL(k_gemm_big_split, dim3(total_blocks), dim3(512), 0, s, probs, total_blocks);
  const int64_t threads = (int64_t)M * (split_sum_ld(N) / 4);
  hipLaunchKernelGGL(k_split_sum, dim3((uint32_t)((threads + 255) / 256)), dim3(256), 0, s, probs);
}

// Gradients of one launch that are stored past the caches: those that a memory-side cache of 256 MB cannot hold until somebody
// reads them, since what it holds instead -- weights, activations -- is read again.  One mini-batch, one group: eight branches with
// 358 MB 241 -> 202 us, 220 MB 204 -> 183, seven towers with 1.9 GB 1594 -> 1481; with 92 MB and less 0 - 1 % slower, and 2 %
// where a second group of the mini-batch adds to them (8 % for that pass alone).  Above the line that second group loses less
// than the first has gained (two groups: 541 -> 492 us, 460 -> 419, 3450 -> 3320).  Where the caller knows that no second group
// follows (a task list with one run of backward passes) every size streams: towers with 78 MB from a graph 243 -> 237 us a
// step, three branches of [244 x 244] 280 -> 268.
bool gemm_dw_group_streams(int64_t gradient_bytes) { return gradient_bytes >= (int64_t)128 << 20; }
void launch_gemm_dw_group(const GemmProb *probs, int n, int total_blocks, int accumulate_dw, int tile_rows, bool stream,
                          const SlotGroup &grp, hipStream_t s) {
  if (total_blocks <= 0 || grp.n <= 0) return;
  const dim3 g(total_blocks), b(256);
  if (tile_rows == 256 || tile_rows > GEMM_RING) {
    launch_gemm_ring_dw(probs, n, total_blocks, accumulate_dw, tile_rows > GEMM_RING ? tile_rows - GEMM_RING : tile_rows, stream, grp, s);
    return;
  }
  if (accumulate_dw) hipLaunchKernelGGL((k_gemm_mid_dw_group<false, true>), g, b, 0, s, probs, n, total_blocks, grp);
  else if (stream) hipLaunchKernelGGL((k_gemm_mid_dw_group<true, false>), g, b, 0, s, probs, n, total_blocks, grp);
  else hipLaunchKernelGGL((k_gemm_mid_dw_group<false, false>), g, b, 0, s, probs, n, total_blocks, grp);
}

}  // namespace gpp
