// Operand tiles copied from memory straight into LDS, for the bf16 GEMM kernels that multiply out of LDS only.
// One copy instruction of a wave fills 1 KB of consecutive LDS (lane l writes 16 bytes at 16 l behind the wave-uniform
// destination), so the layout of a tile in LDS is the order of its 16-byte chunks, and the padding that keeps the operand
// reads free of bank conflicts in the staged loops is replaced by a swizzle: WHICH chunk of memory a lane loads.  The
// copies of later k-steps run while one is multiplied; nothing waits in registers.
#pragma once
#include "gemm_tile_body.h"

namespace gpp {

constexpr int GB_BK = 64;           // contraction elements per k-step

typedef __attribute__((address_space(3))) void lds_void_t;
typedef __attribute__((ext_vector_type(4))) uint32_t rsrc4;   // buffer descriptor as the four scalar registers it is

// A memory instruction may read a scalar register that a vector instruction (the readfirstlanes below) has written five wait states
// later at the earliest.  A tile's two descriptors pass through here behind every such write and before any copy can read them, so
// that no copy has to wait by itself (in each of them the wait cost the passes with ring-buffered GEMMs 0.4 - 1.6 %, here at most 0.3).
// What the compiler could still put in between, a register reloaded from a vector register, tests/test_device_code_cpu.py looks for
// in the built code.
__device__ __forceinline__ void settle(rsrc4 &a, rsrc4 &b) { asm("s_nop 4" : "+s"(a), "+s"(b)); }
// what matrix_rsrc describes: rows beyond the matrix, and chunks steered to OOB_OFFSET, read zero
__device__ __forceinline__ rsrc4 matrix_rsrc4(const void *base, int rows, int64_t ld, int width) {
  const uint64_t a = (uint64_t)base;
  return (rsrc4){(uint32_t)__builtin_amdgcn_readfirstlane((int)(uint32_t)a),
                 (uint32_t)__builtin_amdgcn_readfirstlane((int)((uint32_t)(a >> 32) & 0xffffu)),
                 (uint32_t)__builtin_amdgcn_readfirstlane((int)matrix_bytes(rows, ld, width)), 0x00020000u};
}
// LDS byte address of a pointer into the workgroup's LDS array, in a scalar register
__device__ __forceinline__ uint32_t lds_address(const uint16_t *p) {
  return (uint32_t)__builtin_amdgcn_readfirstlane((int)(uint32_t)(uintptr_t)(lds_void_t *)p);
}
// 16 bytes per lane from byte `off` behind the descriptor's base to LDS byte `dst` + 16 * lane (dst: wave-uniform).
// Written out because the compiler takes the transposing LDS read for a possible reader of ANY copy it knows of and puts
// s_waitcnt vmcnt(0) in front of the first one of a k-step: every kernel whose operand is read that way then waited for the
// copies it had just issued, one memory round trip per k-step whatever the number of LDS buffers (backward-data of
// 4 x [512 x 1000 x 1000] on 128 x 64 tiles 18.9 us with the builtin, 12.7 without that wait).  The instruction has no register
// result; what waits for it is copies_landed_barrier, and the compiler's own counted waits, which do not know of it,
// can only become longer (copies and loads finish in issue order).
// Wait states, which the compiler does not add in front of what it does not know to be a memory instruction: one between the write
// of m0, which holds the destination, and the copy; the five behind a vector write of the descriptor are in settle().
#pragma clang diagnostic push
#pragma clang diagnostic ignored "-Winline-asm"
__device__ __forceinline__ void lds_copy16(rsrc4 rs, uint32_t dst, uint32_t off) {
  asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tbuffer_load_dwordx4 %1, %2, 0 offen lds" ::"s"(dst), "v"(off), "s"(rs) : "m0");
}
#pragma clang diagnostic pop

// The LDS moves 256 bytes per cycle (64 banks of 4 bytes), so what must not collide is:
// k-contiguous operand, tile [EXT][64]: 128-byte rows, two per bank line; a 16-byte operand read serves 16
// lanes per cycle, the same chunk column of 16 consecutive rows.  Chunk c of row r sits at chunk position
// c ^ ((r / 2) % 8): the two rows of a bank line keep their halves, the eight row pairs take eight positions
template <int EXT, int NW>
__device__ __forceinline__ void direct_kmajor(rsrc4 rs, int64_t ld, int r0, int k0, int k_lim, uint32_t tile, int wave, int l) {
  constexpr int ROWS_PER_WAVE = EXT / NW, INSTR = ROWS_PER_WAVE / 8;
  static_assert(EXT % (8 * NW) == 0, "a wave loads whole groups of eight rows");
#pragma unroll
  for (int q = 0; q < INSTR; ++q) {
    const int row = wave * ROWS_PER_WAVE + 8 * q + (l >> 3);
    const int k = k0 + (((l & 7) ^ ((row >> 1) & 7)) << 3);
    const uint32_t oob = (uint32_t)-(int32_t)(k >= k_lim) & OOB_OFFSET;
    lds_copy16(rs, tile + (wave * ROWS_PER_WAVE + 8 * q) * GB_BK * 2, (uint32_t)(((int64_t)(r0 + row) * ld + k) * 2) | oob);
  }
}
__device__ __forceinline__ bf16x8 direct_frag_kmajor(const uint16_t *tile, int row0, int k0) {
  const int l = threadIdx.x & 63;
  const int row = row0 + (l & 31), c = (k0 >> 3) + (l >> 5);
  return *(const bf16x8 *)(tile + row * GB_BK + ((c ^ ((row >> 1) & 7)) << 3));
}
// contraction-major operand, tile [BK][EXT].  The transposing 8-byte read serves 32 lanes per cycle: 64 bytes in each of
// four consecutive rows.  Chunk c of row k sits at chunk position c ^ swizzle(k), which spreads the four rows over the
// four 64-byte quarters of a bank line: of whole lines (EXT 128 and more) by k % 4, of 128-byte rows, which alternate
// between the halves of a line by themselves, by (k / 2) % 2
template <int EXT>
__device__ __forceinline__ int direct_tr_swizzle(int row) {
  static_assert(EXT == 64 || EXT % 128 == 0, "rows of 128 bytes or whole bank lines");
  return EXT >= 128 ? (row & 3) << 2 : ((row >> 1) & 1) << 2;
}
template <int EXT, int NW, int BK = GB_BK>
__device__ __forceinline__ void direct_tr(rsrc4 rs, int64_t ld, int k0, int c0, uint32_t tile, int wave, int l) {
  constexpr int CPR = EXT / 8;                         // chunks per row
  constexpr int INSTR = BK * CPR / 64 / NW;
  static_assert((BK * CPR) % (64 * NW) == 0, "whole load instructions per wave");
#pragma unroll
  for (int q = 0; q < INSTR; ++q) {
    const int first = (wave * INSTR + q) * 64;         // first chunk (in LDS order) of this instruction
    const int row = (first + l) / CPR, pos = (first + l) % CPR;
    const int col = c0 + ((pos ^ direct_tr_swizzle<EXT>(row)) << 3);
    // the whole address in the vector offset: the descriptor's range check (rows at or beyond the contraction
    // length read zero) does not cover a scalar offset
    lds_copy16(rs, tile + first * 16, (uint32_t)(((int64_t)(k0 + row) * ld + col) * 2));
  }
}
template <int COLS>
__device__ __forceinline__ bf16x8 direct_frag_tr(const uint16_t *tile, int col0, int k0) {
  const int l = threadIdx.x & 63;
  const int blk = l >> 4, q = l & 15;
  const int row = k0 + 8 * (blk >> 1) + (q >> 2), col = col0 + 16 * (blk & 1) + 4 * (q & 3);
  const uint16_t *p = tile + row * COLS + ((((col >> 3) ^ direct_tr_swizzle<COLS>(row)) << 3) | (col & 7));
  typedef __attribute__((address_space(3))) s16x4 lds_v4;
  s16x4 lo = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_v4 *)p);
  s16x4 hi = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_v4 *)(p + 4 * COLS));     // row + 4: same swizzle
  return __builtin_bit_cast(bf16x8, __builtin_shufflevector(lo, hi, 0, 1, 2, 3, 4, 5, 6, 7));
}

// End of a k-step: wait until at most VM of this wave's copy instructions are outstanding
// (they land in issue order, so the older k-steps are in LDS) and until its LDS reads have returned, then the
// workgroup barrier.  Written out instead of __syncthreads(): the fence in front of that barrier waits for ALL
// outstanding copies, which would keep only one k-step in flight whatever the number of LDS buffers.  The
// "memory" clobber keeps the compiler from moving LDS accesses across it.
template <int VM>
__device__ __forceinline__ void copies_landed_barrier() {
  asm volatile("s_waitcnt vmcnt(%0) lgkmcnt(0)\n\ts_barrier" ::"n"(VM) : "memory");
}

// Order for the scheduler: one LDS read behind each of the next MF MFMAs (the last MFMA takes the reads left over)
template <int MF, int READS, int Q = 0>
__device__ __forceinline__ void big_mix() {
  if constexpr (Q < MF) {
    __builtin_amdgcn_sched_group_barrier(0x008, 1, 0);
    if constexpr (Q < READS) __builtin_amdgcn_sched_group_barrier(0x100, (Q + 1 == MF && READS > MF) ? READS - MF + 1 : 1, 0);
    big_mix<MF, READS, Q + 1>();
  }
}

// what every tile kernel does first: XCD-aware spreading (consecutive workgroup ids go
// round-robin over the 8 XCDs; give each XCD one contiguous range of tiles instead, so that
// neighbours share operand panels in one L2), then (record, tile) from the records' prefix sums
struct BigTile {
  int pi, m0, n0;
};
// GM > 0: the tiles of a record are numbered in bands of GM tile rows, column by column inside a band, so that
// the tiles in flight on an XCD form a block that is about as wide as it is high (fewest distinct operand panels
// per tile); GM = 0: whole columns of tiles one after the other.
__device__ __forceinline__ int big_spread(int total_blocks) {
  const int bid = blockIdx.x, xcd = bid & 7, idx = bid >> 3, per = total_blocks >> 3, rem = total_blocks & 7;
  return xcd * per + min(xcd, rem) + idx;
}
template <int BM, int BN, int GM = 0>
__device__ __forceinline__ BigTile big_locate(const GemmProb *__restrict__ probs, int n, int total_blocks) {
  const int bid = big_spread(total_blocks);
  BigTile t;
  t.pi = find_prob(probs, n, bid);
  const int tile = bid - probs[t.pi].blk_begin;
  const int tiles_m = cdiv(probs[t.pi].M, BM);
  if constexpr (GM > 0) {
    const int tiles_n = cdiv(probs[t.pi].N, BN), band = tile / (GM * tiles_n), first = band * GM;
    const int rows = min(GM, tiles_m - first), in_band = tile - band * GM * tiles_n;
    t.m0 = (first + in_band % rows) * BM;
    t.n0 = (in_band / rows) * BN;
    return t;
  }
  t.m0 = (tile % tiles_m) * BM;          // consecutive tiles share the B panel
  t.n0 = (tile / tiles_m) * BN;
  return t;
}

}  // namespace gpp
