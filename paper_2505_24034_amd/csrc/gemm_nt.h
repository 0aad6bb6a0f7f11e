// gemm_nt.h -- the MFMA main loop of the large bf16 contractions, and the pieces (tile shapes, schedule, slab loads,
// fragment layout) that the other loops share with it.
//
// C[m,n] = sum_k A[m,k] * B[n,k]   ("NT": both operands are K-contiguous), fp32 accumulate.
//   forward / recompute : A = W [V,d] tile       B = H rows (gathered)   K = d
//   dW = dz^T H         : A = dz^T [V,N]         B = H^T [d,N]           K = N
//   (fp32 only) dH      : A = dz [N,V]           B = W^T [d,V]           K = V
// fp32 runs on the loop of gemm_small.h; the k-major dH contraction of bf16 on that of gemm_tn.h.
//
// gfx950 mapping
//   - one workgroup = 8 wavefronts (2 x 4) = one 256 x 256 output tile; a wavefront owns 128 x 64 of it as
//     8 x 4 blocks of v_mfma_f32_16x16x32_bf16 (128 fp32 accumulator registers per lane).  The 16x16x32 shape is
//     the one to use on this chip: in an MFMA-only loop it sustains 2.0 PFLOP/s where 32x32x16 sustains 1.75 --
//     the chip is power-limited and the smaller shape lets it clock higher.
//   - K advances in slabs of 128 bytes per row (64 bf16 / 32 fp32) = two k-steps of one MFMA depth.  A slab of
//     both operands is 64 KB of LDS; two slabs are resident (128 of the CU's 160 KB).
//   - slabs go HBM/L2 -> LDS with buffer loads that write LDS directly (16 bytes per lane, no VGPR staging).
//     The hardware puts lane i's 16 bytes at LDS base + 16 i, so the bank-conflict swizzle is applied on the
//     global side: physical 16-byte slot p of row r holds logical chunk p ^ ((r >> 1) & 7), which spreads the
//     16 rows that 16 lanes of a ds_read_b128 touch over all 64 LDS banks.
//   - the loop is software-pipelined by hand (see TileGemm::run): every ds_read_b128 and every slab load is
//     issued in the shadow of an MFMA, far ahead of its use, and scheduling fences pin that interleave.
//   - TileGemmWide: the same for 320 columns; TileGemmNarrow: for 128 or 160 (few tokens), three slabs resident.
//   - out-of-range rows and the K tail use the buffer descriptor's bounds check: such lanes read zeros.
//   - kernels are persistent (one workgroup per CU walks a list of tiles) and fetch the first slabs of their next
//     tile before the epilogue of the current one, so the epilogue's VALU work overlaps that latency.
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

#include "tile_rules.h"

namespace llamarl {

typedef __attribute__((__vector_size__(8 * sizeof(__bf16)))) __bf16 bf16x8_t;
typedef __attribute__((__vector_size__(4 * sizeof(float)))) float f32x4_t;

constexpr int SLAB_ROW_BYTES = 128;
constexpr int BLOCK_BYTES = 16 * SLAB_ROW_BYTES;                  // 16 slab rows: one MFMA block of an operand
constexpr uint32_t OOB_OFFSET = 0x80000000u;                      // beyond any descriptor range used here

// A workgroup's output tile: WM x WN wavefronts, each MB_ x NB_ MFMA blocks.  Wavefront w runs on SIMD w % 4.
template <int WM, int WN, int MB_, int NB_>
struct TileShape {
  __device__ __forceinline__ static int wave_row(int wave) { return wave / WN; }
  __device__ __forceinline__ static int wave_col(int wave) { return wave % WN; }
  static constexpr int WAVES_M = WM, WAVES_N = WN, WAVES = WM * WN, THREADS = 64 * WM * WN;
  static constexpr int MB = MB_, NB = NB_, WAVE_M = MB_ * 16, WAVE_N = NB_ * 16;
  static constexpr int BM = WM * WAVE_M, BN = WN * WAVE_N;        // tile rows (A rows), tile columns (B rows)
  static constexpr int SLAB_A_BYTES = BM * SLAB_ROW_BYTES;
  static constexpr int STAGE_BYTES = (BM + BN) * SLAB_ROW_BYTES;  // one K slab of both operands
};
// 256 x 256, 8 wavefronts of 128 x 64, numbered down the columns: the four of a left half sit on four SIMDs, so where the
// last columns are empty the wavefronts with nothing to do (run_idle) leave every SIMD one that has.
struct Shape256 : TileShape<2, 4, 8, 4> {
  __device__ __forceinline__ static int wave_row(int wave) { return wave & 1; }
  __device__ __forceinline__ static int wave_col(int wave) { return wave >> 1; }
};
// 256 rows in two halves of up to 128 columns, 8 wavefronts of 64 x (16 nb): the left half's have eight column blocks, the
// right half's nb1 = 0, 2, .., 8.  A SIMD's two wavefronts (w, w + 4) belong to the two column halves and to row quarters two
// apart: every SIMD has the same work at any width, and keeps a wavefront with work when either edge cuts the tile in half.
struct Shape256Halves : TileShape<4, 2, 4, 8> {
  __device__ __forceinline__ static int wave_row(int wave) { return (wave + 2 * (wave >> 2)) & 3; }
  __device__ __forceinline__ static int wave_col(int wave) { return wave >> 2; }
};
// 256 x 320, as Shape256 with wavefronts of 128 x 80
struct Shape320 : TileShape<2, 4, 8, 5> {
  __device__ __forceinline__ static int wave_row(int wave) { return wave & 1; }
  __device__ __forceinline__ static int wave_col(int wave) { return wave >> 1; }
};
typedef TileShape<2, 2, 4, 4> Shape128;   // 128 x 128, 4 wavefronts of  64 x 64
typedef TileShape<4, 1, 1, 4> Shape64;    //  64 x  64, 4 wavefronts of  16 x 64

// the 256 x 256 loop's own constants
constexpr int MB = Shape256::MB, NB = Shape256::NB;
constexpr int NTHREADS = Shape256::THREADS;
constexpr int SLAB_A_BYTES = Shape256::SLAB_A_BYTES;              // 32 KB
constexpr int STAGE_BYTES = Shape256::STAGE_BYTES;                // 64 KB
constexpr int MAINLOOP_LDS_BYTES = 2 * STAGE_BYTES;               // 128 KB
constexpr int NARROW_STAGE_BYTES = (Shape256::BM + NARROW_BN) * SLAB_ROW_BYTES;      // 52 KB
constexpr int NARROW_LDS_BYTES = 3 * NARROW_STAGE_BYTES;          // 156 KB

struct BF16 {
  typedef uint16_t store_t;
  typedef bf16x8_t frag_t;
  static constexpr int EPC = 8;  // elements per 16-byte chunk
};
struct F32 {
  typedef float store_t;
  typedef f32x4_t frag_t;
  static constexpr int EPC = 4;
};

// A fragment is the 16 bytes a lane reads from its row: row = lane % 16 of the block, chunk = lane / 16 of the
// k-step.  bf16: that is the operand layout of the 16x16x32 MFMA (8 consecutive k per lane).
__device__ __forceinline__ void mma(const bf16x8_t& a, const bf16x8_t& b, f32x4_t& c) {
  c = __builtin_amdgcn_mfma_f32_16x16x32_bf16(a, b, c, 0, 0, 0);
}
// fp32: the 16x16x4 MFMA takes one float per lane (k = lane / 16); four of them consume the lane's chunk.  Which
// k lands in which MFMA does not matter as long as both operands agree, and they do.
__device__ __forceinline__ void mma(const f32x4_t& a, const f32x4_t& b, f32x4_t& c) {
  c = __builtin_amdgcn_mfma_f32_16x16x4f32(a[0], b[0], c, 0, 0, 0);
  c = __builtin_amdgcn_mfma_f32_16x16x4f32(a[1], b[1], c, 0, 0, 0);
  c = __builtin_amdgcn_mfma_f32_16x16x4f32(a[2], b[2], c, 0, 0, 0);
  c = __builtin_amdgcn_mfma_f32_16x16x4f32(a[3], b[3], c, 0, 0, 0);
}

template <int N>
__device__ __forceinline__ void wait_vmcnt() {       // at most N vector-memory operations of this wave in flight
  __builtin_amdgcn_s_waitcnt((N & 15) | ((N >> 4) << 14) | 0x0F70);
}

__device__ __forceinline__ void wait_vmcnt0() { wait_vmcnt<0>(); }

__device__ __forceinline__ float bf16_bits_to_float(uint16_t b) { return __uint_as_float(((uint32_t)b) << 16); }
__device__ __forceinline__ uint16_t float_to_bf16_bits(float f) {  // round to nearest even
  uint32_t u = __float_as_uint(f);
  if ((u & 0x7fffffffu) > 0x7f800000u) return (uint16_t)((u >> 16) | 0x40u);  // NaN stays NaN
  u += 0x7fffu + ((u >> 16) & 1u);
  return (uint16_t)(u >> 16);
}

// Where the accumulator element (ib, jb, r) of this lane sits inside the tile.
// MFMA 16x16 output layout: register r of lane l holds row 4 (l / 16) + r, column l % 16.
template <typename S>
struct LanePos {
  int wm, wn, lane;
  __device__ __forceinline__ explicit LanePos(int tid)
      : wm(S::wave_row(tid >> 6)), wn(S::wave_col(tid >> 6)), lane(tid & 63) {}
  __device__ __forceinline__ int row(int ib, int r) const { return wm * S::WAVE_M + ib * 16 + (lane >> 4) * 4 + r; }
  __device__ __forceinline__ int col(int jb) const { return wn * S::WAVE_N + jb * 16 + (lane & 15); }
  // Neighbouring columns (see tile_row_of): the lane's nb column blocks hold columns col_near(nb) + 0 .. nb - 1, so 16
  // lanes own 16 nb consecutive columns of one row.
  __device__ __forceinline__ int col_near(int nb) const { return wn * S::WAVE_N + nb * (lane & 15); }
};

// Which row of an operand tile the loader puts into LDS row `r`.  The LDS rows of the column operand feed a wavefront's
// 16-column MFMA blocks, WAVE_N rows a wavefront (block jb, MFMA column n = low 4 bits); with NEAR, block jb / column n of
// a wavefront with nb blocks is its tile row nb n + jb, so that acc[.][0 .. nb-1] of a lane are neighbouring output
// columns and an epilogue can store them as one unit.  Rows of blocks it does not have: none.  Only the global side
// changes: LDS layout, swizzle and fragment reads stay.
constexpr int NO_ROW = 1 << 30;
template <bool NEAR, int WAVE_N>
__device__ __forceinline__ int tile_row_of(int r, int nb) {
  const int jb = (r & (WAVE_N - 1)) >> 4;
  return !NEAR ? r : jb < nb ? (r & ~(WAVE_N - 1)) + nb * (r & 15) + jb : NO_ROW;
}

typedef int i32x4_t __attribute__((ext_vector_type(4)));
// buffer_load_dwordx4 ... lds, written out by hand.  The compiler's wait-count pass cannot tell which LDS bytes
// an LDS-direct load will fill: with the builtin, transposing reads (ds_read_b64_tr_b16 carries no memory operand) and
// reads through a computed stage address wait for ALL loads in flight, which serialises the loop.  Issued from inline
// asm the loads are invisible to that pass; the loop's own s_waitcnt vmcnt + barrier order them against the reads.
__device__ __forceinline__ void lds_dma16(uint32_t lds_addr, uint32_t voff, i32x4_t rsrc, uint32_t soff) {
  asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tbuffer_load_dwordx4 %1, %2, %3 offen lds"
               :
               : "s"(lds_addr), "v"(voff), "s"(rsrc), "s"(soff)
               : "memory", "m0");
}

// as lds_dma16, four bytes a lane: 64 neighbouring words of LDS
__device__ __forceinline__ void lds_dma4(uint32_t lds_addr, uint32_t voff, i32x4_t rsrc) {
  asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tbuffer_load_dword %1, %2, 0 offen lds"
               :
               : "s"(lds_addr), "v"(voff), "s"(rsrc)
               : "memory", "m0");
}
__device__ __forceinline__ uint32_t lds_address(const void* p) {
  return (uint32_t)(uintptr_t)(const __attribute__((address_space(3))) char*)(const char*)p;
}

__device__ __forceinline__ int swizzle(int row) { return (row >> 1) & 7; }

// One operand slab stream: ROWS rows x 128 bytes per step; this thread moves ITERS 16-byte chunks of it.
// Wave-instruction `it` of wave w fills rows (it*WAVES + w)*8 .. +7 of the slab; lane l takes row +l/8 and the
// physical 16-byte slot l%8.  Because it*WAVES*8 rows is a multiple of 16, the swizzle (and so the logical chunk this
// lane fetches) is the same for all instructions.
// WAVE_ROWS: rows of a wavefront's blocks (column operand; the last wavefront has nb1 blocks, the others all).
template <typename TT, int ROWS = Shape256::BM, int WAVES = Shape256::WAVES, int WAVE_ROWS = Shape256::WAVE_N>
struct SlabLoader {
  static constexpr int ITERS = ROWS / (8 * WAVES);
  static_assert(ITERS * 8 * WAVES == ROWS && (8 * WAVES) % 16 == 0, "whole wave-instructions, one swizzle for all");
  i32x4_t desc;           // buffer descriptor
  uint32_t voff[ITERS];   // per-lane byte offset of (row, logical chunk) inside the panel at k = 0

  __device__ __forceinline__ void set_base(const void* base, uint32_t bytes) {
    const uint64_t p = reinterpret_cast<uint64_t>(base);
    desc = i32x4_t{__builtin_amdgcn_readfirstlane((int)(uint32_t)p),
                   __builtin_amdgcn_readfirstlane((int)((uint32_t)(p >> 32) & 0xffffu)),
                   __builtin_amdgcn_readfirstlane((int)bytes), 0x00020000};
  }
  // Built once a tile and used as it is: rebuilt for every slab (a dozen scalar instructions) it cost the long contractions
  // 1 - 2 %.  readfirstlane is a no-op on scalar registers; where the compiler has lost track of a word being uniform it
  // is what brings it back.
  __device__ __forceinline__ i32x4_t rsrc() const {
    return i32x4_t{__builtin_amdgcn_readfirstlane(desc[0]), __builtin_amdgcn_readfirstlane(desc[1]),
                   __builtin_amdgcn_readfirstlane(desc[2]), __builtin_amdgcn_readfirstlane(desc[3])};
  }

  __device__ __forceinline__ static int lane_chunk(int wave, int lane) {
    return (lane & 7) ^ swizzle(wave * 8 + (lane >> 3));
  }
  // base: first row of the tile; ld in elements; rows_valid <= ROWS rows exist from base on.
  template <bool NEAR = false>
  __device__ __forceinline__ void init(const void* base, int64_t ld, int rows_valid, int wave, int lane, int nb1 = WAVE_ROWS / 16) {
    const uint32_t row_bytes = (uint32_t)(ld * (int64_t)sizeof(typename TT::store_t));
    set_base(base, row_bytes * (uint32_t)rows_valid);
    const uint32_t c16 = (uint32_t)lane_chunk(wave, lane) * 16u;
#pragma unroll
    for (int it = 0; it < ITERS; ++it) {
      const int row = lane_tile_row<NEAR>(it, wave, lane, nb1);
      voff[it] = (row < rows_valid) ? (uint32_t)row * row_bytes + c16 : OOB_OFFSET;
    }
  }
  // The tile rows this lane fetches (one per wave-instruction).
  template <bool NEAR = false>
  __device__ __forceinline__ static int lane_tile_row(int it, int wave, int lane, int nb1) {
    const int r = (it * WAVES + wave) * 8 + (lane >> 3);
    return tile_row_of<NEAR, WAVE_ROWS>(r, r >= ROWS - WAVE_ROWS ? nb1 : WAVE_ROWS / 16);
  }
  // Gathered panel: tile row r is a row of the whole matrix `base` (total_rows rows, < 2^31 bytes).  Free with per-lane
  // buffer offsets: this is how masked tokens are skipped without a packed copy of H.  The caller loads the gather
  // list entries itself, in one batch and ahead of time.
  // grow[it] = row of the whole matrix that tile row lane_tile_row(it) maps to (any valid row where the tile row
  // is >= rows_valid: it is not fetched).
  template <bool NEAR = false>
  __device__ __forceinline__ void init_gathered(const void* base, int64_t ld, int64_t total_rows, const int (&grow)[ITERS],
                                                int rows_valid, int wave, int lane, int nb1 = WAVE_ROWS / 16) {
    const uint32_t row_bytes = (uint32_t)(ld * (int64_t)sizeof(typename TT::store_t));
    set_base(base, (uint32_t)total_rows * row_bytes);
    const uint32_t c16 = (uint32_t)lane_chunk(wave, lane) * 16u;
#pragma unroll
    for (int it = 0; it < ITERS; ++it)
      voff[it] = (lane_tile_row<NEAR>(it, wave, lane, nb1) < rows_valid) ? (uint32_t)grow[it] * row_bytes + c16 : OOB_OFFSET;
  }
  // One request of a slab (lds_dma16).  k0: first k of the slab (elements); K: contraction length; lds: start of this
  // operand's slab in LDS.  Lanes whose chunk lies past K fetch nothing (zeros); no slab reaches past K if !tail.
  __device__ __forceinline__ void issue_one(const i32x4_t& rs, char* lds, int it, int k0, int K, int wave, int lane,
                                            bool tail = true) const {
    lds_dma16(lds_address(lds) + (uint32_t)((it * WAVES + wave) * 8 * SLAB_ROW_BYTES),
              tail && k0 + lane_chunk(wave, lane) * TT::EPC >= K ? OOB_OFFSET : voff[it], rs,
              (uint32_t)k0 * (uint32_t)sizeof(typename TT::store_t));
  }
  __device__ __forceinline__ void issue(char* lds, int k0, int K, int wave, int lane) const {
    const i32x4_t rs = rsrc();
#pragma unroll
    for (int it = 0; it < ITERS; ++it) issue_one(rs, lds, it, k0, K, wave, lane);
  }
};

__device__ __forceinline__ int wave_id() { return __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6)); }

#define LLAMARL_FENCE() __builtin_amdgcn_sched_barrier(0)

// The loads of one K slab, issued one per MFMA slot after the barrier of a k-step.
template <typename LA, typename LB>
struct SlabFetch {
  const LA* la;
  const LB* lb;
  i32x4_t ra, rb;
  char* dst;      // stage that receives the slab
  int k0, K, wave, lane;
};

// Column block of MFMA slot t: rows of blocks are walked alternately left-to-right and right-to-left, so the column
// operand stays the same across a row change (the row operand changes there).  The chip is power-limited under
// MFMA load and operand switching costs energy: this order measured 0.5 % faster on every contraction kernel than
// restarting each row at column block 0.
__device__ __forceinline__ constexpr int snake(int t) { return ((t >> 2) & 1) ? 3 - (t & 3) : (t & 3); }

// One k-step = one MFMA depth (two per slab): 32 slots, slot t runs block (ib, jb) = (t / 4, snake(t)).
//   a[8]   : the A fragments of this k-step, one register set each.  Block ib is done after slot 4 ib + 3 and its
//            registers take the NEXT k-step's fragment right away (slot 4 ib + 4): 28 slots ahead of its use.
//            a[7] of a k-step is read at its own slot 0.
//   bc, bn : B fragments of this / the next k-step (all four are used by every ib, so they are double-buffered).
//   BAR    : this is the last k-step of a slab that has a successor.  By slot 0 every read of the slab has been
//            issued, so the barrier can sit as early as slot TB = 8: it waits for this thread's share of the next
//            slab (vmcnt) and for its own reads (lgkmcnt), then the 24 MFMAs left run from registers while the
//            next slab's fragments are read and, with FETCH, the slab after that is requested (one load every
//            other slot from slot LS on, into the stage this barrier just freed).  LS = 11 for the logits kernels;
//            the store contraction (dW) asks two slots earlier, which measured 1 - 1.5 % faster for it at three of
//            four shapes and the same at the fourth, while the logits kernels lose 0.5 % with it at the longest
//            batch.  Slots of the same parity as the fragment reads (even) are 4 - 6 % slower.
//   NEXT   : there is a next k-step (pa_nxt / pb_nxt: lane's fragment address of its blocks 0).
//   LS     : a template parameter although only its value matters: every specialisation of this template must be
//            called from ONE function instantiation only -- the host pass of hipcc (ROCm 7.2) rejects a second
//            caller of the same specialisation ("substitution failure", no reason given; the device pass accepts it).
//   YOUNGER: vector-memory operations issued after the next slab's loads that the barrier need not wait for.
//   INIT   : a tile's first k-step; the accumulators start here (as zero), so that no pass clears them.
template <typename TT, bool BAR, bool NEXT, bool FETCH, int LS, int YOUNGER = 0, bool INIT = false>
__device__ __forceinline__ void k_step(typename TT::frag_t (&a)[MB], const typename TT::frag_t (&bc)[NB],
                                       typename TT::frag_t (&bn)[NB], f32x4_t (&acc)[MB][NB], const char* pa_cur,
                                       const char* pa_nxt, const char* pb_nxt, const SlabFetch<SlabLoader<TT>, SlabLoader<TT>>* sf) {
  typedef typename TT::frag_t frag_t;
  constexpr int TB = 8;
  static_assert(MB == 8 && NB == 4, "slot table written for an 8 x 4 wave tile");
#pragma unroll
  for (int t = 0; t < MB * NB; ++t) {
    const int ib = t >> 2, jb = snake(t);
    if (BAR && t == TB) {
      wait_vmcnt<YOUNGER>();      // this thread's share of the next slab has landed in LDS
      __syncthreads();            // everyone's has, and everyone is done reading this slab
      LLAMARL_FENCE();
    }
    if (INIT) acc[ib][jb] = f32x4_t{0.f, 0.f, 0.f, 0.f};
    mma(a[ib], bc[jb], acc[ib][jb]);
    LLAMARL_FENCE();
    if (t == 0) {
      a[7] = *reinterpret_cast<const frag_t*>(pa_cur + 7 * BLOCK_BYTES);
      LLAMARL_FENCE();
    }
    if (NEXT) {
      if (t == TB) a[0] = *reinterpret_cast<const frag_t*>(pa_nxt);
      if (t == TB + 1) a[1] = *reinterpret_cast<const frag_t*>(pa_nxt + BLOCK_BYTES);
      if (t >= 12 && (t & 3) == 0) a[ib - 1] = *reinterpret_cast<const frag_t*>(pa_nxt + (ib - 1) * BLOCK_BYTES);
      if (t == 10) bn[0] = *reinterpret_cast<const frag_t*>(pb_nxt);
      if (t == 14) bn[1] = *reinterpret_cast<const frag_t*>(pb_nxt + BLOCK_BYTES);
      if (t == 18) bn[2] = *reinterpret_cast<const frag_t*>(pb_nxt + 2 * BLOCK_BYTES);
      if (t == 22) bn[3] = *reinterpret_cast<const frag_t*>(pb_nxt + 3 * BLOCK_BYTES);
      LLAMARL_FENCE();
    }
    if (FETCH && t >= LS && t <= LS + 14 && ((t - LS) & 1) == 0) {
      const int n = (t - LS) >> 1;
      if (n < 4) sf->la->issue_one(sf->ra, sf->dst, n, sf->k0, sf->K, sf->wave, sf->lane);
      else sf->lb->issue_one(sf->rb, sf->dst + SLAB_A_BYTES, n - 4, sf->k0, sf->K, sf->wave, sf->lane);
      LLAMARL_FENCE();
    }
  }
}

// The same for a wavefront of 8 x 5 blocks: 40 slots, slot t runs block (t / 5, snake5(t)).  Five column fragments twice leave
// registers for four row fragments: block ib is in a[ib % 4], read when block ib - 4 is done, 14 - 16 slots ahead of its
// use.  So the reads of a slab end at slot 20, its barrier is at slot 22, and the nine loads follow on the odd slots.
__device__ __forceinline__ constexpr int snake5(int t) { return (t / 5 & 1) ? 4 - t % 5 : t % 5; }
template <typename TT, typename Fetch, bool BAR, bool NEXT, bool FETCH, bool INIT = false>
__device__ __forceinline__ void wide_k_step(typename TT::frag_t (&a)[4], const typename TT::frag_t (&bc)[5],
                                            typename TT::frag_t (&bn)[5], f32x4_t (&acc)[8][5], const char* pa_cur,
                                            const char* pa_nxt, const char* pb_nxt, const Fetch* sf) {
  typedef typename TT::frag_t frag_t;
#pragma unroll
  for (int t = 0; t < 40; ++t) {
    const int ib = t / 5, jb = snake5(t);
    if (BAR && t == 22) {
      wait_vmcnt<0>();            // as in k_step
      __syncthreads();
      LLAMARL_FENCE();
    }
    if (INIT) acc[ib][jb] = f32x4_t{0.f, 0.f, 0.f, 0.f};
    mma(a[ib & 3], bc[jb], acc[ib][jb]);
    LLAMARL_FENCE();
    if (t == 0) a[3] = *reinterpret_cast<const frag_t*>(pa_cur + 3 * BLOCK_BYTES);
    if (t == 6) a[0] = *reinterpret_cast<const frag_t*>(pa_cur + 4 * BLOCK_BYTES);
    if (t == 10) a[1] = *reinterpret_cast<const frag_t*>(pa_cur + 5 * BLOCK_BYTES);
    if (t == 16) a[2] = *reinterpret_cast<const frag_t*>(pa_cur + 6 * BLOCK_BYTES);
    if (t == 20) a[3] = *reinterpret_cast<const frag_t*>(pa_cur + 7 * BLOCK_BYTES);
    LLAMARL_FENCE();
    if (NEXT) {
      if (t == 26) a[0] = *reinterpret_cast<const frag_t*>(pa_nxt);
      if (t == 30) a[1] = *reinterpret_cast<const frag_t*>(pa_nxt + BLOCK_BYTES);
      if (t == 36) a[2] = *reinterpret_cast<const frag_t*>(pa_nxt + 2 * BLOCK_BYTES);
      if (t == 22) bn[0] = *reinterpret_cast<const frag_t*>(pb_nxt);
      if (t == 24) bn[1] = *reinterpret_cast<const frag_t*>(pb_nxt + BLOCK_BYTES);
      if (t == 28) bn[2] = *reinterpret_cast<const frag_t*>(pb_nxt + 2 * BLOCK_BYTES);
      if (t == 32) bn[3] = *reinterpret_cast<const frag_t*>(pb_nxt + 3 * BLOCK_BYTES);
      if (t == 34) bn[4] = *reinterpret_cast<const frag_t*>(pb_nxt + 4 * BLOCK_BYTES);
      LLAMARL_FENCE();
    }
    if (FETCH && t >= 23 && (t & 1)) {
      const int n = (t - 23) >> 1;
      if (n < 4) sf->la->issue_one(sf->ra, sf->dst, n, sf->k0, sf->K, sf->wave, sf->lane);
      else sf->lb->issue_one(sf->rb, sf->dst + SLAB_A_BYTES, n - 4, sf->k0, sf->K, sf->wave, sf->lane);
      LLAMARL_FENCE();
    }
  }
}

// Whether the last slab's second half holds anything: past K both operands are zeros, and their k-step is left out (d of
// 520: 8.5 of 9 slabs, logits of 3000 x 40000 142 -> 138 us; 1032: 403 -> 398; whole slabs as before).
template <int BK>
__device__ __forceinline__ bool half_slab_left(int K) { return (unsigned)(K - 1) % BK >= BK / 2; }

// The order in which a logits kernel takes the slabs: the whole ones from `turn` on, wrapping round, then the rest of K.  Rows of
// W and H often lie a power of two apart (d = 4096: 8 KB), and workgroups that walk K together then read the same few
// channels of the memory: 256 workgroups streaming 1 GB of W took 235 us (4.5 TB/s) from slab 0, whatever their slabs in flight,
// and 169 us (6.2) each from a slab of its own.  Workgroups that share a row of patches, and so the panels in their L2, start
// together; the next row starts two slabs (256 bytes) on.  Forward call over a 128256 x 4096 head: 40 tokens 236 -> 181 us, 150
// 228 -> 194, 300 309 -> 294; dz at 225, 500 and 900 tokens 324 -> 271, 470 -> 447, 801 -> 789.  Only where W streams: with more
// than TURN_COLUMNS columns of tiles the panels come from the caches.
constexpr int TURN_COLUMNS = 4;
struct SlabOrder {
  int whole, turn;
  template <int BK>
  __device__ __forceinline__ void init(int K, int row_of_patches) {
    whole = K / BK;
    turn = whole < 2 ? 0 : 2 * row_of_patches & ((1 << (31 - __builtin_clz(whole))) - 1);
  }
  template <int BK>
  __device__ __forceinline__ int k(int kt, int) const {   // first k of the kt-th slab taken; past K where there is none
    const int s = kt + turn;
    return (kt >= whole ? kt : s >= whole ? s - whole : s) * BK;
  }
  __device__ __forceinline__ bool rest_is_last() const { return true; }
};
// Two scalar registers through the main loop and eight scalar operations a slab, which long contractions on 256 columns notice though
// nothing turns: dz of 33001 x 1032 0.3 - 1.6 % (6400 tokens 455 / 461 us, 9500 663 / 671; 128256 x 4096, 8576 tokens: 6434 / 6482), the
// forward up to 0.6 %.  dz has a loop in order beside the turned one.  The forward, whose short calls notice a kernel with one loop more (two
// more: (1700, 5412, 192) 16.3 -> 16.6 us, (128, 98304, 64) 20.1 -> 20.5), wraps round all slabs there, the rest of K among them: one register
// and three operations.  (kt ^ turn, as cheap, breaks up the runs of slabs that share a line where rows are no multiple of 128 bytes:
// (256, 49200, 520) 30.0 / 30.9 us, in order 31.4.)
struct SlabRing {
  int first;                                              // k of the slab taken first
  template <int BK>
  __device__ __forceinline__ void init(int K, int row_of_patches) {
    first = (2 * row_of_patches & ((1 << (31 - __builtin_clz((K + BK - 1) / BK))) - 1)) * BK;
  }
  template <int BK>
  __device__ __forceinline__ int k(int kt, int K) const {
    const uint32_t s = (uint32_t)(kt * BK + first);
    return (int)min(s, s - (uint32_t)((K + BK - 1) & -BK));         // past the end: wrapped; before it the difference is huge
  }
  __device__ __forceinline__ bool rest_is_last() const { return first == 0; }
};
struct InOrder {
  template <int BK>
  __device__ __forceinline__ void init(int, int) {}
  template <int BK>
  __device__ __forceinline__ int k(int kt, int) const { return kt * BK; }
  __device__ __forceinline__ bool rest_is_last() const { return true; }
};

// The main loop, split in two so that a persistent workgroup can start fetching its NEXT tile before it runs the
// epilogue of the current one:
//   prefetch(): set up both operand streams of a tile and issue its first two K slabs.  Only legal once every
//               wave of the workgroup is done reading LDS (a __syncthreads() after the previous run()).
//   run():      the K loop.  Waves leave it at different times: __syncthreads() before reusing LDS.
// smem must hold MAINLOOP_LDS_BYTES.
//
// NEAR: a lane's column blocks hold neighbouring output columns (tile_row_of); the epilogue must then take its columns from
// LanePos::col_near().
// YOUNGER, FIRST_ONLY: see run().
template <typename TT, int LOAD_SLOT, int YOUNGER, bool FIRST_ONLY, typename Order = InOrder>
struct TileGemm {
  typedef TT Type;
  typedef Shape256 Shape;
  typedef typename TT::frag_t frag_t;
  static constexpr bool KMAJOR = false;
  static constexpr bool HAS_IDLE = true, HALVES = false;
  static constexpr bool REQUESTS_PAST_K = false;      // slabs past K may be in flight after run(): to be waited for
  static constexpr int BK = 8 * TT::EPC;
  static constexpr int LDS_BYTES = MAINLOOP_LDS_BYTES;
  static constexpr int GROUPS_PER_CU = 1;      // workgroups of a persistent grid per CU
  SlabLoader<TT> la, lb;
  int K;
  Order order;
  __device__ __forceinline__ static constexpr int width() { return Shape::BN; }

  template <bool NEAR>
  __device__ __forceinline__ void prefetch(const void* A_tile, int64_t lda, int rowsA, const void* B_tile, int64_t ldb,
                                           int rowsB, int64_t K_, char* smem) {
    const int lane = threadIdx.x & 63, wave = wave_id();
    K = (int)K_;
    la.init(A_tile, lda, rowsA, wave, lane);
    lb.template init<NEAR>(B_tile, ldb, rowsB, wave, lane);
    la.issue(smem, 0, K, wave, lane);
    lb.issue(smem + SLAB_A_BYTES, 0, K, wave, lane);
    if (K > BK) {
      la.issue(smem + STAGE_BYTES, BK, K, wave, lane);
      lb.issue(smem + STAGE_BYTES + SLAB_A_BYTES, BK, K, wave, lane);
    }
  }

  // as prefetch, the B panel gathered: B_base is the base of the whole matrix with b_total rows, grow the gather list
  // entries of this lane (SlabLoader::init_gathered), already in registers: no global load stands between the
  // caller's barrier and the first slab request.  The requests are the caller's: issue_first(0) .. (FIRST_PARTS - 1).
  template <bool NEAR>
  __device__ __forceinline__ void setup_gathered(const void* A_tile, int64_t lda, int rowsA, const void* B_base,
                                                 int64_t ldb, int rowsB, int64_t K_, const int (&grow)[4],
                                                 int64_t b_total, int turn) {
    const int lane = threadIdx.x & 63, wave = wave_id();
    K = (int)K_;
    order.template init<BK>(K, turn);
    la.init(A_tile, lda, rowsA, wave, lane);
    lb.template init_gathered<NEAR>(B_base, ldb, b_total, grow, rowsB, wave, lane);
  }
  // Four requests a call, so that a logits kernel can spread them over its epilogue: sixteen at once (128 KB for the
  // workgroup) keep a wavefront from its epilogue for as long as the CU takes to accept them.
  static constexpr int FIRST_PARTS = 4;
  __device__ __forceinline__ void issue_first(char* smem, int part) const {
    const int lane = threadIdx.x & 63, wave = wave_id();
    char* st = smem + (part >> 1) * STAGE_BYTES;
    if (part > 1 && BK >= K) return;
    const int k0 = order.template k<BK>(part >> 1, K);
    if ((part & 1) == 0) la.issue(st, k0, K, wave, lane);
    else lb.issue(st + SLAB_A_BYTES, k0, K, wave, lane);
  }

  // Instead of run() for a wavefront whose whole part of the tile lies past the matrix (wave-uniform; a last column of
  // few tokens): its loads and barriers, nothing else.  The SIMD then belongs to the other wavefront.
  __device__ __forceinline__ void run_idle(char* smem) const {
    const int lane = threadIdx.x & 63, wave = wave_id();
    const int nk = (K + BK - 1) / BK;
    wait_vmcnt0();
    __syncthreads();
    for (int kt = 0; kt < nk - 2; ++kt) {
      char* cur = smem + (kt & 1) * STAGE_BYTES;
      wait_vmcnt0();
      __syncthreads();
      la.issue(cur, order.template k<BK>(kt + 2, K), K, wave, lane);
      lb.issue(cur + SLAB_A_BYTES, order.template k<BK>(kt + 2, K), K, wave, lane);
    }
    if (nk >= 2) {
      wait_vmcnt0();
      __syncthreads();
    }
  }

  static constexpr int COUNTED_STORES = YOUNGER;
  // If `counted` (wave-uniform), at least YOUNGER vector-memory operations -- the previous tile's stores -- were issued
  // after prefetch().  vmcnt counts in order, so slabs 0 and 1 are waited for without them; the stores then drain under
  // the first slabs.  dW over a 128256 x 4096 head: 64 rows 295 -> 273 us, 300 rows 587 -> 528, 1100 rows 1183 -> 1124,
  // 8576 rows -0.8 %.  (No gain for the recompute, whose epilogue is longer than its stores.)
  // FIRST_ONLY: only the first wait is counted, for a few stores (the forward's).
  __device__ __forceinline__ void run(char* smem, f32x4_t (&acc)[MB][NB], bool counted = false) {
    const int lane = threadIdx.x & 63, wave = wave_id();
    const int wm = Shape::wave_row(wave), wn = Shape::wave_col(wave);
    const int nk = (K + BK - 1) / BK;
    // per-lane read addresses of block 0: row = lane % 16, chunk 4 ks + lane / 16 of k-step ks, swizzled.  The
    // swizzle depends on the low four row bits only, so block ib is the same address + ib * BLOCK_BYTES.
    const int g = lane >> 4, l16 = lane & 15;
    const int sw = swizzle(l16);
    int a_addr[2], b_addr[2];
#pragma unroll
    for (int ks = 0; ks < 2; ++ks) {
      a_addr[ks] = (wm * Shape::WAVE_M + l16) * SLAB_ROW_BYTES + (((4 * ks + g) ^ sw) * 16);
      b_addr[ks] = SLAB_A_BYTES + (wn * Shape::WAVE_N + l16) * SLAB_ROW_BYTES + (((4 * ks + g) ^ sw) * 16);
    }
    // Slabs 0 and 1 were issued by prefetch(); stores of a previous epilogue may sit between them and now in the
    // vmcnt queue.  Where their number is not known, wait for everything.
    if (counted) wait_vmcnt<YOUNGER>();
    else wait_vmcnt0();
    __syncthreads();
    frag_t a[MB], b0[NB], b1[NB];
    a[0] = *reinterpret_cast<const frag_t*>(smem + a_addr[0]);
#pragma unroll
    for (int j = 0; j < NB; ++j) b0[j] = *reinterpret_cast<const frag_t*>(smem + b_addr[0] + j * BLOCK_BYTES);
#pragma unroll
    for (int i = 1; i < MB - 1; ++i) a[i] = *reinterpret_cast<const frag_t*>(smem + a_addr[0] + i * BLOCK_BYTES);

    // One turn of the loop: a slab's second k-step, then the next slab's first.  Slabs 0 .. nk-3 fetch slab kt+2 after
    // their barrier; slab nk-2 (nothing left to fetch) and the last slab follow, written out one after the other (a
    // branch inside one loop body makes the compiler copy accumulators)
    LLAMARL_FENCE();
    k_step<TT, false, true, false, LOAD_SLOT, 0, true>(a, b0, b1, acc, smem + a_addr[0], smem + a_addr[1],
                                                       smem + b_addr[1], nullptr);
    int kt0 = 0;
    if (!FIRST_ONLY && nk > 2) {       // slab 0 apart: its barrier waits for slab 1, older than the stores too
      char* cur = smem;
      const char* nxt = smem + STAGE_BYTES;
      const SlabFetch<SlabLoader<TT>, SlabLoader<TT>> sf{&la, &lb, la.rsrc(), lb.rsrc(), cur, order.template k<BK>(2, K), K, wave, lane};
      k_step<TT, true, true, true, LOAD_SLOT, FIRST_ONLY ? 0 : YOUNGER>(a, b1, b0, acc, cur + a_addr[1], nxt + a_addr[0],
                                                                        nxt + b_addr[0], &sf);
      k_step<TT, false, true, false, LOAD_SLOT>(a, b0, b1, acc, nxt + a_addr[0], nxt + a_addr[1], nxt + b_addr[1], nullptr);
      kt0 = 1;
    }
    for (int kt = kt0; kt < nk - 2; ++kt) {
      char* cur = smem + (kt & 1) * STAGE_BYTES;
      const char* nxt = smem + ((kt + 1) & 1) * STAGE_BYTES;
      LLAMARL_FENCE();
      const SlabFetch<SlabLoader<TT>, SlabLoader<TT>> sf{&la, &lb, la.rsrc(), lb.rsrc(), cur, order.template k<BK>(kt + 2, K), K, wave, lane};
      k_step<TT, true, true, true, LOAD_SLOT>(a, b1, b0, acc, cur + a_addr[1], nxt + a_addr[0], nxt + b_addr[0], &sf);
      k_step<TT, false, true, false, LOAD_SLOT>(a, b0, b1, acc, nxt + a_addr[0], nxt + a_addr[1], nxt + b_addr[1], nullptr);
    }
    if (nk >= 2) {
      const char* cur = smem + ((nk - 2) & 1) * STAGE_BYTES;
      const char* nxt = smem + ((nk - 1) & 1) * STAGE_BYTES;
      LLAMARL_FENCE();
      k_step<TT, true, true, false, LOAD_SLOT>(a, b1, b0, acc, cur + a_addr[1], nxt + a_addr[0], nxt + b_addr[0], nullptr);
      k_step<TT, false, true, false, LOAD_SLOT>(a, b0, b1, acc, nxt + a_addr[0], nxt + a_addr[1], nxt + b_addr[1], nullptr);
    }
    if (half_slab_left<BK>(K) || !order.rest_is_last()) {
      const char* cur = smem + ((nk - 1) & 1) * STAGE_BYTES;
      LLAMARL_FENCE();
      k_step<TT, false, false, false, LOAD_SLOT>(a, b1, b0, acc, cur + a_addr[1], nullptr, nullptr, nullptr);
    }
  }
};

// ---- wide tiles: 256 rows x 320 columns -----------------------------------------------------------------------------------
// As TileGemm (see there); two slabs of 72 KB.  A product takes a tenth fewer bytes from L2 and LDS than on 256 x 256, and a
// fifth fewer barriers and epilogues.  247 registers.  (A word of every line of W two slabs ahead, to have it in L2 earlier: 300
// tokens 305 -> 330 us; a barrier that leaves one request in flight for that: the long contractions +2 %.)
template <typename TT>
struct TileGemmWide {
  typedef TT Type;
  typedef Shape320 Shape;
  typedef typename TT::frag_t frag_t;
  typedef SlabLoader<TT> LoaderA;
  typedef SlabLoader<TT, Shape::BN, Shape::WAVES, Shape::WAVE_N> LoaderB;
  typedef SlabFetch<LoaderA, LoaderB> Fetch;
  static constexpr bool KMAJOR = false;
  static constexpr bool HAS_IDLE = true, HALVES = false;
  static constexpr bool REQUESTS_PAST_K = false;
  static constexpr int BK = 8 * TT::EPC;
  static constexpr int LDS_BYTES = 2 * Shape::STAGE_BYTES;
  static constexpr int COUNTED_STORES = 2;
  LoaderA la;
  LoaderB lb;
  int K;
  SlabOrder order;
  __device__ __forceinline__ static constexpr int width() { return Shape::BN; }

  template <bool NEAR>
  __device__ __forceinline__ void setup_gathered(const void* A_tile, int64_t lda, int rowsA, const void* B_base,
                                                 int64_t ldb, int rowsB, int64_t K_, const int (&grow)[LoaderB::ITERS],
                                                 int64_t b_total, int turn) {
    const int lane = threadIdx.x & 63, wave = wave_id();
    K = (int)K_;
    order.init<BK>(K, turn);
    la.init(A_tile, lda, rowsA, wave, lane);
    lb.template init_gathered<NEAR>(B_base, ldb, b_total, grow, rowsB, wave, lane);
  }
  static constexpr int FIRST_PARTS = 4;
  __device__ __forceinline__ void issue_first(char* smem, int part) const {
    const int lane = threadIdx.x & 63, wave = wave_id();
    char* st = smem + (part >> 1) * Shape::STAGE_BYTES;
    if (part > 1 && BK >= K) return;
    const int k0 = order.k<BK>(part >> 1, K);
    if ((part & 1) == 0) la.issue(st, k0, K, wave, lane);
    else lb.issue(st + SLAB_A_BYTES, k0, K, wave, lane);
  }
  __device__ __forceinline__ void run_idle(char* smem) const {
    const int lane = threadIdx.x & 63, wave = wave_id();
    const int nk = (K + BK - 1) / BK;
    wait_vmcnt0();
    __syncthreads();
    for (int kt = 0; kt < nk - 2; ++kt) {
      char* cur = smem + (kt & 1) * Shape::STAGE_BYTES;
      wait_vmcnt0();
      __syncthreads();
      la.issue(cur, order.k<BK>(kt + 2, K), K, wave, lane);
      lb.issue(cur + SLAB_A_BYTES, order.k<BK>(kt + 2, K), K, wave, lane);
    }
    if (nk >= 2) {
      wait_vmcnt0();
      __syncthreads();
    }
  }
  __device__ __forceinline__ void run(char* smem, f32x4_t (&acc)[8][5], bool counted = false) {
    const int lane = threadIdx.x & 63, wave = wave_id();
    const int nk = (K + BK - 1) / BK;
    const int g = lane >> 4, l16 = lane & 15, sw = swizzle(l16);
    int a_addr[2], b_addr[2];
#pragma unroll
    for (int ks = 0; ks < 2; ++ks) {
      a_addr[ks] = (Shape::wave_row(wave) * Shape::WAVE_M + l16) * SLAB_ROW_BYTES + (((4 * ks + g) ^ sw) * 16);
      b_addr[ks] = SLAB_A_BYTES + (Shape::wave_col(wave) * Shape::WAVE_N + l16) * SLAB_ROW_BYTES + (((4 * ks + g) ^ sw) * 16);
    }
    if (counted) wait_vmcnt<COUNTED_STORES>();
    else wait_vmcnt0();
    __syncthreads();
    frag_t a[4], b0[5], b1[5];
    a[0] = *reinterpret_cast<const frag_t*>(smem + a_addr[0]);
#pragma unroll
    for (int j = 0; j < 5; ++j) b0[j] = *reinterpret_cast<const frag_t*>(smem + b_addr[0] + j * BLOCK_BYTES);
#pragma unroll
    for (int i = 1; i < 3; ++i) a[i] = *reinterpret_cast<const frag_t*>(smem + a_addr[0] + i * BLOCK_BYTES);
    LLAMARL_FENCE();
    wide_k_step<TT, Fetch, false, true, false, true>(a, b0, b1, acc, smem + a_addr[0], smem + a_addr[1], smem + b_addr[1], nullptr);
    for (int kt = 0; kt < nk - 2; ++kt) {
      char* cur = smem + (kt & 1) * Shape::STAGE_BYTES;
      const char* nxt = smem + ((kt + 1) & 1) * Shape::STAGE_BYTES;
      LLAMARL_FENCE();
      const Fetch sf{&la, &lb, la.rsrc(), lb.rsrc(), cur, order.k<BK>(kt + 2, K), K, wave, lane};
      wide_k_step<TT, Fetch, true, true, true>(a, b1, b0, acc, cur + a_addr[1], nxt + a_addr[0], nxt + b_addr[0], &sf);
      wide_k_step<TT, Fetch, false, true, false>(a, b0, b1, acc, nxt + a_addr[0], nxt + a_addr[1], nxt + b_addr[1], nullptr);
    }
    if (nk >= 2) {
      const char* cur = smem + ((nk - 2) & 1) * Shape::STAGE_BYTES;
      const char* nxt = smem + ((nk - 1) & 1) * Shape::STAGE_BYTES;
      LLAMARL_FENCE();
      wide_k_step<TT, Fetch, true, true, false>(a, b1, b0, acc, cur + a_addr[1], nxt + a_addr[0], nxt + b_addr[0], nullptr);
      wide_k_step<TT, Fetch, false, true, false>(a, b0, b1, acc, nxt + a_addr[0], nxt + a_addr[1], nxt + b_addr[1], nullptr);
    }
    if (half_slab_left<BK>(K)) {
      const char* cur = smem + ((nk - 1) & 1) * Shape::STAGE_BYTES;
      LLAMARL_FENCE();
      wide_k_step<TT, Fetch, false, false, false>(a, b1, b0, acc, cur + a_addr[1], nullptr, nullptr, nullptr);
    }
  }
};

// ---- narrow tiles: 256 rows x 128 or 160 columns -----------------------------------------------------------------------
// For few tokens against a large vocabulary, where W streams from HBM: with two slabs resident a slab took the 1.6 us of a
// trip to memory whatever its MFMAs; here three are resident and two in flight.  Wavefronts 0 .. 3 are the left half with
// eight column blocks, 4 .. 7 the right half with nb1 = 2 or none.
// The slots of a k-step for a wavefront with nb column blocks: 4 nb slots, slot t runs block (snake(t), t / 4).
struct KSlots {
  int nb;
  constexpr int barrier() const { return nb >= 6 ? 8 : 4; }
  // where the next k-step's fragment of column block j < nb - 1 is read: the block is done after slot 4 j + 3
  constexpr int column(int j) const { return j == 0 ? barrier() : j == 1 && nb >= 6 ? 9 : 4 * (j + 1); }
  constexpr int row(int i) const { return nb >= 6 ? 10 + 4 * i : nb == 4 ? 5 + 3 * i : 4 + i; }     // ... of row block i
  // load n = 0 .. 7 of the slab after next; first: for eight blocks, see k_step
  constexpr int load(int n, int first) const { return nb == 8 ? first + 2 * n : nb == 4 ? 8 + n : 4 + n / 2; }
};

// One k-step, as k_step with the operands' roles exchanged: the column fragments b have one register set each, the four row
// fragments are double-buffered.  LB: loads of the column operand.
template <typename TT, typename Fetch, int nb, bool BAR, bool NEXT, bool FETCH, int YOUNGER, bool INIT, int LB>
__device__ __forceinline__ void narrow_k_step(typename TT::frag_t (&b)[nb], const typename TT::frag_t (&ac)[4],
                                       typename TT::frag_t (&an)[4], f32x4_t (&acc)[4][nb], const char* pb_cur,
                                       const char* pb_nxt, const char* pa_nxt, const Fetch* sf) {
  typedef typename TT::frag_t frag_t;
  constexpr KSlots S{nb};
#pragma unroll
  for (int t = 0; t < 4 * nb; ++t) {
    const int ib = snake(t), jb = t >> 2;
    if (BAR && t == S.barrier()) {
      wait_vmcnt<YOUNGER>();      // this thread's share of the next slab has landed in LDS
      __syncthreads();            // everyone's has, and everyone is done reading this slab
      LLAMARL_FENCE();
    }
    if (INIT) acc[ib][jb] = f32x4_t{0.f, 0.f, 0.f, 0.f};
    mma(ac[ib], b[jb], acc[ib][jb]);
    LLAMARL_FENCE();
    if (t == 0) {
      b[nb - 1] = *reinterpret_cast<const frag_t*>(pb_cur + (nb - 1) * BLOCK_BYTES);
      LLAMARL_FENCE();
    }
    if (NEXT) {
#pragma unroll
      for (int j = 0; j < nb - 1; ++j)
        if (t == S.column(j)) b[j] = *reinterpret_cast<const frag_t*>(pb_nxt + j * BLOCK_BYTES);
#pragma unroll
      for (int i = 0; i < 4; ++i)
        if (t == S.row(i)) an[i] = *reinterpret_cast<const frag_t*>(pa_nxt + i * BLOCK_BYTES);
      LLAMARL_FENCE();
    }
    if (FETCH) {
#pragma unroll
      for (int n = 0; n < 4 + LB; ++n)
        if (t == S.load(n, 11)) {
          if (n < 4) sf->la->issue_one(sf->ra, sf->dst, n, sf->k0, sf->K, sf->wave, sf->lane);
          else sf->lb->issue_one(sf->rb, sf->dst + SLAB_A_BYTES, n - 4, sf->k0, sf->K, sf->wave, sf->lane);
          LLAMARL_FENCE();
        }
    }
  }
}

template <typename TT>
struct TileGemmNarrow {
  typedef TT Type;
  typedef Shape256Halves Shape;
  typedef typename TT::frag_t frag_t;
  typedef SlabLoader<TT> LoaderA;
  typedef SlabLoader<TT, Shape::BN, Shape::WAVES, Shape::WAVE_N> LoaderB;
  typedef SlabFetch<LoaderA, LoaderB> Fetch;
  static constexpr bool KMAJOR = false;
  static constexpr bool HAS_IDLE = true, HALVES = true;
  static constexpr bool REQUESTS_PAST_K = true;
  static constexpr int BK = 8 * TT::EPC;
  static constexpr int LDS_BYTES = NARROW_LDS_BYTES;
  static constexpr int FIRST_PARTS = 2;        // see TileGemm::issue_first
  static constexpr int COUNTED_STORES = 2;     // see TileGemm::run
  LoaderA la;
  LoaderB lb;
  int K;
  SlabOrder order;
  int nb1;
  __device__ __forceinline__ int width() const { return Shape::WAVE_N + 16 * nb1; }
  __device__ __forceinline__ void set_width(int w) { nb1 = (w - Shape::WAVE_N) / 16; }

  template <bool NEAR>
  __device__ __forceinline__ void setup_gathered(const void* A_tile, int64_t lda, int rowsA, const void* B_base,
                                                 int64_t ldb, int rowsB, int64_t K_, const int (&grow)[LoaderB::ITERS],
                                                 int64_t b_total, int turn) {
    const int lane = threadIdx.x & 63, wave = wave_id();
    K = (int)K_;
    order.init<BK>(K, turn);
    la.init(A_tile, lda, rowsA, wave, lane);
    lb.template init_gathered<NEAR>(B_base, ldb, b_total, grow, rowsB, wave, lane, nb1);
  }
  // per-lane read addresses of block 0: row = lane % 16, chunk 4 ks + lane / 16 of k-step ks, swizzled.  The
  // swizzle depends on the low four row bits only, so block i is the same address + i * BLOCK_BYTES.
  __device__ __forceinline__ static void fragment_addresses(int (&a_addr)[2], int (&b_addr)[2]) {
    const int lane = threadIdx.x & 63, wave = wave_id();
    const int g = lane >> 4, l16 = lane & 15, sw = swizzle(l16);
#pragma unroll
    for (int ks = 0; ks < 2; ++ks) {
      a_addr[ks] = (Shape::wave_row(wave) * Shape::WAVE_M + l16) * SLAB_ROW_BYTES + (((4 * ks + g) ^ sw) * 16);
      b_addr[ks] = SLAB_A_BYTES + (Shape::wave_col(wave) * Shape::WAVE_N + l16) * SLAB_ROW_BYTES + (((4 * ks + g) ^ sw) * 16);
    }
  }
  template <int nb>
  __device__ __forceinline__ static void first_fragments(const char* smem, const int (&a_addr)[2], const int (&b_addr)[2],
                                                         frag_t (&b)[nb], frag_t (&a)[4]) {
    b[0] = *reinterpret_cast<const frag_t*>(smem + b_addr[0]);
#pragma unroll
    for (int i = 0; i < 4; ++i) a[i] = *reinterpret_cast<const frag_t*>(smem + a_addr[0] + i * BLOCK_BYTES);
#pragma unroll
    for (int j = 1; j < nb - 1; ++j) b[j] = *reinterpret_cast<const frag_t*>(smem + b_addr[0] + j * BLOCK_BYTES);
  }

  // Column rows of a slab: 128 by two loads of everyone, 32 by a third of wavefronts 0 .. 3; slabs past K are requested
  // like the others (zeros, no traffic), so that the waits can count.
  template <int nb>
  static constexpr int LB_LOADS = nb == 8 ? 3 : 2;      // the left half is wavefronts 0 .. 3
  template <int nb>
  __device__ __forceinline__ void issue(char* st, int kt) const {
    const int lane = threadIdx.x & 63, wave = wave_id();
    const int k0 = order.k<BK>(kt, K);
    la.issue(st, k0, K, wave, lane);
    const i32x4_t rs = lb.rsrc();
#pragma unroll
    for (int it = 0; it < LB_LOADS<nb>; ++it) lb.issue_one(rs, st + SLAB_A_BYTES, it, k0, K, wave, lane);
  }
  template <int nb>
  __device__ __forceinline__ void issue_first(char* smem, int part) const {      // as issue_first
    if (part < 2) issue<nb>(smem + part * NARROW_STAGE_BYTES, part);
  }
  __device__ __forceinline__ static char* stage(char* smem, int s) { return smem + s * NARROW_STAGE_BYTES; }
  template <int nb>
  __device__ __forceinline__ void run_idle(char* smem) const {
    const int nk = (K + BK - 1) / BK;
    wait_vmcnt0();
    __syncthreads();
    issue<nb>(stage(smem, 2), 2);
    int st = 0;
    for (int kt = 0; kt < nk - 1; ++kt) {
      wait_vmcnt<4 + LB_LOADS<nb>>();
      __syncthreads();
      issue<nb>(stage(smem, st), kt + 3);
      st = st == 2 ? 0 : st + 1;
    }
  }
  template <int nb>
  __device__ __forceinline__ void run(char* smem, f32x4_t (&acc)[4][nb], bool counted) {
    const int lane = threadIdx.x & 63, wave = wave_id();
    const int nk = (K + BK - 1) / BK;
    constexpr int LB = LB_LOADS<nb>;
    int a_addr[2], b_addr[2];
    fragment_addresses(a_addr, b_addr);
    if (counted) wait_vmcnt<COUNTED_STORES>();
    else wait_vmcnt0();
    __syncthreads();
    issue<nb>(stage(smem, 2), 2);      // not earlier: an epilogue may use that stage
    frag_t b[nb], a0[4], a1[4];
    first_fragments<nb>(smem, a_addr, b_addr, b, a0);
    LLAMARL_FENCE();
    narrow_k_step<TT, Fetch, nb, false, true, false, 0, true, LB>(b, a0, a1, acc, smem + b_addr[0], smem + b_addr[1],
                                                               smem + a_addr[1], nullptr);
    int st = 0;
    for (int kt = 0; kt < nk - 1; ++kt) {
      char* cur = stage(smem, st);
      st = st == 2 ? 0 : st + 1;
      const char* nxt = stage(smem, st);
      LLAMARL_FENCE();
      const Fetch sf{&la, &lb, la.rsrc(), lb.rsrc(), cur, order.k<BK>(kt + 3, K), K, wave, lane};
      narrow_k_step<TT, Fetch, nb, true, true, true, 4 + LB, false, LB>(b, a1, a0, acc, cur + b_addr[1], nxt + b_addr[0],
                                                                     nxt + a_addr[0], &sf);
      narrow_k_step<TT, Fetch, nb, false, true, false, 0, false, LB>(b, a0, a1, acc, nxt + b_addr[0], nxt + b_addr[1],
                                                                  nxt + a_addr[1], nullptr);
    }
    if (half_slab_left<BK>(K)) {
      const char* cur = stage(smem, st);
      LLAMARL_FENCE();
      narrow_k_step<TT, Fetch, nb, false, false, false, 0, false, LB>(b, a1, a0, acc, cur + b_addr[1], nullptr, nullptr, nullptr);
    }
  }

};

}  // namespace llamarl
