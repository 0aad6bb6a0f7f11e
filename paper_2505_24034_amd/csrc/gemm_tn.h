// gemm_tn.h -- the same main loop for operands that are K-MAJOR in memory (bf16 only):
//
//   C[m,n] = sum_k At[k,m] * Bt[k,n]        At [K][lda], Bt [K][ldb], rows are k, m / n contiguous
//
// Used for dH = dz W with At = dz^T [V][tokens] (the one orientation the recompute kernel writes) and Bt = W [V][d]
// as the caller holds it: no transposed copy of W and no second orientation of dz are ever made.
//
// gfx950 mapping: a K slab of an operand is 64 k-rows x 256 columns x bf16 = 64 rows of 512 bytes in LDS (32 KB,
// same footprint as the K-contiguous slab).  The 16x16x32 MFMA wants, per lane, 8 consecutive k of ONE column
// (column = lane % 16, k group = lane / 16); in this layout they sit 512 bytes apart.  ds_read_b64_tr_b16 does the
// transposition in the LDS pipe: inside each group of 16 lanes, lane 4j+q loads 8 bytes (4 columns) of k-row j,
// and lane i receives column i of the resulting 4 x 16 block, i.e. 4 consecutive k of its own column.  Two such
// reads (k-rows 8g .. 8g+3 and 8g+4 .. 8g+7 for lane group g) make one MFMA fragment.
//
// Bank conflicts: the 32 lanes served together are two lane groups, i.e. k-rows 8g + 0..3 for two values of g, 32
// bytes of each.  Rows are 512 bytes apart (same banks), so 16-byte slot p of row k holds logical chunk
// p ^ (2 (k & 3) | 8 ((k >> 3) & 1)): the four rows of a group land in four different 32-byte positions and the
// two groups in different bank halves.  As in gemm_nt.h the permutation is applied on the global-address side of
// the LDS-direct loads.
#pragma once
#include "gemm_small.h"

namespace llamarl {

typedef __attribute__((__vector_size__(4 * sizeof(short)))) short s16x4_t;
typedef __attribute__((address_space(3))) s16x4_t* lds_s16x4_ptr;
constexpr int KM_ROW_BYTES = 512;        // one k-row of a slab: 256 columns of bf16

// XOR applied to the 16-byte chunk index of k-row k (see the header)
__device__ __forceinline__ int km_swz(int k) { return 2 * (k & 3) | 8 * ((k >> 3) & 1); }

// One k-major operand stream.  The descriptor is re-based at every slab (a K range can span many GiB) and covers
// exactly the k-rows that are left, so the K tail reads zeros.
struct KMajorLoader {
  uint32_t base_lo, base_hi;   // first k-row of the K range, first column of the tile
  uint32_t row_bytes, col0_bytes;
  uint32_t voff;               // this lane's (k-row inside a 16-row group, logical chunk) byte offset

  // origin = element (first k-row of the range, column col0) of a matrix with ld columns; the tile's first `width`
  // columns are fetched
  __device__ __forceinline__ void init(const void* origin, int64_t ld, int64_t col0, int width, int wave, int lane) {
    const uint64_t p = reinterpret_cast<uint64_t>(origin);
    base_lo = (uint32_t)__builtin_amdgcn_readfirstlane((int)(uint32_t)p);
    base_hi = (uint32_t)__builtin_amdgcn_readfirstlane((int)(uint32_t)(p >> 32));
    row_bytes = (uint32_t)__builtin_amdgcn_readfirstlane((int)(uint32_t)(ld * 2));
    col0_bytes = (uint32_t)__builtin_amdgcn_readfirstlane((int)(uint32_t)(col0 * 2));
    // wave-instruction `it` of wave w fills k-rows 2(it*8 + w), +1; lane l: row +l/32, physical slot l%32.
    // Bits 0, 1 and 3 of the row do not depend on `it`, so one offset serves all four instructions.
    const int r = 2 * wave + (lane >> 5);
    const int c = (lane & 31) ^ km_swz(r);
    voff = c * 8 < width ? (uint32_t)r * row_bytes + (uint32_t)c * 16u : OOB_OFFSET;
  }
  // slab kt of a K range of k_len rows -> lds: the descriptor (uniform) once, then four loads
  struct Slab {
    i32x4_t rs;
    uint32_t lds0;
  };
  __device__ __forceinline__ Slab slab(char* lds, int kt, int k_len) const {
    const int rows_left = k_len - kt * 64;
    // the range ends with the last k-row that is left: counted from column col0, that is col0 bytes short of
    // rows * row_bytes (a tile that overhangs the right edge wraps into the next row, never past the matrix)
    const uint32_t rows = (uint32_t)(rows_left <= 0 ? 0 : (rows_left < 64 ? rows_left : 64));
    const uint32_t records = rows ? rows * row_bytes - col0_bytes : 0u;
    const uint64_t b = (((uint64_t)base_hi << 32) | base_lo) + (uint64_t)kt * 64u * row_bytes;
    Slab sl;
    sl.rs = i32x4_t{(int)(uint32_t)b, (int)((uint32_t)(b >> 32) & 0xffffu), (int)records, 0x00020000};
    sl.lds0 = (uint32_t)(uintptr_t)(__attribute__((address_space(3))) char*)lds;
    return sl;
  }
  __device__ __forceinline__ void issue_one(const Slab& sl, int it, int wave) const {
    lds_dma16(sl.lds0 + (uint32_t)((it * 8 + wave) * 2 * KM_ROW_BYTES), voff, sl.rs, it * 16u * row_bytes);
  }
  __device__ __forceinline__ void issue(char* lds, int kt, int k_len, int wave) const {
    const Slab sl = slab(lds, kt, k_len);
#pragma unroll
    for (int it = 0; it < 4; ++it) issue_one(sl, it, wave);
  }
};

struct TileGemmTN {
  typedef BF16 Type;
  typedef Shape256Halves Shape;
  typedef bf16x8_t frag_t;
  static constexpr bool KMAJOR = true;
  static constexpr bool HAS_IDLE = true, HALVES = true;
  static constexpr int LDS_BYTES = MAINLOOP_LDS_BYTES;
  static constexpr int GROUPS_PER_CU = 1;
  KMajorLoader la, lb;
  int k_len;
  int nb1;                                     // column blocks of the right half: 0, 2, .., 8 (Shape256Halves)
  __device__ __forceinline__ int width() const { return Shape::WAVE_N + 16 * nb1; }

  // At_origin / Bt_origin: element (first k-row of the range, first column of the tile).  Columns past the
  // matrix edge read the neighbouring row's finite values: they only reach output rows / columns nobody stores.
  __device__ __forceinline__ void prefetch(const uint16_t* At_origin, int64_t lda, int64_t a_col0,
                                           const uint16_t* Bt_origin, int64_t ldb, int64_t b_col0, int k_len_,
                                           char* smem) {
    const int lane = threadIdx.x & 63, wave = wave_id();
    k_len = k_len_;
    la.init(At_origin, lda, a_col0, Shape::BM, wave, lane);
    lb.init(Bt_origin, ldb, b_col0, width(), wave, lane);
    la.issue(smem, 0, k_len, wave);
    lb.issue(smem + SLAB_A_BYTES, 0, k_len, wave);
    if (k_len > 64) {
      la.issue(smem + STAGE_BYTES, 1, k_len, wave);
      lb.issue(smem + STAGE_BYTES + SLAB_A_BYTES, 1, k_len, wave);
    }
  }

  // one fragment = 8 k-values of this lane's column: two transposing 8-byte reads, 4 k-rows apart
  __device__ __forceinline__ static frag_t read_frag(const char* p) {
    const s16x4_t lo = __builtin_amdgcn_ds_read_tr16_b64_v4i16(
        (lds_s16x4_ptr)(__attribute__((address_space(3))) void*)const_cast<char*>(p));
    const s16x4_t hi = __builtin_amdgcn_ds_read_tr16_b64_v4i16(
        (lds_s16x4_ptr)(__attribute__((address_space(3))) void*)const_cast<char*>(p + 4 * KM_ROW_BYTES));
    typedef __attribute__((__vector_size__(8 * sizeof(short)))) short s16x8_t;
    const s16x8_t v = {lo[0], lo[1], lo[2], lo[3], hi[0], hi[1], hi[2], hi[3]};
    return __builtin_bit_cast(frag_t, v);
  }

  struct Fetch {     // the eight loads of one slab, issued one per MFMA slot after the barrier
    const KMajorLoader* la;
    const KMajorLoader* lb;
    KMajorLoader::Slab sa, sb;
    int wave;
  };

  // Address of block b's fragment: blocks are 32 bytes (two chunks) apart before the chunk swizzle, which XORs bits
  // 1..3 of the chunk index -- bits the block index occupies too -- so it is an XOR, not an add.  B: the 8 blocks
  // of a wave span bits 1..3 (fx = the whole swizzle).  A: the 4 blocks span bits 1..2 and the wave's position
  // bits 3..4, so bit 3 of the swizzle is folded into the base and fx carries bits 1..2 only.
  __device__ __forceinline__ static const char* blk(const char* base, int b, int fx) { return base + ((b * 32) ^ fx); }

  // The slots (KSlots) with the barrier of a slab's last k-step moved up to slot 4 and the slab loads to the odd slots
  // 5 .. 19.  Every fragment is two LDS instructions here, so the 24 reads of the next slab need the room: barrier at slot
  // 8 / loads from slot 11 measured 3.4 % slower for the dH contraction, barrier at slot 6: 0.8 % slower, at slot 2: 0.5 %
  // slower; loads on even slots (where the fragment reads sit): 4 - 6 % slower.  (The K-contiguous loop does not care:
  // +-0.5 % for the same moves.)
  struct Slots {
    int nb;
    constexpr int barrier() const { return 4; }
    constexpr int column(int j) const { return 4 * (j + 1); }
    constexpr int row(int i) const { return KSlots{nb}.row(i); }
    constexpr int load(int n) const { return nb >= 6 ? 5 + 2 * n : KSlots{nb}.load(n, 0); }
  };
  // One k-step (32 k-rows), as narrow_k_step in gemm_nt.h.  pa / pb: slab base + this lane's row and byte offset for the k-step;
  // fx: the lane's chunk swizzle in bytes.
  template <int nb, bool BAR, bool NEXT, bool FETCH, bool INIT = false>
  __device__ __forceinline__ static void k_step(frag_t (&b)[nb], const frag_t (&ac)[4], frag_t (&an)[4],
                                                f32x4_t (&acc)[4][nb], const char* pb_cur, const char* pb_nxt,
                                                const char* pa_nxt, int fx, int fxa, const Fetch* f) {
    constexpr Slots S{nb};
#pragma unroll
    for (int t = 0; t < 4 * nb; ++t) {
      const int ib = snake(t), jb = t >> 2;
      if (BAR && t == S.barrier()) {      // b[nb - 1], the last read of the slab, was issued at slot 0
        wait_vmcnt0();      // this thread's share of the next slab has landed in LDS
        __syncthreads();    // everyone's has, and everyone is done reading this slab
        LLAMARL_FENCE();
      }
      if (INIT) acc[ib][jb] = f32x4_t{0.f, 0.f, 0.f, 0.f};
      mma(ac[ib], b[jb], acc[ib][jb]);
      LLAMARL_FENCE();
      if (t == 0) {
        b[nb - 1] = read_frag(blk(pb_cur, nb - 1, fx));
        LLAMARL_FENCE();
      }
      if (NEXT) {
#pragma unroll
        for (int j = 0; j < nb - 1; ++j)
          if (t == S.column(j)) b[j] = read_frag(blk(pb_nxt, j, fx));
#pragma unroll
        for (int i = 0; i < 4; ++i)
          if (t == S.row(i)) an[i] = read_frag(blk(pa_nxt, i, fxa));
        LLAMARL_FENCE();
      }
      if (FETCH) {
#pragma unroll
        for (int n = 0; n < 8; ++n)
          if (t == S.load(n)) {
            if (n < 4) f->la->issue_one(f->sa, n, f->wave);
            else f->lb->issue_one(f->sb, n - 4, f->wave);
            LLAMARL_FENCE();
          }
      }
    }
  }

  // as TileGemm::run_idle
  __device__ __forceinline__ void run_idle(char* smem) const {
    const int wave = wave_id();
    const int nk = (k_len + 63) / 64;
    wait_vmcnt0();
    __syncthreads();
    for (int kt = 0; kt < nk - 2; ++kt) {
      char* cur = smem + (kt & 1) * STAGE_BYTES;
      wait_vmcnt0();
      __syncthreads();
      la.issue(cur, kt + 2, k_len, wave);
      lb.issue(cur + SLAB_A_BYTES, kt + 2, k_len, wave);
    }
    if (nk >= 2) {
      wait_vmcnt0();
      __syncthreads();
    }
  }

  template <int nb>                            // column blocks of this wavefront
  __device__ __forceinline__ void run(char* smem, f32x4_t (&acc)[4][nb]) {
    const int lane = threadIdx.x & 63, wave = wave_id();
    const int wm = Shape::wave_row(wave), wn = Shape::wave_col(wave);
    const int nk = (k_len + 63) / 64;

    // lane -> what it LOADS for the transposing read: lane group g = lane / 16 serves k-rows 8g .. 8g+7 of a k-step;
    // inside the group lane 4j+q loads k-row j (the second read: j + 4), columns 4q .. 4q+3 of the 16-column block.
    const int g = lane >> 4, jrow = (lane >> 2) & 3, q4 = lane & 3;
    const int krow = 8 * g + jrow;
    const int fx = km_swz(krow) * 16;                  // same for krow + 4; bit 3 of the k-row is g & 1 in both k-steps
    // block 0 of this wave: chunk (column / 8) before the swizzle, + the 8-byte half the lane's 4 columns sit in
    const int b_off = SLAB_A_BYTES + krow * KM_ROW_BYTES + (wn * Shape::WAVE_N / 8 + (q4 >> 1)) * 16 + (q4 & 1) * 8;
    const int fxa = fx & 0x60;
    const int a_off = krow * KM_ROW_BYTES + ((wm * Shape::WAVE_M * 2) ^ (fx & 0x80)) + (q4 >> 1) * 16 + (q4 & 1) * 8;
    constexpr int KS = 32 * KM_ROW_BYTES;              // bytes between the two k-steps of a slab

    wait_vmcnt0();
    __syncthreads();
    frag_t b[nb], a0[4], a1[4];
    b[0] = read_frag(blk(smem + b_off, 0, fx));
#pragma unroll
    for (int i = 0; i < 4; ++i) a0[i] = read_frag(blk(smem + a_off, i, fxa));
#pragma unroll
    for (int j = 1; j < nb - 1; ++j) b[j] = read_frag(blk(smem + b_off, j, fx));

    // as TileGemm::run
    LLAMARL_FENCE();
    k_step<nb, false, true, false, true>(b, a0, a1, acc, smem + b_off, smem + b_off + KS, smem + a_off + KS, fx, fxa, nullptr);
    for (int kt = 0; kt < nk - 2; ++kt) {
      char* cur = smem + (kt & 1) * STAGE_BYTES;
      const char* nxt = smem + ((kt + 1) & 1) * STAGE_BYTES;
      LLAMARL_FENCE();
      const Fetch f{&la, &lb, la.slab(cur, kt + 2, k_len), lb.slab(cur + SLAB_A_BYTES, kt + 2, k_len), wave};
      k_step<nb, true, true, true>(b, a1, a0, acc, cur + b_off + KS, nxt + b_off, nxt + a_off, fx, fxa, &f);
      k_step<nb, false, true, false>(b, a0, a1, acc, nxt + b_off, nxt + b_off + KS, nxt + a_off + KS, fx, fxa, nullptr);
    }
    if (nk >= 2) {
      const char* cur = smem + ((nk - 2) & 1) * STAGE_BYTES;
      const char* nxt = smem + ((nk - 1) & 1) * STAGE_BYTES;
      LLAMARL_FENCE();
      k_step<nb, true, true, false>(b, a1, a0, acc, cur + b_off + KS, nxt + b_off, nxt + a_off, fx, fxa, nullptr);
      k_step<nb, false, true, false>(b, a0, a1, acc, nxt + b_off, nxt + b_off + KS, nxt + a_off + KS, fx, fxa, nullptr);
    }
    {
      const char* cur = smem + ((nk - 1) & 1) * STAGE_BYTES;
      LLAMARL_FENCE();
      k_step<nb, false, false, false>(b, a1, a0, acc, cur + b_off + KS, nullptr, nullptr, fx, fxa, nullptr);
    }
  }
};

// The same contraction on 128 x 128 or 64 x 64 tiles, for outputs too small to give every CU a 256 x 256 tile: the
// pipeline of TileGemmSmall (several workgroups per CU, counted waits, compiler-scheduled fragments) on k-major slabs.
//
// A k-row of a slab has COLS columns.  128 columns = 256 bytes: all rows start at the same bank, as with 256 columns,
// and the same chunk permutation applies.  64 columns = 128 bytes: odd rows sit in the upper bank half already, so the
// permutation separates rows 0 and 2 of a lane group (bit 1 of the row) and the two groups (bit 3).
template <int COLS>
__device__ __forceinline__ int km_swz_of(int k) {
  static_assert(COLS == 128 || COLS == 64, "");
  return COLS == 128 ? km_swz(k) : (2 * ((k >> 1) & 1) | 4 * ((k >> 3) & 1));
}

template <int COLS, int WAVES>
struct KMajorLoaderSmall {
  static constexpr int ROW_BYTES = COLS * 2, LANES_PER_ROW = COLS / 8, ROWS_PER_LOAD = 64 / LANES_PER_ROW;
  static constexpr int ITERS = 64 / (ROWS_PER_LOAD * WAVES);       // loads of one thread per slab
  static_assert(ITERS * ROWS_PER_LOAD * WAVES == 64 && (ROWS_PER_LOAD * WAVES) % 16 == 0,
                "whole wave-instructions, one permutation for all");
  uint32_t base_lo, base_hi, row_bytes, col0_bytes, voff;

  // as KMajorLoader::init
  __device__ __forceinline__ void init(const void* origin, int64_t ld, int64_t col0, int wave, int lane) {
    const uint64_t p = reinterpret_cast<uint64_t>(origin);
    base_lo = (uint32_t)__builtin_amdgcn_readfirstlane((int)(uint32_t)p);
    base_hi = (uint32_t)__builtin_amdgcn_readfirstlane((int)(uint32_t)(p >> 32));
    row_bytes = (uint32_t)__builtin_amdgcn_readfirstlane((int)(uint32_t)(ld * 2));
    col0_bytes = (uint32_t)__builtin_amdgcn_readfirstlane((int)(uint32_t)(col0 * 2));
    const int r = wave * ROWS_PER_LOAD + lane / LANES_PER_ROW;
    voff = (uint32_t)r * row_bytes + (uint32_t)((lane % LANES_PER_ROW) ^ km_swz_of<COLS>(r)) * 16u;
  }
  // slab kt of a K range of k_len rows; past the range every lane is out of the descriptor's range (zeros, no traffic)
  __device__ __forceinline__ void issue(char* lds, int kt, int k_len, int wave) const {
    const int rows_left = k_len - kt * 64;
    const uint32_t rows = (uint32_t)(rows_left <= 0 ? 0 : (rows_left < 64 ? rows_left : 64));
    const uint32_t records = rows ? rows * row_bytes - col0_bytes : 0u;
    const uint64_t b = (((uint64_t)base_hi << 32) | base_lo) + (rows ? (uint64_t)kt * 64u * row_bytes : 0u);
    const i32x4_t rs = {(int)(uint32_t)b, (int)((uint32_t)(b >> 32) & 0xffffu), (int)records, 0x00020000};
    const uint32_t lds0 = (uint32_t)(uintptr_t)(__attribute__((address_space(3))) char*)lds;
#pragma unroll
    for (int it = 0; it < ITERS; ++it)
      lds_dma16(lds0 + (uint32_t)((it * WAVES + wave) * ROWS_PER_LOAD * ROW_BYTES), voff, rs,
                (uint32_t)(it * WAVES * ROWS_PER_LOAD) * row_bytes);
  }
};

template <typename S, int NSTAGE, int GROUPS_PER_CU_>
struct TileGemmTNSmall {
  typedef BF16 Type;
  typedef S Shape;
  typedef bf16x8_t frag_t;
  typedef KMajorLoaderSmall<S::BM, S::WAVES> LoaderA;
  typedef KMajorLoaderSmall<S::BN, S::WAVES> LoaderB;
  static constexpr bool KMAJOR = true;
  static constexpr bool HAS_IDLE = false, HALVES = false;
  static constexpr int LDS_BYTES = NSTAGE * S::STAGE_BYTES;
  static constexpr int GROUPS_PER_CU = GROUPS_PER_CU_;
  static constexpr int LOADS = LoaderA::ITERS + LoaderB::ITERS;
  LoaderA la;
  LoaderB lb;
  int k_len;
  __device__ __forceinline__ static constexpr int width() { return S::BN; }

  __device__ __forceinline__ void issue(char* stage, int kt) const {
    const int wave = wave_id();
    la.issue(stage, kt, k_len, wave);
    lb.issue(stage + S::SLAB_A_BYTES, kt, k_len, wave);
  }
  __device__ __forceinline__ void prefetch(const uint16_t* At_origin, int64_t lda, int64_t a_col0,
                                           const uint16_t* Bt_origin, int64_t ldb, int64_t b_col0, int k_len_,
                                           char* smem) {
    const int lane = threadIdx.x & 63, wave = wave_id();
    k_len = k_len_;
    la.init(At_origin, lda, a_col0, wave, lane);
    lb.init(Bt_origin, ldb, b_col0, wave, lane);
#pragma unroll
    for (int i = 0; i < NSTAGE - 1; ++i) issue(smem + i * S::STAGE_BYTES, i);
  }

  // two transposing reads, 4 k-rows apart (TileGemmTN::read_frag)
  template <int ROW_BYTES>
  __device__ __forceinline__ static frag_t read_frag(const char* p) {
    const s16x4_t lo = __builtin_amdgcn_ds_read_tr16_b64_v4i16(
        (lds_s16x4_ptr)(__attribute__((address_space(3))) void*)const_cast<char*>(p));
    const s16x4_t hi = __builtin_amdgcn_ds_read_tr16_b64_v4i16(
        (lds_s16x4_ptr)(__attribute__((address_space(3))) void*)const_cast<char*>(p + 4 * ROW_BYTES));
    typedef __attribute__((__vector_size__(8 * sizeof(short)))) short s16x8_t;
    const s16x8_t v = {lo[0], lo[1], lo[2], lo[3], hi[0], hi[1], hi[2], hi[3]};
    return __builtin_bit_cast(frag_t, v);
  }

  __device__ __forceinline__ void run(char* smem, f32x4_t (&acc)[S::MB][S::NB]) {
    const int lane = threadIdx.x & 63, wave = wave_id();
    const int wm = S::wave_row(wave), wn = S::wave_col(wave);
    // lane -> k-row and 8-byte piece it loads for the transposing reads: see TileGemmTN::run
    const int g = lane >> 4, jrow = (lane >> 2) & 3, q4 = lane & 3, krow = 8 * g + jrow;
    int a_off[S::MB], b_off[S::NB];
#pragma unroll
    for (int i = 0; i < S::MB; ++i)
      a_off[i] = krow * LoaderA::ROW_BYTES + (((wm * S::WAVE_M / 8 + 2 * i) ^ km_swz_of<S::BM>(krow)) + (q4 >> 1)) * 16 +
                 (q4 & 1) * 8;
#pragma unroll
    for (int j = 0; j < S::NB; ++j)
      b_off[j] = S::SLAB_A_BYTES + krow * LoaderB::ROW_BYTES +
                 (((wn * S::WAVE_N / 8 + 2 * j) ^ km_swz_of<S::BN>(krow)) + (q4 >> 1)) * 16 + (q4 & 1) * 8;
#pragma unroll
    for (int i = 0; i < S::MB; ++i)
#pragma unroll
      for (int j = 0; j < S::NB; ++j) acc[i][j] = f32x4_t{0.f, 0.f, 0.f, 0.f};
    const int nk = (k_len + 63) / 64;
    wait_vmcnt0();
    __syncthreads();
    int st = 0;
    for (int kt = 0; kt < nk; ++kt) {
      if (kt > 0) {
        wait_vmcnt<LOADS * (NSTAGE - 2)>();
        __syncthreads();
      }
      issue(smem + (st == 0 ? NSTAGE - 1 : st - 1) * S::STAGE_BYTES, kt + NSTAGE - 1);
      const char* cur = smem + st * S::STAGE_BYTES;
#pragma unroll
      for (int ks = 0; ks < 2; ++ks) {
        frag_t a[S::MB], b[S::NB];
#pragma unroll
        for (int j = 0; j < S::NB; ++j) b[j] = read_frag<LoaderB::ROW_BYTES>(cur + b_off[j] + ks * 32 * LoaderB::ROW_BYTES);
#pragma unroll
        for (int i = 0; i < S::MB; ++i) a[i] = read_frag<LoaderA::ROW_BYTES>(cur + a_off[i] + ks * 32 * LoaderA::ROW_BYTES);
#pragma unroll
        for (int i = 0; i < S::MB; ++i)
#pragma unroll
          for (int j = 0; j < S::NB; ++j) mma(a[i], b[j], acc[i][j]);
      }
      st = st == NSTAGE - 1 ? 0 : st + 1;
    }
  }
};

}  // namespace llamarl
