// gemm_small.h -- K-contiguous contraction loops on 128 x 128 and 64 x 64 tiles, C[m,n] = sum_k A[m,k] * B[n,k]: TileGemmSmall
// (bf16) and TileGemmSplit (fp32).
//
// fp32 operands go through the bf16 matrix pipes: every value is written as a sum of three bf16 numbers,
// x = h + m + l (h = bf16(x), m = bf16(x - h), l = bf16(x - h - m): 3 x 8 significant bits, so nothing of a normal fp32
// number is lost), and a product is taken as  hh + hm + mh + mm + hl + lh + ml + lm  in fp32 accumulators.  bf16 products
// are exact in fp32; the term left out, ll, is below 2^-34 of the product (|l| <= 2^-17 of a number's leading power of
// two).  hh is summed apart from the seven small terms, whose rounding errors are 2^-8 smaller, so 32 k cost the main
// accumulator one rounding where eight 16x16x4 fp32 MFMAs cost it eight; a contraction with a single product is within
// 0.506 ulp of it (without ml and lm, up to 2^-24 of the product together, 0.96 ulp; fp32 MFMAs 0.5).  Eight 16x16x32
// bf16 MFMAs take half the time of the eight fp32 ones.
//   - bf16 has fp32's exponents (subnormals are not flushed), but a value below 2^-110 can have bits below 2^-133, the
//     last one of l.  (The gradient of a very unlikely vocabulary row would be such a value, 76 nats under its token's: dz
//     is stored scaled up, dz_scale_for.)
//   - Infinities, NaN and values that round to infinity in bf16 cannot be split (inf - inf): they make the
//     accumulator non-finite, and so does an honest overflow.
// A tile whose operands lost a bit or that has a non-finite sum is contracted again with fp32 MFMAs, whose results it
// keeps.
//
// gfx950 mapping: four wavefronts a tile, two or three workgroups per CU, whose main loops and epilogues cover each other's waits:
// no hand-written slot table.  bf16: 128-byte slab rows with the XOR swizzle of gemm_nt.h, slabs fetched straight into LDS.
// fp32: an operation on the VALU takes 2.4 cycles from the matrix pipe of its SIMD even where another wavefront owns that, and a
// split is 48 of them for 8 x 64 values; so a workgroup splits each value once, in registers on its way to LDS (192 operations a
// slab and wavefront beside 128 MFMAs), where each of the two wavefronts that multiply it did it for itself (384).  The next row
// block's parts are read under this one's MFMAs.  Forward call / dz / dH / dW, every wavefront splitting / now, us: (N, V, d) = (3600,
// 20011, 516) 539 / 591 / 635 / 653 -> 467 / 548 / 551 / 569, (1024, 32000, 2048) - / 927 / 863 / 888 -> - / 813 / 792 / 814, (1000, 3000, 516)
// 46 / 49 / 53 / 52 -> 45 / 47 / 43 / 45, (300, 16400, 260) - / 43 / 48 / 42 -> - / 37 / 43 / 38; the same bits.  (Parts read where they are
// used: 512 for 467; the split of the next slab between the last row block's MFMAs: 496, its loads then have less time;
// v_dot2_f32_bf16 for x - h: not exact; either workgroup of a CU preferred by s_setprio or started later: no change.)
// Relative error against 64 bits over 60 shapes (32 .. 8192 tokens, 300 .. 40000 entries, d 64 .. 2048), fp32 MFMAs / split: logp 7.1e-8
// / 3.1e-8, dH 4.3e-7 / 1.9e-7, dW 2.2e-7 / 1.2e-7, and smaller at every one of them.
#pragma once
#include "gemm_nt.h"

namespace llamarl {

typedef __bf16 bf16x2_t __attribute__((ext_vector_type(2)));
typedef float f32x2_t __attribute__((ext_vector_type(2)));

__device__ __forceinline__ uint32_t pack_bf16(float lo, float hi) {   // v_cvt_pk_bf16_f32: round to nearest even
  f32x2_t v = {lo, hi};
  return __builtin_bit_cast(uint32_t, __builtin_convertvector(v, bf16x2_t));
}

struct Split3 {
  bf16x8_t h, m, l;
};
// lost: bits that l has no room for are collected in its low half (0 as long as every split is exact)
__device__ __forceinline__ Split3 split3(const f32x4_t& x0, const f32x4_t& x1, uint32_t& lost) {
  typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));
  u32x4 h, m, l;
#pragma unroll
  for (int i = 0; i < 4; ++i) {
    const float a = i < 2 ? x0[2 * i] : x1[2 * i - 4], b = i < 2 ? x0[2 * i + 1] : x1[2 * i - 3];
    h[i] = pack_bf16(a, b);
    const float ra = a - __uint_as_float(h[i] << 16), rb = b - __uint_as_float(h[i] & 0xffff0000u);
    m[i] = pack_bf16(ra, rb);
    const float sa = ra - __uint_as_float(m[i] << 16), sb = rb - __uint_as_float(m[i] & 0xffff0000u);
    l[i] = pack_bf16(sa, sb);
    // one instruction, here: left to itself the compiler gathers the 64 parts of a slab first, and spills
    asm("v_or3_b32 %0, %0, %1, %2" : "+v"(lost) : "v"(sa), "v"(sb));
  }
  return Split3{__builtin_bit_cast(bf16x8_t, h), __builtin_bit_cast(bf16x8_t, m), __builtin_bit_cast(bf16x8_t, l)};
}

// bf16.  Same interface as TileGemm (prefetch / setup_gathered, issue_first / run).  NSTAGE slabs are resident, NSTAGE - 1 of
// them in flight; smem must hold LDS_BYTES.
template <typename TT, typename S, int NSTAGE, int GROUPS_PER_CU_>
struct TileGemmSmall {
  typedef TT Type;
  typedef S Shape;
  typedef typename TT::frag_t frag_t;
  typedef SlabLoader<TT, S::BM, S::WAVES, S::WAVE_N> LoaderA;
  typedef SlabLoader<TT, S::BN, S::WAVES, S::WAVE_N> LoaderB;
  static constexpr bool KMAJOR = false;
  static constexpr bool HAS_IDLE = false, HALVES = false;
  static constexpr bool REQUESTS_PAST_K = true;
  static constexpr int BK = 8 * TT::EPC;
  static constexpr int LDS_BYTES = NSTAGE * S::STAGE_BYTES;
  static constexpr int GROUPS_PER_CU = GROUPS_PER_CU_;
  static constexpr int LOADS = LoaderA::ITERS + LoaderB::ITERS;      // of one thread per slab
  LoaderA la;
  LoaderB lb;
  int K;
  __device__ __forceinline__ static constexpr int width() { return S::BN; }

  // A slab past K fetches nothing (every lane out of the descriptor's range: zeros land in LDS), so the number of
  // loads in flight is the same in every iteration and the waits can count them.
  __device__ __forceinline__ void issue(char* stage, int kt) const {
    const int lane = threadIdx.x & 63, wave = wave_id();
    la.issue(stage, kt * BK, K, wave, lane);
    lb.issue(stage + S::SLAB_A_BYTES, kt * BK, K, wave, lane);
  }
  __device__ __forceinline__ void first_slabs(char* smem) const {
#pragma unroll
    for (int i = 0; i < NSTAGE - 1; ++i) issue(smem + i * S::STAGE_BYTES, i);
  }

  template <bool NEAR>
  __device__ __forceinline__ void prefetch(const void* A_tile, int64_t lda, int rowsA, const void* B_tile, int64_t ldb,
                                           int rowsB, int64_t K_, char* smem) {
    const int lane = threadIdx.x & 63, wave = wave_id();
    K = (int)K_;
    la.init(A_tile, lda, rowsA, wave, lane);
    lb.template init<NEAR>(B_tile, ldb, rowsB, wave, lane);
    first_slabs(smem);
  }
  template <bool NEAR>
  __device__ __forceinline__ void setup_gathered(const void* A_tile, int64_t lda, int rowsA, const void* B_base,
                                                 int64_t ldb, int rowsB, int64_t K_, const int (&grow)[LoaderB::ITERS],
                                                 int64_t b_total, int) {
    const int lane = threadIdx.x & 63, wave = wave_id();
    K = (int)K_;
    la.init(A_tile, lda, rowsA, wave, lane);
    lb.template init_gathered<NEAR>(B_base, ldb, b_total, grow, rowsB, wave, lane);
  }
  static constexpr int FIRST_PARTS = 1;
  __device__ __forceinline__ void issue_first(char* smem, int) const { first_slabs(smem); }

  __device__ __forceinline__ static void clear(f32x4_t (&acc)[S::MB][S::NB]) {
#pragma unroll
    for (int i = 0; i < S::MB; ++i)
#pragma unroll
      for (int j = 0; j < S::NB; ++j) acc[i][j] = f32x4_t{0.f, 0.f, 0.f, 0.f};
  }

  // the MFMAs of one slab; a_addr / b_addr: this lane's chunk of block 0 in either half of a slab row
  __device__ __forceinline__ static void slab(const char* st, const int (&a_addr)[2], const int (&b_addr)[2],
                                              f32x4_t (&acc)[S::MB][S::NB]) {
#pragma unroll
    for (int ks = 0; ks < 2; ++ks) {
      frag_t b[S::NB], a[S::MB];
#pragma unroll
      for (int j = 0; j < S::NB; ++j) b[j] = *reinterpret_cast<const frag_t*>(st + b_addr[ks] + j * BLOCK_BYTES);
#pragma unroll
      for (int i = 0; i < S::MB; ++i) a[i] = *reinterpret_cast<const frag_t*>(st + a_addr[ks] + i * BLOCK_BYTES);
#pragma unroll
      for (int i = 0; i < S::MB; ++i)
#pragma unroll
        for (int j = 0; j < S::NB; ++j) mma(a[i], b[j], acc[i][j]);
    }
  }

  __device__ __forceinline__ void run(char* smem, f32x4_t (&acc)[S::MB][S::NB]) {
    const int lane = threadIdx.x & 63, wave = wave_id();
    const int wm = S::wave_row(wave), wn = S::wave_col(wave);
    const int g = lane >> 4, l16 = lane & 15, sw = swizzle(l16);
    int a_addr[2], b_addr[2];
#pragma unroll
    for (int ks = 0; ks < 2; ++ks) {
      a_addr[ks] = (wm * S::WAVE_M + l16) * SLAB_ROW_BYTES + (((4 * ks + g) ^ sw) * 16);
      b_addr[ks] = S::SLAB_A_BYTES + (wn * S::WAVE_N + l16) * SLAB_ROW_BYTES + (((4 * ks + g) ^ sw) * 16);
    }
    clear(acc);
    const int nk = (K + BK - 1) / BK;
    wait_vmcnt0();                     // the first slabs (and stores of a previous epilogue, which may sit between)
    __syncthreads();
    int st = 0;                        // stage of slab kt
    for (int kt = 0; kt < nk; ++kt) {
      if (kt > 0) {
        wait_vmcnt<LOADS * (NSTAGE - 2)>();      // this thread's share of slab kt has landed
        __syncthreads();                         // everyone's has, and everyone is done with slab kt - 1
      }
      // slab kt - 1's stage is free now
      issue(smem + (st == 0 ? NSTAGE - 1 : st - 1) * S::STAGE_BYTES, kt + NSTAGE - 1);
      slab(smem + st * S::STAGE_BYTES, a_addr, b_addr, acc);
      st = st == NSTAGE - 1 ? 0 : st + 1;
    }
  }
};

// fp32 on 128 x 128 and 64 x 64 tiles, see the header.  A slab (32 k) goes through registers: a wavefront loads 16-row blocks of
// one operand (half of the wavefronts A, half B), splits them and writes the three parts to LDS as the fragments the MFMAs
// read, 16 bytes a lane.
// STAGES: 2 where LDS has room for the parts of two slabs in every workgroup (64 x 64 tiles, few of them: a chain of slabs with
// nothing to cover it).  The next slab is split and written behind this one's fragment reads, and a slab has one barrier instead of
// two: (N, V, d), fp32, us, backward (100, 5000, 1024) 88.6 / 80.3, (256, 1024, 256) 30.9 / 28.9, (512, 2048, 512) 59.5 / 55.1; log-probs 38.4 /
// 35.5, 17.8 / 17.1, 25.1 / 23.6.  (Loads two or three slabs ahead gained nothing on that; on 128 x 128 tiles they spill: 467 -> 990 us.)
template <typename S, int GROUPS_PER_CU_, int STAGES>
struct TileGemmSplit {
  typedef F32 Type;
  typedef S Shape;
  static constexpr bool KMAJOR = false;
  static constexpr bool HAS_IDLE = false, HALVES = false;
  static constexpr bool REQUESTS_PAST_K = false;
  static constexpr int BK = 32;
  static constexpr int BLOCKS_A = S::BM / 16, BLOCKS = (S::BM + S::BN) / 16, PER = BLOCKS / S::WAVES;      // of a wavefront
  static_assert(BLOCKS % S::WAVES == 0 && BLOCKS_A % PER == 0, "a wavefront's blocks are of one operand");
  static constexpr int FRAG_BYTES = 1024, SPLIT_BYTES = 3 * FRAG_BYTES;
  static constexpr int STAGE_BYTES = BLOCKS * SPLIT_BYTES, LDS_BYTES = STAGES * STAGE_BYTES + 16;      // + a flag (redo this tile)
  static constexpr int GROUPS_PER_CU = GROUPS_PER_CU_;
  struct Rows {                                                      // which tile rows a lane fetches, see SlabLoader
    static constexpr int ITERS = PER;
    template <bool NEAR>
    __device__ __forceinline__ static int lane_tile_row(int it, int wave, int lane, int nb) {
      return tile_row_of<NEAR, S::WAVE_N>(max((wave * PER + it - BLOCKS_A) * 16 + (lane & 15), 0), nb);
    }
  } lb;
  uint64_t base;          // of this wavefront's operand
  uint32_t bytes;
  uint32_t voff[PER];     // byte offset of (row, chunk lane / 16)
  int K;
  float unscale;          // run<true> only
  __device__ __forceinline__ static constexpr int width() { return S::BN; }
  __device__ __forceinline__ static bool holds_a(int wave) { return wave * PER < BLOCKS_A; }

  __device__ __forceinline__ void set_rows(const void* p, uint32_t size, int it, int row, bool valid, uint32_t row_bytes, int lane) {
    base = reinterpret_cast<uint64_t>(p);
    bytes = size;
    voff[it] = valid ? (uint32_t)row * row_bytes + (uint32_t)(lane >> 4) * 16u : OOB_OFFSET;
  }
  __device__ __forceinline__ void set_a(const void* A_tile, int64_t lda, int rowsA, int wave, int lane) {
    const uint32_t row_bytes = (uint32_t)(lda * 4);
#pragma unroll
    for (int it = 0; it < PER; ++it) {
      const int row = (wave * PER + it) * 16 + (lane & 15);
      set_rows(A_tile, row_bytes * (uint32_t)rowsA, it, row, row < rowsA, row_bytes, lane);
    }
  }
  template <bool NEAR>
  __device__ __forceinline__ void prefetch(const void* A_tile, int64_t lda, int rowsA, const void* B_tile, int64_t ldb,
                                           int rowsB, int64_t K_, char*) {
    int tid = threadIdx.x;                           // opaque per tile: what depends on the lane alone is not kept for the next
    asm volatile("" : "+v"(tid));                    // one, which took two or three registers more than there are (scratch)
    const int lane = tid & 63, wave = wave_id();
    K = (int)K_;
    if (holds_a(wave)) {                             // wave-uniform
      set_a(A_tile, lda, rowsA, wave, lane);
    } else {
      const uint32_t row_bytes = (uint32_t)(ldb * 4);
#pragma unroll
      for (int it = 0; it < PER; ++it) {
        const int row = Rows::template lane_tile_row<NEAR>(it, wave, lane, S::NB);
        set_rows(B_tile, row_bytes * (uint32_t)rowsB, it, row, row < rowsB, row_bytes, lane);
      }
    }
  }
  template <bool NEAR>
  __device__ __forceinline__ void setup_gathered(const void* A_tile, int64_t lda, int rowsA, const void* B_base,
                                                 int64_t ldb, int rowsB, int64_t K_, const int (&grow)[PER],
                                                 int64_t b_total, int) {
    const int lane = threadIdx.x & 63, wave = wave_id();
    K = (int)K_;
    if (holds_a(wave)) {
      set_a(A_tile, lda, rowsA, wave, lane);
    } else {
      const uint32_t row_bytes = (uint32_t)(ldb * 4);
#pragma unroll
      for (int it = 0; it < PER; ++it)
        set_rows(B_base, row_bytes * (uint32_t)b_total, it, grow[it],
                 Rows::template lane_tile_row<NEAR>(it, wave, lane, S::NB) < rowsB, row_bytes, lane);
    }
  }
  static constexpr int FIRST_PARTS = 0;              // the other workgroups of the CU cover a tile's first slab
  __device__ __forceinline__ void issue_first(char*, int) const {}

  // A lane's 2 x 4 elements of its row in each block: chunks lane / 16 and lane / 16 + 4 of the slab.  Which k sits at which
  // position of a fragment does not matter as long as both operands agree.
  __device__ __forceinline__ void load(int k0, f32x4_t (&x)[PER][2]) const {
    const uint64_t b = ((uint64_t)(uint32_t)__builtin_amdgcn_readfirstlane((int)(uint32_t)(base >> 32)) << 32) |
                       (uint32_t)__builtin_amdgcn_readfirstlane((int)(uint32_t)base);
    const __amdgpu_buffer_rsrc_t rs =
        __builtin_amdgcn_make_buffer_rsrc(reinterpret_cast<void*>(b), 0, __builtin_amdgcn_readfirstlane((int)bytes), 0x00020000);
    const int left = K - k0 - 4 * (int)((threadIdx.x & 63) >> 4);      // of this lane's first chunk on
#pragma unroll
    for (int it = 0; it < PER; ++it)
#pragma unroll
      for (int c = 0; c < 2; ++c)
        x[it][c] = __builtin_bit_cast(f32x4_t, __builtin_amdgcn_raw_buffer_load_b128(
                                                   rs, left > 16 * c ? voff[it] + 64u * c : OOB_OFFSET, k0 * 4, 0));
  }
  // LDS traffic of this wavefront is over, and everyone's.  (Not __syncthreads(): the loads of the next slab stay in flight.)
  __device__ __forceinline__ static void lds_barrier() { asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory"); }

  __device__ __forceinline__ static void clear(f32x4_t (&acc)[S::MB][S::NB]) {
#pragma unroll
    for (int i = 0; i < S::MB; ++i)
#pragma unroll
      for (int j = 0; j < S::NB; ++j) acc[i][j] = f32x4_t{0.f, 0.f, 0.f, 0.f};
  }
  __device__ __forceinline__ static bf16x8_t frag(const char* block, int part, int lane) {
    return *reinterpret_cast<const bf16x8_t*>(block + part * FRAG_BYTES + lane * 16);
  }

  // low: sums of the seven small terms of split products
  __device__ __forceinline__ void split_slabs(char* smem, f32x4_t (&acc)[S::MB][S::NB], f32x4_t (&low)[S::MB][S::NB],
                                              uint32_t& lost) const {
    const int lane = threadIdx.x & 63, wave = wave_id(), nk = (K + BK - 1) / BK;
    const int pa = S::wave_row(wave) * S::MB * SPLIT_BYTES, pb = (BLOCKS_A + S::wave_col(wave) * S::NB) * SPLIT_BYTES;
    const int mine = wave * PER * SPLIT_BYTES + lane * 16;
    f32x4_t x[PER][2];
    Split3 sp[PER];
    auto split = [&] {
#pragma unroll
      for (int it = 0; it < PER; ++it) sp[it] = split3(x[it][0], x[it][1], lost);
    };
    auto write = [&](char* st) {
#pragma unroll
      for (int it = 0; it < PER; ++it) {
        *reinterpret_cast<bf16x8_t*>(st + mine + it * SPLIT_BYTES) = sp[it].h;
        *reinterpret_cast<bf16x8_t*>(st + mine + it * SPLIT_BYTES + FRAG_BYTES) = sp[it].m;
        *reinterpret_cast<bf16x8_t*>(st + mine + it * SPLIT_BYTES + 2 * FRAG_BYTES) = sp[it].l;
      }
    };
    auto parts = [&](const char* q) { return Split3{frag(q, 0, lane), frag(q, 1, lane), frag(q, 2, lane)}; };
    // j innermost: consecutive MFMAs do not wait for each other's accumulator
    auto products = [&](const Split3& a, const Split3 (&b)[S::NB], int i) {
#pragma unroll
      for (int j = 0; j < S::NB; ++j) mma(a.m, b[j].l, low[i][j]);
#pragma unroll
      for (int j = 0; j < S::NB; ++j) mma(a.l, b[j].m, low[i][j]);
#pragma unroll
      for (int j = 0; j < S::NB; ++j) mma(a.l, b[j].h, low[i][j]);
#pragma unroll
      for (int j = 0; j < S::NB; ++j) mma(a.h, b[j].l, low[i][j]);
#pragma unroll
      for (int j = 0; j < S::NB; ++j) mma(a.m, b[j].m, low[i][j]);
#pragma unroll
      for (int j = 0; j < S::NB; ++j) mma(a.m, b[j].h, low[i][j]);
#pragma unroll
      for (int j = 0; j < S::NB; ++j) mma(a.h, b[j].m, low[i][j]);
#pragma unroll
      for (int j = 0; j < S::NB; ++j) mma(a.h, b[j].h, acc[i][j]);
    };
    load(0, x);
    if constexpr (STAGES == 2) {
      static_assert(S::MB == 1, "all parts of a slab are read before its products");
      split();
      write(smem);
      if (nk > 1) load(BK, x);
      lds_barrier();
      char *cur = smem, *other = smem + STAGE_BYTES;
      for (int kt = 0; kt < nk; ++kt) {
        Split3 b[S::NB];
#pragma unroll
        for (int j = 0; j < S::NB; ++j) b[j] = parts(cur + pb + j * SPLIT_BYTES);
        const Split3 a = parts(cur + pa);
        LLAMARL_FENCE();
        if (kt + 1 < nk) {                             // everyone was done with that stage at the last barrier
          split();
          write(other);
          if (kt + 2 < nk) load((kt + 2) * BK, x);
        }
        LLAMARL_FENCE();
        products(a, b, 0);
        lds_barrier();
        char* t = cur;
        cur = other;
        other = t;
      }
    } else {
      for (int kt = 0; kt < nk; ++kt) {
        split();
        lds_barrier();                                 // everyone is done with the previous slab's parts
        write(smem);
        if (kt + 1 < nk) load((kt + 1) * BK, x);
        lds_barrier();
        Split3 b[S::NB];
  #pragma unroll
        for (int j = 0; j < S::NB; ++j) b[j] = parts(smem + pb + j * SPLIT_BYTES);
        // The next row block is read under this one's MFMAs; left to itself the compiler reads it where it is used.
        Split3 next = parts(smem + pa);
  #pragma unroll
        for (int i = 0; i < S::MB; ++i) {
          const Split3 a = next;
          LLAMARL_FENCE();
          if (i + 1 < S::MB) next = parts(smem + pa + (i + 1) * SPLIT_BYTES);
          LLAMARL_FENCE();
          products(a, b, i);
          LLAMARL_FENCE();
        }
      }
    }
  }
  // the operands' own MFMAs, A times a_factor; a block takes two fragments of LDS
  __device__ __forceinline__ void native_slabs(char* smem, f32x4_t (&acc)[S::MB][S::NB], float a_factor) const {
    const int lane = threadIdx.x & 63, wave = wave_id(), nk = (K + BK - 1) / BK;
    const float factor = holds_a(wave) ? a_factor : 1.f;
    auto at = [&](int block, int c) { return reinterpret_cast<f32x4_t*>(smem + (block * 2 + c) * FRAG_BYTES + lane * 16); };
    for (int kt = 0; kt < nk; ++kt) {
      f32x4_t x[PER][2];
      load(kt * BK, x);
      lds_barrier();
#pragma unroll
      for (int it = 0; it < PER; ++it)
#pragma unroll
        for (int c = 0; c < 2; ++c) *at(wave * PER + it, c) = x[it][c] * factor;
      lds_barrier();
#pragma unroll
      for (int c = 0; c < 2; ++c)
#pragma unroll
        for (int i = 0; i < S::MB; ++i) {
          const f32x4_t a = *at(S::wave_row(wave) * S::MB + i, c);
#pragma unroll
          for (int j = 0; j < S::NB; ++j) mma(a, *at(BLOCKS_A + S::wave_col(wave) * S::NB + j, c), acc[i][j]);
        }
    }
  }

  // A_SCALED: A holds its values divided by `unscale`, a power of two; the sums come out unscaled.  The native pass
  // unscales the operand itself: what it is there for may be a sum that only overflows scaled.
  template <bool A_SCALED = false>
  __device__ __forceinline__ void run(char* smem, f32x4_t (&acc)[S::MB][S::NB]) {
    const float factor = A_SCALED ? unscale : 1.f;
    int* redo = reinterpret_cast<int*>(smem + STAGES * STAGE_BYTES);
    if (threadIdx.x == 0) *redo = 0;
    wait_vmcnt0();                                   // token words (TokenWords) are there after the first barrier
    f32x4_t low[S::MB][S::NB];
    uint32_t lost = 0;
    clear(acc);
    clear(low);
    split_slabs(smem, acc, low, lost);
    bool bad = (lost & 0xffffu) != 0;
#pragma unroll
    for (int i = 0; i < S::MB; ++i)
#pragma unroll
      for (int j = 0; j < S::NB; ++j)
#pragma unroll
        for (int r = 0; r < 4; ++r) {
          acc[i][j][r] += low[i][j][r];
          bad |= !(fabsf(acc[i][j][r]) < INFINITY);
          if constexpr (A_SCALED) acc[i][j][r] *= factor;
        }
    if (bad) *redo = 1;
    __syncthreads();
    if (*redo) {                                     // workgroup-uniform
      clear(acc);
      native_slabs(smem, acc, factor);
    }
  }
};

}  // namespace llamarl
