// gemm_small.h -- K-contiguous contraction loop on 128 x 128 and 64 x 64 tiles, C[m,n] = sum_k A[m,k] * B[n,k].
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
// gfx950 mapping: four wavefronts, 128-byte slab rows with the XOR swizzle of gemm_nt.h, slabs fetched straight into
// LDS.  The tiles are small enough for two or more workgroups per CU, whose main loops, splits and epilogues cover
// each other's waits: the loop needs no hand-written slot table.  Bound by the VALU work of the splits (48 operations
// per fragment, 8 fragments per 128 MFMAs of a wavefront) beside the MFMAs.  Measured against a 256 x 256 loop of
// 16x16x4 fp32 MFMAs, per contraction of (N, V, d): (4096, 20011, 516) 690 - 930 -> 630 - 705 us, (1024, 32000, 2048)
// 940 - 1020 -> 830 - 885 us (without ml and lm 545 - 585 and 705 - 750, with them but without `lost` 620 - 680 and
// 820 - 865); (256, 1024, 256) on 64 x 64 tiles 45 - 97 -> 15 - 18 us.  Relative error against 64 bits over 60 shapes
// (32 .. 8192 tokens, 300 .. 40000 entries, d 64 .. 2048): logp 7.1e-8 -> 3.1e-8, dH 4.3e-7 -> 1.9e-7, dW 2.2e-7 ->
// 1.2e-7, and smaller than before at every one of them.
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

// Same interface as TileGemm (prefetch / setup_gathered, issue_first / run).  NSTAGE slabs are resident, NSTAGE - 1 of them in
// flight; smem must hold LDS_BYTES.
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
  static constexpr int LDS_BYTES = NSTAGE * S::STAGE_BYTES + 16;     // + a flag (fp32: redo this tile)
  static constexpr int GROUPS_PER_CU = GROUPS_PER_CU_;
  static constexpr int LOADS = LoaderA::ITERS + LoaderB::ITERS;      // of one thread per slab
  LoaderA la;
  LoaderB lb;
  int K;
  __device__ __forceinline__ static constexpr int width() { return S::BN; }
  float unscale;     // run<true> only

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

  // the MFMAs of one slab; a_addr / b_addr: this lane's chunk of block 0 in either half of a slab row.
  // low: sums of the seven small terms of split products; lost: see split3.  SPLIT = false: the operands' own MFMAs, A
  // times a_factor
  template <bool SPLIT>
  __device__ __forceinline__ static void slab(const char* st, const int (&a_addr)[2], const int (&b_addr)[2],
                                              f32x4_t (&acc)[S::MB][S::NB], f32x4_t (&low)[S::MB][S::NB], uint32_t& lost,
                                              float a_factor) {
    if constexpr (sizeof(typename TT::store_t) == 2) {
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
    } else if constexpr (!SPLIT) {
#pragma unroll
      for (int ks = 0; ks < 2; ++ks)
#pragma unroll
        for (int i = 0; i < S::MB; ++i) {
          frag_t a = *reinterpret_cast<const frag_t*>(st + a_addr[ks] + i * BLOCK_BYTES);
#pragma unroll
          for (int r = 0; r < 4; ++r) a[r] *= a_factor;
#pragma unroll
          for (int j = 0; j < S::NB; ++j)
            mma(a, *reinterpret_cast<const frag_t*>(st + b_addr[ks] + j * BLOCK_BYTES), acc[i][j]);
        }
    } else {
      // The 32 k of a slab are one k-step of the 16x16x32 MFMA.  Which k sits at which position of the fragment does
      // not matter as long as both operands agree: a lane takes the chunks of the two conflict-free reads.
      Split3 b[S::NB];
#pragma unroll
      for (int j = 0; j < S::NB; ++j)
        b[j] = split3(*reinterpret_cast<const frag_t*>(st + b_addr[0] + j * BLOCK_BYTES),
                      *reinterpret_cast<const frag_t*>(st + b_addr[1] + j * BLOCK_BYTES), lost);
#pragma unroll
      for (int i = 0; i < S::MB; ++i) {
        const Split3 a = split3(*reinterpret_cast<const frag_t*>(st + a_addr[0] + i * BLOCK_BYTES),
                                *reinterpret_cast<const frag_t*>(st + a_addr[1] + i * BLOCK_BYTES), lost);
        // j innermost: consecutive MFMAs do not wait for each other's accumulator
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
      }
    }
  }

  // the K loop; the first slabs are on their way
  template <bool SPLIT>
  __device__ __forceinline__ void slabs(char* smem, const int (&a_addr)[2], const int (&b_addr)[2],
                                        f32x4_t (&acc)[S::MB][S::NB], f32x4_t (&low)[S::MB][S::NB], uint32_t& lost,
                                        float a_factor) const {
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
      slab<SPLIT>(smem + st * S::STAGE_BYTES, a_addr, b_addr, acc, low, lost, a_factor);
      st = st == NSTAGE - 1 ? 0 : st + 1;
    }
  }

  // A_SCALED (fp32): A holds its values divided by `unscale`, a power of two; the sums come out unscaled.  The native pass
  // unscales the operand itself: what it is there for may be a sum that only overflows scaled.
  template <bool A_SCALED = false>
  __device__ __forceinline__ void run(char* smem, f32x4_t (&acc)[S::MB][S::NB]) {
    constexpr bool SPLIT = sizeof(typename TT::store_t) == 4;
    const float factor = A_SCALED ? unscale : 1.f;
    const int lane = threadIdx.x & 63, wave = wave_id();
    const int wm = S::wave_row(wave), wn = S::wave_col(wave);
    const int g = lane >> 4, l16 = lane & 15, sw = swizzle(l16);
    int a_addr[2], b_addr[2];
#pragma unroll
    for (int ks = 0; ks < 2; ++ks) {
      a_addr[ks] = (wm * S::WAVE_M + l16) * SLAB_ROW_BYTES + (((4 * ks + g) ^ sw) * 16);
      b_addr[ks] = S::SLAB_A_BYTES + (wn * S::WAVE_N + l16) * SLAB_ROW_BYTES + (((4 * ks + g) ^ sw) * 16);
    }
    int* redo = reinterpret_cast<int*>(smem + NSTAGE * S::STAGE_BYTES);
    if (SPLIT && threadIdx.x == 0) *redo = 0;
    f32x4_t low[S::MB][S::NB];
    uint32_t lost = 0;
    clear(acc);
    clear(low);
    slabs<SPLIT>(smem, a_addr, b_addr, acc, low, lost, 1.f);
    if constexpr (SPLIT) {
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
      wait_vmcnt0();                   // slabs past K that are still in flight would overwrite the ones fetched below
      __syncthreads();
      if (*redo) {                     // workgroup-uniform
        clear(acc);
        first_slabs(smem);
        slabs<false>(smem, a_addr, b_addr, acc, low, lost, factor);
      }
    }
  }
};

}  // namespace llamarl
