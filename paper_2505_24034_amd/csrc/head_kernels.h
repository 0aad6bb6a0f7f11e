// head_kernels.h -- the four contractions of the path and their fused epilogues.
//
//   k_fwd_partials   logits tile -> per-(vocab tile, token) online-softmax partial (max, sum of exp) and the
//                    target logit: the [N,V] logits never leave the accumulators (paper Sec. 6: log pi(y_t|.))
//   k_merge_logp     partials -> lse[t], logp[t]
//   k_bwd_dz         recomputed logits tile -> dz = g * coef * (onehot - softmax), written in both orientations
//   k_gemm_store     plain contraction with a store epilogue: dW = dz^T H (K-contiguous operands) and
//                    dH = dz W (k-major operands: dz^T as written, W as the caller holds it; bf16)
//   k_gemm_store_pair   both of them, where neither is on 256-tiles;  k_reduce_tail, k_reduce_tail_pair: sums of split tiles
//   k_transpose      [R,C] -> [C,R] with zero padding and row gather (H^T panel of the active tokens)
//   k_compact_rows   ascending list of active token rows (the backward's is part of k_bwd_setup)
//   k_bwd_setup      the backward's list, zeroed inactive dH rows, fp32: W^T, and H^T of up to SETUP_HT_ROWS rows
//
// In the two logits kernels the MFMA "row" operand is W (vocab) and the "column" operand is H (tokens): an
// accumulator lane then holds ONE token per column block (column = lane % 16) and 4 vocab entries per 16x16
// block, 32 per token over the wave's 8 row blocks, so the softmax reductions over the vocabulary run inside the
// lane's own registers and finish with two cross-lane steps (lane groups l/16 hold different rows).
//
// Every kernel is a template over its main loop G (TileGemm, TileGemmSmall, TileGemmTN), which brings element type,
// tile shape and LDS size; the rules of tile_rules.h pick the loop.
#pragma once
#include "gemm_nt.h"
#include "gemm_small.h"
#include "gemm_tn.h"

#include <type_traits>

namespace llamarl {

constexpr float LOG2E = 1.4426950408889634f;

// Row pitch (elements) of the two panels that live in list-position space, dz^T [V][.] and H^T [d][.]: the number
// of active rows rounded up to 64, made an ODD multiple of 64.  It is derived on the device from the active count,
// so the panels are as narrow as the batch's valid tokens allow (the k-major dH contraction walks one row pitch per
// k: a pitch sized for all N rows spreads every 64-row slab over 2 MiB of address space), and an odd multiple of
// 128 bytes never lines rows up on a power-of-two stride.  The workspace is sized for packed_pitch(N).
__host__ __device__ __forceinline__ int64_t packed_pitch(int64_t n_rows) {
  const int64_t p = (n_rows + 63) / 64;
  return ((p & 1) ? p : p + 1) * 64;
}
constexpr int STORE_LOAD_SLOT = 9;      // first slab-load slot of the K-contiguous store contraction (see k_step)
// Patch rows of dW (see PATCH_ROWS_LOGITS): 8 (4: +1.6 %, 2: +5 %); dH: see PATCH_ROWS_KMAJOR.
constexpr int PATCH_ROWS_STORE = 8;
// dH on k-major operands, whole tiles of K = V, when the output is at most 16 tiles wide (d <= 4096): 16 x 2
// patches (8 x 4: +0.8 %, 4 x 8: +1.7 %).  Wider outputs (d = 8192, 16384) keep 8 x 4 (16 x 2: +2 - 3 % there).
constexpr int PATCH_ROWS_KMAJOR = 16;

typedef unsigned int u32x2_t __attribute__((ext_vector_type(2)));
// v_exp_f32 without the denormal-range fix-up of exp2f(): arguments here are <= 0 up to rounding, results that
// underflow are exact zeros in the sums they feed.
__device__ __forceinline__ float fast_exp2(float x) { return __builtin_amdgcn_exp2f(x); }
// Four values over the four lane groups l / 16, without the LDS pipe.  v_permlane16_swap / v_permlane32_swap exchange the odd
// 16-lane rows of one register with the even ones of another (the upper half of one with the lower of the other): combining
// the two registers then combines neighbouring rows of BOTH values in one instruction, and after two such steps row g holds
// value g over all rows.
struct Swapped {
  float a, b;
};
__device__ __forceinline__ Swapped swap16(float x, float y) {      // {x0 y0 x2 y2}, {x1 y1 x3 y3}
  const auto p = __builtin_amdgcn_permlane16_swap(__float_as_uint(x), __float_as_uint(y), false, false);
  return {__uint_as_float(p[0]), __uint_as_float(p[1])};
}
__device__ __forceinline__ Swapped swap32(float x, float y) {      // {x0 x1 y0 y1}, {x2 x3 y2 y3}
  const auto p = __builtin_amdgcn_permlane32_swap(__float_as_uint(x), __float_as_uint(y), false, false);
  return {__uint_as_float(p[0]), __uint_as_float(p[1])};
}
template <typename F>
__device__ __forceinline__ float rows_combine(const float (&v)[4], F f) {
  const Swapped p = swap16(v[0], v[1]), q = swap16(v[2], v[3]);
  const Swapped r = swap32(f(p.a, p.b), f(q.a, q.b));
  return f(r.a, r.b);
}
__device__ __forceinline__ void rows_spread(float x, float (&v)[4]) {      // v[g] = row g of x, in every row
  const Swapped p = swap16(x, x), q = swap32(p.a, p.a), r = swap32(p.b, p.b);
  v[0] = q.a;
  v[1] = r.a;
  v[2] = q.b;
  v[3] = r.b;
}

// second launch bound: wavefronts per SIMD that the register allocation has to leave room for
template <typename G>
constexpr int MIN_WAVES = G::GROUPS_PER_CU * G::Shape::WAVES / 4;

struct FwdArgs {
  const void* H;
  const void* W;
  const int32_t* targets;
  int64_t N, d, V;        // V: rows of W as passed (the whole vocabulary, or a shard's slice of it)
  int64_t v_off;          // vocabulary index of row 0 of W (0 unless W is a slice): targets are global indices
  int tiles_v;            // tiles over the vocabulary (MFMA rows)
  int64_t n_pad;          // row stride of the partial arrays
  float* part_m;          // [tiles_v][n_pad] max of the tile's logits of a token
  float* part_s;          // [tiles_v][n_pad] sum of exp(logit - max)
  float* zt;              // [n_pad] target logit, written by the one tile that holds vocab row y_t
  const int32_t* rows;    // [n_act] active token rows, ascending: position p of the compacted list is token rows[p]
  const int32_t* n_act;   // device scalar
};  // partials and zt are indexed by compacted position, not by token

typedef TileGemm<BF16, 11, 2, true> Logits256;      // counted: the two stores of a token's partials
typedef TileGemm<BF16, 11, 2, true, SlabOrder> Logits256Turned;
typedef TileGemm<BF16, 11, 2, true, SlabRing> Logits256Ring;
typedef TileGemmWide<BF16> LogitsWide;
// zeros from an opaque register: as constants the compiler sets them ahead of the branch, for every tile
template <int M, int N>
__device__ __forceinline__ void clear(f32x4_t (&acc)[M][N]) {
  float z = 0.f;
  asm volatile("" : "+v"(z));
#pragma unroll
  for (int i = 0; i < M; ++i)
#pragma unroll
    for (int j = 0; j < N; ++j) acc[i][j] = f32x4_t{z, z, z, z};
}
// One tile's main loop; a wavefront with no part in the tile only takes part in its loads (256-row loops).  nb: its column
// blocks; counted: the loop's COUNTED_STORES were issued since the tile was fetched (TileGemm::run).
template <typename G, int nb>
__device__ __forceinline__ void run_tile(G& g, char* smem, f32x4_t (&acc)[G::Shape::MB][nb > 0 ? nb : 1], bool idle,
                                         bool counted = false) {
  if constexpr (G::HAS_IDLE) {
    if (nb == 0 || idle) {                           // wave-uniform
      clear(acc);
      if constexpr (G::HALVES && !G::KMAJOR) g.template run_idle<nb>(smem);
      else g.run_idle(smem);
      return;
    }
  }
  if constexpr (nb == 0) {
  } else if constexpr (std::is_same<G, Logits256>::value || std::is_same<G, Logits256Turned>::value ||
                       std::is_same<G, Logits256Ring>::value || std::is_same<G, LogitsWide>::value) g.run(smem, acc, counted);
  else if constexpr (G::HALVES && !G::KMAJOR) g.template run<nb>(smem, acc, counted);
  else if constexpr (G::HALVES) g.template run<nb>(smem, acc);
  else g.run(smem, acc);
}
// column blocks of this wavefront
template <typename G>
__device__ __forceinline__ int column_blocks(const G& g) {
  if constexpr (G::HALVES) return G::Shape::wave_col(wave_id()) == 0 ? G::Shape::NB : g.nb1;
  else return G::Shape::NB;
}
template <typename G>
__device__ __forceinline__ int last_blocks(const G& g) {      // ... of the tile's last column of wavefronts
  if constexpr (G::HALVES) return g.nb1;
  else return G::Shape::NB;
}

template <typename G, int nb>
__device__ __forceinline__ void issue_first(const G& g, char* smem, int part) {
  if constexpr (G::HALVES) g.template issue_first<nb>(smem, part);
  else g.issue_first(smem, part);
}

// A tile of the logits kernels: rows [BM tv, ..) of W, list positions [width tt, ..).
struct LogitsTile {
  int tv, tt;
  __device__ __forceinline__ void take(TileSchedule<PATCH_ROWS_LOGITS>& sch) {
    sch.take(tv, tt);
    asm volatile("" : "+s"(tv), "+s"(tt));           // divided out here, under an epilogue, not where they are used
  }
};
// What a tile of the logits kernels needs per token goes through LDS, a word a list position: list 0 the token rows of the
// NEXT tile's columns, further lists this tile's words out of arrays by token (targets; lse, coef), fetched with the tile's first
// slabs -- their rows came with the tile before -- and there when its main loop starts: no global load stands between two
// tiles.  Loaded at the boundary, through the row list, they were two dependent trips to memory; with accumulators that are
// not cleared, requests spread over the epilogue and no wait but the loop's own, a tile of 10188 tokens x 128256 entries takes 1.1 - 2 us less (forward / dz: d = 256 900 / 1015
// -> 817 / 909 us, 696 1945 / 1970 -> 1785 / 1830, 1024 2240 / 2388 -> 2128 / 2277, 4096 -0.7 / -0.4 %).
// Positions past the list repeat its last word.
template <typename S, int LISTS>
struct TokenWords {
  // a wavefront fetches 64 words at a time, always of the same 64 positions (of which the last may lie past a wide tile)
  static constexpr int PIECES = S::BN <= 64 ? 1 : S::BN <= 128 ? 2 : S::BN <= 256 ? 4 : 8, BYTES = LISTS * PIECES * 256;
  static_assert(S::WAVES % PIECES == 0, "");
  __device__ __forceinline__ static int position() { return wave_id() % PIECES * 64 + (int)(threadIdx.x & 63); }
  // rows: the row list; next: first position of the next tile; row: the token row of this lane's position of this tile;
  // by_token: the arrays of lists 1 .., N words each
  __device__ __forceinline__ static void fetch(const int32_t* rows, int next, int n_act, int row,
                                               const void* const (&by_token)[LISTS - 1], int64_t N, char* lds) {
    const int wave = wave_id();
#pragma unroll
    for (int i = 0; i < (LISTS * PIECES + S::WAVES - 1) / S::WAVES; ++i) {
      const int piece = i * S::WAVES + wave, l = piece / PIECES;
      if (LISTS * PIECES % S::WAVES != 0 && piece >= LISTS * PIECES) break;      // wave-uniform
      uint64_t base = reinterpret_cast<uint64_t>(rows);
#pragma unroll
      for (int q = 1; q < LISTS; ++q) base = l == q ? reinterpret_cast<uint64_t>(by_token[q - 1]) : base;
      const i32x4_t rs = {__builtin_amdgcn_readfirstlane((int)(uint32_t)base),
                          __builtin_amdgcn_readfirstlane((int)((uint32_t)(base >> 32) & 0xffffu)),
                          __builtin_amdgcn_readfirstlane((l == 0 ? n_act : (int)N) * 4), 0x00020000};
      lds_dma4(lds_address(lds) + (uint32_t)piece * 256u, (uint32_t)(l == 0 ? min(next + position(), n_act - 1) : row) * 4u, rs);
    }
  }
  template <typename V>
  __device__ __forceinline__ static V word(const char* lds, int list, int pos) {
    return *reinterpret_cast<const V*>(lds + (list * (PIECES * 64) + pos) * 4);
  }
};
// The logits kernels gather their column operand (H rows) through the active-row list: the rows a lane fetches.
template <bool NEAR, typename G>
__device__ __forceinline__ void gather_rows(const G& g, const char* words, int (&grow)[decltype(G::lb)::ITERS]) {
  const int lane = threadIdx.x & 63, wave = wave_id();
#pragma unroll
  for (int it = 0; it < decltype(G::lb)::ITERS; ++it)
    grow[it] = *reinterpret_cast<const int*>(
        words + min(decltype(G::lb)::template lane_tile_row<NEAR>(it, wave, lane, last_blocks(g)), G::Shape::BN - 1) * 4);
}
template <bool NEAR, typename G, typename Args>
__device__ __forceinline__ void gather_rows_of_first(const G& g, const Args& a, const LogitsTile& t, int n_act,
                                                     int (&grow)[decltype(G::lb)::ITERS]) {
  const int lane = threadIdx.x & 63, wave = wave_id();
#pragma unroll
  for (int it = 0; it < decltype(G::lb)::ITERS; ++it)
    grow[it] = a.rows[min(t.tt * g.width() + decltype(G::lb)::template lane_tile_row<NEAR>(it, wave, lane, last_blocks(g)),
                          n_act - 1)];
}
// both operand streams of a tile (rows = W tile, columns = gathered H rows); issue_first() requests the first slabs
template <bool NEAR, typename G, typename Args>
__device__ __forceinline__ void logits_setup(G& g, const Args& a, const LogitsTile& t, int n_act,
                                             const int (&grow)[decltype(G::lb)::ITERS]) {
  typedef typename G::Type::store_t st;
  constexpr int BM = G::Shape::BM;
  const int width = g.width();
  g.template setup_gathered<NEAR>((const st*)a.W + (int64_t)t.tv * BM * a.d, a.d,
                                     (int)min((int64_t)BM, a.V - (int64_t)t.tv * BM), a.H, a.d,
                                     min(width, n_act - t.tt * width), a.d, grow, a.N,
                                     n_act <= TURN_COLUMNS * width ? t.tv / PATCH_ROWS_LOGITS : 0);
}

// f(std::integral_constant<int, column blocks of this wavefront>()): a kernel's walk over its tiles.  The wavefronts of a
// workgroup may take different branches; all of them meet the same barriers.
template <typename G, typename F>
__device__ __forceinline__ void with_blocks(const G& g, F&& f) {
  if constexpr (!G::HALVES) {
    f(std::integral_constant<int, G::Shape::NB>());
  } else {                                           // wave-uniform
    const int nb = column_blocks(g);
    constexpr bool ANY = G::KMAJOR;                  // the narrow loop has right halves of two or no blocks
    if (nb == 8) f(std::integral_constant<int, 8>());
    else if (ANY && nb == 6) f(std::integral_constant<int, ANY ? 6 : 0>());
    else if (ANY && nb == 4) f(std::integral_constant<int, ANY ? 4 : 0>());
    else if (nb == 2) f(std::integral_constant<int, 2>());
    else f(std::integral_constant<int, 0>());
  }
}
// LDS of the logits kernels: slabs, the token words and, in the forward, per-token (max, sum) of the wave rows.  Narrow
// tiles have those inside their third slab, which is empty during an epilogue.
template <typename G>
constexpr int FWD_SUMS_BYTES = 2 * G::Shape::WAVES_M * G::Shape::BN * 4;
template <typename G>
constexpr int fwd_sums_at = G::HALVES ? 2 * NARROW_STAGE_BYTES : G::LDS_BYTES;
static_assert(FWD_SUMS_BYTES<TileGemmNarrow<BF16>> <= NARROW_STAGE_BYTES, "");
template <typename G>
constexpr int fwd_words_at = G::LDS_BYTES + (G::HALVES ? 0 : FWD_SUMS_BYTES<G>);
template <typename G>
constexpr int fwd_bytes_of = fwd_words_at<G> + TokenWords<typename G::Shape, 2>::BYTES;
template <typename G>
constexpr int dz_bytes_of = G::LDS_BYTES + TokenWords<typename G::Shape, 4>::BYTES;
// a kernel of 256-row tiles holds both loops
typedef TileGemmNarrow<BF16> LogitsNarrow;
template <typename G>
constexpr bool HAS_NARROW = std::is_same<G, Logits256>::value;
template <typename G>
constexpr int fwd_lds_bytes = HAS_NARROW<G> ? (fwd_bytes_of<LogitsNarrow> > fwd_bytes_of<LogitsWide> ? fwd_bytes_of<LogitsNarrow> : fwd_bytes_of<LogitsWide>) : fwd_bytes_of<G>;
static_assert(fwd_lds_bytes<Logits256> <= 160 * 1024, "");
template <typename G>
constexpr int dz_lds_bytes = HAS_NARROW<G> ? (dz_bytes_of<LogitsNarrow> > dz_bytes_of<G> ? dz_bytes_of<LogitsNarrow> : dz_bytes_of<G>) : dz_bytes_of<G>;

template <typename G, int nb>
__device__ __forceinline__ void fwd_tiles(const FwdArgs& a, G& g, TileSchedule<PATCH_ROWS_LOGITS>& sch, int n_act, char* smem) {
  typedef typename G::Shape S;
  constexpr int BM = S::BM, BN = S::BN, MB = S::MB;
  const int width = g.width();
  float* s_m = reinterpret_cast<float*>(smem + fwd_sums_at<G>);   // [waves along the vocabulary][tokens of the tile]
  float* s_s = s_m + S::WAVES_M * BN;                           // not in the stages of the next tile's first slabs

  typedef TokenWords<S, 2> Words;
  char* words = smem + fwd_words_at<G>;

  LogitsTile cur, next;
  cur.take(sch);
  int grow[decltype(g.lb)::ITERS];
  gather_rows_of_first<false>(g, a, cur, n_act, grow);
  int first_row = a.rows[min(cur.tt * width + Words::position(), n_act - 1)];
  logits_setup<false>(g, a, cur, n_act, grow);
  asm volatile("" : "+v"(first_row));             // waited for here, with the others, not behind the slab requests
#pragma unroll
  for (int q = 0; q < G::FIRST_PARTS; ++q) issue_first<G, nb>(g, smem, q);
  bool more = sch.has_tile();
  next = cur;
  if (more) next.take(sch);
  const void* const by_token[] = {a.targets};
  Words::fetch(a.rows, next.tt * width, n_act, first_row, by_token, a.N, words);
  bool counted = false;
  while (true) {
    f32x4_t acc[MB][nb > 0 ? nb : 1];
    run_tile<G, nb>(g, smem, acc, S::wave_col(wave_id()) * S::WAVE_N >= n_act - cur.tt * width, counted);
    // The lane's position is rebuilt from an opaque copy of the thread id after every main loop: otherwise all the
    // per-lane constants of the epilogue stay live through the loop, are spilled, and every reload waits (vmcnt) for
    // the slab requests of the next tile as well.
    int tid = threadIdx.x;
    asm volatile("" : "+v"(tid));
    const LanePos<S> lp(tid);
    const int tv = cur.tv, tt = cur.tt;
    const int64_t v0 = (int64_t)tv * BM, t0 = (int64_t)tt * width;
    const int rowsV = (int)min((int64_t)BM, a.V - v0);
    const int rowsT = min(width, n_act - tt * width);
    const bool last = !more;
    gather_rows<false>(g, words, grow);
    const int word_row = Words::template word<int>(words, 0, Words::position());
    int ytok[nb > 0 ? nb : 1];
#pragma unroll
    for (int j = 0; j < nb; ++j) ytok[j] = Words::template word<int>(words, 1, lp.col(j));
    if constexpr (G::REQUESTS_PAST_K) wait_vmcnt0();    // they must not land in what is fetched or written next
    __syncthreads();                                 // every wave is done reading the slab buffers and the token words
    LLAMARL_FENCE();
    if (!last) {                                     // start the next tile's first slabs; the epilogue hides them
      cur = next;
      logits_setup<false>(g, a, cur, n_act, grow);
      issue_first<G, nb>(g, smem, 0);
      more = sch.has_tile();
      if (more) next.take(sch);
      Words::fetch(a.rows, next.tt * width, n_act, word_row, by_token, a.N, words);
    }
    // From here to the next main loop nothing may wait on vmcnt: the counter is in order, so a wait for any load
    // (or spill reload) issued before the slab requests turns into a wait for the requests themselves, and the
    // epilogue would start only when the slabs have arrived.
    LLAMARL_FENCE();

    if (rowsV < BM) {   // last vocab tile only (block-uniform): rows past V must not enter the softmax
#pragma unroll
      for (int i = 0; i < MB; ++i)
#pragma unroll
        for (int r = 0; r < 4; ++r)
          if (lp.row(i, r) >= rowsV) {
#pragma unroll
            for (int j = 0; j < nb; ++j) acc[i][j][r] = -INFINITY;
          }
    }
    auto issue_part = [&](int part) {
      if (part > 0 && part < G::FIRST_PARTS && !last) issue_first<G, nb>(g, smem, part);
    };
    // Four tokens at a time.  VALU-bound: per logit half a max, an fma, an exponential (two issue cycles) and an add; what a
    // token costs beyond its logits is shared by the four.
#pragma unroll
    for (int j0 = 0; j0 < nb; j0 += 4) {
      float m[4], s[4];
#pragma unroll
      for (int q = 0; q < 4; ++q) {
        m[q] = -INFINITY;
        if (j0 + q < nb) {
#pragma unroll
          for (int i = 0; i < MB; ++i)
#pragma unroll
            for (int r = 0; r < 4; ++r) m[q] = fmaxf(m[q], acc[i][j0 + q][r]);
        }
      }
      const float top = rows_combine(m, [](float x, float y) { return fmaxf(x, y); });    // row g: token j0 + g
      rows_spread(top, m);
#pragma unroll
      for (int q = 0; q < 4; ++q) {
        issue_part(j0 + q);
        s[q] = 0.f;
        if (j0 + q < nb) {
          const float mb = (m[q] == -INFINITY) ? 0.f : m[q] * LOG2E;
#pragma unroll
          for (int i = 0; i < MB; ++i)
#pragma unroll
            for (int r = 0; r < 4; ++r) s[q] += fast_exp2(fmaf(acc[i][j0 + q][r], LOG2E, -mb));   // exp2(-inf) = 0
          asm volatile("" : "+v"(s[q]));             // here, between the requests: the compiler sinks it past them all
        }
      }
      const float sum = rows_combine(s, [](float x, float y) { return x + y; });
      // row g of the wavefront holds token j0 + g: position 16 (j0 + g) + l % 16 = 16 j0 + l of its columns
      if (nb - j0 >= 4 || lp.lane < 16 * (nb - j0)) {
        const int at = lp.wm * BN + lp.wn * S::WAVE_N + 16 * j0 + lp.lane;
        s_m[at] = top;
        s_s[at] = sum;
      }
    }
#pragma unroll
    for (int part = (nb + 3) / 4 * 4; part < G::FIRST_PARTS; ++part) issue_part(part);
    // target logits: a token's is held by one lane of one wavefront of one vocab tile; most wavefronts hold none
    {
      const int first = (int)a.v_off + (int)v0 + lp.wm * S::WAVE_M;     // the wavefront's first row (a global index)
      bool any = false;
#pragma unroll
      for (int j = 0; j < nb; ++j) any |= (uint32_t)(ytok[j] - first) < (uint32_t)S::WAVE_M;
      if (__any(any)) {                              // wave-uniform
        const int lane_row0 = lp.row(0, 0);          // rows of this lane: lane_row0 + 16 ib + r
#pragma unroll
        for (int j = 0; j < nb; ++j) {
          const int tok = lp.col(j);
          const int yrow = ytok[j] - (int)a.v_off - (int)v0;      // vocab row of the target inside this tile
          const int yrel = yrow - lane_row0;                      // ... relative to this lane's first row
          float zy = 0.f;
#pragma unroll
          for (int i = 0; i < MB; ++i)
#pragma unroll
            for (int r = 0; r < 4; ++r) zy = (yrel == i * 16 + r) ? acc[i][j][r] : zy;
          if (tok < rowsT && yrow < rowsV && yrel >= 0 && yrel < S::WAVE_M && (yrel & 12) == 0) a.zt[t0 + tok] = zy;
        }
      }
    }
    __syncthreads();
    if (tid < rowsT) {
      float M = s_m[tid];
#pragma unroll
      for (int w = 1; w < S::WAVES_M; ++w) M = fmaxf(M, s_m[w * BN + tid]);
      const float Mb = (M == -INFINITY) ? 0.f : M;
      float sum = s_s[tid] * __expf(s_m[tid] - Mb);
#pragma unroll
      for (int w = 1; w < S::WAVES_M; ++w) sum += s_s[w * BN + tid] * __expf(s_m[w * BN + tid] - Mb);
      a.part_m[(int64_t)tv * a.n_pad + t0 + tid] = M;
      a.part_s[(int64_t)tv * a.n_pad + t0 + tid] = sum;
    }
    if (last) break;
    counted = (wave_id() * 64) < rowsT;              // this wavefront has just issued its two stores
  }
}

template <typename G>
__global__ __launch_bounds__(G::Shape::THREADS, MIN_WAVES<G>) void k_fwd_partials(FwdArgs a) {
  extern __shared__ __attribute__((aligned(1024))) char smem[];
  const int n_act = *a.n_act;
  auto walk = [&](auto g) __attribute__((always_inline)) {
    TileSchedule<PATCH_ROWS_LOGITS> sch;
    // token tiles that hold active rows only
    sch.init(a.tiles_v, (n_act + g.width() - 1) / g.width(), blockIdx.x, gridDim.x);
    if (!sch.has_tile()) return;                     // block-uniform
    with_blocks(g, [&](auto blocks) { fwd_tiles<decltype(g), decltype(blocks)::value>(a, g, sch, n_act, smem); });
  };
  if constexpr (HAS_NARROW<G>) {
    const int width = fwd_width(a.tiles_v, n_act, a.d, gridDim.x).width;
    if (width == LogitsWide::width()) return walk(LogitsWide());
    if (width <= NARROW_BN) {
      LogitsNarrow g;
      g.set_width(width);
      return walk(g);
    }
    walk(Logits256Ring());
  } else {
    walk(G());
  }
}

// lse[t] = log sum over vocab tiles; logp[t] = z[t,y_t] - lse[t], for the active tokens (the compaction pass
// already wrote 0 for masked / bad-target rows).  8 bytes per token and vocab tile.  A block of 1024 threads takes
// TOKENS list positions x 1024 / TOKENS slices of the vocab tiles: 32 tokens read whole 128-byte lines and stream; where
// that leaves most CUs without a block (few tokens) 8 tokens and 128 slices shorten the chain instead.
constexpr int MERGE_THREADS = 1024, MERGE_BATCH = 8;
struct MergeArgs {
  const float* part_m;
  const float* part_s;
  const float* zt;
  const int32_t* rows;
  const int32_t* n_act;
  int tiles_v;
  int64_t n_pad;
  float* out0;            // full vocabulary: logp           shard: m   (max of the shard's logits)
  float* out1;            //                  lse                   s   (sum of exp(z - m) over the shard)
  float* out2;            //                  unused                zt  (target logit if the shard owns it, else 0)
  const int32_t* targets; // shard only
  int64_t v_off, V;       // shard only: its vocabulary range is [v_off, v_off + V)
};
// PARTIAL: W is a shard of a vocabulary-parallel head; the per-token (m, s, zt) are what the shards would
// all-reduce (paper Sec. 8.2, Table 3: trainer model parallelism 8-32), see k_merge_shards.
template <bool PARTIAL, int TOKENS>
__global__ __launch_bounds__(MERGE_THREADS) void k_merge_logp(MergeArgs a) {
  constexpr int SLICES = MERGE_THREADS / TOKENS, WAVES = MERGE_THREADS / 64;
  static_assert(TOKENS == 32 || TOKENS == 8, "cross-lane steps written for these");
  __shared__ float s_M[WAVES][TOKENS], s_S[WAVES][TOKENS];
  const int tok = threadIdx.x % TOKENS, sl = threadIdx.x / TOKENS;
  const int64_t p = (int64_t)blockIdx.x * TOKENS + tok;
  const int64_t n = *a.n_act;
  if ((int64_t)blockIdx.x * TOKENS >= n) return;        // block-uniform
  float M = -INFINITY, S = 0.f;
  if (p < n) {
    // MERGE_BATCH tiles' loads in flight at a time: the running (M, S) is a serial chain, the loads need not be
    for (int j0 = sl; j0 < a.tiles_v; j0 += SLICES * MERGE_BATCH) {
      float mb[MERGE_BATCH], sb[MERGE_BATCH];
#pragma unroll
      for (int q = 0; q < MERGE_BATCH; ++q) {
        const int64_t at = (int64_t)min(j0 + q * SLICES, a.tiles_v - 1) * a.n_pad + p;
        mb[q] = a.part_m[at];
        sb[q] = a.part_s[at];
      }
#pragma unroll
      for (int q = 0; q < MERGE_BATCH; ++q) {
        if (j0 + q * SLICES >= a.tiles_v) break;
        const float m = mb[q], s = sb[q];
        if (m > M) {
          S = S * __expf(M - m) + s;      // exp(-inf) = 0 on the first tile
          M = m;
        } else if (m != -INFINITY) {
          S += s * __expf(m - M);
        }
      }
    }
  }
  // the slices of a wavefront meet across its lanes (the sum is the same in both lanes of a pair), wavefronts in LDS
  auto merge = [&](float m2, float s2) {
    const float m = fmaxf(M, m2), b = (m == -INFINITY) ? 0.f : m;
    S = S * expf(M - b) + s2 * expf(m2 - b);
    M = m;
  };
  if constexpr (TOKENS == 8)
    merge(__uint_as_float((uint32_t)__builtin_amdgcn_update_dpp(0, (int)__float_as_uint(M), 0x128, 0xf, 0xf, true)),   // lane ^ 8
          __uint_as_float((uint32_t)__builtin_amdgcn_update_dpp(0, (int)__float_as_uint(S), 0x128, 0xf, 0xf, true)));
  if constexpr (TOKENS == 8) {
    const bool up = (threadIdx.x & 16) != 0;                                                                            // lane ^ 16
    const auto m = __builtin_amdgcn_permlane16_swap(__float_as_uint(M), __float_as_uint(M), false, false);
    const auto t = __builtin_amdgcn_permlane16_swap(__float_as_uint(S), __float_as_uint(S), false, false);
    merge(__uint_as_float(up ? m[0] : m[1]), __uint_as_float(up ? t[0] : t[1]));
  }
  {
    const bool up = (threadIdx.x & 32) != 0;                                                                            // lane ^ 32
    const auto m = __builtin_amdgcn_permlane32_swap(__float_as_uint(M), __float_as_uint(M), false, false);
    const auto t = __builtin_amdgcn_permlane32_swap(__float_as_uint(S), __float_as_uint(S), false, false);
    merge(__uint_as_float(up ? m[0] : m[1]), __uint_as_float(up ? t[0] : t[1]));
  }
  if ((threadIdx.x & 63) < TOKENS) {
    s_M[threadIdx.x >> 6][tok] = M;
    s_S[threadIdx.x >> 6][tok] = S;
  }
  __syncthreads();
  if (sl == 0 && p < n) {
    float Mx = s_M[0][tok];
#pragma unroll
    for (int q = 1; q < WAVES; ++q) Mx = fmaxf(Mx, s_M[q][tok]);
    float Sx = 0.f;
#pragma unroll
    for (int q = 0; q < WAVES; ++q) Sx += (s_M[q][tok] == -INFINITY) ? 0.f : s_S[q][tok] * expf(s_M[q][tok] - Mx);
    const int64_t t = a.rows[p];
    if constexpr (PARTIAL) {
      const int64_t y = (int64_t)a.targets[t] - a.v_off;
      a.out0[t] = Mx;
      a.out1[t] = Sx;
      a.out2[t] = (y >= 0 && y < a.V) ? a.zt[p] : 0.f;
    } else {
      // in double: lse and logp each carry one fp32 rounding, at the size of the result
      const double l = (double)Mx + log((double)Sx);
      a.out1[t] = (float)l;
      a.out0[t] = (float)((double)a.zt[p] - l);
    }
  }
}

// The all-reduce of a vocabulary-parallel head, done here for shards that ran one after another on one GPU:
//   M = max_p m_p,  lse = M + log sum_p s_p exp(m_p - M),  logp = sum_p zt_p - lse        (m, s, zt: [shards][N])
// Rows whose every m_p is -inf (masked / bad target in every shard) get logp = lse = 0.  Shards are summed in
// ascending order: deterministic.
__global__ __launch_bounds__(256) void k_merge_shards(const float* m, const float* s, const float* zt, int shards,
                                                       int64_t N, float* logp, float* lse) {
  for (int64_t t = (int64_t)blockIdx.x * 256 + threadIdx.x; t < N; t += (int64_t)gridDim.x * 256) {
    float M = -INFINITY;
    for (int p = 0; p < shards; ++p) M = fmaxf(M, m[(int64_t)p * N + t]);
    float l = 0.f, lp = 0.f;
    if (M != -INFINITY) {
      float S = 0.f, Z = 0.f;
      for (int p = 0; p < shards; ++p) {
        const float mp = m[(int64_t)p * N + t];
        S += (mp == -INFINITY) ? 0.f : s[(int64_t)p * N + t] * expf(mp - M);
        Z += zt[(int64_t)p * N + t];
      }
      l = M + logf(S);
      lp = Z - l;
    }
    lse[t] = l;
    logp[t] = lp;
  }
}

// Active-row list.  mode 0 (forward): row t is active if mask[t] != 0 (mask == nullptr: always) and its target
// is inside [0,V); inactive rows get out0 = out1 = 0 (logp, lse) here.  mode 2 (forward of a shard): the same
// list, inactive rows get (out0, out1, out2) = (-inf, 0, 0), the shard's (m, s, zt).  mode 1 (backward): active
// if coef[t] != 0.
// The list is ascending, so every later kernel is deterministic.  Block b owns rows [b, b+1) * COMPACT_BLOCK_ROWS, four
// neighbouring rows a thread (16-byte loads of targets / coef, 4 bytes of mask; token by token where the arrays are
// not aligned for that or the batch ends inside the group).  It first counts the active rows in front of its range by
// evaluating the predicate over them (5 bytes a row, served by L2 -- cheaper than a second launch or a cross-block
// wait for the batch sizes of a trainer step), then places its own in one scan.  The last block stores the total.
// Bound by latency; with four scans of one row a thread and its list walked a row at a time the log-prob call on a tiny
// head took 18 us at 4097 rows and 29 us at 40000, now 12 and 18 (partial merge included, see MERGE_BATCH).
constexpr int COMPACT_THREADS = 1024;
constexpr int COMPACT_BLOCK_ROWS = 4 * COMPACT_THREADS;

struct CompactArgs {
  int mode;
  const uint8_t* mask;
  const int32_t* targets;
  const float* coef;
  int64_t V, N;
  int aligned;               // targets / coef 16-byte, mask 4-byte aligned
  int32_t* rows;
  int32_t* n_act;
  float* out0;
  float* out1;
  float* out2;
  float g;                   // mode 1, fp32: the upstream scalar (or *g_device) and where the scale of dz goes
  const float* g_device;
  float* dz_scale;
};

// bit i: row t0 + i is active (t0 a multiple of 4); mode 1: top = max(top, |coef|)
__device__ __forceinline__ uint32_t active_rows4(const CompactArgs& a, int64_t t0, float& top) {
  uint32_t bits = 0;
  if (a.aligned && t0 + 4 <= a.N) {
    if (a.mode == 1) {
      const float4 c = *reinterpret_cast<const float4*>(a.coef + t0);
      top = fmaxf(fmaxf(top, fmaxf(fabsf(c.x), fabsf(c.y))), fmaxf(fabsf(c.z), fabsf(c.w)));
      return (c.x != 0.f ? 1u : 0u) | (c.y != 0.f ? 2u : 0u) | (c.z != 0.f ? 4u : 0u) | (c.w != 0.f ? 8u : 0u);
    }
    const int4 y = *reinterpret_cast<const int4*>(a.targets + t0);
    const uchar4 k = a.mask != nullptr ? *reinterpret_cast<const uchar4*>(a.mask + t0) : make_uchar4(1, 1, 1, 1);
    bits |= (k.x != 0 && y.x >= 0 && (int64_t)y.x < a.V) ? 1u : 0u;
    bits |= (k.y != 0 && y.y >= 0 && (int64_t)y.y < a.V) ? 2u : 0u;
    bits |= (k.z != 0 && y.z >= 0 && (int64_t)y.z < a.V) ? 4u : 0u;
    bits |= (k.w != 0 && y.w >= 0 && (int64_t)y.w < a.V) ? 8u : 0u;
    return bits;
  }
#pragma unroll
  for (int i = 0; i < 4; ++i) {
    const int64_t t = t0 + i;
    if (t >= a.N) continue;
    bool on;
    if (a.mode == 1) {
      on = a.coef[t] != 0.f;
      top = fmaxf(top, fabsf(a.coef[t]));
    } else {
      const int y = a.targets[t];
      on = (a.mask == nullptr || a.mask[t] != 0) && y >= 0 && (int64_t)y < a.V;
    }
    bits |= on ? 1u << i : 0u;
  }
  return bits;
}

// fp32 keeps dz multiplied by a power of two that lifts the largest |upstream * coef| to 2^60: the contractions split
// their operands into bf16 parts that end at 2^-133 (gemm_small.h), and entries c p with p down to 2^-126 then stay clear of
// that for any coef within 2^-40 of the largest one.  Exact in both directions; large gradients are left alone.
__device__ __forceinline__ float dz_scale_for(float c) {
  const int e = (int)(__float_as_uint(c) >> 23 & 0xffu) - 127;      // a subnormal c counts as 2^-127
  return (c == 0.f || e >= 60) ? 1.f : __uint_as_float((uint32_t)(min(60 - e, 126) + 127) << 23);
}

// put(position, row) for the active rows of block's range; returns the active rows up to its end.  want_top (of the last block,
// block-uniform): top = the largest |coef| of the batch.
template <typename Put>
__device__ __forceinline__ int place_rows(const CompactArgs& a, int block, bool want_top, float& top, Put put) {
  constexpr int WAVES = COMPACT_THREADS / 64;
  __shared__ int s_front[WAVES], s_own[WAVES];
  __shared__ float s_top[WAVES];
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int64_t first = (int64_t)block * COMPACT_BLOCK_ROWS, t0 = first + 4 * tid;
  top = 0.f;
  const uint32_t act = t0 < a.N ? active_rows4(a, t0, top) : 0u;
  int front = 0;
#pragma unroll 4
  for (int64_t t = 4 * tid; t < first; t += COMPACT_BLOCK_ROWS) front += __popc(active_rows4(a, t, top));
  if (a.mode != 1) {
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      const int64_t t = t0 + i;
      if (t < a.N && !(act >> i & 1u)) {
        a.out0[t] = (a.mode == 2) ? -INFINITY : 0.f;
        a.out1[t] = 0.f;
        if (a.mode == 2) a.out2[t] = 0.f;
      }
    }
  }
  const int own = __popc(act);
  int upto = own;                                   // active rows of lanes 0 .. lane of this wavefront
#pragma unroll
  for (int o = 1; o < 64; o <<= 1) {
    const int v = __shfl_up(upto, o);
    upto += lane >= o ? v : 0;
  }
#pragma unroll
  for (int o = 32; o > 0; o >>= 1) front += __shfl_xor(front, o);
  if (want_top) {
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) top = fmaxf(top, __shfl_xor(top, o));
    if (lane == 0) s_top[wave] = top;
  }
  if (lane == 63) s_own[wave] = upto;
  if (lane == 0) s_front[wave] = front;
  __syncthreads();
  int base = 0, total = 0;
#pragma unroll
  for (int w = 0; w < WAVES; ++w) {
    base += s_front[w] + (w < wave ? s_own[w] : 0);
    total += s_front[w] + s_own[w];
  }
  int at = base + upto - own;
#pragma unroll
  for (int i = 0; i < 4; ++i)
    if (act >> i & 1u) put(at++, (int32_t)(t0 + i));
  if (want_top)
    for (int w = 0; w < WAVES; ++w) top = fmaxf(top, s_top[w]);
  return total;
}
__device__ __forceinline__ void compact_rows(const CompactArgs& a, int block, int nblocks) {
  const bool last = block == nblocks - 1;           // has seen every row
  float top;
  const int total = place_rows(a, block, last && a.dz_scale != nullptr, top, [&](int at, int32_t row) { a.rows[at] = row; });
  if (threadIdx.x == 0 && last) {
    *a.n_act = total;
    if (a.dz_scale != nullptr) *a.dz_scale = dz_scale_for(fabsf((a.g_device != nullptr ? *a.g_device : a.g) * top));
  }
}
__global__ __launch_bounds__(COMPACT_THREADS) void k_compact_rows(CompactArgs a) { compact_rows(a, blockIdx.x, gridDim.x); }

struct DzArgs {
  const void* H;
  const void* W;
  const int32_t* targets;
  const float* lse;
  const float* coef;
  float g;
  const float* g_device;  // non-null: the upstream scalar is *g_device instead of g
  const float* dz_scale;  // fp32: dz is stored times this (dz_scale_for)
  int64_t N, d, V;
  int64_t v_off;          // vocabulary index of row 0 of W (0 unless W is a shard's slice); lse is always global
  int tiles_v;
  void* dz;     // [N][ldz]  token-major (type of H/W); columns V..ldz-1 written as zero
  int64_t ldz;
  void* dzt;    // [V][packed_pitch(n_act)] vocab-major; columns past the active rows written as zero
  const int32_t* rows;    // active token rows (coef != 0), ascending; dz / dzt are indexed by list position
  const int32_t* n_act;
};
template <typename G, int nb>
__device__ __forceinline__ void dz_tiles(const DzArgs& a, G& g, TileSchedule<PATCH_ROWS_LOGITS>& sch, int n_act, char* smem) {
  typedef typename G::Shape S;
  constexpr int BM = S::BM, MB = S::MB;
  const int width = g.width();
  const int64_t ldzt = packed_pitch(n_act);
  const float upstream = a.g_device != nullptr ? *a.g_device : a.g;
  float scale = 1.f;
  if constexpr (sizeof(typename G::Type::store_t) == 4) scale = *a.dz_scale;
  // a lane's column blocks are neighbouring tokens, so the vocab-major dz^T leaves straight from registers, 16 bytes per
  // lane and whole lines per 16 lanes
  typedef TokenWords<S, 4> Words;
  char* words = smem + G::LDS_BYTES;
  LogitsTile cur, next;
  cur.take(sch);
  int grow[decltype(g.lb)::ITERS];
  gather_rows_of_first<true>(g, a, cur, n_act, grow);
  int first_row = a.rows[min(cur.tt * width + Words::position(), n_act - 1)];
  logits_setup<true>(g, a, cur, n_act, grow);
  asm volatile("" : "+v"(first_row));             // waited for here, with the others, not behind the slab requests
#pragma unroll
  for (int q = 0; q < G::FIRST_PARTS; ++q) issue_first<G, nb>(g, smem, q);
  bool more = sch.has_tile();
  next = cur;
  if (more) next.take(sch);
  const void* const by_token[] = {a.targets, a.lse, a.coef};
  Words::fetch(a.rows, next.tt * width, n_act, first_row, by_token, a.N, words);
  while (true) {
    f32x4_t acc[MB][nb > 0 ? nb : 1];
    run_tile<G, nb>(g, smem, acc, S::wave_col(wave_id()) * S::WAVE_N >= n_act - cur.tt * width);
    int tid = threadIdx.x;                           // opaque per tile: see k_fwd_partials
    asm volatile("" : "+v"(tid));
    const LanePos<S> lp(tid);
    const int tv = cur.tv, tt = cur.tt;
    const int64_t v0 = (int64_t)tv * BM, t0 = (int64_t)tt * width;
    const int rowsV = (int)min((int64_t)BM, a.V - v0);
    const int rowsT = min(width, n_act - tt * width), tok0 = lp.col_near(nb);
    const bool last = !more;
    gather_rows<true>(g, words, grow);
    const int word_row = Words::template word<int>(words, 0, Words::position());
    float tcoef[nb > 0 ? nb : 1], tlse[nb > 0 ? nb : 1];
    int ttgt[nb > 0 ? nb : 1];
#pragma unroll
    for (int j = 0; j < nb; ++j) {
      const int tok = tok0 + j;
      ttgt[j] = Words::template word<int>(words, 1, tok);
      tlse[j] = Words::template word<float>(words, 2, tok);
      tcoef[j] = Words::template word<float>(words, 3, tok);
    }
    if constexpr (G::REQUESTS_PAST_K) wait_vmcnt0();    // they must not land in what is fetched or written next
    __syncthreads();                                 // every wave is done reading the slab buffers and the token words
    LLAMARL_FENCE();
    if (!last) {                                     // the epilogue uses no LDS: fetch the next tile under it
      cur = next;
      logits_setup<true>(g, a, cur, n_act, grow);
      issue_first<G, nb>(g, smem, 0);
      more = sch.has_tile();
      if (more) next.take(sch);
      Words::fetch(a.rows, next.tt * width, n_act, word_row, by_token, a.N, words);
    }
    LLAMARL_FENCE();                                 // nothing may wait on vmcnt from here on: see k_fwd_partials

    // dz in place of the logits; per-token scalars live in registers (one token per lane and j)
    const int lane_row0 = lp.row(0, 0);
    auto issue_part = [&](int part) {
      if (part > 0 && part < G::FIRST_PARTS && !last) issue_first<G, nb>(g, smem, part);
    };
    float nc[nb > 0 ? nb : 1];                               // - upstream * coef; 0 past the active rows
    bool dead = false, any = false;
    const int first = (int)a.v_off + (int)v0 + lp.wm * S::WAVE_M;       // the wavefront's first row (a global index)
#pragma unroll
    for (int j = 0; j < nb; ++j) {
      const bool in = tok0 + j < rowsT;
      float c = in ? upstream * tcoef[j] : 0.f;
      if constexpr (sizeof(typename G::Type::store_t) == 4) c *= scale;
      nc[j] = -c;
      dead |= c == 0.f;
      any |= (uint32_t)(ttgt[j] - first) < (uint32_t)S::WAVE_M;
    }
    if (__any(dead)) {                                       // wave-uniform
      // a row whose upstream * coef is 0 is exactly 0, whatever its logits are (they may be infinite or NaN), and so is a
      // position past the active rows: dW contracts over the last 64 of them, and the zeros fetched for H there meet a -inf
      // of W in a NaN
      asm volatile("");                                      // a branch, not 128 selects of every tile
#pragma unroll
      for (int j = 0; j < nb; ++j)
#pragma unroll
        for (int i = 0; i < MB; ++i)
#pragma unroll
          for (int r = 0; r < 4; ++r) acc[i][j][r] = nc[j] != 0.f ? acc[i][j][r] : 0.f;
    }
#pragma unroll
    for (int j = 0; j < nb; ++j) {
      issue_part(j);
      const float lb = (nc[j] != 0.f) ? tlse[j] * LOG2E : 0.f;
#pragma unroll
      for (int i = 0; i < MB; ++i)
#pragma unroll
        for (int r = 0; r < 4; ++r) acc[i][j][r] = nc[j] * fast_exp2(fmaf(acc[i][j][r], LOG2E, -lb));
    }
#pragma unroll
    for (int part = nb; part < G::FIRST_PARTS; ++part) issue_part(part);
    if (__any(any)) {                                        // wave-uniform; most wavefronts hold no token's target
#pragma unroll
      for (int j = 0; j < nb; ++j) {
        // + coef at the target's own vocab row: one lane of one wave of one vocab tile per token
        const int yrel = ttgt[j] - (int)a.v_off - (int)v0 - lane_row0;          // far out of range: another shard's
        const bool mine = nc[j] != 0.f && yrel >= 0 && yrel < S::WAVE_M && (yrel & 12) == 0;
#pragma unroll
        for (int i = 0; i < MB; ++i)
#pragma unroll
          for (int r = 0; r < 4; ++r) acc[i][j][r] += (mine && yrel == i * 16 + r) ? -nc[j] : 0.f;
      }
    }

    // how far the zero padding of each orientation reaches inside this tile
    const int dzt_cols = (int)min((int64_t)width, ldzt - t0);   // dzt[vocab][token]: vocab < V, token < ldzt
    if constexpr (nb == 0) {
    } else if constexpr (sizeof(typename G::Type::store_t) == 2) {
      // bf16: only the vocab-major orientation exists (both gradient contractions read it).
      // Uniform 64-bit tile base + 32-bit lane offset, made opaque once per tile so that the row offsets are
      // not hoisted out of the persistent loop into scratch memory (a 256-row panel of dz^T is < 2 GiB).
      char* tile_base = reinterpret_cast<char*>(a.dzt) + (v0 * ldzt + t0) * 2;
      const uint32_t ld_b = (uint32_t)ldzt * 2u;
      uint32_t lane_off = (uint32_t)lane_row0 * ld_b + (uint32_t)tok0 * 2u;
      asm volatile("" : "+v"(lane_off));
      const bool in_cols = tok0 < dzt_cols;          // ldzt is a multiple of 64: it cuts no group of 2, 4 or 8 neighbours
      typedef uint32_t words_t __attribute__((ext_vector_type(nb / 2), aligned(4)));
#pragma unroll
      for (int i = 0; i < MB; ++i) {
        LLAMARL_FENCE();
#pragma unroll
        for (int r = 0; r < 4; ++r) {
          const int rel = i * 16 + r;
          if (lane_row0 + rel < rowsV && in_cols) {
            words_t v;
#pragma unroll
            for (int j = 0; j < nb / 2; ++j) {
              if constexpr (nb == 2) v = pack_bf16(acc[i][0][r], acc[i][1][r]);
              else v[j] = pack_bf16(acc[i][2 * j][r], acc[i][2 * j + 1][r]);
            }
            // non-temporal: dz^T is gigabytes that the gradient contractions stream later; written normally it
            // pushes the H and W panels this kernel re-reads out of the Infinity Cache (-5 % kernel time at
            // 21 k active rows, where the active H rows alone are 174 MB; neutral at 8.6 k)
            __builtin_nontemporal_store(v, reinterpret_cast<words_t*>(tile_base + (lane_off + (uint32_t)rel * ld_b)));
          }
        }
      }
    } else {
      // fp32: both orientations.  A lane holds four neighbouring vocabulary rows (r) of four neighbouring tokens (j):
      // 16-byte stores along either.  ldz and ldzt are multiples of 64, so no group of four is cut.
      const int dz_cols = (int)min((int64_t)BM, a.ldz - v0);   // dz[token][vocab]:  token < N, vocab < ldz
      float* dz = reinterpret_cast<float*>(a.dz);
      float* dzt = reinterpret_cast<float*>(a.dzt);
#pragma unroll
      for (int i = 0; i < MB; ++i) {
        LLAMARL_FENCE();
        const int vr0 = lp.row(i, 0);
#pragma unroll
        for (int r = 0; r < 4; ++r)
          if (vr0 + r >= rowsV) {                              // padded vocab rows of the token-major copy are 0
#pragma unroll
            for (int j = 0; j < nb; ++j) acc[i][j][r] = 0.f;
          }
#pragma unroll
        for (int j = 0; j < nb; ++j)
          if (tok0 + j < rowsT && vr0 < dz_cols)
            *reinterpret_cast<f32x4_t*>(dz + (t0 + tok0 + j) * a.ldz + v0 + vr0) = acc[i][j];
#pragma unroll
        for (int r = 0; r < 4; ++r)
          if (vr0 + r < rowsV && tok0 < dzt_cols)
            *reinterpret_cast<float4*>(dzt + (v0 + vr0 + r) * ldzt + t0 + tok0) =
                make_float4(acc[i][0][r], acc[i][1][r], acc[i][2][r], acc[i][3][r]);
      }
    }
    if (last) break;
  }
}

template <typename G>
__global__ __launch_bounds__(G::Shape::THREADS, MIN_WAVES<G>) void k_bwd_dz(DzArgs a) {
  extern __shared__ __attribute__((aligned(1024))) char smem[];
  const int n_act = *a.n_act;
  auto walk = [&](auto g) __attribute__((always_inline)) {
    TileSchedule<PATCH_ROWS_LOGITS> sch;
    // token tiles that hold active rows only
    sch.init(a.tiles_v, (n_act + g.width() - 1) / g.width(), blockIdx.x, gridDim.x);
    if (!sch.has_tile()) return;                     // block-uniform
    with_blocks(g, [&](auto blocks) { dz_tiles<decltype(g), decltype(blocks)::value>(a, g, sch, n_act, smem); });
  };
  if constexpr (HAS_NARROW<G>) {
    const int width = dz_width(a.tiles_v, n_act, a.d, gridDim.x).width;
    if (width <= NARROW_BN) {
      LogitsNarrow g;
      g.set_width(width);
      return walk(g);
    }
    if (n_act <= TURN_COLUMNS * width) return walk(Logits256Turned());
  }
  walk(G());
}

struct StoreArgs {
  const void* A;
  const float* a_scale;     // fp32: A holds its values times *a_scale, a power of two
  int64_t lda;
  const void* B;
  int64_t ldb;
  int64_t M, Nn, K;
  int tiles_n;
  void* C;
  int64_t ldc;
  int c_is_f32;
  int accumulate;
  const int32_t* m_count;   // non-null: M = *m_count (device scalar)
  const int32_t* k_count;   // non-null: K = dz_columns(*k_count) (the operands are zero-padded that far)
  const int32_t* c_rows;    // non-null: output row r goes to row c_rows[r] of C
  const int32_t* pitch_count;  // non-null: operands flagged below have the row pitch packed_pitch(*pitch_count)
  int packed_a, packed_b;   // A / B is such a panel (lda / ldb are then ignored)
  int group_m;              // rows of a 32-tile patch (see TileSchedule)
  int width, nb1;           // columns of a tile; column blocks of its right half (TileGemmTN)
  int max_splits;           // the tiles of the last, partial round may be split this many ways along K (1: never)
  int max_parts;            // blocks that `part` has room for
  float* part;              // [splits][tail tiles][tile] fp32 partial products of split tiles
  int32_t* plan_out;        // [4] {whole, rem, splits, tiles_m}: what k_reduce_tail has to finish
  int grid;                 // workgroups of this contraction
  int tail_blocks;          // ... and of its reduction (0: no tile is ever split)
};

struct StoreStrides {       // row strides of A and B
  int64_t a, b;
};

// Work list of a store contraction.  T tiles on a persistent grid of G workgroups: the first floor(T / G) * G tiles
// are contracted whole, one per workgroup and round, and stored in their final form.  The rem = T mod G tiles left
// would occupy only rem of the G workgroups for a whole tile time; instead each is split along K (at most
// max_splits ways, at least four K slabs each) so that the parts fill the grid in a few short rounds, leave fp32
// partial products in the workspace, and k_reduce_tail adds them in split order.  This is what keeps a
// contraction with few output tiles and a long K (dH: 34 x 16 tiles, K = V) on all CUs without a split-K round trip
// for every tile, and what trims the last round of dW (8016 tiles on 256 CUs).  The assignment is fixed by the
// sizes alone: results stay bitwise reproducible.
constexpr int STORE_TAIL_ROUNDS = 4;      // rounds of split parts at the end of a store contraction, at most
constexpr int STORE_REDUCE_COST = 3 * 256;    // launch and latency of k_reduce_tail, ~4 us, in 1/256 of a 1.5 us slab
// A block of BM x BN floats written and read at ~5 TB/s against the time the whole grid takes for a slab: 256 x 256
// bf16 0.105 of 1.47 us; the 128-tiles' block is a quarter and their slab 0.9 us (bf16) or 3.5 us (fp32).
template <typename G>
constexpr int STORE_PART_COST = G::Shape::BM == 256 ? 18 : G::Shape::BM == 128 ? (sizeof(typename G::Type::store_t) == 2 ? 7 : 2) : 1;
struct StorePlan {
  int tiles_m, tiles_n, group_m;
  int whole, rem, splits, n_items;
  int full, last;      // items of whole rounds; this workgroup's item of the last one
  int next, stride;
  // b: this workgroup of G; part_cost: what writing one part's fp32 block and reading it back costs, in 1/256 of a slab of the
  // whole grid
  __device__ __forceinline__ void init(int tiles_m_, int tiles_n_, int group_m_, int nk, int max_splits, int max_parts, int part_cost,
                                       int b, int G) {
    tiles_m = tiles_m_;
    tiles_n = tiles_n_;
    group_m = group_m_;
    const int T = tiles_m * tiles_n;
    whole = T / G * G;
    rem = T - whole;
    // split factor of the tail: the one that makes the tail shortest -- ceil(rem s / G) rounds of nk / s slabs each, the
    // traffic of the rem s partial blocks and the reduction's launch -- among those that keep four K slabs per part
    // and at most STORE_TAIL_ROUNDS rounds of parts, for which the workspace has room; the smallest such factor on ties.
    // Counting rounds alone cut the dW of (N, V, d) = (7000, 33001, 1032) into 931 parts (0.5 GB of blocks): 515 us instead of 487; (3000, 60000, 1504) 545 instead of 485, (4000, 128256, 2560) 2022 instead of 1944.
    // One factor a lane, cost and factor in one word: 31 factors one after the other, two divisions each, took 6 us.
    const int sp = (threadIdx.x & 31) + 1;             // STORE_MAX_SPLITS lanes
    const int rounds = (rem * sp + G - 1) / G;
    // nk < 2^16 (a 256-row panel is < 2 GiB): costs are below 2^26
    const unsigned cost = sp == 1 ? nk * 256 : rounds * nk * 256 / sp + rem * sp * part_cost + STORE_REDUCE_COST;
    unsigned best = sp == 1 || (sp <= max_splits && nk / sp >= 4 && rounds <= STORE_TAIL_ROUNDS &&
                                      rem * sp <= max_parts) ? cost * 32 + (sp - 1) : ~0u;
#pragma unroll
    for (int m = 16; m > 0; m >>= 1) best = min(best, (unsigned)__shfl_xor((int)best, m));
    splits = rem > 0 ? __builtin_amdgcn_readfirstlane((int)(best & 31)) + 1 : 1;
    n_items = whole + rem * splits;
    // 32 consecutive items per XCD and round (see TileSchedule): workgroup b sits on XCD b % 8.  The items of a last round
    // that does not fill the grid are dealt to all XCDs alike.
    full = n_items / G * G;
    const int left = n_items - full, per = (left + 7) >> 3, mine = (b & 7) * per + (b >> 3);
    last = (G & 7) != 0 ? full + b : (b >> 3) < per && mine < left ? full + mine : n_items;
    next = full == 0 ? last : (G & 7) == 0 ? (b & 7) * (G >> 3) + (b >> 3) : b;
    stride = G;
  }
  __device__ __forceinline__ bool has_item() const { return next < n_items; }
  __device__ __forceinline__ int take() {
    const int it = next;
    next = it >= full ? n_items : it + stride < full ? it + stride : last;
    return it;
  }
  // item -> tile id, K split and number of splits; tail items are split-major, so the 32 items an XCD holds in
  // the last round are neighbouring tiles of one K range and share operand panels like whole tiles do
  __device__ __forceinline__ void decode(int item, int& tile, int& split, int& nsplit) const {
    if (item < whole) {
      tile = item;
      split = 0;
      nsplit = 1;
    } else {
      const int j = item - whole;
      split = j / rem;
      tile = whole + (j - split * rem);
      nsplit = splits;
    }
  }
  __device__ __forceinline__ void coords(int id, int& tm, int& tn) const {   // as TileSchedule::take, without the turn
    const int per_group = group_m * tiles_n;
    const int g = id / per_group;
    const int first_m = g * group_m;
    const int gsize = min(tiles_m - first_m, group_m);
    const int in_g = id - g * per_group;
    tm = first_m + in_g % gsize;
    tn = in_g / gsize;
  }
};

template <typename G>
struct StoreTile {     // what one work item of k_gemm_store contracts and where it goes
  int64_t row0, col0, k_lo, k_len;
  int rowsA, rowsB, split, nsplit, tail_index;
  __device__ __forceinline__ void set(const StoreArgs& a, const StorePlan& plan, int64_t M, int64_t K, int item) {
    constexpr int BK = 8 * G::Type::EPC, BM = G::Shape::BM, BN = G::Shape::BN;
    int tile, tm, tn;
    plan.decode(item, tile, split, nsplit);
    plan.coords(tile, tm, tn);
    tail_index = tile - plan.whole;
    row0 = (int64_t)tm * BM;
    const int width = G::HALVES ? a.width : BN;
    col0 = (int64_t)tn * width;
    rowsA = (int)min((int64_t)BM, M - row0);
    rowsB = (int)min((int64_t)width, a.Nn - col0);
    k_lo = 0;
    k_len = K;
    if (nsplit > 1) {
      const int nk = (int)((K + BK - 1) / BK);       // 32-bit: slabs per contraction fit an int by far
      k_lo = (int64_t)(nk * split / nsplit) * BK;
      k_len = min(K, (int64_t)(nk * (split + 1) / nsplit) * BK) - k_lo;
    }
  }
};

template <typename G>
__device__ __forceinline__ StoreTile<G> store_tile_of(const StorePlan& plan, const StoreArgs& a, int item, int64_t M,
                                                      int64_t K) {
  StoreTile<G> t;
  t.set(a, plan, M, K, item);
  return t;
}
// (nothing to contract, k_len = 0: every request lies past K)
template <typename G>
__device__ __forceinline__ void store_fetch(G& g, const StorePlan& plan, const StoreArgs& a, const StoreStrides& ld, int item,
                                            int64_t M, int64_t K, char* smem) {
  typedef typename G::Type::store_t st;
  const StoreTile<G> t = store_tile_of<G>(plan, a, item, M, K);
  if constexpr (G::KMAJOR)   // A is At [K][lda] (output rows are its columns), B is Bt [K][ldb]
    g.prefetch((const uint16_t*)a.A + t.k_lo * ld.a + t.row0, ld.a, t.row0,
               (const uint16_t*)a.B + t.k_lo * ld.b + t.col0, ld.b, t.col0, (int)t.k_len, smem);
  else
    g.template prefetch<true>((const st*)a.A + t.row0 * ld.a + t.k_lo, ld.a, t.rowsA,
                              (const st*)a.B + t.col0 * ld.b + t.k_lo, ld.b, t.rowsB, t.k_len, smem);
}

// Four neighbouring output elements in their final form.  MODE: 1 fp32, 2 fp32 accumulate, 3 bf16, 4 bf16 accumulate.
template <int MODE>
__device__ __forceinline__ void store_final(char* q, const float (&x)[4]) {
  if constexpr (MODE <= 2) {
    f32x4_t v = {x[0], x[1], x[2], x[3]};
    if (MODE == 2) v += *reinterpret_cast<const f32x4_t*>(q);
    *reinterpret_cast<f32x4_t*>(q) = v;
  } else {
    float y[4] = {x[0], x[1], x[2], x[3]};
    if constexpr (MODE == 4) {
      const u32x2_t w = *reinterpret_cast<const u32x2_t*>(q);
#pragma unroll
      for (int j = 0; j < 4; ++j) y[j] += bf16_bits_to_float((uint16_t)(w[j >> 1] >> (16 * (j & 1))));
    }
    *reinterpret_cast<u32x2_t*>(q) = u32x2_t{pack_bf16(y[0], y[1]), pack_bf16(y[2], y[3])};
  }
}
template <int MODE>
__device__ __forceinline__ void store_final1(char* q, float v) {
  if (MODE <= 2) {
    float* f = reinterpret_cast<float*>(q);
    if (MODE == 2) v += *f;
    *f = v;
  } else {
    uint16_t* h = reinterpret_cast<uint16_t*>(q);
    if (MODE == 4) v += bf16_bits_to_float(*h);
    *h = float_to_bf16_bits(v);
  }
}

// MODE (compile time): the final form of the output, see store_final.  Split tiles of the last round leave fp32
// partial products instead (k_reduce_tail finishes them in the same MODE).
typedef TileGemm<BF16, STORE_LOAD_SLOT, 32, false> Store256;      // counted: its epilogue's stores, one unit per row of a lane
template <typename G, int MODE, int nb>
__device__ __forceinline__ void store_tiles(const StoreArgs a, const StoreStrides ld, G g, StorePlan plan, int64_t M, int64_t K, char* smem) {
  typedef typename G::Shape S;
  constexpr bool KMAJOR = G::KMAJOR;
  constexpr int BM = S::BM, BN = S::BN, MB = S::MB;
  int id = plan.take();
  store_fetch(g, plan, a, ld, id, M, K, smem);
  bool counted = false;
  while (true) {
    f32x4_t acc[MB][nb > 0 ? nb : 1];
    const int cur_id = id;
    if (store_tile_of<G>(plan, a, cur_id, M, K).k_len > 0) {
      const StoreTile<G> t = store_tile_of<G>(plan, a, cur_id, M, K);
      if constexpr (G::HALVES)
        run_tile<G, nb>(g, smem, acc,
                        S::wave_row(wave_id()) * S::WAVE_M >= t.rowsA || S::wave_col(wave_id()) * S::WAVE_N >= t.rowsB, counted);
      else if constexpr (std::is_same<G, Store256>::value)
        g.run(smem, acc, counted);
      else if constexpr (sizeof(typename G::Type::store_t) == 4)
        g.template run<true>(smem, acc);
      else
        g.run(smem, acc);
    } else {
      clear(acc);                                    // nothing to contract: the product is zero
    }
    const bool more = plan.has_item();
    wait_vmcnt0();                                   // nothing may wait on vmcnt after the slab requests: see k_fwd_partials
    __syncthreads();                                 // every wave is done reading the slab buffers
    if (more) {                                      // the store epilogue uses no LDS: fetch the next tile under it
      id = plan.take();
      store_fetch(g, plan, a, ld, id, M, K, smem);
    }
    LLAMARL_FENCE();

    const StoreTile<G> t = store_tile_of<G>(plan, a, cur_id, M, K);
    // no store of a lane is left out (a wavefront without columns has none)
    counted = nb > 0 && (t.nsplit > 1 || (t.rowsA == BM && t.rowsB == g.width()));
    if constexpr (nb > 0) {
      int tid = threadIdx.x;                           // opaque per tile: see k_fwd_partials (a spilled per-lane constant
      asm volatile("" : "+v"(tid));                    // reloaded here would wait for the slab requests above)
      const LanePos<S> lp(tid);
      // Store epilogue, one 16-row block at a time (fences keep the unrolled blocks from piling up address registers).
      // Addresses are a uniform 64-bit tile base plus a 32-bit per-lane byte offset (a 256-row panel is < 2 GiB).
      // The offset passes through an empty asm once per tile: otherwise the 32 row offsets of a lane, which do not
      // depend on the tile, are hoisted out of the persistent loop and live in scratch memory.
      const int row_l = lp.row(0, 0);                                // lane's first row; (ib, r) adds 16 ib + r
      if (t.nsplit > 1) {
        // a split tile of the last round (block-uniform): the whole BM x BN fp32 block goes to the workspace,
        // rows and columns past the matrix edge included (they hold zeros or values nobody reads)
        char* blk = reinterpret_cast<char*>(a.part + ((int64_t)t.split * plan.rem + t.tail_index) * (BM * BN));
        uint32_t lane_off = (uint32_t)row_l * (BN * 4) + (uint32_t)(KMAJOR ? lp.col(0) : lp.col_near(nb)) * 4u;
        asm volatile("" : "+v"(lane_off));
#pragma unroll
        for (int i = 0; i < MB; ++i) {
          LLAMARL_FENCE();
#pragma unroll
          for (int r = 0; r < 4; ++r) {
            char* q = blk + (lane_off + (uint32_t)(i * 16 + r) * (BN * 4));
            float x[nb];
#pragma unroll
            for (int j = 0; j < nb; ++j) x[j] = acc[i][j][r];
            if constexpr (!KMAJOR) {
              store_final<1>(q, x);
            } else {
#pragma unroll
              for (int j = 0; j < nb; ++j) reinterpret_cast<float*>(q)[j * 16] = x[j];
            }
          }
        }
      } else {
        constexpr int esz = (MODE >= 3) ? 2 : 4;
        char* Cb = reinterpret_cast<char*>(a.C);
        const bool scatter = a.c_rows != nullptr;
        const uint32_t ldc_b = (uint32_t)a.ldc * esz;
        char* tile_base = Cb + (t.row0 * a.ldc + t.col0) * esz;
        if constexpr (!KMAJOR) {
          // A lane's four column blocks are neighbouring columns c .. c + 3, stored as one unit, 8 bytes of bf16; 16 lanes
          // cover 128 consecutive bytes of a row -- whole lines with no cross-lane traffic (stores that split a line over
          // lanes of different rows measured ~0.5 ms per GB slower).  The number of columns is a multiple of 4 (checked on the
          // host), so no unit is cut.
          static_assert(nb == 4, "a unit of four columns");
          const int c = lp.col_near(nb);
          uint32_t lane_off = (uint32_t)row_l * ldc_b + (uint32_t)c * esz;
          asm volatile("" : "+v"(lane_off));
#pragma unroll
          for (int i = 0; i < MB; ++i) {
            LLAMARL_FENCE();
#pragma unroll
            for (int r = 0; r < 4; ++r) {
              const int rel = i * 16 + r;
              const int rib = row_l + rel;
              if (rib < t.rowsA && c < t.rowsB) {
                char* q = scatter ? Cb + ((int64_t)a.c_rows[t.row0 + rib] * a.ldc + t.col0 + c) * esz
                                  : tile_base + (lane_off + (uint32_t)rel * ldc_b);
                float x[nb];
#pragma unroll
                for (int j = 0; j < nb; ++j) x[j] = acc[i][j][r];
                store_final<MODE>(q, x);
              }
            }
          }
        } else {
          // k-major operands keep the plain column order: one element per lane and column block
          uint32_t lane_off = (uint32_t)row_l * ldc_b + (uint32_t)lp.col(0) * esz;
          asm volatile("" : "+v"(lane_off));
#pragma unroll
          for (int i = 0; i < MB; ++i) {
            LLAMARL_FENCE();
#pragma unroll
            for (int r = 0; r < 4; ++r) {
              const int rel = i * 16 + r;
              const int rib = row_l + rel;
              if (rib < t.rowsA) {
                char* rowq = scatter ? Cb + ((int64_t)a.c_rows[t.row0 + rib] * a.ldc + t.col0 + lp.col(0)) * esz
                                     : tile_base + (lane_off + (uint32_t)rel * ldc_b);
#pragma unroll
                for (int j = 0; j < nb; ++j)
                  if (lp.col(j) < t.rowsB) store_final1<MODE>(rowq + j * 16 * esz, acc[i][j][r]);
              }
            }
          }
        }
      }
    }
    if (!more) break;
  }
}

// workgroup `block` of a contraction's a.grid
template <typename G, int MODE>
__device__ __forceinline__ void gemm_store(const StoreArgs& a, int block, char* smem) {
  constexpr int BK = 8 * G::Type::EPC, BM = G::Shape::BM;
  const int64_t M = a.m_count ? (int64_t)*a.m_count : a.M;
  const int64_t K = a.k_count ? dz_columns(*a.k_count, sizeof(typename G::Type::store_t) == 2) : a.K;
  // a later pass of a chunked backward that found no active rows: nothing to add to what the output holds
  if ((MODE == 2 || MODE == 4) && a.k_count != nullptr && K == 0) {
    if (block == 0 && threadIdx.x == 0) {
      a.plan_out[0] = 0; a.plan_out[1] = 0; a.plan_out[2] = 1; a.plan_out[3] = 0;
    }
    return;
  }
  const int64_t pitch = a.pitch_count != nullptr ? packed_pitch(*a.pitch_count) : 0;
  const StoreStrides ld{a.packed_a ? pitch : a.lda, a.packed_b ? pitch : a.ldb};
  const int tiles_m = (int)((M + BM - 1) / BM);
  StorePlan plan;
  plan.init(tiles_m, a.tiles_n, a.group_m, (int)((K + BK - 1) / BK), a.max_splits, a.max_parts, STORE_PART_COST<G>,
            block, a.grid);
  if (block == 0 && threadIdx.x == 0) {
    a.plan_out[0] = plan.whole; a.plan_out[1] = plan.rem; a.plan_out[2] = plan.splits; a.plan_out[3] = tiles_m;
  }
  if (!plan.has_item()) return;                      // block-uniform
  G g;
  if constexpr (G::HALVES) g.nb1 = a.nb1;
  if constexpr (sizeof(typename G::Type::store_t) == 4)
    g.unscale = __uint_as_float((254u << 23) - __float_as_uint(*a.a_scale));       // 1 / *a.a_scale
  if constexpr (G::HALVES)
    with_blocks(g, [&](auto blocks) { store_tiles<G, MODE, decltype(blocks)::value>(a, ld, g, plan, M, K, smem); });
  else
    store_tiles<G, MODE, G::Shape::NB>(a, ld, g, plan, M, K, smem);
}
template <typename G, int MODE>
__global__ __launch_bounds__(G::Shape::THREADS, MIN_WAVES<G>) void k_gemm_store(const StoreArgs a) {
  extern __shared__ __attribute__((aligned(1024))) char smem[];
  gemm_store<G, MODE>(a, blockIdx.x, smem);
}
// dH and dW in one launch, where both run on small tiles: neither needs the other's result, and what bounds a small one is the
// launch, the first loads and the stores, which the other's products cover (figures at plan_store).
template <typename GH, int MODE_H, typename GW, int MODE_W>
__global__ __launch_bounds__(GH::Shape::THREADS, MIN_WAVES<GH> < MIN_WAVES<GW> ? MIN_WAVES<GH> : MIN_WAVES<GW>)
void k_gemm_store_pair(const StoreArgs h, const StoreArgs w) {
  extern __shared__ __attribute__((aligned(1024))) char smem[];
  if ((int)blockIdx.x < h.grid) gemm_store<GH, MODE_H>(h, blockIdx.x, smem);
  else gemm_store<GW, MODE_W>(w, (int)blockIdx.x - h.grid, smem);
}

// Finishes the split tiles of a store contraction's last round: C tile = sum over splits (ascending) of the fp32
// partial blocks, stored in the contraction's MODE (dtype, accumulate, row scatter); the plan is the one k_gemm_store
// wrote.  Bound by memory latency: a work unit is a few rows of one tail tile (one float4 per thread and split), all
// of a thread's loads, up to sixteen, are in flight before the first is added, and the units of all tail tiles are dealt to a bounded
// grid -- bounded because the number of tail tiles is only known on the device and a launch that finds none must
// stay cheap.  Against one block per 32-row stripe, whose threads walked eight rows and their splits one dependent
// load after the other: 18.0 -> 5.4 us for one tile in eight parts, 19.5 -> 5.4 us for 15, 52.8 -> 32 us for the dW
// of a 33001 x 1032 head (~200 MB of partial blocks, now near copy rate).
template <typename S>
struct TailUnit {
  static constexpr int THREADS_PER_ROW = S::BN / 4, ROWS = 256 / THREADS_PER_ROW;   // 256 threads, one float4 each
  static constexpr int PER_TILE = S::BM / ROWS;
};
constexpr int TAIL_MAX_BLOCKS = 2048;
static_assert(STORE_MAX_SPLITS <= 32, "StorePlan::init weighs 32 factors");
// The parts in ascending order, MOST loads of a thread in flight.  More than eight parts are few tiles, bound by latency: 32
// of them eight at a time took 13 us.  All 32 at once, though, leave too few wavefronts for the many tiles of eight parts.
template <int MOST>
__device__ __forceinline__ void add_parts(float4& s, const float* p, int64_t plane, int splits) {
  float4 v[MOST];
#pragma unroll
  for (int q = 0; q < MOST; ++q)
    if (q < splits) v[q] = *reinterpret_cast<const float4*>(p + q * plane);
#pragma unroll
  for (int q = 0; q < MOST; ++q)
    if (q < splits) {
      s.x += v[q].x; s.y += v[q].y; s.z += v[q].z; s.w += v[q].w;
    }
}
template <typename S, int MODE>
__device__ __forceinline__ void reduce_tail(const StoreArgs& a, int block) {
  const int whole = a.plan_out[0], rem = a.plan_out[1], splits = a.plan_out[2], tiles_m = a.plan_out[3];
  if (splits <= 1) return;                           // block-uniform
  const int64_t M = a.m_count ? (int64_t)*a.m_count : a.M;
  StorePlan plan;
  plan.tiles_m = tiles_m;
  plan.tiles_n = a.tiles_n;
  plan.group_m = a.group_m;
  constexpr int esz = (MODE >= 3) ? 2 : 4, BM = S::BM, BN = S::BN;
  typedef TailUnit<S> U;
  char* Cb = reinterpret_cast<char*>(a.C);
  const int c = (int)(threadIdx.x % U::THREADS_PER_ROW) * 4;
  const int64_t plane = (int64_t)rem * (BM * BN);
  for (int u = block; u < rem * U::PER_TILE; u += a.tail_blocks) {
    const int j = u / U::PER_TILE;
    const int row = (u - j * U::PER_TILE) * U::ROWS + (int)(threadIdx.x / U::THREADS_PER_ROW);
    int tm, tn;
    plan.coords(whole + j, tm, tn);
    const int64_t row0 = (int64_t)tm * BM, col0 = (int64_t)tn * a.width;
    const int rowsA = (int)min((int64_t)BM, M - row0), rowsB = (int)min((int64_t)a.width, a.Nn - col0);
    if (row >= rowsA || c >= rowsB) continue;
    const float* p = a.part + (int64_t)j * (BM * BN) + row * BN + c;
    const int64_t orow = a.c_rows ? (int64_t)a.c_rows[row0 + row] : row0 + row;
    float4 s = make_float4(0.f, 0.f, 0.f, 0.f);
    if (splits <= 8) {
      add_parts<8>(s, p, plane, splits);
    } else {
      for (int q = 0; q < splits; q += 16) add_parts<16>(s, p + q * plane, plane, splits - q);
    }
    const float x[4] = {s.x, s.y, s.z, s.w};
    store_final<MODE>(Cb + (orow * a.ldc + col0 + c) * esz, x);
  }
}
template <typename S, int MODE>
__global__ __launch_bounds__(256) void k_reduce_tail(StoreArgs a) { reduce_tail<S, MODE>(a, blockIdx.x); }
template <typename SH, int MODE_H, typename SW, int MODE_W>      // of k_gemm_store_pair
__global__ __launch_bounds__(256) void k_reduce_tail_pair(StoreArgs h, StoreArgs w) {
  if ((int)blockIdx.x < h.tail_blocks) reduce_tail<SH, MODE_H>(h, blockIdx.x);
  else reduce_tail<SW, MODE_W>(w, (int)blockIdx.x - h.tail_blocks);
}

// out[c][p] = in[src(p)][c] for p < R, c < C; out[c][p] = 0 for R <= p < ld_out, one 64 x 64 tile (origin r0, c0) by a
// workgroup of THREADS: 16-byte loads and stores along both matrices' rows (of 16-byte multiples, aligned: the host has checked
// H, W and the workspace, and d), the transposition through LDS in between.  The LDS row is padded by one chunk: the columns a
// wavefront gathers for its stores then start in different banks.
template <typename ST, int THREADS, typename Src>
__device__ __forceinline__ void transpose_tile(const ST* in, int64_t R, int64_t C, int64_t ld_in, ST* out, int64_t ld_out, Src src,
                                               int64_t r0, int64_t c0) {
  constexpr int EPV = 16 / sizeof(ST);                          // elements of a 16-byte chunk
  constexpr int CHUNKS = 64 / EPV, LINES = THREADS / CHUNKS;    // chunks along a tile row; rows taken at a time
  __shared__ __attribute__((aligned(16))) ST t[64][64 + EPV];
  const int q = threadIdx.x % CHUNKS, line = threadIdx.x / CHUNKS;
#pragma unroll
  for (int h = 0; h < 64; h += LINES) {
    const int rr = line + h;
    const int64_t r = r0 + rr, c = c0 + q * EPV;
    uint4 v = make_uint4(0, 0, 0, 0);
    if (rr < 64 && r < R && c < C) v = *reinterpret_cast<const uint4*>(in + src(r) * ld_in + c);
    if (rr < 64) *reinterpret_cast<uint4*>(&t[rr][q * EPV]) = v;
  }
  __syncthreads();
#pragma unroll
  for (int h = 0; h < 64; h += LINES) {
    const int cc = line + h;
    const int64_t c = c0 + cc, r = r0 + q * EPV;
    if (cc < 64 && c < C && r < ld_out) {
      ST w[EPV];
#pragma unroll
      for (int j = 0; j < EPV; ++j) w[j] = t[q * EPV + j][cc];
      uint4 v;
      __builtin_memcpy(&v, w, 16);
      *reinterpret_cast<uint4*>(out + c * ld_out + r) = v;
    }
  }
}

// H^T panel of a pass's active tokens: R = *r_count, the row pitch of `out` is packed_pitch(R), and only the first R
// rounded up to 64 columns of `out` are written (the contraction that reads it stops there or before).
template <typename ST>
__global__ __launch_bounds__(256) void k_transpose(const ST* in, int64_t C, int64_t ld_in, ST* out, const int32_t* rows,
                                                    const int32_t* r_count) {
  const int64_t R = *r_count, r0 = (int64_t)blockIdx.x * 64;
  if (r0 >= R) return;                                          // block-uniform
  transpose_tile<ST, 256>(in, R, C, ld_in, out, packed_pitch(R), [&](int64_t r) { return (int64_t)rows[r]; }, r0, (int64_t)blockIdx.y * 64);
}

// What the backward prepares before it knows the active rows, in one launch: the active-row list (first blocks), zeros
// in the dH rows of inactive tokens (coef == 0: the dH contraction only writes the active ones; a wavefront takes a
// row), fp32 only, W^T [d][ldz] (64 x 64 tiles), and, for up to SETUP_HT_ROWS rows, the H^T panel
// that is k_transpose's otherwise: its blocks place the rows again for themselves.  Launches of a few microseconds each otherwise.
template <typename ST>
struct SetupArgs {
  CompactArgs compact;
  int compact_blocks, ht_blocks, zero_blocks;
  const ST* H;
  ST* ht;
  int ht_tiles_r;            // tiles of H^T along the list; a block takes every ht_blocks / ht_tiles_r-th along d
  ST* dH;
  int64_t d;
  const ST* W;               // fp32 only
  int64_t V, ldz;
  ST* wt;
  int64_t wt_tiles, wt_tiles_r;        // tiles of W^T, along V of them
  int wt_blocks;
};
constexpr int SETUP_MAX_WT_BLOCKS = 1 << 20;           // a launch has fewer than 2^32 threads: 2^22 blocks
constexpr int SETUP_HT_ROWS = 2048, SETUP_HT_BLOCKS = 512;             // two a CU; more tiles take turns
constexpr int SETUP_ROWS = COMPACT_THREADS / 64;       // dH rows of a block
template <typename ST>
__global__ __launch_bounds__(COMPACT_THREADS) void k_bwd_setup(SetupArgs<ST> a) {
  int block = blockIdx.x;
  if (block < a.compact_blocks) {
    compact_rows(a.compact, block, a.compact_blocks);
    return;
  }
  block -= a.compact_blocks;
  if (block < a.ht_blocks) {
    __shared__ int32_t s_rows[64];
    const int tc = block / a.ht_tiles_r, r0 = (block - tc * a.ht_tiles_r) * 64;
    float top;
    const int R = place_rows(a.compact, 0, false, top, [&](int at, int32_t row) {
      if ((uint32_t)(at - r0) < 64u) s_rows[at - r0] = row;
    });
    if (r0 >= R) return;                               // block-uniform
    for (int64_t c0 = (int64_t)tc * 64; c0 < a.d; c0 += (int64_t)(a.ht_blocks / a.ht_tiles_r) * 64) {
      __syncthreads();                                 // the rows are there; everyone is done with the previous tile's LDS
      transpose_tile<ST, COMPACT_THREADS>(a.H, R, a.d, a.d, a.ht, packed_pitch(R), [&](int64_t r) { return (int64_t)s_rows[r - r0]; },
                                          r0, c0);
    }
    return;
  }
  block -= a.ht_blocks;
  if (block < a.zero_blocks) {
    const int64_t t = (int64_t)block * SETUP_ROWS + (threadIdx.x >> 6);
    if (t >= a.compact.N || a.compact.coef[t] != 0.f) return;
    uint4* p = reinterpret_cast<uint4*>(a.dH + t * a.d);
    const int64_t n16 = a.d * (int64_t)sizeof(ST) / 16;
    for (int64_t i = threadIdx.x & 63; i < n16; i += 64) p[i] = make_uint4(0, 0, 0, 0);
    return;
  }
  block -= a.zero_blocks;
  if constexpr (sizeof(ST) == 4) {
    for (int64_t tile = block; tile < a.wt_tiles; tile += a.wt_blocks) {
      const int64_t tc = tile / a.wt_tiles_r, tr = tile - tc * a.wt_tiles_r;
      if (tile != block) __syncthreads();              // everyone is done with the previous tile's LDS
      transpose_tile<ST, COMPACT_THREADS>(a.W, a.V, a.d, a.d, a.wt, a.ldz, [](int64_t r) { return r; }, tr * 64, tc * 64);
    }
  }
}

}  // namespace llamarl
