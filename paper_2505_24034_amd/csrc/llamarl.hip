// llamarl.hip -- host side of the C ABI declared in include/llamarl.h: argument validation, workspace
// layout and kernel launches.  No allocation, no synchronisation, no state between calls.
#include "../../include/llamarl.h"

#include <hip/hip_runtime.h>

#include <algorithm>
#include <cmath>
#include <cstdarg>
#include <cstdio>
#include <cstring>
#include <mutex>

#include "ceiling_kernel.h"
#include "head_kernels.h"
#include "loss_kernels.h"

using namespace llamarl;

namespace {

thread_local char g_err[512] = "";

llamarl_status fail(llamarl_status s, const char* fmt, ...) {
  va_list ap;
  va_start(ap, fmt);
  vsnprintf(g_err, sizeof(g_err), fmt, ap);
  va_end(ap);
  return s;
}

inline int64_t round_up(int64_t x, int64_t m) { return (x + m - 1) / m * m; }
inline bool aligned16(const void* p) { return (reinterpret_cast<uintptr_t>(p) & 15u) == 0; }
inline size_t esize(llamarl_dtype dt) { return dt == LLAMARL_BF16 ? 2 : 4; }

// ---- main loops of the tiles that tile_rules.h picks --------------------------------------------------------
typedef TileGemmSmall<BF16, Shape128, 2, 2> Bf16Loop128;
typedef TileGemmSmall<BF16, Shape64, 4, 2> Bf16Loop64;
typedef TileGemmTNSmall<Shape128, 2, 2> Bf16LoopTN128;
typedef TileGemmTNSmall<Shape64, 4, 2> Bf16LoopTN64;
typedef TileGemmSplit<Shape128, 2, 1> F32Loop128;
typedef TileGemmSplit<Shape64, 3, 2> F32Loop64;

// ---- workspace layouts (every block 256-byte aligned) ----------------------------------------------------
struct FwdWs {
  int tiles_v;
  int64_t n_pad;
  size_t off_m, off_s, off_zt, off_rows, off_nact, total;
};
FwdWs fwd_ws(int64_t N, int64_t d, int64_t V, llamarl_dtype dt) {
  FwdWs w;
  const int tile = tile_edge(logits_tile(N, V, d, dt == LLAMARL_BF16));
  w.tiles_v = (int)((V + tile - 1) / tile);
  w.n_pad = round_up(N, 256);
  // Smaller tiles leave more partials per token, so the planes of a call can be larger than those of a call with more
  // tokens (or vocabulary rows) on larger tiles.  A workspace sized for the larger call has to serve the smaller one as
  // well: room for whatever any N' <= N, V' <= V can need.  A call on tiles of edge e has fewer than LOGITS_MIN_TILES
  // of edge 2e, each of them two rows of partials of at most 256 tokens: at most `small` floats, 0.4 MB.
  const int64_t largest = dt == LLAMARL_BF16 ? 256 : 128, small = 2 * 256 * (LOGITS_MIN_TILES - 1);
  static_assert(LOGITS_MIN_TILES_BF16_128 <= LOGITS_MIN_TILES, "`small` covers both edges");
  const int64_t reserve = std::max((V + largest - 1) / largest * w.n_pad, std::min((V + 63) / 64 * w.n_pad, small));
  const size_t plane = (size_t)reserve * sizeof(float);
  w.off_m = 0;
  w.off_s = round_up((int64_t)plane, 256);
  w.off_zt = w.off_s + round_up((int64_t)plane, 256);
  w.off_rows = w.off_zt + (size_t)round_up(w.n_pad * (int64_t)sizeof(float), 256);
  w.off_nact = w.off_rows + (size_t)round_up(w.n_pad * (int64_t)sizeof(int32_t), 256);
  w.total = w.off_nact + 256;
  return w;
}

struct LossWs {
  int threads, nblocks;     // of k_loss_tokens
  size_t off_len, off_bad, off_part, off_ticket, total;
};
LossWs loss_ws(int64_t N, int64_t B) {  // B generations, N = B * T tokens
  LossWs w;
  w.threads = N > (int64_t)LOSS_MAX_BLOCKS * 256 * LOSS_ITEMS ? 1024 : 256;
  w.nblocks = (int)std::min<int64_t>((N + w.threads * LOSS_ITEMS - 1) / (w.threads * LOSS_ITEMS), LOSS_MAX_BLOCKS);
  w.off_len = 0;
  w.off_bad = (size_t)round_up(B * 4, 256);
  w.off_part = w.off_bad + (size_t)round_up(B * 4, 256);
  // room for the partial sums of the narrower blocks (more of them): the size does not fall where the width changes
  const int64_t most = std::min<int64_t>((N + 256 * LOSS_ITEMS - 1) / (256 * LOSS_ITEMS), LOSS_MAX_BLOCKS);
  w.off_ticket = w.off_part + (size_t)round_up(most * LOSS_NSUM * 8, 256);
  w.total = w.off_ticket + 256;
  return w;
}


// Scratch of llamarl_offpolicy_loss_fwd_static: room for the LossWs layout at the entry point's stated maximum
// (2 x 65536 per-generation counters, LOSS_MAX_BLOCKS x LOSS_NSUM partial sums, the ticket): about 0.5 MB that every
// GPU the library runs on holds until the process ends.  In host code the array's name is only a handle for
// hipGetSymbolAddress(); kernels get the device address that call returns.
constexpr int64_t STATIC_MAX_TOKENS = (int64_t)1 << 22;
constexpr int64_t STATIC_MAX_GENERATIONS = (int64_t)1 << 16;
constexpr size_t STATIC_SCRATCH_BYTES =
    2 * (size_t)STATIC_MAX_GENERATIONS * 4 + ((size_t)LOSS_MAX_BLOCKS * LOSS_NSUM * 8 + 255) / 256 * 256 + 256;
static __device__ __align__(256) unsigned char scratch[STATIC_SCRATCH_BYTES];

constexpr int STATIC_MAX_DEVICES = 64;
std::mutex g_scratch_mutex;
void* g_scratch_ptr[STATIC_MAX_DEVICES] = {};      // device address of `scratch` on each GPU, looked up once

struct BwdWs {
  int64_t R;          // active rows one pass takes (a multiple of 256, or N): dz, the operand panels and the split
                      // partials are sized for R rows; more active rows than that are taken in further passes
  int n_pass;         // passes the host enqueues = ceil(N / R); passes past the active rows find nothing to do
  int64_t ldz, ldzt;  // padded leading dimensions (elements): V rounded up to 64; packed_pitch(R)
  size_t off_dz, off_dzt, off_wt, off_ht, off_rows, off_nact, off_plan, off_part, part, total;
};
// Most workgroups a persistent grid has (one per CU of an MI355X); also the most split items the last round of a
// store contraction can hold, each leaving one BM x BN fp32 block in the workspace.
constexpr int MAX_GRID = 256;
BwdWs bwd_ws(int64_t N, int64_t d, int64_t V, llamarl_dtype dt, int64_t max_rows_per_pass) {
  BwdWs w;
  const size_t es = esize(dt);
  w.R = (max_rows_per_pass <= 0 || max_rows_per_pass >= N) ? N : std::min(N, round_up(max_rows_per_pass, 256));
  w.n_pass = (int)((N + w.R - 1) / w.R);
  w.ldz = round_up(V, 64);
  w.ldzt = packed_pitch(w.R);        // the kernels use packed_pitch(active rows of the pass) <= this
  // bf16: dz exists in the vocab-major orientation only and W is read as it is (k-major dH contraction);
  // fp32 keeps a token-major dz and a transposed copy of W as well
  const bool both = dt == LLAMARL_F32;
  w.off_dz = 0;
  w.off_dzt = w.off_dz + (both ? (size_t)round_up(w.R * w.ldz * (int64_t)es, 256) : 0);
  w.off_wt = w.off_dzt + (size_t)round_up(V * w.ldzt * (int64_t)es, 256);
  w.off_ht = w.off_wt + (both ? (size_t)round_up(d * w.ldz * (int64_t)es, 256) : 0);
  w.off_rows = w.off_ht + (size_t)round_up(d * w.ldzt * (int64_t)es, 256);
  w.off_nact = w.off_rows + (size_t)round_up(round_up(N, 64) * (int64_t)sizeof(int32_t), 256);
  w.off_plan = w.off_nact + (size_t)round_up((int64_t)(1 + w.n_pass) * (int64_t)sizeof(int32_t), 256);
  w.off_part = w.off_plan + 256;
  // fp32 partial blocks of the split tiles at the end of a store contraction (see StorePlan): STORE_TAIL_ROUNDS per workgroup of
  // the grid at most, and room for RESERVED_SPLITS per tile.  A tile is cut into more parts where the room, which is the
  // larger of the two contractions', allows it (StoreArgs::max_parts): few tokens against a long vocabulary, where dW's many
  // tiles have reserved it.  Reserving 32 a tile would make it four times as large for small heads, whose K is too short
  // for them.
  constexpr int RESERVED_SPLITS = 8;
  auto part_bytes = [&](int64_t M, int64_t edge) {
    const int64_t grid = (int64_t)MAX_GRID * (edge == 256 ? 1 : 2);
    return std::min(STORE_TAIL_ROUNDS * grid, tile_count(M, d, edge) * RESERVED_SPLITS) * edge * edge * 4;
  };
  // passes of different lengths may run on different tiles: room for any
  int64_t part = 0;
  for (const int64_t M : {w.R, V})
    for (const int64_t edge : {256, 128, 64})
      if (edge != 256 || dt == LLAMARL_BF16) part = std::max(part, part_bytes(M, edge));
  w.part = (size_t)part;
  w.total = w.off_part + (size_t)part;
  return w;
}

llamarl_status check_head_shape(int64_t N, int64_t d, int64_t V, llamarl_dtype dt) {
  if (dt != LLAMARL_F32 && dt != LLAMARL_BF16) return fail(LLAMARL_ERR_INVALID_ARG, "unknown dtype %d", (int)dt);
  if (N <= 0 || d <= 0 || V <= 0)
    return fail(LLAMARL_ERR_INVALID_ARG, "N, d, V must be positive (got %lld, %lld, %lld)", (long long)N,
                (long long)d, (long long)V);
  const int epc = dt == LLAMARL_BF16 ? 8 : 4;
  if (d % epc != 0)
    return fail(LLAMARL_ERR_UNSUPPORTED, "d = %lld must be a multiple of %d for this dtype (16-byte rows)",
                (long long)d, epc);
  // one 256-row operand panel must stay below 2^31 bytes (32-bit buffer offsets)
  const int64_t widest = (d > V ? d : V) > N ? (d > V ? d : V) : N;
  if (round_up(widest, 64) * (int64_t)esize(dt) * 256 >= (int64_t)1 << 31)
    return fail(LLAMARL_ERR_UNSUPPORTED, "a 256-row panel of %lld elements per row exceeds 2 GiB", (long long)widest);
  if (N * d * (int64_t)esize(dt) >= (int64_t)1 << 31)
    return fail(LLAMARL_ERR_UNSUPPORTED, "H must be smaller than 2 GiB (its rows are gathered with 32-bit offsets)");
  if (tile_count(N, V, tile_edge(logits_tile(N, V, d, dt == LLAMARL_BF16))) >= (int64_t)1 << 31 || V >= (int64_t)1 << 31)
    return fail(LLAMARL_ERR_UNSUPPORTED, "too many tiles");
  return LLAMARL_OK;
}

template <typename K>
hipError_t set_lds(K kernel, int bytes) {
  return hipFuncSetAttribute(reinterpret_cast<const void*>(kernel), hipFuncAttributeMaxDynamicSharedMemorySize,
                             bytes);
}

// `per_cu` persistent workgroups per CU (256 on MI355X); a smaller problem gets one workgroup per tile.
int persistent_grid(int64_t tiles, int per_cu = 1) {
  static int cus = 0;   // a device property, not call state: read once
  if (cus == 0) {
    int dev = 0, n = 0;
    if (hipGetDevice(&dev) == hipSuccess &&
        hipDeviceGetAttribute(&n, hipDeviceAttributeMultiprocessorCount, dev) == hipSuccess && n > 0)
      cus = n;
    else
      cus = MAX_GRID;
    if (cus > MAX_GRID) cus = MAX_GRID;
  }
  return (int)std::min<int64_t>(tiles, (int64_t)cus * per_cu);
}

// Blocks of one launch where a block takes one generation or a few prompts (of 256 or 1024 threads): a launch has fewer than
// 2^32 threads, and HIP gives one that asks for more the count modulo 2^32.  A multiple of 4, so that a later launch's
// tokens start as aligned as the batch.
constexpr int64_t LAUNCH_BLOCKS = (int64_t)1 << 20;

#define HIP_TRY(expr)                                                                              \
  do {                                                                                             \
    hipError_t e_ = (expr);                                                                        \
    if (e_ != hipSuccess) return fail(LLAMARL_ERR_HIP, "%s failed: %s", #expr, hipGetErrorString(e_)); \
  } while (0)

// Dynamic LDS beyond 64 KB has to be asked for.
template <typename K>
hipError_t set_lds_if_large(K kernel, int bytes) {
  return bytes > 65536 ? set_lds(kernel, bytes) : hipSuccess;
}

// C [M,Nn] (+)= A B^T, see StoreArgs; a: the caller's part of the arguments (operands, counts, output, workspace); workgroups: at
// most so many of them.
template <typename G>
llamarl_status plan_store(StoreArgs& a, size_t part_bytes, int workgroups) {
  constexpr int BM = G::Shape::BM, BN = G::Shape::BN, BK = 8 * G::Type::EPC;
  // the store epilogue of the K-contiguous loop writes four neighbouring columns per lane as one unit, and so
  // does the tail reduction
  if (a.Nn % 4 != 0 || a.ldc % 4 != 0)
    return fail(LLAMARL_ERR_UNSUPPORTED, "output columns and row stride must be multiples of 4");
  a.max_splits = STORE_MAX_SPLITS;
  a.max_parts = (int)(part_bytes / (BM * BN * 4));
  const int tiles_m = (int)((a.M + BM - 1) / BM);      // worst case: every row active
  a.width = BN;
  a.nb1 = 0;
  if constexpr (G::HALVES) {
    a.width = store_width(a.Nn);
    a.nb1 = (a.width - G::Shape::WAVE_N) / 16;
  }
  a.tiles_n = (int)((a.Nn + a.width - 1) / a.width);
  a.group_m = (G::KMAJOR && a.tiles_n <= 16) ? PATCH_ROWS_KMAJOR : PATCH_ROWS_STORE;
  const int tiles = tiles_m * a.tiles_n;
  constexpr int64_t PART_K = 4 * BK;                         // a part has four slabs or more
  // a small contraction still gets a workgroup per split
  const int64_t items = (int64_t)tiles * std::min<int64_t>(STORE_MAX_SPLITS, std::max<int64_t>(1, (a.K + PART_K - 1) / PART_K));
  a.grid = (int)std::min<int64_t>(items, workgroups);
  // the split tiles of the last round, if the device-side sizes left any: fewer than `grid` of them.  A contraction
  // whose longest K leaves no two parts of four slabs is never split (StorePlan::init).
  a.tail_blocks = (a.K + BK - 1) / BK < 8 ? 0 : std::min(std::min(a.grid - 1, tiles) * TailUnit<typename G::Shape>::PER_TILE, TAIL_MAX_BLOCKS);
  return LLAMARL_OK;
}

template <typename G, int MODE>
llamarl_status launch_store_mode(const StoreArgs& a, hipStream_t st) {
  HIP_TRY(set_lds_if_large(k_gemm_store<G, MODE>, G::LDS_BYTES));
  k_gemm_store<G, MODE><<<dim3((unsigned)a.grid), dim3(G::Shape::THREADS), G::LDS_BYTES, st>>>(a);
  HIP_TRY(hipGetLastError());
  if (a.tail_blocks > 0) {
    k_reduce_tail<typename G::Shape, MODE><<<dim3((unsigned)a.tail_blocks), dim3(256), 0, st>>>(a);
    HIP_TRY(hipGetLastError());
  }
  return LLAMARL_OK;
}
// f(std::integral_constant<int, MODE>()), see store_final.  k-major operands are bf16's dH, which is bf16 and never accumulates.
template <typename G, typename F>
llamarl_status with_mode(const StoreArgs& a, F&& f) {
  if constexpr (G::KMAJOR) {
    return f(std::integral_constant<int, 3>());
  } else {
    if (a.c_is_f32) return a.accumulate ? f(std::integral_constant<int, 2>()) : f(std::integral_constant<int, 1>());
    if constexpr (sizeof(typename G::Type::store_t) == 2)
      return a.accumulate ? f(std::integral_constant<int, 4>()) : f(std::integral_constant<int, 3>());
    else
      return fail(LLAMARL_ERR_INVALID_ARG, "a 16-bit output needs a 16-bit input type");
  }
}
template <typename G>
llamarl_status launch_store(StoreArgs a, size_t part_bytes, hipStream_t st) {
  const llamarl_status s = plan_store<G>(a, part_bytes, persistent_grid((int64_t)1 << 30, G::GROUPS_PER_CU));
  if (s != LLAMARL_OK) return s;
  return with_mode<G>(a, [&](auto mode) { return launch_store_mode<G, decltype(mode)::value>(a, st); });
}

bool overlap(const void* a, int64_t a_bytes, const void* b, int64_t b_bytes) {
  const uintptr_t x = reinterpret_cast<uintptr_t>(a), y = reinterpret_cast<uintptr_t>(b);
  return x < y + (uint64_t)b_bytes && y < x + (uint64_t)a_bytes;
}

// dH (h, which never accumulates) and dW (w) in one launch, and their split tiles in another; parts: the workspace's blocks,
// of which each contraction takes what its parts can need, dH at least half.
template <typename GH, typename GW>
llamarl_status launch_store_pair(StoreArgs h, StoreArgs w, float* parts, size_t part_bytes, hipStream_t st) {
  constexpr size_t BLOCK_H = GH::Shape::BM * GH::Shape::BN * 4, BLOCK_W = GW::Shape::BM * GW::Shape::BN * 4;
  constexpr int BK = 8 * GW::Type::EPC;                // both have operands of one type
  const int64_t most_w = tile_count(w.M, w.Nn, GW::Shape::BM) * std::min<int64_t>(STORE_MAX_SPLITS, (w.K + BK - 1) / BK / 4);
  const size_t for_w = std::min(part_bytes / 2, (size_t)most_w * BLOCK_W);
  const size_t for_h = (part_bytes - for_w) / BLOCK_H * BLOCK_H;
  h.part = parts;
  w.part = parts + for_h / 4;
  const bool h_long = h.K >= PAIR_LONG_SLABS * BK, w_long = w.K >= PAIR_LONG_SLABS * BK;
  const int cus = persistent_grid((int64_t)1 << 30);
  llamarl_status s = plan_store<GH>(h, for_h, pair_workgroups(cus, GH::GROUPS_PER_CU, GW::GROUPS_PER_CU, h_long, w_long));
  if (s == LLAMARL_OK) s = plan_store<GW>(w, part_bytes - for_h, pair_workgroups(cus, GW::GROUPS_PER_CU, GH::GROUPS_PER_CU, w_long, h_long));
  if (s != LLAMARL_OK) return s;
  return with_mode<GW>(w, [&](auto mode) -> llamarl_status {
    constexpr int MODE_H = sizeof(typename GH::Type::store_t) == 2 ? 3 : 1, MODE_W = decltype(mode)::value;
    constexpr int LDS = GH::LDS_BYTES > GW::LDS_BYTES ? GH::LDS_BYTES : GW::LDS_BYTES;
    const auto kernel = k_gemm_store_pair<GH, MODE_H, GW, MODE_W>;
    HIP_TRY(set_lds_if_large(kernel, LDS));
    kernel<<<dim3((unsigned)(h.grid + w.grid)), dim3(GH::Shape::THREADS), LDS, st>>>(h, w);
    HIP_TRY(hipGetLastError());
    const int tails = h.tail_blocks + w.tail_blocks;
    if (tails > 0) {
      k_reduce_tail_pair<typename GH::Shape, MODE_H, typename GW::Shape, MODE_W><<<dim3((unsigned)tails), dim3(256), 0, st>>>(h, w);
      HIP_TRY(hipGetLastError());
    }
    return LLAMARL_OK;
  });
}

CompactArgs compact_args(CompactArgs a) {
  a.aligned = aligned16(a.targets) && aligned16(a.coef) && (reinterpret_cast<uintptr_t>(a.mask) & 3u) == 0;
  return a;
}
int compact_blocks(int64_t N) { return (int)((N + COMPACT_BLOCK_ROWS - 1) / COMPACT_BLOCK_ROWS); }

template <typename G>
llamarl_status launch_fwd_partials(const FwdArgs& a, hipStream_t st) {
  HIP_TRY(set_lds_if_large(k_fwd_partials<G>, fwd_lds_bytes<G>));
  constexpr int narrowest = HAS_NARROW<G> ? 128 : G::Shape::BN;      // the kernel picks a width
  const int64_t tiles_t = (a.N + narrowest - 1) / narrowest;
  k_fwd_partials<G><<<dim3((unsigned)persistent_grid((int64_t)a.tiles_v * tiles_t, G::GROUPS_PER_CU)),
                      dim3(G::Shape::THREADS), fwd_lds_bytes<G>, st>>>(a);
  HIP_TRY(hipGetLastError());
  return LLAMARL_OK;
}
template <typename G>
llamarl_status launch_bwd_dz(DzArgs a, int64_t rows, hipStream_t st) {
  a.tiles_v = (int)((a.V + G::Shape::BM - 1) / G::Shape::BM);
  constexpr int narrowest = HAS_NARROW<G> ? 128 : G::Shape::BN;      // the kernel picks a width
  const int64_t tiles_t = (rows + narrowest - 1) / narrowest;
  HIP_TRY(set_lds_if_large(k_bwd_dz<G>, dz_lds_bytes<G>));
  k_bwd_dz<G><<<dim3((unsigned)persistent_grid((int64_t)a.tiles_v * tiles_t, G::GROUPS_PER_CU)),
                dim3(G::Shape::THREADS), dz_lds_bytes<G>, st>>>(a);
  HIP_TRY(hipGetLastError());
  return LLAMARL_OK;
}

// W holds the vocabulary rows [v_off, v_off + V) of a head with V_total rows (the whole head: v_off = 0, V = V_total).
// partial == 0: out0 = logp, out1 = lse.  partial != 0: (out0, out1, out2) = the shard's (m, s, zt).
template <typename TT>
llamarl_status run_logprobs(const void* H, const void* W, const int32_t* targets, const uint8_t* mask, int64_t N,
                            int64_t d, int64_t V, int64_t v_off, int64_t V_total, int partial, float* out0,
                            float* out1, float* out2, char* ws, hipStream_t st) {
  constexpr llamarl_dtype dt = sizeof(typename TT::store_t) == 2 ? LLAMARL_BF16 : LLAMARL_F32;
  const FwdWs w = fwd_ws(N, d, V, dt);
  FwdArgs a;
  a.H = H; a.W = W; a.targets = targets; a.N = N; a.d = d; a.V = V; a.v_off = v_off;
  a.tiles_v = w.tiles_v; a.n_pad = w.n_pad;
  a.part_m = reinterpret_cast<float*>(ws + w.off_m);
  a.part_s = reinterpret_cast<float*>(ws + w.off_s);
  a.zt = reinterpret_cast<float*>(ws + w.off_zt);
  int32_t* rows = reinterpret_cast<int32_t*>(ws + w.off_rows);
  int32_t* n_act = reinterpret_cast<int32_t*>(ws + w.off_nact);
  a.rows = rows; a.n_act = n_act;
  // active-token list (mask and target range); inactive rows get their outputs here
  k_compact_rows<<<dim3((unsigned)compact_blocks(N)), dim3(COMPACT_THREADS), 0, st>>>(
      compact_args({partial ? 2 : 0, mask, targets, nullptr, V_total, N, 0, rows, n_act, out0, out1, out2, 0.f, nullptr,
                    nullptr}));
  HIP_TRY(hipGetLastError());
  llamarl_status s;
  const Tile tile = logits_tile(N, V, d, dt == LLAMARL_BF16);
  if constexpr (dt == LLAMARL_BF16)
    s = (tile == TILE_256   ? launch_fwd_partials<Logits256>
         : tile == TILE_128 ? launch_fwd_partials<Bf16Loop128>
                            : launch_fwd_partials<Bf16Loop64>)(a, st);
  else
    s = (tile == TILE_128 ? launch_fwd_partials<F32Loop128> : launch_fwd_partials<F32Loop64>)(a, st);
  if (s != LLAMARL_OK) return s;
  MergeArgs m;
  m.part_m = a.part_m; m.part_s = a.part_s; m.zt = a.zt; m.rows = rows; m.n_act = n_act; m.tiles_v = w.tiles_v;
  m.n_pad = w.n_pad; m.out0 = out0; m.out1 = out1; m.out2 = out2; m.targets = targets; m.v_off = v_off; m.V = V;
  // the log-prob call with d = 8 at (N, V), 8 / 32 tokens a block: (300, 128256) 24.2 / 26.0 us, (1041, 5003) 14.4 / 15.8,
  // (4097, 32000) 42.7 / 42.8, (8192, 60000) 109 / 103
  const int tokens = N <= 2048 ? 8 : 32;
  const auto merge = tokens == 8 ? (partial ? k_merge_logp<true, 8> : k_merge_logp<false, 8>)
                                 : (partial ? k_merge_logp<true, 32> : k_merge_logp<false, 32>);
  merge<<<dim3((unsigned)((N + tokens - 1) / tokens)), dim3(MERGE_THREADS), 0, st>>>(m);
  HIP_TRY(hipGetLastError());
  return LLAMARL_OK;
}

// active rows of each pass: cnt[c] = clamp(n_act - c * R, 0, R)
__global__ void k_pass_counts(const int32_t* n_act, int64_t R, int n_pass, int32_t* cnt) {
  const int c = blockIdx.x * blockDim.x + threadIdx.x;
  if (c >= n_pass) return;
  const int64_t left = (int64_t)*n_act - (int64_t)c * R;
  cnt[c] = (int32_t)(left < 0 ? 0 : (left > R ? R : left));
}

template <typename TT>
llamarl_status run_bwd(const void* H, const void* W, const int32_t* targets, const float* lse, const float* coef,
                       float g, const float* g_device, int64_t N, int64_t d, int64_t V, int64_t v_off,
                       llamarl_dtype dt, void* dH, void* dW, llamarl_dtype dW_dt, int accumulate_dW, int64_t max_rows_per_pass, char* ws, hipStream_t st,
                       void* const* ev) {
  typedef typename TT::store_t stt;
  const BwdWs w = bwd_ws(N, d, V, dt, max_rows_per_pass);
  // ev (optional, 6 caller-owned hipEvent_t): recorded on the stream at the phase boundaries of a one-pass backward
#define PHASE_EVENT(i) \
  do { if (ev) HIP_TRY(hipEventRecord(reinterpret_cast<hipEvent_t>(ev[i]), st)); } while (0)
  PHASE_EVENT(0);
  stt* dz = reinterpret_cast<stt*>(ws + w.off_dz);
  stt* dzt = reinterpret_cast<stt*>(ws + w.off_dzt);
  stt* wt = reinterpret_cast<stt*>(ws + w.off_wt);
  stt* ht = reinterpret_cast<stt*>(ws + w.off_ht);
  int32_t* all_rows = reinterpret_cast<int32_t*>(ws + w.off_rows);
  int32_t* n_act_all = reinterpret_cast<int32_t*>(ws + w.off_nact);
  int32_t* pass_cnt = n_act_all + 1;

  constexpr bool kBf16 = sizeof(stt) == 2;
  // tokens that carry gradient (coef != 0), exact zeros for the dH rows of all the others, fp32: W^T for the
  // K-contiguous dH contraction
  SetupArgs<stt> u;
  int32_t* plan = reinterpret_cast<int32_t*>(ws + w.off_plan);
  float* dz_scale = kBf16 ? nullptr : reinterpret_cast<float*>(plan + 16);     // plan: StoreArgs::plan_out, 4 entries of dH, 4 of dW
  u.compact = compact_args({1, nullptr, nullptr, coef, V, N, 0, all_rows, n_act_all, nullptr, nullptr, nullptr, g, g_device,
                            dz_scale});
  u.compact_blocks = compact_blocks(N);
  u.zero_blocks = (int)((N + SETUP_ROWS - 1) / SETUP_ROWS);
  u.H = reinterpret_cast<const stt*>(H); u.ht = ht;
  u.ht_tiles_r = (int)(w.ldzt / 64);
  // Backward at (N, V, d), k_transpose / here, us: bf16 (128, 1000, 128) 18.2 / 16.8, (1041, 5003, 520) 46.2 / 44.2, (2048, 4096, 264)
  // 44.9 / 42.7, (4096, 3000, 512) 63.4 / 64.6 (every block reads all of coef); fp32 (512, 2048, 512) 63.0 / 59.7
  static_assert(SETUP_HT_ROWS <= COMPACT_BLOCK_ROWS, "a block places all rows");
  const bool ht_in_setup = N <= SETUP_HT_ROWS && w.n_pass == 1;
  u.ht_blocks = ht_in_setup ? u.ht_tiles_r * (int)std::min<int64_t>((d + 63) / 64, std::max(SETUP_HT_BLOCKS / u.ht_tiles_r, 1)) : 0;
  u.dH = reinterpret_cast<stt*>(dH); u.d = d;
  u.W = reinterpret_cast<const stt*>(W); u.V = V; u.ldz = w.ldz; u.wt = wt;
  u.wt_tiles_r = w.ldz / 64;
  u.wt_tiles = kBf16 ? 0 : u.wt_tiles_r * ((d + 63) / 64);
  u.wt_blocks = (int)std::min<int64_t>(u.wt_tiles, SETUP_MAX_WT_BLOCKS);
  const int64_t setup_blocks = (int64_t)u.compact_blocks + u.ht_blocks + u.zero_blocks + u.wt_blocks;
  k_bwd_setup<stt><<<dim3((unsigned)setup_blocks), dim3(COMPACT_THREADS), 0, st>>>(u);
  HIP_TRY(hipGetLastError());
  if (w.n_pass > 1) {
    k_pass_counts<<<dim3((unsigned)((w.n_pass + 255) / 256)), dim3(256), 0, st>>>(n_act_all, w.R, w.n_pass, pass_cnt);
    HIP_TRY(hipGetLastError());
  }
  llamarl_status s;
  for (int c = 0; c < w.n_pass; ++c) {
    // this pass: list positions [c R, c R + n_act), n_act = the pass's own count (device scalar)
    const int32_t* rows = all_rows + (int64_t)c * w.R;
    const int32_t* n_act = w.n_pass > 1 ? pass_cnt + c : n_act_all;
    const int64_t Rc = std::min(w.R, N - (int64_t)c * w.R);       // rows the pass can hold at most
    // operand panel H^T [d][pitch] of the pass's tokens (dW contraction)
    if (!ht_in_setup) {
      k_transpose<stt><<<dim3((unsigned)(w.ldzt / 64), (unsigned)((d + 63) / 64)), dim3(256), 0, st>>>(
          reinterpret_cast<const stt*>(H), d, d, ht, rows, n_act);
      HIP_TRY(hipGetLastError());
    }
    if (c == 0) PHASE_EVENT(1);

    // recompute logits tile by tile, turn them into dz (rows / columns = list positions of the pass)
    DzArgs a;
    a.H = H; a.W = W; a.targets = targets; a.lse = lse; a.coef = coef; a.g = g; a.g_device = g_device; a.N = N; a.d = d; a.V = V;
    a.dz_scale = dz_scale;
    a.v_off = v_off;
    a.dz = dz; a.ldz = w.ldz; a.dzt = dzt; a.rows = rows; a.n_act = n_act;
    const Tile logits = dz_tile(Rc, V, d, kBf16);
    if constexpr (kBf16)
      s = (logits == TILE_256   ? launch_bwd_dz<Logits256>
           : logits == TILE_128 ? launch_bwd_dz<Bf16Loop128>
                                : launch_bwd_dz<Bf16Loop64>)(a, Rc, st);
    else
      s = (logits == TILE_128 ? launch_bwd_dz<F32Loop128> : launch_bwd_dz<F32Loop64>)(a, Rc, st);
    if (s != LLAMARL_OK) return s;
    if (c == 0) PHASE_EVENT(2);

    // dH [active rows, d] = dz [n_act,V] . W [V,d], scattered to the token rows.
    //   bf16: k-major operands dz^T [V][n_act] and W [V][d], K = V exactly
    //   fp32: K-contiguous operands dz [n_act][ldz] and W^T [d][ldz], K zero-padded to ldz
    float* part = reinterpret_cast<float*>(ws + w.off_part);
    const Tile dh_tile = store_tile(Rc, d, V, kBf16), dw_tile = store_tile(V, d, Rc, kBf16);
    StoreArgs h = {};
    h.M = Rc; h.Nn = d; h.C = dH; h.ldc = d; h.c_is_f32 = !kBf16; h.m_count = n_act; h.c_rows = rows; h.part = part; h.plan_out = plan;
    h.a_scale = dz_scale;
    if constexpr (kBf16) {
      h.A = dzt; h.packed_a = 1; h.pitch_count = n_act; h.B = W; h.ldb = d; h.K = V;
    } else {
      h.A = dz; h.lda = w.ldz; h.B = wt; h.ldb = w.ldz; h.K = w.ldz;
    }
    // dW [V,d] (+)= dz^T [V,n_act] . H^T[d,n_act]^T      (K = dz_columns(n_act), zero-padded); passes after
    // the first add to what the earlier ones stored
    StoreArgs o = {};
    o.A = dzt; o.B = ht; o.packed_a = o.packed_b = 1; o.pitch_count = o.k_count = n_act; o.M = V; o.Nn = d; o.K = w.ldzt;
    o.C = dW; o.ldc = d; o.c_is_f32 = dW_dt == LLAMARL_F32; o.accumulate = c == 0 ? accumulate_dW : 1; o.part = part;
    o.plan_out = plan + 4; o.a_scale = dz_scale;
    // bf16's dH reads W: a dW that is W itself (weights updated in place) is written when that is over
    const bool dw_over_w = kBf16 && overlap(W, V * d * 2, dW, V * d * (o.c_is_f32 ? 4 : 2));
    if (dh_tile != TILE_256 && dw_tile != TILE_256 && !dw_over_w) {
      const bool h128 = dh_tile == TILE_128, w128 = dw_tile == TILE_128;
      if (c == 0) PHASE_EVENT(3);
      if (c == 0) PHASE_EVENT(4);
      if constexpr (kBf16)
        s = (h128 ? (w128 ? launch_store_pair<Bf16LoopTN128, Bf16Loop128> : launch_store_pair<Bf16LoopTN128, Bf16Loop64>)
                  : (w128 ? launch_store_pair<Bf16LoopTN64, Bf16Loop128> : launch_store_pair<Bf16LoopTN64, Bf16Loop64>))(
            h, o, part, w.part, st);
      else
        s = (h128 ? (w128 ? launch_store_pair<F32Loop128, F32Loop128> : launch_store_pair<F32Loop128, F32Loop64>)
                  : (w128 ? launch_store_pair<F32Loop64, F32Loop128> : launch_store_pair<F32Loop64, F32Loop64>))(
            h, o, part, w.part, st);
      if (s != LLAMARL_OK) return s;
    } else if constexpr (kBf16) {                      // fp32 has no other tiles
      s = (dh_tile == TILE_256   ? launch_store<TileGemmTN>
           : dh_tile == TILE_128 ? launch_store<Bf16LoopTN128>
                                 : launch_store<Bf16LoopTN64>)(h, w.part, st);
      if (s != LLAMARL_OK) return s;
      if (c == 0) PHASE_EVENT(3);
      if (c == 0) PHASE_EVENT(4);
      s = (dw_tile == TILE_256   ? launch_store<Store256>
           : dw_tile == TILE_128 ? launch_store<Bf16Loop128>
                                 : launch_store<Bf16Loop64>)(o, w.part, st);
      if (s != LLAMARL_OK) return s;
    }
    if (c == 0) PHASE_EVENT(5);
  }
#undef PHASE_EVENT
  return LLAMARL_OK;
}

typedef void (*ceiling_traffic_kernel_t)(int, float*, const void*);
llamarl_status launch_ceiling_traffic(ceiling_traffic_kernel_t kernel, int grid, int iters, float* sink,
                                      const void* panels, hipStream_t st) {
  HIP_TRY(set_lds(kernel, MAINLOOP_LDS_BYTES));
  kernel<<<dim3((unsigned)grid), dim3(NTHREADS), MAINLOOP_LDS_BYTES, st>>>(iters, sink, panels);
  HIP_TRY(hipGetLastError());
  return LLAMARL_OK;
}

}  // namespace

extern "C" {

const char* llamarl_last_error(void) { return g_err; }
const char* llamarl_version(void) { return "llamarl-mi355x 0.1 (gfx950)"; }

size_t llamarl_workspace_bytes(int64_t N, int64_t d, int64_t V, llamarl_dtype dt, llamarl_pass pass) {
  if (N <= 0) return 0;
  switch (pass) {
    case LLAMARL_PASS_LOGPROBS:
      if (V <= 0) return 0;
      return fwd_ws(N, d, V, dt).total;
    case LLAMARL_PASS_LOSS_FWD:
      return loss_ws(N, N).total;     // sized for the worst case B = N
    case LLAMARL_PASS_LOSS_BWD:
      if (V <= 0 || d <= 0 || (dt != LLAMARL_F32 && dt != LLAMARL_BF16)) return 0;
      return bwd_ws(N, d, V, dt, 0).total;
    default:
      return 0;
  }
}

static llamarl_status logprobs_entry(const void* H, const void* W, const int32_t* targets, const uint8_t* mask, int64_t N,
                                     int64_t d, int64_t V, int64_t v_off, int64_t V_total, llamarl_dtype dt, int partial,
                                     float* out0, float* out1, float* out2, void* ws, size_t ws_bytes, void* stream) {
  if (!H || !W || !targets || !out0 || !out1 || (partial && !out2))
    return fail(LLAMARL_ERR_INVALID_ARG, "null pointer argument");
  llamarl_status s = check_head_shape(N, d, V, dt);
  if (s != LLAMARL_OK) return s;
  if (v_off < 0 || V_total >= ((int64_t)1 << 31) || v_off + V > V_total)
    return fail(LLAMARL_ERR_INVALID_ARG, "vocabulary slice [%lld, %lld) does not lie inside [0, %lld)", (long long)v_off,
                (long long)(v_off + V), (long long)V_total);
  if (!aligned16(H) || !aligned16(W)) return fail(LLAMARL_ERR_INVALID_ARG, "H and W must be 16-byte aligned");
  const size_t need = fwd_ws(N, d, V, dt).total;
  if (!ws || ws_bytes < need)
    return fail(LLAMARL_ERR_WORKSPACE, "workspace of %zu bytes given, %zu needed", ws ? ws_bytes : (size_t)0, need);
  if (!aligned16(ws)) return fail(LLAMARL_ERR_INVALID_ARG, "workspace must be 16-byte aligned");
  hipStream_t st = reinterpret_cast<hipStream_t>(stream);
  if (dt == LLAMARL_BF16)
    return run_logprobs<BF16>(H, W, targets, mask, N, d, V, v_off, V_total, partial, out0, out1, out2,
                              reinterpret_cast<char*>(ws), st);
  return run_logprobs<F32>(H, W, targets, mask, N, d, V, v_off, V_total, partial, out0, out1, out2,
                           reinterpret_cast<char*>(ws), st);
}

llamarl_status llamarl_token_logprobs(const void* H, const void* W, const int32_t* targets, const uint8_t* mask,
                                      int64_t N, int64_t d, int64_t V, llamarl_dtype dt, float* logp, float* lse,
                                      void* ws, size_t ws_bytes, void* stream) {
  return logprobs_entry(H, W, targets, mask, N, d, V, 0, V, dt, 0, logp, lse, nullptr, ws, ws_bytes, stream);
}

llamarl_status llamarl_token_logprobs_partial(const void* H, const void* W_slice, const int32_t* targets,
                                              const uint8_t* mask, int64_t N, int64_t d, int64_t V_slice, int64_t v0,
                                              int64_t V_total, llamarl_dtype dt, float* m, float* s, float* zt,
                                              void* ws, size_t ws_bytes, void* stream) {
  return logprobs_entry(H, W_slice, targets, mask, N, d, V_slice, v0, V_total, dt, 1, m, s, zt, ws, ws_bytes, stream);
}

llamarl_status llamarl_merge_partials(const float* m, const float* s, const float* zt, int shards, int64_t N,
                                      float* logp, float* lse, void* stream) {
  if (!m || !s || !zt || !logp || !lse) return fail(LLAMARL_ERR_INVALID_ARG, "null pointer argument");
  if (shards <= 0 || N <= 0) return fail(LLAMARL_ERR_INVALID_ARG, "shards and N must be positive");
  if (N >= ((int64_t)1 << 39)) return fail(LLAMARL_ERR_UNSUPPORTED, "too many tokens");
  k_merge_shards<<<dim3((unsigned)std::min((N + 255) / 256, LAUNCH_BLOCKS)), dim3(256), 0, reinterpret_cast<hipStream_t>(stream)>>>(
      m, s, zt, shards, N, logp, lse);
  HIP_TRY(hipGetLastError());
  return LLAMARL_OK;
}

static llamarl_status check_loss_args(const float* logp, const float* mu_logp, const float* adv, const uint8_t* mask,
                                      const int32_t* targets, int64_t V, int64_t B, int64_t T,
                                      const llamarl_loss_params* p, const float* loss, const float* coef,
                                      const float* stats) {
  if (!logp || !mu_logp || !adv || !p || !loss || !coef || !stats)
    return fail(LLAMARL_ERR_INVALID_ARG, "null pointer argument");
  if (B <= 0 || T <= 0) return fail(LLAMARL_ERR_INVALID_ARG, "B and T must be positive");
  if (B >= ((int64_t)1 << 31) || T >= ((int64_t)1 << 31) || B * T >= ((int64_t)1 << 40))
    return fail(LLAMARL_ERR_UNSUPPORTED, "batch too large");
  if (p->clip_mode != LLAMARL_CLIP_AIPO && p->clip_mode != LLAMARL_CLIP_PPO)
    return fail(LLAMARL_ERR_INVALID_ARG, "unknown clip_mode %d", p->clip_mode);
  if (p->norm_mode < 0 || p->norm_mode > 2) return fail(LLAMARL_ERR_INVALID_ARG, "unknown norm_mode %d", p->norm_mode);
  if (p->clip_mode == LLAMARL_CLIP_AIPO && !(p->rho > 0.f))
    return fail(LLAMARL_ERR_INVALID_ARG, "rho must be positive (got %g)", (double)p->rho);
  if (p->clip_mode == LLAMARL_CLIP_PPO && (!(p->eps_lo >= 0.f) || !(p->eps_hi >= 0.f) || p->eps_lo > 1.f))
    return fail(LLAMARL_ERR_INVALID_ARG, "PPO mode needs 0 <= eps_lo <= 1 and eps_hi >= 0");
  if (targets && V <= 0) return fail(LLAMARL_ERR_INVALID_ARG, "targets given but V <= 0");
  if (!aligned16(logp) || !aligned16(mu_logp) || !aligned16(coef) || !aligned16(adv) || !aligned16(targets) ||
      (reinterpret_cast<uintptr_t>(mask) & 3u) != 0)
    return fail(LLAMARL_ERR_INVALID_ARG, "logp, mu_logp, adv, targets and coef must be 16-byte aligned, mask 4-byte");
  return LLAMARL_OK;
}

// the launches of the loss forward; wsb holds a LossWs layout for (B*T, B)
static llamarl_status launch_loss_fwd(const float* logp, const float* mu_logp, const float* adv, int adv_per_token,
                                      const uint8_t* mask, const int32_t* targets, int64_t V, int64_t B, int64_t T,
                                      const llamarl_loss_params* p, float* loss, float* coef, float* stats, char* wsb,
                                      const LossWs& w, hipStream_t st) {
  LossArgs a;
  a.logp = logp; a.mu_logp = mu_logp; a.adv = adv; a.mask = mask; a.targets = targets; a.V = V; a.B = B; a.T = T;
  a.adv_per_token = adv_per_token; a.rho = p->rho; a.clip_mode = p->clip_mode; a.eps_lo = p->eps_lo;
  a.eps_hi = p->eps_hi; a.norm_mode = p->norm_mode;
  a.seq_len = reinterpret_cast<int32_t*>(wsb + w.off_len);
  a.seq_bad = reinterpret_cast<int32_t*>(wsb + w.off_bad);
  a.partials = reinterpret_cast<double*>(wsb + w.off_part);
  a.ticket = reinterpret_cast<unsigned int*>(wsb + w.off_ticket);
  a.nblocks = w.nblocks; a.coef = coef; a.loss = loss; a.stats = stats;
  if (B <= LOSS_SMALL_GENERATIONS && B * T <= LOSS_SMALL_TOKENS) {
    k_loss_small<<<dim3(1), dim3(LOSS_SMALL_THREADS), 0, st>>>(a);
    HIP_TRY(hipGetLastError());
    return LLAMARL_OK;
  }
  const int seq_threads = T > 4096 ? 1024 : 256;
  for (int64_t b = 0; b < B; b += LAUNCH_BLOCKS) {
    LossArgs part = a;
    part.B = std::min(B - b, LAUNCH_BLOCKS);
    if (mask) part.mask += b * T;
    if (targets) part.targets += b * T;
    part.seq_len += b;
    part.seq_bad += b;
    (seq_threads == 1024 ? k_seq_lengths<1024> : k_seq_lengths<256>)<<<dim3((unsigned)part.B), dim3((unsigned)seq_threads), 0,
                                                                       st>>>(part);   // also clears the ticket
    HIP_TRY(hipGetLastError());
  }
  (w.threads == 1024 ? k_loss_tokens<1024> : k_loss_tokens<256>)<<<dim3((unsigned)w.nblocks), dim3((unsigned)w.threads), 0,
                                                                   st>>>(a);   // its last block writes loss, stats
  HIP_TRY(hipGetLastError());
  return LLAMARL_OK;
}

llamarl_status llamarl_offpolicy_loss_fwd(const float* logp, const float* mu_logp, const float* adv,
                                          int adv_per_token, const uint8_t* mask, const int32_t* targets, int64_t V,
                                          int64_t B, int64_t T, const llamarl_loss_params* p, float* loss,
                                          float* coef, float* stats, void* ws, size_t ws_bytes, void* stream) {
  llamarl_status s = check_loss_args(logp, mu_logp, adv, mask, targets, V, B, T, p, loss, coef, stats);
  if (s != LLAMARL_OK) return s;
  const LossWs w = loss_ws(B * T, B);
  if (!ws || ws_bytes < w.total)
    return fail(LLAMARL_ERR_WORKSPACE, "workspace of %zu bytes given, %zu needed", ws ? ws_bytes : (size_t)0, w.total);
  if (!aligned16(ws)) return fail(LLAMARL_ERR_INVALID_ARG, "workspace must be 16-byte aligned");
  return launch_loss_fwd(logp, mu_logp, adv, adv_per_token, mask, targets, V, B, T, p, loss, coef, stats,
                         reinterpret_cast<char*>(ws), w, reinterpret_cast<hipStream_t>(stream));
}

// Device address of this GPU's copy of `scratch` (each GPU has its own, at its own address).
static llamarl_status scratch_of_current_device(char** out) {
  int dev = -1;
  HIP_TRY(hipGetDevice(&dev));
  if (dev < 0 || dev >= STATIC_MAX_DEVICES) return fail(LLAMARL_ERR_UNSUPPORTED, "device ordinal %d not supported", dev);
  std::lock_guard<std::mutex> lock(g_scratch_mutex);
  if (g_scratch_ptr[dev] == nullptr) {
    void* p = nullptr;
    HIP_TRY(hipGetSymbolAddress(&p, HIP_SYMBOL(scratch)));
    if (p == nullptr) return fail(LLAMARL_ERR_HIP, "hipGetSymbolAddress returned a null address");
    g_scratch_ptr[dev] = p;
  }
  *out = static_cast<char*>(g_scratch_ptr[dev]);
  return LLAMARL_OK;
}

llamarl_status llamarl_offpolicy_loss_fwd_static(const float* logp, const float* mu_logp, const float* adv,
                                                 int adv_per_token, const uint8_t* mask, const int32_t* targets,
                                                 int64_t V, int64_t B, int64_t T, const llamarl_loss_params* p,
                                                 float* loss, float* coef, float* stats, void* stream) {
  llamarl_status s = check_loss_args(logp, mu_logp, adv, mask, targets, V, B, T, p, loss, coef, stats);
  if (s != LLAMARL_OK) return s;
  if (B > STATIC_MAX_GENERATIONS || B * T > STATIC_MAX_TOKENS)
    return fail(LLAMARL_ERR_UNSUPPORTED,
                "B = %lld, B*T = %lld exceed the static scratch of this entry point (at most %lld generations, %lld "
                "tokens): use llamarl_offpolicy_loss_fwd with a workspace",
                (long long)B, (long long)(B * T), (long long)STATIC_MAX_GENERATIONS, (long long)STATIC_MAX_TOKENS);
  const LossWs w = loss_ws(B * T, B);
  if (w.total > STATIC_SCRATCH_BYTES) return fail(LLAMARL_ERR_UNSUPPORTED, "static scratch too small for this batch");
  char* base = nullptr;
  s = scratch_of_current_device(&base);
  if (s != LLAMARL_OK) return s;
  // nothing in the scratch has to start at zero: k_seq_lengths overwrites the counters and clears the ticket
  return launch_loss_fwd(logp, mu_logp, adv, adv_per_token, mask, targets, V, B, T, p, loss, coef, stats, base, w,
                         reinterpret_cast<hipStream_t>(stream));
}

static llamarl_status bwd_entry(const void* H, const void* W, const int32_t* targets, const float* lse,
                                const float* coef, float grad_loss, const float* grad_loss_device, int64_t N,
                                int64_t d, int64_t V, int64_t v_off, llamarl_dtype dt, void* dH, void* dW, llamarl_dtype dW_dt, int accumulate_dW,
                                int64_t max_rows_per_pass, void* ws, size_t ws_bytes, void* stream, void* const* ev) {
  if (!H || !W || !targets || !lse || !coef || !dH || !dW) return fail(LLAMARL_ERR_INVALID_ARG, "null pointer argument");
  llamarl_status s = check_head_shape(N, d, V, dt);
  if (s != LLAMARL_OK) return s;
  if (dW_dt != LLAMARL_F32 && dW_dt != dt)
    return fail(LLAMARL_ERR_INVALID_ARG, "dW_dt must be LLAMARL_F32 or equal to dt");
  if (!aligned16(H) || !aligned16(W) || !aligned16(dH) || !aligned16(dW))
    return fail(LLAMARL_ERR_INVALID_ARG, "H, W, dH, dW must be 16-byte aligned");
  if (!std::isfinite(grad_loss)) return fail(LLAMARL_ERR_INVALID_ARG, "grad_loss must be finite");
  if (v_off < 0 || v_off + V >= ((int64_t)1 << 31)) return fail(LLAMARL_ERR_INVALID_ARG, "bad vocabulary offset");
  if (max_rows_per_pass < 0) return fail(LLAMARL_ERR_INVALID_ARG, "max_rows_per_pass must not be negative");
  const size_t need = bwd_ws(N, d, V, dt, max_rows_per_pass).total;
  if (!ws || ws_bytes < need)
    return fail(LLAMARL_ERR_WORKSPACE, "workspace of %zu bytes given, %zu needed", ws ? ws_bytes : (size_t)0, need);
  if (!aligned16(ws)) return fail(LLAMARL_ERR_INVALID_ARG, "workspace must be 16-byte aligned");
  hipStream_t st = reinterpret_cast<hipStream_t>(stream);
  if (dt == LLAMARL_BF16)
    return run_bwd<BF16>(H, W, targets, lse, coef, grad_loss, grad_loss_device, N, d, V, v_off, dt, dH, dW, dW_dt, accumulate_dW,
                         max_rows_per_pass,
                         reinterpret_cast<char*>(ws), st, ev);
  return run_bwd<F32>(H, W, targets, lse, coef, grad_loss, grad_loss_device, N, d, V, v_off, dt, dH, dW, dW_dt, accumulate_dW,
                      max_rows_per_pass,
                      reinterpret_cast<char*>(ws), st, ev);
}

llamarl_status llamarl_offpolicy_loss_bwd(const void* H, const void* W, const int32_t* targets, const float* lse,
                                          const float* coef, float grad_loss, int64_t N, int64_t d, int64_t V,
                                          llamarl_dtype dt, void* dH, void* dW, llamarl_dtype dW_dt,
                                          int accumulate_dW, void* ws, size_t ws_bytes, void* stream) {
  return bwd_entry(H, W, targets, lse, coef, grad_loss, nullptr, N, d, V, 0, dt, dH, dW, dW_dt, accumulate_dW, 0, ws, ws_bytes,
                   stream, nullptr);
}

llamarl_status llamarl_offpolicy_loss_bwd_device_scale(const void* H, const void* W, const int32_t* targets,
                                                       const float* lse, const float* coef, const float* grad_loss,
                                                       int64_t N, int64_t d, int64_t V, llamarl_dtype dt, void* dH,
                                                       void* dW, llamarl_dtype dW_dt, int accumulate_dW, void* ws,
                                                       size_t ws_bytes, void* stream) {
  if (!grad_loss || (reinterpret_cast<uintptr_t>(grad_loss) & 3u) != 0)
    return fail(LLAMARL_ERR_INVALID_ARG, "grad_loss must be a 4-byte aligned device pointer");
  return bwd_entry(H, W, targets, lse, coef, 1.f, grad_loss, N, d, V, 0, dt, dH, dW, dW_dt, accumulate_dW, 0, ws,
                   ws_bytes, stream, nullptr);
}

size_t llamarl_bwd_workspace_bytes(int64_t N, int64_t d, int64_t V, llamarl_dtype dt, int64_t max_rows_per_pass) {
  if (N <= 0 || V <= 0 || d <= 0 || max_rows_per_pass < 0 || (dt != LLAMARL_F32 && dt != LLAMARL_BF16)) return 0;
  return bwd_ws(N, d, V, dt, max_rows_per_pass).total;
}

llamarl_status llamarl_offpolicy_loss_bwd_chunked(const void* H, const void* W, const int32_t* targets,
                                                  const float* lse, const float* coef, float grad_loss, int64_t N,
                                                  int64_t d, int64_t V, llamarl_dtype dt, void* dH, void* dW,
                                                  llamarl_dtype dW_dt, int accumulate_dW, int64_t max_rows_per_pass,
                                                  void* ws, size_t ws_bytes, void* stream) {
  return bwd_entry(H, W, targets, lse, coef, grad_loss, nullptr, N, d, V, 0, dt, dH, dW, dW_dt, accumulate_dW, max_rows_per_pass,
                   ws, ws_bytes, stream, nullptr);
}

llamarl_status llamarl_offpolicy_loss_bwd_slice(const void* H, const void* W_slice, const int32_t* targets,
                                                const float* lse, const float* coef, float grad_loss, int64_t N,
                                                int64_t d, int64_t V_slice, int64_t v0, llamarl_dtype dt,
                                                void* dH_partial, void* dW_slice, llamarl_dtype dW_dt,
                                                int accumulate_dW, void* ws, size_t ws_bytes, void* stream) {
  return bwd_entry(H, W_slice, targets, lse, coef, grad_loss, nullptr, N, d, V_slice, v0, dt, dH_partial, dW_slice, dW_dt,
                   accumulate_dW, 0, ws, ws_bytes, stream, nullptr);
}

llamarl_status llamarl_offpolicy_loss_bwd_phases(const void* H, const void* W, const int32_t* targets,
                                                 const float* lse, const float* coef, float grad_loss, int64_t N,
                                                 int64_t d, int64_t V, llamarl_dtype dt, void* dH, void* dW,
                                                 llamarl_dtype dW_dt, int accumulate_dW, void* ws, size_t ws_bytes,
                                                 void* stream, void* const* phase_events) {
  if (!phase_events) return fail(LLAMARL_ERR_INVALID_ARG, "phase_events is null");
  for (int i = 0; i < 6; ++i)
    if (!phase_events[i]) return fail(LLAMARL_ERR_INVALID_ARG, "phase_events[%d] is null", i);
  return bwd_entry(H, W, targets, lse, coef, grad_loss, nullptr, N, d, V, 0, dt, dH, dW, dW_dt, accumulate_dW, 0, ws, ws_bytes,
                   stream, phase_events);
}

llamarl_status llamarl_mfma_ceiling(int iters, float* sink, double* flops, void* stream) {
  if (!sink || !flops) return fail(LLAMARL_ERR_INVALID_ARG, "null pointer argument");
  if (iters <= 0) return fail(LLAMARL_ERR_INVALID_ARG, "iters must be positive");
  const int grid = persistent_grid((int64_t)1 << 30);      // one workgroup per CU
  k_mfma_ceiling<<<dim3((unsigned)grid), dim3(NTHREADS), 0, reinterpret_cast<hipStream_t>(stream)>>>(iters, sink);
  HIP_TRY(hipGetLastError());
  // 16x16x32 MFMA = 2 * 16 * 16 * 32 flop; CEILING_MB x CEILING_NB of them per k-step and wavefront
  *flops = (double)grid * (NTHREADS / 64) * (double)iters * CEILING_KSTEPS_PER_ITER * (CEILING_MB * CEILING_NB) * (2.0 * 16 * 16 * 32);
  return LLAMARL_OK;
}

llamarl_status llamarl_mfma_ceiling_traffic(int traffic, int iters, const void* panels, size_t panel_bytes,
                                            float* sink, double* flops, void* stream) {
  if (!sink || !flops || !panels) return fail(LLAMARL_ERR_INVALID_ARG, "null pointer argument");
  if (iters <= 0) return fail(LLAMARL_ERR_INVALID_ARG, "iters must be positive");
  if (traffic < 0 || traffic > 3) return fail(LLAMARL_ERR_INVALID_ARG, "traffic must be 0 .. 3");
  if (panel_bytes < CEILING_PANEL_BYTES || !aligned16(panels))
    return fail(LLAMARL_ERR_INVALID_ARG, "panels must be 16-byte aligned and hold %zu bytes (got %zu)",
                CEILING_PANEL_BYTES, panel_bytes);
  const int grid = persistent_grid((int64_t)1 << 30);      // one workgroup per CU
  hipStream_t st = reinterpret_cast<hipStream_t>(stream);
  static const ceiling_traffic_kernel_t kernels[4] = {k_mfma_ceiling_schedule, k_mfma_ceiling_lds_reads,
                                                      k_mfma_ceiling_slab_loads, k_mfma_ceiling_reads_and_loads};
  const llamarl_status s = launch_ceiling_traffic(kernels[traffic], grid, iters, sink, panels, st);
  if (s != LLAMARL_OK) return s;
  *flops = (double)grid * (NTHREADS / 64) * (double)iters * CEILING_KSTEPS_PER_ITER * (CEILING_MB * CEILING_NB) * (2.0 * 16 * 16 * 32);
  return LLAMARL_OK;
}

llamarl_status llamarl_group_advantages(const float* rewards, int64_t P, int64_t n, int normalise_std, float eps,
                                        float* adv, void* stream) {
  if (!rewards || !adv) return fail(LLAMARL_ERR_INVALID_ARG, "null pointer argument");
  if (P <= 0 || n <= 0) return fail(LLAMARL_ERR_INVALID_ARG, "P and n must be positive");
  if (P >= ((int64_t)1 << 31) * 4) return fail(LLAMARL_ERR_UNSUPPORTED, "too many prompts");
  if (normalise_std && !(eps >= 0.f)) return fail(LLAMARL_ERR_INVALID_ARG, "eps must be non-negative");
  for (int64_t p = 0; p < P; p += LAUNCH_BLOCKS * 4) {
    const int64_t prompts = std::min(P - p, LAUNCH_BLOCKS * 4);
    k_group_advantages<<<dim3((unsigned)((prompts + 3) / 4)), dim3(256), 0, reinterpret_cast<hipStream_t>(stream)>>>(
        rewards + p * n, prompts, n, normalise_std, eps, adv + p * n);
    HIP_TRY(hipGetLastError());
  }
  return LLAMARL_OK;
}

llamarl_status llamarl_kl_shaped_rewards(const float* rewards, const float* logp, const float* base_logp,
                                         const uint8_t* mask, int64_t B, int64_t T, float lambda_kl, float* shaped,
                                         float* kl, void* stream) {
  if (!rewards || !logp || !base_logp || !shaped) return fail(LLAMARL_ERR_INVALID_ARG, "null pointer argument");
  if (B <= 0 || T <= 0) return fail(LLAMARL_ERR_INVALID_ARG, "B and T must be positive");
  if (B >= (int64_t)1 << 31) return fail(LLAMARL_ERR_UNSUPPORTED, "too many generations");
  if (!(lambda_kl == lambda_kl)) return fail(LLAMARL_ERR_INVALID_ARG, "lambda_kl is NaN");
  const int aligned = aligned16(logp) && aligned16(base_logp) && (reinterpret_cast<uintptr_t>(mask) & 3u) == 0;
  const int threads = T > 2048 ? 1024 : 256;
  for (int64_t b = 0; b < B; b += LAUNCH_BLOCKS) {
    const int64_t n = std::min(B - b, LAUNCH_BLOCKS), t = b * T;
    (threads == 1024 ? k_kl_shaped_rewards<1024> : k_kl_shaped_rewards<256>)<<<
        dim3((unsigned)n), dim3((unsigned)threads), 0, reinterpret_cast<hipStream_t>(stream)>>>(
        rewards + b, logp + t, base_logp + t, mask ? mask + t : nullptr, n, T, aligned, lambda_kl, shaped + b,
        kl ? kl + b : nullptr);
    HIP_TRY(hipGetLastError());
  }
  return LLAMARL_OK;
}

}  // extern "C"
