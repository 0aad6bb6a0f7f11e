// tile_rules.h -- which tiles a contraction is cut into and who takes which: plain arithmetic, the same in the kernels, in the
// host code that launches them and in native.cpp, through which the tests ask for it without a GPU.
#pragma once
#include <stdint.h>

#ifdef __HIP__
#define LLAMARL_RULE __host__ __device__ __forceinline__
#else
#define LLAMARL_RULE inline
#endif

namespace llamarl {

// Patch rows of the logits kernels (TileSchedule::init), measured at the Llama-3-8B shape with patches dealt round-robin over
// the XCDs: 4 and 8 tie (2: +1 %).
constexpr int PATCH_ROWS_LOGITS = 4;

// Persistent tile schedule.  The grid has one workgroup per CU (every tile is taken once by a grid of any size;
// tests/test_tile_rules.py walks them on the CPU); the hardware deals workgroups round-robin to the 8 XCDs, each with a private L2.  Tile ids are ordered so that 32 consecutive ones form a patch
// (group_m x 32/group_m tiles) that shares A and B panels; the workgroups of one XCD take one patch at a time, so
// those panels are shared in its L2, and the eight patches in flight on the chip are consecutive in id order, so
// they share panels through the Infinity Cache (against giving every XCD a contiguous eighth of the ids: -3.5 %
// step time, -6.5 % for the dH contraction whose two operands both stream from HBM).  tiles_m x tiles_n is the
// number of tiles that exist once the device-side active-row count is known.
template <int GROUP_M>     // rows of a patch
struct TileSchedule {
  int tiles_m, tiles_n;
  int next_id, end_id, stride;
  bool turn;               // see take
  int group, in_group;     // of next_id: its group of GROUP_M rows of tiles, and its place there
  int group_step, in_group_step, round;
  // The 32 workgroups of an XCD work on 32 consecutive ids = GROUP_M x (32 / GROUP_M)
  // tiles, which load GROUP_M A panels and 32 / GROUP_M B panels: a B panel is shared by GROUP_M tiles, an A panel
  // by 32 / GROUP_M.  Give the larger share to the operand that has to come from HBM.
  LLAMARL_RULE void init(int tiles_m_, int tiles_n_, int bid, int nblk) {
    tiles_m = tiles_m_;
    tiles_n = tiles_n_;
    const int ntiles = tiles_m * tiles_n;
    const int xcd = bid & 7, local = bid >> 3;
    turn = (nblk & 7) == 0 && nblk % (GROUP_M * tiles_n) == 0;
    if ((nblk & 7) == 0 || nblk < 8) {
      // Patches dealt round-robin over the XCDs: in round k XCD x works on patch 8 k + x, so the eight patches in
      // flight are neighbours in id order and share operand panels through the Infinity Cache.
      const int per = nblk >> 3;                            // workgroups per XCD = tiles per patch
      next_id = nblk < 8 ? bid : xcd * per + local;         // few: not every XCD has a workgroup
      stride = nblk;
      end_id = ntiles;
    } else {
      const int base = ntiles >> 3, rem = ntiles & 7;
      const int start = xcd * base + (xcd < rem ? xcd : rem);
      end_id = start + base + (xcd < rem ? 1 : 0);
      next_id = start + local;
      stride = (nblk >> 3) + ((nblk & 7) > xcd ? 1 : 0);    // workgroups of this grid that sit on my XCD
    }
    const int per_group = GROUP_M * tiles_n;
    group = next_id / per_group;
    in_group = next_id - group * per_group;
    group_step = stride / per_group;
    in_group_step = stride - group_step * per_group;
    round = 0;
  }
  LLAMARL_RULE bool has_tile() const { return next_id < end_id; }
  // coordinates of the next tile; advance.  No division while the group is whole: this stands in every tile's epilogue.
  LLAMARL_RULE void take(int& tm, int& tn) {
    const int first_m = group * GROUP_M, left = tiles_m - first_m, gsize = left < GROUP_M ? left : GROUP_M;
    tn = gsize == GROUP_M ? in_group / GROUP_M : in_group / gsize;
    tm = first_m + in_group - tn * gsize;
    // Where a round of the grid is a whole number of groups, a workgroup would get the same column in every round:
    // turn the columns by one a round (a whole group is in one round, so each of its tiles is still taken once), so that
    // nobody is left with all the narrow last columns (two columns, 300 tokens: half of the workgroups had four full tiles, the other half four of 44 tokens).
    if (turn) tn = (tn + round) % tiles_n;
    ++round;
    next_id += stride;
    group += group_step;
    in_group += in_group_step;
    const int per_group = GROUP_M * tiles_n;
    if (in_group >= per_group) {
      in_group -= per_group;
      ++group;
    }
  }
};

// Tiles of at most NARROW_BN columns: three resident slabs instead of two.
constexpr int NARROW_BN = 160;
// Which tiles a logits kernel of 256 vocabulary rows takes: 256 columns wide, 128 or 160 (TileGemmNarrow), or, in the forward,
// 320 (TileGemmWide), by what the rounds of the grid cost.  Costs in 1/256 of the time of a slab of the 256 x 256 forward
// (1.4 us), for 128, 160, 256 and 320 columns, measured over (6720, 128256, 512 .. 2048):
//   slab, tile      a slab of d; what a tile costs besides (dz stores its tile, in partial lines where it is narrow)
//   unaligned       rows of d that are no multiple of 128 bytes: a slab row touches two lines, and the requests bound a slab
//   one, two, few   W comes from HBM: a slab where there are 1, 2 or 3 - 4 columns of tiles (more share W in the caches)
// 320 columns read a tenth less per product from LDS and L2 and have a fifth fewer tiles to wait for.  Long contractions, which the
// power limit bounds, hardly gain (7600 .. 10600 tokens of a 128256 x 4096 head: -3 .. +3 % of 256 columns, by the tokens that fill
// the last column); few rounds do where a fifth fewer tiles fit them, and one or two columns that read W once.  As much at
// short K, 320 columns against the best of the others: (300, 49200, 72) 21.0 / 19.3 us, (320, 128256, 128) 32.5 / 29.2, (3200, 50304, 128) 101 / 73,
// (600, 128256, 256) 62.4 / 55.6, (8000, 33001, 264) 170 / 167, (300, 49200, 520) 36.4 / 34.1, (2300, 16032, 576) 56.2 / 50.7; worse
// at one of 86 such sizes by more than 3 %: (1600, 32000, 520) 70.7 / 73.7.
// Forward at (N, V, d), 320 / 256 / 160 / 128 columns, us: (150, 128256, 4096) 223 / 230 / 188 / 248, (225, ..) 266 / 246 / 272 / 269,
// (300, ..) 279 / 366 / 304 / 364, (450, ..) 434 / 426 / 423 / 475, (600, ..) 500 / 550 / 524 / 592, (1250, ..) 955 / 991 / 1044 / 1128,
// (8576, ..) 6190 / 6348 / 6849 / 7153; (7125, 33001, 1032) 400 / 428 / 465 / 508; (2300, 16032, 8192) 449 / 540 / 486 / 529;
// (2012, 16032, 8192) 442 / 388 / 464 / 450; (640, 128256, 776) 118 / 127 / 134 / 148.  dz, 256 / 160 / 128: (150, 128256, 4096) 261 / 231 / 267,
// (225, ..) 265 / 277 / 280, (450, ..) 442 / 429 / 480, (600, ..) 560 / 526 / 597.
constexpr int WIDTHS = 4, LOGITS_WIDTHS[WIDTHS] = {128, 160, 256, 320};
struct WidthCosts {
  int widths, slab[WIDTHS], tile[WIDTHS], one[WIDTHS], two[WIDTHS], few[WIDTHS];       // the first `widths` of them
};
constexpr WidthCosts FWD_COSTS = {4, {167, 184, 256, 318}, {328, 474, 765, 1000}, {235, 240, 315, 365}, {185, 200, 300, 330}, {0, 0, 300, 0}};
constexpr WidthCosts DZ_COSTS = {3, {177, 201, 261}, {440, 640, 1000}, {318, 318, 363}, {193, 206, 300}, {0, 0, 300}};
constexpr int UNALIGNED_SLAB[WIDTHS] = {220, 239, 294, 355};
struct LogitsWidth {
  int width;
  int64_t cost;
};
LLAMARL_RULE LogitsWidth logits_width(const WidthCosts& c, int tiles_v, int n_act, int64_t d, int grid) {
  const int nk = (int)((d + 63) / 64);
  // Every workgroup does this before anything else.  All widths together, without branches: the divisions by the grid share one
  // reciprocal; one after the other they were 0.1 us of a forward call.
  int cols[WIDTHS];
  uint32_t rounds[WIDTHS];
  bool fits[WIDTHS];
#pragma unroll
  for (int h = 0; h < WIDTHS; ++h) {
    cols[h] = (int)((uint32_t)(n_act + LOGITS_WIDTHS[h] - 1) / (uint32_t)LOGITS_WIDTHS[h]);
    const int64_t tiles = (int64_t)tiles_v * cols[h];
    fits[h] = tiles + grid < (1ll << 31);                    // 32-bit division; so many rounds are 256 wide
    rounds[h] = ((uint32_t)tiles + (uint32_t)grid - 1u) / (uint32_t)grid;
  }
  LogitsWidth best = {256, 0};
#pragma unroll
  for (int i = 0; i < WIDTHS; ++i) {
    const int h = i == 0 ? 2 : i == 3 ? 3 : 2 - i;           // 256 columns, then whatever costs less
    if (h >= c.widths) continue;
    int slab = c.slab[h];
    slab = d % 64 != 0 && slab < UNALIGNED_SLAB[h] ? UNALIGNED_SLAB[h] : slab;
    const int stream = cols[h] == 1 ? c.one[h] : cols[h] == 2 ? c.two[h] : cols[h] <= 4 ? c.few[h] : 0;
    slab = slab < stream ? stream : slab;
    const int64_t cost = (int64_t)rounds[h] * (nk * slab + c.tile[h]);
    const bool take = fits[h] & ((i == 0) | ((best.cost != 0) & (cost < best.cost)));
    best.width = take ? LOGITS_WIDTHS[h] : best.width;
    best.cost = take ? cost : best.cost;
  }
  return best;
}
LLAMARL_RULE LogitsWidth fwd_width(int tiles_v, int n_act, int64_t d, int grid) {
  return logits_width(FWD_COSTS, tiles_v, n_act, d, grid);
}
LLAMARL_RULE LogitsWidth dz_width(int tiles_v, int n_act, int64_t d, int grid) {
  return logits_width(DZ_COSTS, tiles_v, n_act, d, grid);
}
// Columns of dz^T, zeros past the active rows, that the dW contraction reads: the next 32 in bf16, half of its last slab.  Every
// width is a multiple of that, so the columns of tiles that hold tokens write all of it.  Up to the next 64, tiles 160 wide
// needed one more of zeros for 129 .. 160 rows, which the costs did not see.
// dz at (150, 128256, d) before / now: d = 512 47 / 40 us, 1024 88 / 84, 4096 296 / 271 (on 256 columns 46, 89 and 301);
// (470, 33000, 1024) 55.5 / 45, (780, 128256, 512) 140 / 134.
LLAMARL_RULE int dz_columns(int n_act, bool bf16) { return bf16 ? (n_act + 31) / 32 * 32 : (n_act + 63) / 64 * 64; }

// ---- which main loop a contraction runs on ---------------------------------------------------------------
// The choice depends on host-side sizes only (workspace sizes follow from it).  A large contraction runs fastest on the
// largest tiles (bf16: 256 x 256, 1.2 - 1.3 times as fast as 128 x 128 when both fill the chip), a small one on the
// tiles that give most CUs something to do.
enum Tile { TILE_256, TILE_128, TILE_64 };
LLAMARL_RULE int tile_edge(Tile t) { return t == TILE_256 ? 256 : t == TILE_128 ? 128 : 64; }
LLAMARL_RULE int64_t tile_count(int64_t rows, int64_t cols, int64_t edge) {
  return ((rows + edge - 1) / edge) * ((cols + edge - 1) / edge);
}
// Logits kernels (forward, recompute): N x V outputs.  bf16 takes tiles of 256 vocabulary rows where 256 x 256 ones come to
// LOGITS_MIN_TILES, and below that where they cost less in rounds of the grid than 128 x 128 ones: a round of those takes the
// slabs of two workgroups a CU, or of one where less than half of it is left, and a tile's remainder; `launch` is what the
// first round takes less (their epilogues cover each other).  128 x 128 ones win where K is short, in dz up to longer K: narrow
// tiles leave it partial lines to write.  Forward call / dz at (N, V, d), 256 rows : 128 x 128, us:
//   (882, 10487, 7808) 127 : 204 / 129 : 226    (1700, 5412, 1888) 43 : 67 / 40 : 64       (1024, 8192, 1024) 27.2 : 28.3 / 24.6 : 24.0
//   (1024, 8192, 256) 16.3 : 15.6 / 15.4 : 13.0 (2048, 4096, 264) 18.0 : 17.6 / 17.1 : 14.6 (512, 12000, 2048) 35.6 : 38.0 / 32.3 : 34.0
//   (256, 33000, 1024) 38.5 : 35.3 / 37.6 : 31.5 (600, 7000, 512) 18.6 : 18.0 / 18.0 : 15.5 (512, 24000, 1024) 36.8 : 43.2 / 33.8 : 38.6
//   bf16, dz at (N, V, d) on 128- / 64-tiles: (512, 2048, 512) 16 / 12 us, (512, 8192, 1024) 18 / 22, (1041, 5003, 520) 18 / 26.
//   fp32, dz on 128- / 64-tiles: (512, 2048, 512) 44 / 26 us, (512, 4096, 512) 45 / 34, (1024, 4096, 512) 48 / 57,
//   (2048, 8192, 512) 127 / 206.
constexpr int LOGITS_MIN_TILES = 192, LOGITS_MIN_TILES_BF16_128 = 128;   // of the larger edge; fewer: the next smaller one
struct SmallCosts {       // of 128 x 128 tiles, in logits_width's units
  int slab_two, slab_one, tile, launch;
};
constexpr SmallCosts FWD_SMALL = {186, 131, 550, 400}, DZ_SMALL = {202, 142, 400, 500};
LLAMARL_RULE Tile logits_tile_by(const SmallCosts& c, const WidthCosts& wide, int64_t N, int64_t V, int64_t d, bool bf16) {
  const int64_t t128 = tile_count(N, V, 128);
  if (bf16) {
    const int64_t tiles_v = (V + 255) / 256;
    if (tile_count(N, V, 256) >= LOGITS_MIN_TILES) return TILE_256;
    if (tiles_v * ((N + 127) / 128) >= LOGITS_MIN_TILES_BF16_128) {
      const int64_t nk = (d + 63) / 64, full = t128 / 512, left = t128 % 512;
      const int64_t last = left == 0 ? 0 : nk * (left > 256 ? c.slab_two : c.slab_one) + c.tile;
      if (logits_width(wide, (int)tiles_v, (int)N, d, 256).cost < full * (nk * c.slab_two + c.tile) + last - c.launch) return TILE_256;
    }
  }
  return t128 >= (bf16 ? LOGITS_MIN_TILES_BF16_128 : LOGITS_MIN_TILES) ? TILE_128 : TILE_64;
}
LLAMARL_RULE Tile logits_tile(int64_t N, int64_t V, int64_t d, bool bf16) { return logits_tile_by(FWD_SMALL, FWD_COSTS, N, V, d, bf16); }
LLAMARL_RULE Tile dz_tile(int64_t N, int64_t V, int64_t d, bool bf16) { return logits_tile_by(DZ_SMALL, DZ_COSTS, N, V, d, bf16); }

// Most parts a tail tile is cut into.  Eight left most CUs idle where few tokens meet a long vocabulary: dH of
// (300, 128256, 1032), 27 tiles of 128, 250 -> 133 us; (1024, 128256, 520) 243 -> 153.
constexpr int STORE_MAX_SPLITS = 32;
// Store contractions: M x Nn outputs over K, split along K where tiles are few; counted in parts of 16 slabs, which
// still pay for their partial blocks.  Up to eight parts a tile the tiles of a count decide; beyond, where K is long and
// the output small, 256-tiles of more than 128 rows if they fill the chip, 128-tiles by the output they hold (the rest of
// an edge tile is padding).  bf16 dH on 256- / 128- / 64-tiles with up to 32 parts, and now against eight parts and the rule
// of then:
//   (64, 128256, 1024) 86 / 60 / 54, 80 -> 51; (300, 128256, 520) 105 / 96 / 130, 110 -> 90; (64, 128256, 4096) 203 / 193 / 225,
//   231 -> 186; (300, 128256, 1032) 141 / 145 / 231, 250 -> 133; (150, 128256, 2048) 124 / 170 / 247, 225 -> 117;
//   (1024, 128256, 520) 163 / 203 / 373, 243 -> 153; (600, 60000, 1032) 100 / 102 / 195, 112 -> 90;
//   fp32 on 128- / 64-tiles (300, 16400, 260) 62 / 47, 65 -> 41; (300, 40000, 1024) 289 -> 190.
// With up to eight parts:
//   bf16, dH at (N, V, d) on 256- / 128- / 64-tiles: (512, 2048, 512) 23 / 17.5 / 17 us, (1041, 5003, 520) 33 / 26 / 29,
//   (1024, 8192, 1024) 42 / 36 / 43, (64, 128256, 4096) 337 / 236 / 229, (1024, 16032, 2048) 77 / 79 / 125;
//   dW: (512, 2048, 512) 23 / 19 / 16, (512, 8192, 1024) 38 / 17 / 25, (1024, 16032, 2048) 67 / 73 / 131.
//   fp32 on 128- / 64-tiles, dH: (512, 4096, 512) 45 / 35, (1024, 4096, 512) 49 / 57, (300, 16400, 260) 137 / 69;
//   dW: (512, 4096, 512) 35 / 31, (1024, 4096, 512) 48 / 52, (300, 16400, 260) 43 / 54.
LLAMARL_RULE Tile store_tile(int64_t M, int64_t Nn, int64_t K, bool bf16) {
  const int64_t slab_k = bf16 ? 64 : 32;
  const int64_t most = K / (16 * slab_k), parts = most < 1 ? 1 : most < STORE_MAX_SPLITS ? most : STORE_MAX_SPLITS;
  const int64_t few = parts < 8 ? parts : 8;
  if (bf16) {
    const int64_t t256 = tile_count(M, Nn, 256);
    if (t256 * few >= 256 || (M > 128 && t256 * parts >= 256)) return TILE_256;
  }
  if (tile_count(M, Nn, 128) * few >= (bf16 ? 128 : 256)) return TILE_128;
  return M * Nn / (128 * 128) * parts >= 256 ? TILE_128 : TILE_64;
}

// Width of the tiles of the k-major store contraction (dH): the narrowest that takes no more columns of tiles than 256.  (The
// empty columns of a wide tile multiply zeros and cost a power-limited chip less than their share.  dW keeps 256: at
// 6720 rows a narrow last column made it slower.)
//   (6720, 40000, d), 256 / narrow: d = 264 223 / 213 us, 520 319 / 307, 1032 587 / 562, 1288 618 / 601
LLAMARL_RULE int store_width(int64_t Nn) {
  const int64_t cols = (Nn + 255) / 256;
  const int width = (int)(((Nn + cols - 1) / cols + 31) / 32 * 32);
  return width < 128 ? 128 : width;
}

// Workgroups of a contraction in a launch of two (dH and dW on small tiles): `own` and `other` are what a CU holds of either by
// itself, long: K has PAIR_LONG_SLABS slabs or more (with every row active).  Each takes half of the workgroups (both have the same
// products to form) and cuts its tiles into fewer parts, except where a tile is few slabs: its first loads and its stores want
// workgroups.  Backward at (N, V, d), three quarters of the rows active, one contraction after the other / together, each cut for
// the whole grid / as here, us:
//   fp32 (256, 1024, 256) 42.2 / 33.0 / 33.0, (1024, 4096, 512) 129 / 119 / 111, (300, 16400, 260) 117 / 120 / 114 (130 on halves),
//   (4800, 20011, 516) 1622 / 1622 / 1593; bf16 (1041, 5003, 520) 58.8 / 52.8 / 46.4, (512, 8192, 1024) 58.9 / 52.0 / 50.1,
//   (2048, 4096, 264) 64.6 / 48.3 / 44.6, (4096, 3000, 512) 74.7 / 68.2 / 63.2, (300, 16400, 264) 43.8 / 40.0 / 38.9.
// The grid is the host's, who does not know how many rows are active; with few of them halves and whole grids are the same within
// -2 .. +10 %: a tenth active, bf16 (2048, 4096, 264) 38.9 / 30.3 / 31.1, a fifth, fp32 (2048, 8192, 512) 155 / 137 / 125.
// The kernel's registers are those of the larger body, so two long ones share what a CU holds of that (fp32, three workgroups with
// 64 x 64 tiles and two with 128 x 128): halves of what each could have alone put a third more workgroups into the plan than run at
// once.  fp32, halves of its own / as here: (1359, 21070, 68) 255 / 225, (351, 24111, 332) 253 / 213, (2030, 869, 1592) 204 / 180,
// (346, 3658, 1432) 168 / 146, (700, 3000, 1032) 171 / 167, but (3593, 5092, 76) 159 / 166.  Where one is short the plan is too
// coarse for either to win everywhere: (66, 11647, 1124) 141 / 134, (79, 18054, 452) 96 / 99, (2452, 219, 1780) 119 / 132.
constexpr int PAIR_LONG_SLABS = 12;
LLAMARL_RULE int pair_workgroups(int cus, int own, int other, bool own_long, bool other_long) {
  return !own_long ? cus * own : cus * (other_long && other < own ? other : own) / 2;
}

}  // namespace llamarl
