// Host side of the projection: the tile plan for a row bound, and the
// dispatch to the kernel variant it names.
#include <algorithm>

#include "rpd_launch.h"

namespace rpd {

ProjPlan plan_projection(int dtype, long long rows_cap, int V) {
  ProjPlan p{};
  if (rows_cap < 1) rows_cap = 1;
  if (dtype == 1) {   // fp32
    // The tile height (32..128 rows) whose padded rows cost least, a row of a
    // shorter tile costing more (it reads W_U more often: 1024 rows at d = 4096,
    // V = 126464 in tiles of 128, 96, 64 and 32 rows 8.15, 8.38 per padded row,
    // 8.17 and 8.79 ms; 4096 rows at d = 1024, V = 32000 2.17, 2.21, 2.21 and
    // 2.33); the tallest of equals. A launch that would leave most of the 256
    // CUs idle takes 64 x 32 tiles instead.
    static constexpr struct {
      int rows;
      double cost;   // of a row, against the tallest tile's
    } kHeights[] = {{128, 1.0}, {96, 1.02}, {64, 1.02}, {32, 1.07}};
    p.variant = PROJ_F32;
    p.vocab_cap = kF32TileVocab;
    double best = 0.0;
    for (const auto& h : kHeights) {
      const double cost = (double)((rows_cap + h.rows - 1) / h.rows * h.rows) * h.cost;
      if (best == 0.0 || cost < best) {
        best = cost;
        p.rows_per_tile = h.rows;
      }
    }
    p.nvt = (V + p.vocab_cap - 1) / p.vocab_cap;
    if ((long long)p.nvt * ((rows_cap + p.rows_per_tile - 1) / p.rows_per_tile) < 256) {
      p.vocab_cap = kF32TileVocabSmall;
      p.rows_per_tile = 32;
      p.nvt = (V + p.vocab_cap - 1) / p.vocab_cap;
    }
  } else if (rows_cap <= kStreamMaxRows) {
    // HBM-bound: one row tile holding every projected row, so W_U is read
    // once; a multiple of 256 equal vocabulary tiles, so every CU streams the
    // same share
    p.variant = rows_cap <= 32 ? PROJ_BF16_S32 : PROJ_BF16_S64;
    p.rows_per_tile = rows_cap <= 32 ? 32 : 64;
    p.vocab_cap = kStreamTileVocab;
    int nvt = (V + p.vocab_cap - 1) / p.vocab_cap;
    nvt = ((nvt + 255) / 256) * 256;
    p.nvt = nvt < V ? nvt : V;
  } else if (rows_cap <= kBigTileRowsMid) {
    // one MFMA tile of 256 vocabulary rows x 128 projected rows per vocabulary tile
    p.variant = PROJ_BF16_BIG128;
    p.rows_per_tile = kBigTileRowsMid;
    p.vocab_cap = kBigTileVocab;
    p.nvt = (V + p.vocab_cap - 1) / p.vocab_cap;
  } else {
    // MFMA tiles of 256 vocabulary rows x 256 or 192 projected rows, whichever
    // pads the rows less (ties to 256)
    const long long pad256 = (rows_cap + kBigTileRows - 1) / kBigTileRows * kBigTileRows;
    const long long pad192 = (rows_cap + kBigTileRowsSmall - 1) / kBigTileRowsSmall * kBigTileRowsSmall;
    p.variant = pad192 < pad256 ? PROJ_BF16_BIG192 : PROJ_BF16_BIG;
    p.rows_per_tile = pad192 < pad256 ? kBigTileRowsSmall : kBigTileRows;
    p.vocab_cap = kBigTileVocab;
    p.nvt = (V + p.vocab_cap - 1) / p.vocab_cap;
  }
  p.nrt = (int)((rows_cap + p.rows_per_tile - 1) / p.rows_per_tile);
  // fp32: the XCDs own whole row tiles only where each gets as many, else
  // ranges of the vocabulary (nine row tiles at d = 4096, V = 126464: 864 rows
  // 13.2 -> 7.0 ms, 1136 rows 17.2 -> 9.2; 32 of them at d = 1024, V = 32000:
  // 2.15 ms against 2.16)
  p.split_rows = p.nrt >= 8 && (dtype != 1 || p.nrt % 8 == 0) ? 1 : 0;
  p.per_xcd = p.split_rows ? ((p.nrt + 7) / 8) * p.nvt : ((p.nvt + 7) / 8) * p.nrt;
  p.grid = 8 * p.per_xcd;
  return p;
}

// ---------------------------------------------------------- lazy passes --
//
// How many layers a lazy pass takes, and whether a call walks at all, is decided
// before anything is known about the walk: positions may stop at the first layer
// below the final one or agree on down to the last. The two rules below bound
// what a call loses against one pass per layer where all stop at once.

// Streaming W_U (6.9 TB/s in bf16, 5.6 in fp32), and one row's matrix time (at 256
// rows 1.05 PFLOP/s in bf16, 128 TFLOP/s in fp32).
static double stream_us(int dtype, int d, int V) { return (double)V * d * (dtype == 1 ? 4 / 5.6e6 : 2 / 6.9e6); }
static double row_us(int dtype, int d, int V) { return 2.0 * V * d / (dtype == 1 ? 128e6 : 1050e6); }

// What a pass costs beside the projection that runs (its listing, reduction and
// up to three projections that exit at once), and what a pass does that finds no
// position (100 and 256 positions at d = 4096, V = 126464 that all stop at the
// first layer: 377 and 517 us with K = 2, 400 and 530 with K = 4, 436 and 551 with
// K = 8; the projections of the first two passes take 2 * 171 and 2 * 240).
static constexpr double kPassUs = 17.0, kEmptyPassUs = 11.0;

// Rows up to which layers taken along in vain cost at most half of a pass over
// few rows, which is what each saves where its positions walk on. At d = 4096,
// V = 126464 (246 rows), K = 4, half of the positions in the band, one layer a
// pass -> so: all stopping at once 125 positions 375 -> 445 us, 200 455 -> 510;
// all agreeing 125 positions 695 -> 460, 200 800 -> 680. Passes of up to twice as
// many rows lose as much as they gain (200 and 256 positions 600 and 630 us
// whether they stop or walk; one layer a pass 455 and 455 to 800 and 800).
int lazy_pass_rows(int dtype, int d, int V) {
  const double r = (1.5 * stream_us(dtype, d, V) + kPassUs) / row_us(dtype, d, V);
  const int n = (int)std::min(std::max(r, 1.0), dtype == 1 ? 128.0 : (double)kBigTileRows);   // one row tile
  // whole fp32 tiles: there the matrix time of the rows that pad the last one counts
  return dtype == 1 && n > 32 ? n / 32 * 32 : n;
}

// A pass over `rows` rows, in tiles of which the busiest XCD has its share. In
// bf16 a fit: the MFMA tiles read W_U 12% slower than the streaming kernel, and
// padding rows cost two thirds of a row (d = 4096, V = 126464, the projection alone:
// 64 rows 153 us, 128 171, 192 193, 256 240, 384 352, 400 418, 512 436, 576 506, 768
// 634, 1024 822; the fit 156, 174, 191, 240, 339, 410, 437, 486, 634, 831. d = 2048,
// V = 32000: 64 rows 26, 256 39, 512 53, 1024 111; the fit 25, 36, 60, 110).
static double pass_us(int dtype, long long rows, int d, int V) {
  const ProjPlan p = plan_projection(dtype, rows, V);
  const double st = stream_us(dtype, d, V);
  const double padded = (double)(p.split_rows ? (p.nrt + 7) / 8 * 8 : p.nrt) * p.rows_per_tile;
  if (dtype == 1) return 6.0 + std::max(st, padded * row_us(dtype, d, V));
  const double matrix = 0.25 * st + (0.68 * padded + 0.32 * (double)rows) * 2.0 * V * d / 1345e6;
  return 6.0 + std::max(rows <= kStreamMaxRows ? st : 1.12 * st, matrix);
}

// Whether one pass over every layer of every position takes the place of
// walking. Where every position walks (walk_all): if it costs at most a fifth
// more than the least that walking with one layer a pass can, the final layer, one more
// pass and passes that find no position. (d = 4096, V = 126464, K = 4: 100
// positions 425 us against 395 where they stop at once and 740 where all agree, 125
// positions 445 against 385 and 725. At 150 and 200 one pass takes 615 and 790,
// walking 431 and 510 to 830 and 1000.) In the band: if it costs no more than the
// final layer, 30 us for the next pass, which takes more as soon as a single
// position is in the band, and passes that find none.
bool lazy_one_pass(int dtype, int K, long long cap, int d, int V, bool walk_all) {
  if (K == 1) return true;
  const int n = (int)std::max(cap, 1LL), pr = lazy_pass_rows(dtype, d, V);
  const double one = pass_us(dtype, (long long)K * n, d, V), final_layer = pass_us(dtype, n, d, V);
  if (walk_all) return one <= 1.2 * (2 * final_layer + kPassUs + (K - 2) * kEmptyPassUs);
  int passes = 0;
  for (int rem = K - 1; rem > 0;) rem -= lazy_group(n, rem, lazy_min_group(++passes), pr);
  return one <= final_layer + 30.0 + (passes - 1) * kEmptyPassUs;
}

hipError_t launch_projection(const Launch& a, hipStream_t s) {
  if (a.max_masked <= 0) return hipSuccess;
  switch (a.plan.variant) {
    case PROJ_BF16_S32:
    case PROJ_BF16_S64: return launch_proj_stream(a, s);
    case PROJ_BF16_BIG:
    case PROJ_BF16_BIG192:
    case PROJ_BF16_BIG128: return launch_proj_big(a, s);
    case PROJ_F32: return launch_proj_f32(a, s);
  }
  return hipErrorInvalidValue;
}

}  // namespace rpd
