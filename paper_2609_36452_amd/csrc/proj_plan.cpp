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

// Time of one projection pass, for the lazy rules below: streaming W_U at the
// rate the smallest row counts reach (6.7 TB/s in bf16, 5.6 in fp32), or the
// rows' matrix time at the rate of 256 rows (1.05 PFLOP/s in bf16; 128 TFLOP/s
// in fp32), whichever is more. kPassUs: what a pass costs besides, its
// launches (up to four projections of which one runs, reduction, listing:
// about 5 us each on the stream).
static constexpr double kPassUs = 30.0;
static double stream_us(int dtype, int d, int V) { return (double)V * d * (dtype == 1 ? 4 / 5.6e6 : 2 / 6.7e6); }
static double row_us(int dtype, int d, int V) { return 2.0 * V * d / (dtype == 1 ? 128e6 : 1050e6); }

int lazy_pass_rows(int dtype, int d, int V) {
  const double r = (stream_us(dtype, d, V) + kPassUs) / row_us(dtype, d, V);
  return r < 1.0 ? 1 : (r > 1e6 ? 1000000 : (int)r);
}

// A pass over `rows` rows: in bf16 above the ridge an affine fit (at d = 4096,
// V = 126464: 244 us at 256 rows, 440 at 512, 600 at 768, 815 at 1024).
static double pass_us(int dtype, double rows, int d, int V) {
  const double st = stream_us(dtype, d, V);
  if (dtype == 1) return std::max(st, rows * row_us(dtype, d, V));
  return std::max(st, 0.38 * st + rows * 2.0 * V * d / 1440e6);
}

bool lazy_one_pass(int dtype, int K, long long cap, int d, int V, bool walk_all) {
  // One pass over everything against walking. In the band few positions walk:
  // one pass if it costs no more than the least that walking can, the final
  // layer of every position and then empty passes. Where every position walks
  // (walk_all) the least is one more layer of each, the most every layer of
  // each: one pass if it costs no more than the middle of the two. It then
  // loses less against walking that ends at once than it gains against walking
  // that does not (200 positions, K = 4: one pass 655 us; walking 510 to 990).
  if (K == 1) return true;
  const double one = pass_us(dtype, (double)K * (double)cap, d, V);
  const int n = (int)std::max(cap, 1LL), pr = lazy_pass_rows(dtype, d, V);
  double least = pass_us(dtype, n, d, V), most = least;
  if (walk_all) least += least;
  for (int rem = K - 1, g = 1; rem > 0; g *= 2) {
    const int take = lazy_group(n, rem, g, pr);
    most += kPassUs + pass_us(dtype, (double)n * take, d, V);
    least += kPassUs;
    rem -= take;
  }
  return one <= (walk_all ? 0.5 * (least + most) : least);
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
