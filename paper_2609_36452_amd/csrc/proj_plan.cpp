// Host side of the projection: the tile plan for a row bound, and the
// dispatch to the kernel variant it names.
#include <algorithm>

#include "rpd_launch.h"

namespace rpd {

// Rounds of tiles that the 32 CUs of the busiest XCD take, the XCDs owning row
// tiles (by_rows) or ranges of the vocabulary; past a few rounds tiles start
// apart and the last round is seldom a whole one.
static double tile_rounds(long long nrt, int nvt, bool by_rows) {
  const long long tiles = by_rows ? (nrt + 7) / 8 * nvt : (nvt + 7) / 8 * nrt;
  const double whole = (double)((tiles + 31) / 32);
  return tiles > 128 ? std::min(whole, tiles / 32.0 + 0.4) : whole;
}

ProjPlan plan_projection(int dtype, long long rows_cap, int V) {
  ProjPlan p{};
  bool f32_by_rows = false;
  if (rows_cap < 1) rows_cap = 1;
  if (dtype == 1) {   // fp32
    // The tile height (32..128 rows), and whether the XCDs own row tiles or
    // ranges of the vocabulary, by the rounds of tiles that the busiest XCD
    // takes (tile_rounds) and what a row costs, a row of a shorter tile costing
    // more (it reads W_U more often: 1024 rows at d = 4096, V = 126464 in tiles of
    // 128, 96, 64 and 32 rows 8.15, 8.38 per padded row, 8.17 and 8.79 ms; 4096
    // rows at d = 1024, V = 32000 2.17, 2.21, 2.21 and 2.33). Of equals the
    // tallest, and row tiles (32 of them there: 2.15 ms against 2.16). Dealing
    // whole row tiles wherever there are eight took as long for nine as for
    // sixteen (864 rows at d = 4096, V = 126464 13.2 ms, 7.0 so). 64 x 32 tiles, which
    // take 0.84 of a 128 x 32 tile's time, where the launch would leave CUs idle.
    static constexpr struct {
      int rows;
      double cost;   // of a row, against the tallest tile's
    } kHeights[] = {{128, 1.0}, {96, 1.02}, {64, 1.02}, {32, 1.07}};
    p.variant = PROJ_F32;
    p.vocab_cap = kF32TileVocab;
    p.nvt = (V + p.vocab_cap - 1) / p.vocab_cap;
    double best = 0.0;
    for (const auto& h : kHeights) {
      const long long nrt = (rows_cap + h.rows - 1) / h.rows;
      for (int by_rows = nrt >= 8 ? 1 : 0; by_rows >= 0; --by_rows) {
        const double cost = tile_rounds(nrt, p.nvt, by_rows != 0) * h.rows * h.cost;
        if (best == 0.0 || cost < 0.995 * best) {
          best = cost;
          p.rows_per_tile = h.rows;
          f32_by_rows = by_rows != 0;
        }
      }
    }
    const int nvt_small = (V + kF32TileVocabSmall - 1) / kF32TileVocabSmall;
    if (tile_rounds((rows_cap + 31) / 32, nvt_small, false) * 32 * 0.84 < best) {
      p.vocab_cap = kF32TileVocabSmall;
      p.rows_per_tile = 32;
      p.nvt = nvt_small;
      f32_by_rows = false;
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
  split_over_xcds(p, dtype == 1 ? f32_by_rows : p.nrt >= 8);
  return p;
}

void split_over_xcds(ProjPlan& p, bool rows) {
  p.split_rows = rows ? 1 : 0;
  p.per_xcd = rows ? ((p.nrt + 7) / 8) * p.nvt : ((p.nvt + 7) / 8) * p.nrt;
  p.grid = 8 * p.per_xcd;
}

// ---------------------------------------------------------- lazy passes --
//
// How many layers the first pass below the final layer takes, and whether a call
// walks at all, is decided before anything is known about the walk: positions
// may stop at once or agree on down to the last layer. The two rules below bound
// what a call loses against one pass per layer where all stop at once.

// A pass over `rows` rows: the rounds of tiles that the busiest XCD's 32 CUs
// take, each a k-loop over d and a first load and epilogue, or streaming W_U
// (6.9 TB/s in bf16, 4.6 where its rows are not whole 128-byte lines, by the MFMA
// tiles 12% less; 5.6 in fp32) if that is more.
// Fitted to the projection alone at 12 shapes from d = 264 to 4096 and V = 5003 to
// 152064, 8 to 4096 rows: 402 of 447 times within 25% (at d = 4096, V = 126464 64,
// 128, 256, 512 and 1024 rows 160, 169, 226, 417 and 800 us, the fit 159, 176, 222,
// 399 and 792; at d = 656, V = 21723 20, 27, 36, 38 and 63, the fit 19, 41, 46, 36
// and 66).
static double pass_us(int dtype, long long rows, int d, int V) {
  const ProjPlan p = plan_projection(dtype, rows, V);
  const double st = (double)V * d * (dtype == 1 ? 4 / 5.6e6 : 2 / (d % 64 ? 4.6e6 : 6.9e6));
  const double rounds = tile_rounds(p.nrt, p.nvt, p.split_rows != 0);
  if (dtype == 1) {
    const double loop = d / 32.0 * (p.vocab_cap == kF32TileVocabSmall ? 0.42 : 0.5 / 32 * p.rows_per_tile);
    return 6.0 + std::max(st, rounds * (loop + 5.5));
  }
  const double chunks = d / 64.0;
  if (rows <= kStreamMaxRows) return 9.0 + std::max(st, chunks * (rows <= 32 ? 0.78 : 0.95));
  const double from_hbm = p.nrt > 1 ? 1.0 : (d % 64 ? 1.8 : 1.12);   // one row tile: no chunk of W_U is found in L2
  const double chunk = p.rows_per_tile == kBigTileRows ? 1.27 : (p.rows_per_tile == kBigTileRowsSmall ? 1.08 : 0.95);
  return 6.0 + std::max(1.12 * st, rounds * (chunks * chunk * from_hbm + 17.0));
}

// What a pass costs beside the projection that runs (its listing, reduction and
// up to three projections that exit at once), and what a pass does that finds no
// position (100 and 256 positions at d = 4096, V = 126464 that all stop at the
// first layer: 377 and 517 us with K = 2, 400 and 530 with K = 4, 436 and 551 with
// K = 8; the projections of the first two passes take 2 * 171 and 2 * 240); what a
// call costs besides its passes.
static constexpr double kPassUs = 25.0, kEmptyPassUs = 11.0, kCallUs = 20.0;

// Rows up to which a pass takes further layers of its positions: it then costs
// at most three quarters more than a pass over few rows, and each layer taken
// along saves a pass where the positions walk on. (d = 4096, V = 126464: 256 rows.
// Twice a pass over few rows there, 200 and 256 positions, half of them in the
// band, that stop at once, K = 4: 600 and 630 us; so 505 and 525; one layer a pass
// 452 and 452. Agreeing on down to the last layer: 600 and 630; 680 and 705; 800.)
int lazy_pass_rows(int dtype, int d, int V) {
  const int step = dtype == 1 ? 32 : 64, most = 7 * (dtype == 1 ? 128 : kBigTileRows);
  const double limit = 1.75 * pass_us(dtype, step, d, V) + kPassUs;
  int n = step;
  for (int r = step; r <= most; r += step)
    if (pass_us(dtype, r, d, V) <= limit) n = r;
  return n;
}

// In the band of positions that walk: whether one pass over every layer of every
// position, by its bytes and operations alone, costs no more than the final layer
// and 30 us for each further pass. That leaves out the rounds of tiles and so takes
// one pass of few rows rather often, as it should: a position in the band is
// likely, and then the next pass streams W_U again (17 positions, K = 8, d = 1928,
// V = 136547: 244 us in one pass, 331 walking; 8 in fp32, K = 5, d = 1015, V = 101190:
// 228 and 281; 64 at d = 4096, V = 126464, K = 4, which walk: 245 against 345, and
// 196 with none in the band).
static bool band_in_one_pass(int dtype, int K, long long n, int d, int V) {
  const double st = (double)V * d * (dtype == 1 ? 4 / 5.6e6 : 2 / 6.7e6), row = 2.0 * V * d;
  auto us = [&](double rows) {
    return std::max(st, dtype == 1 ? rows * row / 128e6 : 0.38 * st + rows * row / 1440e6);
  };
  const long long worth = std::max(1LL, (long long)((st + 30.0) / (row / (dtype == 1 ? 128e6 : 1050e6))));
  double least = us((double)n);
  for (long long rem = K - 1, g = 1; rem > 0; g *= 2, least += 30.0)
    rem -= n * rem <= 2 * worth ? rem : std::min(std::max(worth / n, g), rem);
  return us((double)K * n) <= least;
}

// Whether one pass over every layer of every position takes the place of
// walking. Where every position walks (walk_all), walking costs least if all
// stop at the first layer, and most if all agree down to the last: one pass is
// taken up to the middle of the two, but costs no more than 1.3 times the least.
// (d = 4096, V = 126464, K = 4: 100 positions 415 us in one pass, with one layer a
// pass 394 to 758; 125 440, 385 to 725; 150 607 and 200 781, where walking, 420 and
// 480 to 760 and 906, is taken.)
bool lazy_one_pass(int dtype, int K, long long cap, int d, int V, bool walk_all) {
  if (K == 1 || (walk_all && K == 2)) return true;   // two layers are projected whatever they hold
  const int n = (int)std::max(cap, 1LL);
  if (!walk_all) return band_in_one_pass(dtype, K, n, d, V);
  const int pr = lazy_pass_rows(dtype, d, V);
  const double one = pass_us(dtype, (long long)K * n, d, V), final_layer = pass_us(dtype, n, d, V);
  double least = final_layer + kCallUs, most = least;
  for (int t = 1, rem = K - 1; rem > 0; ++t) {
    const int g = lazy_group(n, rem, lazy_min_group(t), pr);
    const double walk = kPassUs + pass_us(dtype, (long long)g * n, d, V);
    least += t > 1 ? kEmptyPassUs : walk;
    most += walk;
    rem -= g;
  }
  return one + kCallUs <= std::min(0.5 * (least + most), 1.3 * least);
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
