// Internal interface between the C ABI (rpd_api.cpp), the projection plan
// (proj_plan.cpp) and the gfx950 kernels (proj_*.hip, score_commit.hip).
// Not installed; no torch or HIP types beyond hipStream_t.
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

namespace rpd {

// Projection kernel shapes. A "row" is one (masked position, layer) pair:
// row r = p*K + l for compacted masked position p. A "vocab tile" is a
// contiguous range of W_U rows; tile t covers [t*V/NVT, (t+1)*V/NVT).
enum ProjVariant {
  PROJ_BF16_S32 = 0,    // <= 32 rows: W_U streamed through wave-private LDS, hidden rows shared
  PROJ_BF16_S64 = 1,    // <= 64 rows, same kernel family
  PROJ_F32 = 3,         // fp32 inputs: fp32 MFMA tiles
  PROJ_BF16_BIG = 4,    // MFMA-bound: 256 x 256 tiles, both operands staged through LDS
  PROJ_BF16_BIG192 = 6, // the same kernel with 256 x 192 tiles (where they pad the rows less)
  PROJ_BF16_BIG128 = 7, // the same kernel with 256 x 128 tiles, for 65..128 rows
};

// tile of the large-row variant: vocabulary rows x projected rows
constexpr int kBigTileVocab = 256, kBigTileRows = 256;
// vocabulary rows of one workgroup of the streaming variants (all of them)
constexpr int kStreamTileVocab = 256;
// most projected rows a streaming variant takes; above, the MFMA tiles are
// faster (256 x 128 measured 7-12% faster than 128-row streaming at 68-128
// rows, 256 x 192 3-8% faster than 192-row streaming at 132-192 rows,
// 256 x 256 7-9% faster than 256-row streaming at 224 and 256; at 48 and 64
// rows the 64-row streaming form is 11% faster than 256 x 128)
constexpr int kStreamMaxRows = 64;
// rows of the smaller MFMA tiles
constexpr int kBigTileRowsSmall = 192, kBigTileRowsMid = 128;
// vocabulary rows of the fp32 tiles: the ordinary ones and, for launches that
// would leave CUs idle, the small one
constexpr int kF32TileVocab = 128, kF32TileVocabSmall = 64;
// largest bound on a lazy call's positions below which the host reads no count back
constexpr int kLazyGateRows = 256;
// size classes of a lazy pass whose row count only the device knows: the
// largest count of each class but the last (which holds the rest), by type;
// each is the largest count of a projection variant
constexpr int kLazyClasses = 5;
struct LazyClasses {
  int cap[kLazyClasses - 1];
};
inline LazyClasses lazy_classes(int dtype) {
  return dtype == 1 ? LazyClasses{{32, 64, 96, 128}} : LazyClasses{{64, 128, 192, 256}};
}
// largest canvas (B * L) whose compaction the projection does itself with a single row tile
constexpr int kFusedCompactMax = 2048;
// and with several, in fp32, or the normalization does
constexpr int kFusedCompactTwoRounds = 512;

struct ProjPlan {
  ProjVariant variant;
  int rows_per_tile;   // TR
  int vocab_cap;       // max vocab rows one tile can hold
  int nvt;             // number of vocab tiles
  int nrt;             // number of row tiles (for the row bound)
  int per_xcd;         // workgroups per XCD slot in the launch
  int split_rows;      // 1: XCDs own row tiles; 0: XCDs own vocab tiles
  int grid;            // workgroups launched
};

// the shape plan for `rows_cap` rows (K * max masked positions)
ProjPlan plan_projection(int dtype, long long rows_cap, int V);
// the XCDs own row tiles (rows) or ranges of the vocabulary
void split_over_xcds(ProjPlan& p, bool rows);

// Lazy projection (proj_plan.cpp): the rows up to which a pass takes further
// layers of its positions
int lazy_pass_rows(int dtype, int d, int V);
// whether a lazy call over at most `cap` positions projects all K layers of
// every position in one pass
bool lazy_one_pass(int dtype, int K, long long cap, int d, int V, bool walk_all);
// Layers that the next lazy pass takes of each of its m positions, `rem`
// layers being left: as many as a pass is worth, at least min_group. Never
// fewer for fewer positions.
__host__ __device__ inline int lazy_group(int m, int rem, int min_group, int pass_rows) {
  if (m <= 0 || rem <= 0) return 0;
  int g = pass_rows / m;
  g = g < min_group ? min_group : g;
  return g < rem ? g : rem;
}

// The fewest layers that pass t (from 1) takes of each position: 1, then 2, 4
// and so on. One layer shows which positions stop at once; those that are left
// have agreed, and few passes are made, and enqueued, where K is large.
inline int lazy_min_group(int t) { return t < 7 ? 1 << (t - 1) : 64; }

// per-position state of the lazy layerwise projection (lazy.hip)
struct LazyState {
  int32_t* act;        // [cap] compacted positions listed for the current pass
  long long* rowoff;   // [cap] element offsets into hidden of their rows at the pass's first layer
  int32_t* y;          // [cap] final-layer token
  float* c;            // [cap] final-layer top probability
  float* h;            // [cap] final-layer entropy
  int32_t* k;          // [cap] agreement suffix length so far
  float* pmax;         // [cap] peak top probability over the suffix
  int32_t* alive;      // [cap] 1 while the walk continues
  int32_t* depth;      // [cap] layers projected
  int32_t* m;          // [1] positions in the current pass
  int32_t* grp;        // [1] layers it takes of each
  int32_t* top;        // [1] the first (highest) of these layers
  int32_t* nrow;       // [1] rows in the current pass (m * grp)
  int32_t* tier;       // [kLazyClasses] the row count in its size class, 0 in the others
};

struct LazyScoreArgs {
  int K, B, L;
  float theta_h, theta_c, theta_s, w;
  int k_max;
  int walk_all;        // every position with a finite confidence walked (else only the band)
  int32_t* token;
  float* entropy;
  float* confidence;
  int32_t* persistence;
  float* drop;
  float* stability;
  uint8_t* flags;
  int32_t* layer_argmax;
  float* layer_conf;
  float* layer_entropy;
};

struct Launch {
  int K, B, L, d, V;
  const void* hidden;
  const void* w_u;
  const uint8_t* mask;
  int max_masked;        // bound used for the launches (>= 0)
  // workspace pieces
  int32_t* n_masked;     // [1] device count (clamped to max_masked)
  int32_t* dev_status;   // [1] internal status word
  bool fused_compact;    // the normalization, or without one the projection, does the compaction (no launch_compact)
  int32_t* rows;         // [max_masked] compacted b*L+i
  float4* partials;      // [K*max_masked][nvt]
  // final normalization (norm_weight NULL: none): the projection then reads
  // projected row r at xrows + r * d (normalized, compacted) instead of
  // gathering it from hidden
  const void* norm_weight;
  float norm_eps;
  int norm_final;
  void* xrows;
  // explicit row list (lazy passes): projected row r = j * G + g, with G at
  // lazy.grp, is layer g below the pass's first one of listed position j, at
  // hidden + rowoff[j] - g * B * L * d (n_masked points at the row count);
  // NULL: gathered
  const long long* rowoff;
  LazyState lazy;
  ProjPlan plan;
  // params
  float theta_h, theta_c, theta_s, w, beta;
  int k_max, window;
  int block;             // 0: full RPD; > 0: RPD-block
  float logit_scale;     // multiplies every logit before the softmax statistics
  bool lazy_all;         // lazy projection: every masked position walks its layers (RPD_PARAM_LAZY_ALL)
  bool lazy_score;       // a lazy call projected in one pass: the scoring reports what the walk would have
  // outputs
  uint8_t* commit; int32_t* token; float* entropy; float* confidence;
  int32_t* persistence; float* drop; float* stability; uint8_t* flags;
  float* upstream_entropy; int32_t* n_commit;
  int32_t* layer_argmax; float* layer_conf; float* layer_entropy;
  int32_t* user_status;
};

// enqueue, in this order: compaction, projection, reduction + scoring,
// commitment (the last three use a.plan and a.max_masked)
// lazy_list: also list the first lazy pass (a.lazy), of type dtype
// host_n: host memory to store the count in as well (or NULL)
hipError_t launch_compact(const Launch& a, bool lazy_list, int dtype, int32_t* host_n, hipStream_t s);
hipError_t launch_projection(const Launch& a, hipStream_t s);
hipError_t launch_reduce_score(const Launch& a, hipStream_t s);
hipError_t launch_commit(const Launch& a, hipStream_t s);

// lazy layerwise projection: list the next pass (the positions still walking
// and the layers it takes of each, lazy_group), reduce a pass, score from the
// per-position state
// (host_m: host memory to store the positions' count in as well, or NULL)
hipError_t launch_lazy_next(const Launch& a, int dtype, int min_group, int pass_rows, int32_t* host_m, hipStream_t s);
// m_cap: bound on the pass's positions; class_plans: the plans of the size
// classes, when the pass ran once per class (NULL: a.plan)
hipError_t launch_lazy_reduce(const Launch& a, int dtype, int m_cap, const ProjPlan* class_plans, hipStream_t s);
hipError_t launch_lazy_score(const Launch& a, hipStream_t s);
// the projection or the normalization does the compaction itself (needs a.plan and a.max_masked
// >= 0): the call then launches no compaction kernel
bool compact_fused(const Launch& a);

// the projection variants, dispatched by launch_projection on a.plan.variant
// the final normalization of the compacted rows into a.xrows (before the projection)
hipError_t launch_norm_rows(const Launch& a, hipStream_t s);
hipError_t launch_proj_stream(const Launch& a, hipStream_t s);  // PROJ_BF16_S32, PROJ_BF16_S64
hipError_t launch_proj_big(const Launch& a, hipStream_t s);     // PROJ_BF16_BIG
hipError_t launch_proj_f32(const Launch& a, hipStream_t s);     // PROJ_F32

// end of an iteration: fill the canvas with the committed tokens, unmask them
hipError_t launch_apply_commit(long long BL, uint8_t* mask, int32_t* canvas, const uint8_t* commit,
                               const int32_t* token, int32_t* progress, int progress_len, int32_t* step,
                               hipStream_t s);

// scoring + commitment from caller-supplied per-layer statistics
hipError_t launch_gate_commit(const Launch& a, const int32_t* layer_argmax, const float* layer_conf,
                              const float* layer_entropy, hipStream_t s);

}  // namespace rpd
