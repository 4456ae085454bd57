// Lazy layerwise projection (Appendix A.6 "Layerwise projection"): a
// position's intermediate layers are projected from the final one down, and
// no further than its first disagreeing layer, where its agreement suffix
// (Eq. 2) is known.
//
// Projection passes, from the final layer down:
//   pass 0      the final layer of every masked position;
//   pass t > 0  the next layers of the positions still "alive": those that
//               walk (every position with a finite final confidence with
//               RPD_PARAM_LAZY_ALL, the procedure as the paper states it;
//               otherwise only those in the band theta_c <= c < theta_h, the
//               only ones whose candidacy the stability test decides, Eq. 5,
//               a further saving that leaves every decision unchanged) and
//               whose layers so far all agreed with the final token.
// A pass takes several layers of each of its positions while its rows are few
// (up to the ridge a pass costs the one stream of W_U, whatever its rows), and
// at least 1, 2, 4, .. of them (lazy_group): a position's layers below its
// first disagreement are then projected and not used. Each pass is the ordinary
// projection over an explicit list of rows (a table of element offsets into
// the hidden states, or normalized rows), followed by k_lazy_reduce (merge
// the tile states, walk each position through the pass's layers, in order)
// and, before the next one, k_lazy_next (list the positions still alive, the
// layers taken of each, and the counts; the host plans the pass for a bound on
// them or reads the positions' count back). k_lazy_score then evaluates
// Eq. 2-5 from the per-position state, with persistence exact for every
// position that walked; elsewhere stability is not evaluated (persistence -1,
// drop and stability NaN). The commitment follows as usual.
//
// Against one pass for each layer, at d = 4096, V = 126464, K = 4: a call over
// 256 positions, those in the band (about 60) walking, 757 -> 467 us (one pass
// of 3 layers instead of three, and two sets of empty launches fewer);
// iterations over 190-230 positions that all walk, 987 -> 909 us.
#include "reduce_device.h"

namespace rpd {
namespace {

// One workgroup of four waves per listed position j < m: wave w merges the
// rows of the pass's layers w, w+4, .. (with exact argmax ties resolved after
// a projection whose tiles sum in different orders: bit c of tie_cls for size
// class c), then one thread walks the layers in order and updates the
// position's state.
struct LazyPlans {
  int nvt[kLazyClasses];
  LazyClasses cls;
  int tie_cls;
};
constexpr int kLazyReduceWaves = 4;
__global__ __launch_bounds__(64 * kLazyReduceWaves) void k_lazy_reduce(
    const float4* __restrict__ partials, LazyPlans pl, TieArgs ta, const uint16_t* __restrict__ hidden,
    const uint16_t* __restrict__ xrows, int d, LazyState st, int K, int B, int L, const int32_t* __restrict__ rows,
    float theta_c, float theta_h, int walk_all, int32_t* __restrict__ layer_argmax, float* __restrict__ layer_conf,
    float* __restrict__ layer_entropy) {
  __shared__ int ly[64];
  __shared__ float lc[64], lh[64];
  const int j = blockIdx.x, lane = threadIdx.x & 63, wid = threadIdx.x >> 6;
  // the counts and the position are loaded together (j < m_cap stays inside
  // act), and the position's state with the tile states (unused in the
  // final-layer pass): two memory round trips before the update instead of
  // four. A workgroup beyond the count exits before reading anything else.
  const int m = *st.m, G = *st.grp, top = *st.top;
  const int p = st.act[j];
  if (j >= m) return;
  // the partials follow the plan of the size class the row count is in
  int cls = 0;
#pragma unroll
  for (int c = 0; c < kLazyClasses - 1; ++c) cls += m * G > pl.cls.cap[c] ? 1 : 0;
  int nvt = pl.nvt[0];
#pragma unroll
  for (int c = 1; c < kLazyClasses; ++c) nvt = cls == c ? pl.nvt[c] : nvt;
  const int y_fin = st.y[p], k_prev = st.k[p];
  const float pmax_prev = st.pmax[p];
  const int pos = layer_argmax ? rows[p] : 0;
  const long long off = xrows ? 0 : st.rowoff[j];
  for (int g = wid; g < G; g += kLazyReduceWaves) {
    const long long r = (long long)j * G + g;
    const float4* src = partials + r * nvt;
    float4 keep[8];
    Soft s = wave_merge_row(src, nvt, lane, keep);
    if ((pl.tie_cls >> cls) & 1) {
      const uint16_t* x = xrows ? xrows + r * d : hidden + off - g * ((long long)B * L * d);
      s.idx = resolve_tie(s, keep, src, nvt, ta, x, lane);
    }
    if (lane == 0) state_stats(s, ly[g], lc[g], lh[g]);
  }
  __syncthreads();
  if (threadIdx.x != 0) return;
  const int b = pos / L, i = pos - b * L;
  auto show = [&](int g) {
    if (!layer_argmax) return;
    const long long ol = ((long long)(top - g) * B + b) * L + i;
    layer_argmax[ol] = ly[g];
    layer_conf[ol] = lc[g];
    layer_entropy[ol] = lh[g];
  };
  if (top == K - 1) {   // the final-layer pass (one layer)
    const float c = lc[0];
    st.y[p] = ly[0];
    st.c[p] = c;
    st.h[p] = lh[0];
    st.k[p] = 1;
    st.pmax[p] = c;
    // NaN fails both tests
    st.alive[p] = (K > 1 && (walk_all ? c == c : (c >= theta_c && c < theta_h))) ? 1 : 0;
    st.depth[p] = 1;
    show(0);
    return;
  }
  int k = k_prev, g = 0;
  float pmax = pmax_prev;
  bool agree = true;
  for (; g < G && agree; ++g) {   // down to the first disagreeing layer, which is the last one seen
    agree = ly[g] == y_fin;
    if (agree) {
      ++k;
      pmax = fmaxf(pmax, lc[g]);
    }
    show(g);
  }
  st.k[p] = k;
  st.pmax[p] = pmax;
  st.alive[p] = agree && top - G >= 0 ? 1 : 0;
  st.depth[p] = K - (top - (g - 1));
}

// one workgroup: lists the pass below the last one: the positions still
// alive, in order, with the element offsets of their rows at the pass's first
// layer, and the counts (list_pass). The final-layer pass, every masked
// position, is listed by the compaction.
constexpr int kLazyNextThreads = 1024;
__global__ __launch_bounds__(kLazyNextThreads) void k_lazy_next(const int32_t* __restrict__ n_ptr, LazyState st,
                                                                const int32_t* __restrict__ rows, int cap, int B, int L,
                                                                int d, int min_group, int pass_rows, LazyClasses cls,
                                                                int32_t* host_m) {
  __shared__ int wsum[kLazyNextThreads / 64];
  const int lane = threadIdx.x & 63, wid = threadIdx.x >> 6, nw = blockDim.x >> 6;
  // the first chunk's state and row are loaded with the counts (p < cap stays
  // inside both buffers; entries at or beyond the count are not used)
  const bool in0 = (int)threadIdx.x < cap;
  const int alive0 = in0 ? st.alive[threadIdx.x] : 0;
  const int row0 = in0 ? rows[threadIdx.x] : 0;
  const int n = *n_ptr;
  const int l = *st.top - *st.grp;   // below the last layer, or negative with nothing alive
  __syncthreads();                   // every thread has read the counts that the last lines replace
  int carry = 0;
  for (int base = 0; base < n; base += blockDim.x) {
    const int p = base + threadIdx.x;
    const int alive = base == 0 ? alive0 : (p < n ? st.alive[p] : 0);
    const bool f = p < n && alive != 0;
    const unsigned long long bal = __ballot(f);
    const int before = __popcll(bal & ((1ull << lane) - 1ull));
    if (lane == 0) wsum[wid] = __popcll(bal);
    __syncthreads();
    int off = 0, tot = 0;
    for (int w = 0; w < nw; ++w) {
      const int c = wsum[w];
      off += (w < wid) ? c : 0;
      tot += c;
    }
    if (f) {
      const int j = carry + off + before;
      const int pos = base == 0 ? row0 : rows[p];
      const int b = pos / L, i = pos - b * L;
      st.act[j] = p;
      st.rowoff[j] = (((long long)l * B + b) * L + i) * (long long)d;
    }
    carry += tot;
    __syncthreads();
  }
  if (threadIdx.x == 0) {
    // with no position alive the pass is empty and the walk over: the layer
    // stays where it is, so that later passes find nothing either
    const int g = lazy_group(carry, l + 1, min_group, pass_rows);
    if (host_m) __hip_atomic_store(host_m, g > 0 ? carry : 0, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_SYSTEM);
    list_pass(st, g > 0 ? carry : 0, g > 0 ? g : 1, g > 0 ? l : 0, cls);
  }
}

// Eq. 2-5 from the per-position state, one thread per masked position
__global__ __launch_bounds__(256) void k_lazy_score(const int32_t* __restrict__ n_ptr, LazyState st,
                                                    const int32_t* __restrict__ rows, LazyScoreArgs a) {
  const int p = blockIdx.x * blockDim.x + threadIdx.x;
  if (p >= *n_ptr) return;
  const int pos = rows[p];
  const int b = pos / a.L, i = pos - b * a.L;
  const long long o = (long long)b * a.L + i;
  const float c = st.c[p];
  const bool band = c >= a.theta_c && c < a.theta_h;
  const bool walked = a.walk_all ? c == c : band;
  const bool high = c >= a.theta_h;
  float r = NAN, s = NAN;
  int k = -1;
  bool stab = false;
  if (walked) {
    k = st.k[p];
    r = st.pmax[p] - c;
    s = fmaf(-a.w, r, (float)min(k, a.k_max));
    stab = band && s >= a.theta_s;
  }
  a.token[o] = st.y[p];
  a.entropy[o] = st.h[p];
  a.confidence[o] = c;
  a.persistence[o] = k;
  a.drop[o] = r;
  a.stability[o] = s;
  a.flags[o] = (uint8_t)((high || stab ? kFlagCandidate : 0u) | (high ? kFlagHigh : 0u) | (stab ? kFlagStable : 0u));
  if (a.layer_argmax)   // layers never projected
    for (int l = 0; l < a.K - st.depth[p]; ++l) {
      const long long ol = ((long long)l * a.B + b) * a.L + i;
      a.layer_argmax[ol] = -1;
      a.layer_conf[ol] = NAN;
      a.layer_entropy[ol] = NAN;
    }
}

}  // namespace

hipError_t launch_lazy_next(const Launch& a, int dtype, int min_group, int pass_rows, int32_t* host_m, hipStream_t s) {
  hipLaunchKernelGGL(k_lazy_next, dim3(1), dim3(kLazyNextThreads), 0, s, a.n_masked, a.lazy, a.rows, a.max_masked, a.B,
                     a.L, a.d, min_group, pass_rows, lazy_classes(dtype), host_m);
  return hipGetLastError();
}

hipError_t launch_lazy_reduce(const Launch& a, int dtype, int m_cap, const ProjPlan* class_plans, hipStream_t s) {
  if (m_cap <= 0) return hipSuccess;
  LazyPlans pl{};
  pl.cls = lazy_classes(dtype);
  for (int c = 0; c < kLazyClasses; ++c) {
    const ProjPlan& p = class_plans ? class_plans[c] : a.plan;
    pl.nvt[c] = p.nvt;
    pl.tie_cls |= tie_args(a, p).w_u ? 1 << c : 0;
  }
  const TieArgs ta{static_cast<const uint16_t*>(a.w_u), a.d, a.logit_scale};
  hipLaunchKernelGGL(k_lazy_reduce, dim3(m_cap), dim3(64 * kLazyReduceWaves), 0, s, a.partials, pl, ta,
                     static_cast<const uint16_t*>(a.hidden), static_cast<const uint16_t*>(a.xrows), a.d, a.lazy, a.K,
                     a.B, a.L, a.rows, a.theta_c, a.theta_h, a.lazy_all ? 1 : 0, a.layer_argmax, a.layer_conf,
                     a.layer_entropy);
  return hipGetLastError();
}

hipError_t launch_lazy_score(const Launch& a, hipStream_t s) {
  if (a.max_masked <= 0) return hipSuccess;
  LazyScoreArgs sa{a.K,          a.B,          a.L,         a.theta_h,     a.theta_c,    a.theta_s,
                   a.w,          a.k_max,      a.lazy_all ? 1 : 0,        a.token,      a.entropy,
                   a.confidence, a.persistence, a.drop,     a.stability,   a.flags,      a.layer_argmax,
                   a.layer_conf, a.layer_entropy};
  hipLaunchKernelGGL(k_lazy_score, dim3((unsigned)((a.max_masked + 255) / 256)), dim3(256), 0, s, a.n_masked,
                     a.lazy, a.rows, sa);
  return hipGetLastError();
}

}  // namespace rpd
