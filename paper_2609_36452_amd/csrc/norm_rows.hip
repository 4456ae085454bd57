// The model's final normalization applied to the projected rows before the
// output head (Appendix A.2 "Intermediate-layer readout", A.6 "Layerwise
// projection"): RMS normalization g * x / sqrt(mean(x^2) + eps) of every
// (masked position, layer) row, in the compacted row order, written to the
// workspace; the projection then reads these rows instead of gathering from
// the hidden states. The final layer's native state is copied unchanged
// unless norm_final is set.
//
// The sum of squares, the scale and the product are evaluated in float64
// (each x^2 of a bf16 value is exact there), and the result is rounded once
// to the input type, round to nearest with ties to even, so the normalized
// rows the output head sees are reproducible to the last bit.
#include "rpd_device.h"

namespace rpd {
namespace {

__device__ __forceinline__ double load_f64(const uint16_t* p, long long k) {
  return (double)__uint_as_float((uint32_t)p[k] << 16);
}
__device__ __forceinline__ double load_f64(const float* p, long long k) { return (double)p[k]; }

// float64 -> bfloat16 bits, round to nearest, ties to even, in one step
// (8 significant bits; below 2^-126 the bfloat16 grid is 2^-133)
__device__ __forceinline__ uint16_t f64_to_bf16(double v) {
  const unsigned long long u = (unsigned long long)__double_as_longlong(v);
  const uint16_t sign = (uint16_t)((u >> 63) << 15);
  const int e = (int)((u >> 52) & 0x7FF);
  const unsigned long long m = u & ((1ull << 52) - 1);
  if (e == 0x7FF) return (uint16_t)(sign | 0x7F80 | (m ? 0x40 : 0));   // inf, NaN
  int be = e - 1023 + 127;
  if (be <= 0) {   // bfloat16 subnormal (or zero): a multiple of 2^-133
    const double q = rint(fabs(v) * 0x1p133);                        // ties to even
    return (uint16_t)(sign | (uint16_t)q);                           // q == 128 is the smallest normal
  }
  unsigned long long keep = m >> 45;
  const unsigned long long rem = m & ((1ull << 45) - 1), half = 1ull << 44;
  if (rem > half || (rem == half && (keep & 1))) ++keep;
  if (keep == 128) {
    keep = 0;
    ++be;
  }
  if (be >= 255) return (uint16_t)(sign | 0x7F80);
  return (uint16_t)(sign | (be << 7) | keep);
}
__device__ __forceinline__ void store_f64(uint16_t* p, long long k, double v) { p[k] = f64_to_bf16(v); }
__device__ __forceinline__ void store_f64(float* p, long long k, double v) { p[k] = (float)v; }

constexpr int kNormThreads = 256;
constexpr int kNormKeep = 4;   // pieces of a thread kept between the two passes (the whole row to d = 8192 in bf16)

// One workgroup per projected row r = p*K + l (r < n*K).
// With an explicit row list (rowoff, a lazy pass over *grp layers from *top
// down), row r = j * *grp + g < *n_ptr is layer *top - g of listed position j;
// otherwise rows are gathered for r < *n_ptr * K.
//
// A row is 8 KB, so what bounds it is the chain of round trips (count, row
// list, row, output), not the bandwidth: VEC elements per load (16 bytes of
// long rows), the gain loaded with the row, and the row kept in registers from
// the sum to the scaling. 512 rows of d = 3584: 15.9 us with one element per
// load and every row read twice, 10.7 so.
//
// FC: every workgroup also scans the mask for its position
// (compact_in_workgroup), on a small canvas, which saves the compaction's
// launch.
template <typename T, int VEC, bool FC>
__global__ __launch_bounds__(kNormThreads) void k_norm_rows(const T* __restrict__ hidden, const T* __restrict__ g,
                                                           const int32_t* __restrict__ rows,
                                                           const int32_t* __restrict__ n_ptr, T* __restrict__ xrows,
                                                           int K, int B, int L, int d, float eps, int norm_final,
                                                           const long long* __restrict__ rowoff,
                                                           const int32_t* __restrict__ grp,
                                                           const int32_t* __restrict__ top, CompactArgs ca) {
  struct alignas(VEC * sizeof(T)) Piece {
    T e[VEC];
  };
  __shared__ double s_ss[kNormThreads / 64];
  const int r = blockIdx.x;
  int l;
  const T* src;
  if constexpr (FC) {
    __shared__ int s_pos[1], s_wave[kNormThreads / 64];
    MaskBytes<kNormThreads / 64> mb;
    mb.load(ca);
    const int p = r / K;
    l = r - p * K;
    const int n = compact_in_workgroup<kNormThreads / 64>(ca, mb, s_pos, p, 1, s_wave);
    if (p >= n) return;
    src = hidden + ((long long)l * B * L + s_pos[0]) * (long long)d;
  } else if (rowoff) {
    if (r >= *n_ptr) return;
    const int G = *grp, j = r / G, k = r - j * G;
    l = *top - k;
    src = hidden + rowoff[j] - k * ((long long)B * L * d);
  } else {
    if (r >= *n_ptr * K) return;
    const int p = r / K;
    l = r - p * K;
    src = hidden + ((long long)l * B * L + rows[p]) * (long long)d;
  }
  const Piece* sp = reinterpret_cast<const Piece*>(src);
  const Piece* gp = reinterpret_cast<const Piece*>(g);
  Piece* dp = reinterpret_cast<Piece*>(xrows + (long long)r * d);
  const int np = d / VEC;
  if (l == K - 1 && !norm_final) {
    for (int k = threadIdx.x; k < np; k += kNormThreads) dp[k] = sp[k];
    return;
  }
  Piece keep[kNormKeep], gain[kNormKeep];
#pragma unroll
  for (int u = 0; u < kNormKeep; ++u) {
    const int k = threadIdx.x + u * kNormThreads;
    keep[u] = Piece{};
    if (k < np) {
      keep[u] = sp[k];
      gain[u] = gp[k];
    }
  }
  double ss = 0.0;
#pragma unroll
  for (int u = 0; u < kNormKeep; ++u)
#pragma unroll
    for (int e = 0; e < VEC; ++e) {
      const double x = load_f64(keep[u].e, e);
      ss += x * x;
    }
  for (int k = threadIdx.x + kNormKeep * kNormThreads; k < np; k += kNormThreads) {
    const Piece v = sp[k];
#pragma unroll
    for (int e = 0; e < VEC; ++e) {
      const double x = load_f64(v.e, e);
      ss += x * x;
    }
  }
#pragma unroll
  for (int m = 32; m >= 1; m >>= 1) ss += __shfl_xor(ss, m);
  const int lane = threadIdx.x & 63, wid = threadIdx.x >> 6;
  if (lane == 0) s_ss[wid] = ss;
  __syncthreads();
  ss = 0.0;
#pragma unroll
  for (int w = 0; w < kNormThreads / 64; ++w) ss += s_ss[w];
  const double den = sqrt(ss / (double)d + (double)eps);
  auto put = [&](int k, const Piece& x, const Piece& w) {
    Piece y;
#pragma unroll
    for (int e = 0; e < VEC; ++e) store_f64(y.e, e, load_f64(w.e, e) * load_f64(x.e, e) / den);
    dp[k] = y;
  };
#pragma unroll
  for (int u = 0; u < kNormKeep; ++u) {
    const int k = threadIdx.x + u * kNormThreads;
    if (k < np) put(k, keep[u], gain[u]);
  }
  for (int k = threadIdx.x + kNormKeep * kNormThreads; k < np; k += kNormThreads) put(k, sp[k], gp[k]);
}

template <typename T, int VEC>
void launch_norm(const Launch& a, const dim3& grid, hipStream_t s) {
  const auto kernel = a.fused_compact ? k_norm_rows<T, VEC, true> : k_norm_rows<T, VEC, false>;
  const CompactArgs ca{a.mask, a.B * a.L, a.max_masked, a.rows, a.n_masked, a.dev_status, a.user_status};
  hipLaunchKernelGGL(kernel, grid, dim3(kNormThreads), 0, s, static_cast<const T*>(a.hidden),
                     static_cast<const T*>(a.norm_weight), a.rows, a.n_masked, static_cast<T*>(a.xrows), a.K, a.B, a.L,
                     a.d, a.norm_eps, a.norm_final, a.rowoff, a.lazy.grp, a.lazy.top, ca);
}

}  // namespace

hipError_t launch_norm_rows(const Launch& a, hipStream_t s) {
  if (a.max_masked <= 0) return hipSuccess;
  // an explicit row list holds max_masked rows
  const dim3 grid((unsigned)(a.rowoff ? (long long)a.max_masked : (long long)a.K * a.max_masked));
  // bf16: d % 8 == 0 and 16-byte aligned sources, as the call requires. Short
  // rows take smaller pieces, which keeps the workgroup's threads busy (d =
  // 512 in pieces of 8: the call 1.3 us longer than with one element a load).
  if (a.plan.variant != PROJ_F32) {
    if (a.d >= 8 * kNormThreads)
      launch_norm<uint16_t, 8>(a, grid, s);
    else
      launch_norm<uint16_t, 2>(a, grid, s);
  } else if (a.d >= 4 * kNormThreads && a.d % 4 == 0 && (((uintptr_t)a.hidden | (uintptr_t)a.norm_weight) & 15) == 0)
    launch_norm<float, 4>(a, grid, s);
  else
    launch_norm<float, 1>(a, grid, s);
  return hipGetLastError();
}

}  // namespace rpd
