// K1 projection for fp32 inputs, on the fp32 matrix cores.
#include <type_traits>

#include "rpd_device.h"

namespace rpd {
namespace {

// s_waitcnt immediate: vmcnt <= n, lgkmcnt == 0, expcnt unconstrained
constexpr unsigned vm_lgkm_wait(int n) { return (unsigned)((n & 15) | ((n >> 4) << 14) | (7 << 4)); }

// A tile of TV = 32*WV vocabulary rows x TR = 32*NB projected rows over the
// full hidden dimension, one wave per 32 vocabulary rows, with
// v_mfma_f32_32x32x2_f32 (IEEE fp32 products and sums).
//
// What bounds it: the fp32 matrix rate (157 TFLOP/s nominal, 152 by the
// vendor's 8192^3 product on this card) is met by streaming W_U at about 45
// projected rows, so up to 32 rows HBM bounds the tile and from 64 rows on
// the MFMAs do (64 cycles each). A wave reads 1 + NB fragments for 4 * NB
// MFMAs, so LDS is busy for an eighth of the MFMA time or less and one
// wave-row layout serves every TR.
//
// Operands go from global memory straight into LDS in 32-wide k-chunks (rows
// of 128 bytes, the eight 16-byte pieces of row r XOR-swizzled by
// (r >> 1) & 7: fragment reads are free of bank conflicts), NS stages, one
// barrier per chunk: at the top of chunk c its loads have landed (the newest
// (NS - 2) chunks' may be outstanding), the barrier publishes them and frees
// chunk c - 1's stage for chunk c + NS - 1. A stage holds both operands, and
// the stages of every form fit twice into a CU's LDS, so that two workgroups
// share it and one's first loads and epilogue run under the other's MFMAs.
//
// A fragment read takes four consecutive k of a row (16 bytes): lanes 0-31
// hold k 8s .. 8s+3 and lanes 32-63 k 8s+4 .. 8s+7, and MFMA j of the step
// multiplies element j of both operands, i.e. the pair k = 8s+j, 8s+4+j.
// Every vocabulary row is summed in this one order, so equal rows give equal
// logits.
//
// The next step's fragments are read under this step's MFMAs, and a chunk's
// loads are issued before its MFMAs (the compiler, left alone, sank them to
// the end of the chunk: 4% slower).
//
// Measured at d = 4096, V = 126464 (whole call, against the vector-ALU kernel
// this replaces): 32 rows 1935 -> 380 us (HBM 5.6 TB/s in the projection),
// 256 rows 13.84 -> 2.10 ms (128 TFLOP/s; the matrix cores busy 81% of the
// active cycles, of which the last, partly filled round of tiles takes 6%);
// 120 rows at d = 256, V = 4096: 36.8 -> 19.1 us. A rotated chunk order
// (against HBM channel crowding) changed nothing at either size; 256 rows in tiles
// of 64 and 32 rows, with three or four stages, took 2.20 and 2.52 ms.
//
// V16: 16-byte loads (d % 4 == 0 and 16-byte aligned sources); else 4-byte
// loads, a quarter of the bytes per instruction.
//
// FC: the workgroup compacts the mask itself (compact_in_workgroup), on a
// small canvas: the first chunk of W_U is loaded while it does, and the
// positions sit in the stage loaded last (from chunk 0's barrier on).
template <int WV, int NB, int NS, bool V16, bool FC>
__global__ __launch_bounds__(WV * 64, 2) void k_proj_f32(
    const float* __restrict__ hidden, const float* __restrict__ w_u, const int32_t* __restrict__ rows,
    const int32_t* __restrict__ n_ptr, float4* __restrict__ partials, int K, int B, int L, int d, int V, int nvt,
    int nrt, int split_rows, const float* __restrict__ xrows, const long long* __restrict__ rowoff,
    const int32_t* __restrict__ grp, float scale, CompactArgs ca) {
  constexpr int TV = 32 * WV, TR = 32 * NB, KC = 32;
  constexpr int RPI = V16 ? 8 : 2;             // rows per load instruction
  constexpr int AL = 32 / RPI;                 // W_U load instructions per wave per chunk
  constexpr int BLD = TR / RPI / WV;           // hidden-row load instructions per wave per chunk
  static_assert(TR % (RPI * WV) == 0 && NS >= 2 && NS <= 4 && (NS - 2) * (AL + BLD) < 64, "load schedule");
  __shared__ __attribute__((aligned(1024))) float st0[TV + TR][KC], st1[TV + TR][KC];
  __shared__ __attribute__((aligned(1024))) float st2[NS > 2 ? TV + TR : 1][KC], st3[NS > 3 ? TV + TR : 1][KC];
#define RPD_ST(X) ((X) == 0 ? st0 : (X) == 1 ? st1 : (X) == 2 ? st2 : st3)
  float4 (*red)[TR] = reinterpret_cast<float4 (*)[TR]>(&st0[0][0]);   // used after the loop only

  int rt = 0, vt = 0;
  const bool has_job = map_job(blockIdx.x, nvt, nrt, split_rows, rt, vt);
  if (!has_job && !(FC && blockIdx.x == 0)) return;   // workgroup 0 always publishes the compaction
  const int r0 = rt * TR;
  int R = 0;
  if (!FC) {
    R = rowoff ? *n_ptr : *n_ptr * K;   // an explicit row list counts rows, not positions
    if (r0 >= R) return;
  }
  const int per = !FC && rowoff ? *grp : K;   // rows (layers) of a position
  const int vb = (int)((long long)vt * V / nvt);
  const int ve = (int)((long long)(vt + 1) * V / nvt);
  const int tid = threadIdx.x, lane = tid & 63, wid = tid >> 6;

#define RPD_FLOAD1(SRC, DST)                                                                               \
  do { /* the builtin's size is a literal */                                                               \
    if constexpr (V16)                                                                                     \
      __builtin_amdgcn_global_load_lds((const void*)(SRC), (__attribute__((address_space(3))) void*)(DST), 16, 0, 0); \
    else                                                                                                   \
      __builtin_amdgcn_global_load_lds((const void*)(SRC), (__attribute__((address_space(3))) void*)(DST), 4, 0, 0);  \
  } while (0)
#define RPD_FLOADA(X, chunk)                                                                               \
  do {                                                                                                     \
    const long long k0_ = (long long)(chunk)*KC;                                                           \
    _Pragma("unroll") for (int u_ = 0; u_ < AL; ++u_)                                                     \
      RPD_FLOAD1(pa[u_] + k0_, &RPD_ST(X)[32 * wid + RPI * u_][0]);                                        \
  } while (0)
#define RPD_FLOADB(X, chunk)                                                                               \
  do {                                                                                                     \
    const long long k0_ = (long long)(chunk)*KC;                                                           \
    _Pragma("unroll") for (int u_ = 0; u_ < BLD; ++u_)                                                    \
      RPD_FLOAD1(pb[u_] + k0_, &RPD_ST(X)[TV + (TR / WV) * wid + RPI * u_][0]);                            \
  } while (0)
#define RPD_FLOAD(X, chunk)                                                                                \
  do {                                                                                                     \
    RPD_FLOADA(X, chunk);                                                                                  \
    RPD_FLOADB(X, chunk);                                                                                  \
  } while (0)
  // Load sources. Instruction u of this wave covers tile rows 32*wid + RPI*u
  // .. of W_U and (TR/WV)*wid + RPI*u .. of the hidden rows; the lane lands at
  // row + lane / (64/RPI), LDS float lk of the row, and fetches the global
  // float that belongs there. Rows past the tile re-read its last vocabulary
  // row, rows past the last projected row re-read row r0 (both discarded).
  const int lrow = lane / (64 / RPI), lk = V16 ? (lane & 7) * 4 : (lane & 31);
  const float* pa[AL];
  const float* pb[BLD];
  int ka[AL], kb[BLD];   // first k of the lane's piece within a chunk
#pragma unroll
  for (int u = 0; u < AL; ++u) {
    const int tr = 32 * wid + RPI * u + lrow;
    ka[u] = (((lk >> 2) ^ ((tr >> 1) & 7)) << 2) + (lk & 3);
    pa[u] = w_u + (long long)min(vb + tr, ve - 1) * d + ka[u];
  }
  const int nchf = d / KC;
  int* s_pos = reinterpret_cast<int*>(&RPD_ST(NS - 1)[0][0]);   // the stage loaded last
  if constexpr (FC) {
    MaskBytes<WV> mb;
    mb.load(ca);   // ahead of the loads below (loads return in order)
    if (has_job && nchf > 0) RPD_FLOADA(0, 0);
    R = compact_in_workgroup<WV>(ca, mb, s_pos, r0 / K, TR, s_pos + TR) * K;
    if (!has_job || r0 >= R) {
      __builtin_amdgcn_s_waitcnt(0);   // the loads above write this workgroup's LDS
      return;
    }
  }
#pragma unroll
  for (int u = 0; u < BLD; ++u) {
    const int tr = (TR / WV) * wid + RPI * u + lrow;
    kb[u] = (((lk >> 2) ^ ((tr >> 1) & 7)) << 2) + (lk & 3);
    const int r = r0 + tr < R ? r0 + tr : r0;
    if (!FC && xrows) {   // normalized rows, already in projected-row order
      pb[u] = xrows + (long long)r * d + kb[u];
    } else {
      const int p = r / per, l = r - p * per;
      if (!FC && rowoff)   // an explicit row list, its layers from the first one down
        pb[u] = hidden + rowoff[p] - l * ((long long)B * L * d) + kb[u];
      else
        pb[u] = hidden + ((long long)l * B * L + (FC ? s_pos[p - r0 / K] : rows[p])) * (long long)d + kb[u];
    }
  }
  // fragment reads: row base + (lane & 31), logical piece 2s + (lane >> 5)
  const int fr = lane & 31, fsw = (fr >> 1) & 7, fhi = lane >> 5;

  f32x16 acc[NB];
#pragma unroll
  for (int nb = 0; nb < NB; ++nb)
#pragma unroll
    for (int q = 0; q < 16; ++q) acc[nb][q] = 0.f;

#define RPD_FFRAG(F, X, S)                                                                                 \
  do {                                                                                                     \
    const int fc_ = 4 * ((2 * (S) + fhi) ^ fsw);                                                           \
    F[NB] = *reinterpret_cast<const f32x4*>(&RPD_ST(X)[32 * wid + fr][fc_]);                               \
    _Pragma("unroll") for (int nb_ = 0; nb_ < NB; ++nb_)                                                  \
      F[nb_] = *reinterpret_cast<const f32x4*>(&RPD_ST(X)[TV + 32 * nb_ + fr][fc_]);                       \
    __builtin_amdgcn_sched_barrier(0);                                                                     \
  } while (0)
#define RPD_FMMA(F)                                                                                        \
  do {                                                                                                     \
    _Pragma("unroll") for (int j_ = 0; j_ < 4; ++j_)                                                      \
      _Pragma("unroll") for (int nb_ = 0; nb_ < NB; ++nb_)                                                \
        acc[nb_] = __builtin_amdgcn_mfma_f32_32x32x2f32(F[NB][j_], F[nb_][j_], acc[nb_], 0, 0, 0);         \
    __builtin_amdgcn_sched_barrier(0);                                                                     \
  } while (0)
  // chunk c in stage X (c % NS); chunks past the end repeat the last one (never multiplied)
#define RPD_FCHUNK(c, X)                                                                                   \
  do {                                                                                                     \
    __builtin_amdgcn_s_waitcnt(vm_lgkm_wait((NS - 2) * (AL + BLD)));                                       \
    __builtin_amdgcn_s_barrier();                                                                          \
    __builtin_amdgcn_sched_barrier(0);                                                                     \
    RPD_FFRAG(f0, X, 0);                                                                                   \
    RPD_FFRAG(f1, X, 1);                                                                                   \
    RPD_FLOAD(((X) + NS - 1) % NS, min((c) + NS - 1, nchf - 1));                                           \
    __builtin_amdgcn_sched_barrier(0);                                                                     \
    RPD_FMMA(f0);                                                                                          \
    RPD_FFRAG(f0, X, 2);                                                                                   \
    RPD_FMMA(f1);                                                                                          \
    RPD_FFRAG(f1, X, 3);                                                                                   \
    RPD_FMMA(f0);                                                                                          \
    RPD_FMMA(f1);                                                                                          \
  } while (0)

  f32x4 f0[NB + 1], f1[NB + 1];   // a k-step's fragments: NB of hidden rows, then W_U's
  if (nchf > 0) {
    if (!FC) RPD_FLOADA(0, 0);
    RPD_FLOADB(0, 0);
    if constexpr (NS > 2) RPD_FLOAD(1, min(1, nchf - 1));
    if constexpr (NS > 3) RPD_FLOAD(2, min(2, nchf - 1));
    int c = 0;
    for (; c + NS <= nchf; c += NS) {
      RPD_FCHUNK(c, 0);
      RPD_FCHUNK(c + 1, 1);
      if constexpr (NS > 2) RPD_FCHUNK(c + 2, 2);
      if constexpr (NS > 3) RPD_FCHUNK(c + 3, 3);
    }
    if (c < nchf) RPD_FCHUNK(c, 0);
    if (NS > 2 && c + 1 < nchf) RPD_FCHUNK(c + 1, 1);
    if constexpr (NS > 3)
      if (c + 2 < nchf) RPD_FCHUNK(c + 2, 2);
    __builtin_amdgcn_s_waitcnt(vm_lgkm_wait(0));   // no load outstanding past the loop
    __syncthreads();
  }
  if (d % KC != 0) {   // partial last chunk, zero-filled past d
    const long long k0 = (long long)nchf * KC;
    using piece = typename std::conditional<V16, f32x4, float>::type;
#pragma unroll
    for (int u = 0; u < AL; ++u) {
      piece v{};
      if (k0 + ka[u] < d) v = *reinterpret_cast<const piece*>(pa[u] + k0);
      *reinterpret_cast<piece*>(&st0[32 * wid + RPI * u + lrow][lk]) = v;
    }
#pragma unroll
    for (int u = 0; u < BLD; ++u) {
      piece v{};
      if (k0 + kb[u] < d) v = *reinterpret_cast<const piece*>(pb[u] + k0);
      *reinterpret_cast<piece*>(&st0[TV + (TR / WV) * wid + RPI * u + lrow][lk]) = v;
    }
    __syncthreads();
#pragma unroll
    for (int s4 = 0; s4 < 4; ++s4) {
      RPD_FFRAG(f0, 0, s4);
      RPD_FMMA(f0);
    }
    __syncthreads();   // red aliases stage 0
  }
#undef RPD_FCHUNK
#undef RPD_FMMA
#undef RPD_FFRAG
#undef RPD_FLOAD
#undef RPD_FLOADA
#undef RPD_FLOADB
#undef RPD_FLOAD1
#undef RPD_ST

  // epilogue: lane holds projected row 32*nb + (lane & 31) against vocabulary
  // rows 32*wid + 8*(q >> 2) + 4*(lane >> 5) + (q & 3) of the tile
#pragma unroll
  for (int nb = 0; nb < NB; ++nb) {
    float z[16];
    int vi[16];
    bool ok[16];
#pragma unroll
    for (int q = 0; q < 16; ++q) {
      const int v = vb + 32 * wid + (q >> 2) * 8 + (lane >> 5) * 4 + (q & 3);
      z[q] = acc[nb][q] * scale;
      vi[q] = v;
      ok[q] = v < ve;
    }
    Soft sst = soft_from_values(z, vi, ok);
    sst = soft_merge(sst, soft_shfl_xor(sst, 32));
    if (lane < 32) red[wid][32 * nb + lane] = soft_pack(sst);
  }
  __syncthreads();
  for (int t = tid; t < TR; t += WV * 64) {
    const int r = r0 + t;
    if (r < R) {
      Soft s = soft_unpack(red[0][t]);
#pragma unroll
      for (int w = 1; w < WV; ++w) s = soft_merge(s, soft_unpack(red[w][t]));
      partials[(long long)r * nvt + vt] = soft_pack(s);
    }
  }
}

template <int WV, int NB, int NS>
void launch_f32(const Launch& a, hipStream_t s) {
  const ProjPlan& p = a.plan;
  const void* src = a.xrows ? a.xrows : a.hidden;
  const bool v16 = a.d % 4 == 0 && (((uintptr_t)src | (uintptr_t)a.w_u) & 15) == 0;
  const auto kernel = a.fused_compact && !a.xrows ? (v16 ? k_proj_f32<WV, NB, NS, true, true> : k_proj_f32<WV, NB, NS, false, true>)
                                      : (v16 ? k_proj_f32<WV, NB, NS, true, false> : k_proj_f32<WV, NB, NS, false, false>);
  const CompactArgs ca{a.mask, a.B * a.L, a.max_masked, a.rows, a.n_masked, a.dev_status, a.user_status};
  hipLaunchKernelGGL(kernel, dim3(p.grid), dim3(WV * 64), 0, s, static_cast<const float*>(a.hidden),
                     static_cast<const float*>(a.w_u), a.rows, a.n_masked, a.partials, a.K, a.B, a.L, a.d, a.V, p.nvt,
                     p.nrt, p.split_rows, static_cast<const float*>(a.xrows), a.rowoff, a.lazy.grp,
                     a.logit_scale, ca);
}

}  // namespace

hipError_t launch_proj_f32(const Launch& a, hipStream_t s) {
  // stages: (TV + TR) * 128 B each, at most 80 KB in all (two workgroups per CU)
  if (a.plan.vocab_cap == kF32TileVocabSmall) {
    if (a.plan.rows_per_tile != 32) return hipErrorInvalidValue;
    launch_f32<2, 1, 4>(a, s);
  } else {
    switch (a.plan.rows_per_tile) {
      case 32: launch_f32<4, 1, 4>(a, s); break;
      case 64: launch_f32<4, 2, 3>(a, s); break;
      case 96: launch_f32<4, 3, 2>(a, s); break;
      case 128: launch_f32<4, 4, 2>(a, s); break;
      default: return hipErrorInvalidValue;
    }
  }
  return hipGetLastError();
}

}  // namespace rpd
