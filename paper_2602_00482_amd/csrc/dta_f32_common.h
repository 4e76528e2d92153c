// What the fp32 kernels share: dta_f32_kernels.hip (products on the fp32 matrix
// instruction) and dta_f32_planes.hip (products on the bf16 one, operands in three parts).
#pragma once

#include <hip/hip_runtime.h>

#include "dta_internal.h"
#include "dta_mfma.h"

namespace dta {

// D(16x16) += A(16x4) * B(4x16), fp32.  Lane l = (n = l % 16, g = l / 16):
//   A: row n, k = g     B: column n, k = g     D: column n, row = 4*g + v, v = 0..3
__device__ __forceinline__ f32x4 mfma16_f32(float a, float b, f32x4 c) {
  return __builtin_amdgcn_mfma_f32_16x16x4f32(a, b, c, 0, 0, 0);
}

// sum / max over the four lane groups that share a column
__device__ __forceinline__ float column_sum(float x) {
  x += __shfl_xor(x, 16);
  x += __shfl_xor(x, 32);
  return x;
}
__device__ __forceinline__ float column_max(float x) {
  x = fmaxf(x, __shfl_xor(x, 16));
  return fmaxf(x, __shfl_xor(x, 32));
}

// The forward of single rows (query qrow of this lane's column), key by key: acc = columns
// 16 * j + 4 * (lane group) .. + 3 of sum w v over the keys the row sees, with w = exp(s - m) * inv.  For rows that a
// V row they do not see has spoilt (a masked key's probability 0 times a value that is not finite).
// Called by whole waves.
template <int HD>
__device__ __forceinline__ void row_by_keys(const QTile& tile, const KeySeg* segs, const int32_t* kend, int qrow,
                                            const float* q_row, const float* kbase, const float* vbase,
                                            size_t kv_stride, float scale, float m, float inv, f32x4 (&acc)[HD / 16]) {
  constexpr int NB = HD / 16;
  const int lg = (threadIdx.x >> 4) & 3;
  f32x4 Qr[NB];
#pragma unroll
  for (int j = 0; j < NB; ++j) {
    Qr[j] = *reinterpret_cast<const f32x4*>(q_row + 4 * lg + 16 * j);
    acc[j] = f32x4{0.f, 0.f, 0.f, 0.f};
  }
  for (int si = tile.seg_begin; si <= tile.seg_end; ++si) {
    const bool own = si == tile.seg_end;
    const int start = own ? tile.t0 : segs[si].start, end = own ? tile.t1 : segs[si].end;
    const bool all = !own && segs[si].full;
#pragma unroll 1
    for (int key = start; key < end; ++key) {
      const size_t at = (size_t)key * kv_stride + 4 * lg;
      float s = 0.f;
#pragma unroll
      for (int j = 0; j < NB; ++j) {
        const f32x4 kx = *reinterpret_cast<const f32x4*>(kbase + at + 16 * j);
#pragma unroll
        for (int e = 0; e < 4; ++e) s = fmaf(kx[e], Qr[j][e], s);
      }
      s = column_sum(s) * scale;
      if (!all && !(key <= qrow && qrow < kend[key])) continue;
      const float w = expf(s - m) * inv;
#pragma unroll
      for (int j = 0; j < NB; ++j) {
        const f32x4 vx = *reinterpret_cast<const f32x4*>(vbase + at + 16 * j);
#pragma unroll
        for (int e = 0; e < 4; ++e) acc[j][e] = fmaf(w, vx[e], acc[j][e]);
      }
    }
  }
}

// What the backward kernels read and write.
struct F32BwdArgs {
  const QTile* tiles;
  const KeySeg* segs;
  const KvItem* items;
  const int32_t* kend;
  const float *q, *k, *v, *d_o, *o, *lse;
  float *delta, *dq, *dk, *dv, *partial;
  int accumulate, Hq, Hkv, HB, hblocks;
  float scale;
  int dkdv_blocks;   // blocks [0, dkdv_blocks) of a launch of both do dK/dV, the rest dQ
};

// Launchers of dta_f32_planes.hip; they return a DTA status.  (dkdv: the partial sums are
// added by the caller's reduce launch, if any)
int launch_fwd_f32_planes(const LaunchArgs& a, size_t blocks);
int launch_dq_f32_planes(const LaunchArgs& a, const F32BwdArgs& args, size_t blocks);
int launch_dkdv_f32_planes(const LaunchArgs& a, const F32BwdArgs& args, size_t blocks);

}  // namespace dta
