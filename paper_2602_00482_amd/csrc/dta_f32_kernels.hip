// fp32 tree attention for gfx950: forward, dQ and dK/dV with every product, sum
// and exponential in fp32, for callers that need ~1e-6 relative accuracy.  Here: launches
// that do not fill the chip; the others are in dta_f32_planes.hip (f32_planes in
// dta_tree.cpp has the rule).
//
// What is computed follows the attention inside the paper's FWD / BWD
// primitives (pseudocode appendix) for all segments of the tree at once: a
// query sees key k iff  k <= t < kend[k]  in packed DFS coordinates.
//
// All products run on the fp32 matrix instruction (v_mfma_f32_16x16x4_f32: fused
// multiply-adds in fp32, nothing is rounded to a shorter type), twice the rate
// of the vector ALU without packed arithmetic.  A
// 16x16x4 product holds a SIMD for 32 cycles and needs one operand of 256 bytes
// from LDS, a quarter of what LDS delivers.  A wave
// owns 16 query rows (forward, dQ) or 16 keys (dK/dV): with 32 the stationary
// operands and accumulators of dK/dV (four 32 x 128 matrices) would not fit in
// 256 registers, and small trees would have half as many waves to spread.
//   The scores of a tile come out with the streamed rows (keys, or queries) in
// registers and the wave's own 16 in lanes: register v of lane group l / 16 is
// streamed row 4 * (l / 16) + v, which is exactly the operand layout of the next
// product with that row as the contraction index, so P and dS never move.
//
//   Products that contract over head_dim sum its two halves apart: one chain of
// head_dim / 4 instructions rounds more than the chains per quarter of head_dim that
// four lanes per row on the vector ALU had.  It costs 1 to 2 % of each kernel, and quarters cost dQ 4 %.
//
// Measured on MI355X, four lanes per row on the vector ALU before, and now:
//   384 tokens in 13 nodes, 4/4 heads of 64 (latency of a chain of dependent steps):
//     forward 71 -> 11 us, dQ 64 and dK/dV 146 -> 17 us together (two launches)
#include <hip/hip_runtime.h>

#include "dta_f32_common.h"
#include "dta_launch.h"
#include "dta_tile_walk.h"

namespace dta {
namespace {

// ---- 32-row tiles of HD floats filled by direct global-to-LDS loads -------------
// One wave-wide 16-byte load fills 1 KB = kRowsPerGroup consecutive rows; groups
// start 1056 bytes apart.  Matrix position x (0..31) uses row
//   kRowsPerGroup * (x % kGroups) + x / kGroups
// so that 8 consecutive positions lie in 8 different groups, 32 bytes of bank
// offset apart: a 16-byte row read of 8 lanes touches 8 different bank quads.
template <int HD>
struct Rows32 {
  static_assert(HD == 128 || HD == 64, "head_dim 64 or 128");
  static constexpr int kRowsPerGroup = 256 / HD;
  static constexpr int kGroups = 32 / kRowsPerGroup;
  static constexpr int kPitch = 256 + 8;             // floats between groups
  static constexpr int kTile = kGroups * kPitch;     // floats per tile
  static constexpr int NB = HD / 16;                 // 16-wide output blocks; also float4 per lane and row

  __device__ __forceinline__ static int row_of_pos(int x) {
    return kRowsPerGroup * (x % kGroups) + x / kGroups;
  }
  // row of position 16*mb + 4*g + v
  __device__ __forceinline__ static int row_of_acc(int mb, int g, int v) {
    return HD == 128 ? 8 * g + 2 * v + mb : 16 * (g & 1) + 4 * v + (g >> 1) + 2 * mb;
  }
  // per-lane base of row operands: float4 j of position 16*mb + n is at
  //   tile + row_lane_off() + 128 * mb + 16 * j      (columns 16*j + 4*g .. +3)
  __device__ __forceinline__ static int row_lane_off() {
    const int n = threadIdx.x & 15, g = (threadIdx.x >> 4) & 3;
    return (n % kGroups) * kPitch + (n / kGroups) * HD + 4 * g;
  }
  // per-lane base of column operands: lane n owns columns NB*n .. NB*n + NB-1 (one per
  // output block), of position 16*mb + 4*g + v:
  //   tile + col_lane_off() + 128 * mb + kPitch * v
  __device__ __forceinline__ static int col_lane_off() {
    const int n = threadIdx.x & 15, g = (threadIdx.x >> 4) & 3;
    return ((4 * g) % kGroups) * kPitch + ((4 * g) / kGroups) * HD + NB * n;
  }
};

// Starts the copy of ROWS rows of HD floats (row pitch stride_bytes, base uniform
// over the block) into ROWS / 32 consecutive tiles; rows >= nvalid re-read row
// nvalid - 1.  NW waves take part.  Completion: async_wait_all(), then a barrier.
template <int HD, int ROWS, int NW>
__device__ __forceinline__ void rows_async_load(float* tiles, const float* base, uint32_t stride_bytes,
                                                int nvalid) {
  using RL = Rows32<HD>;
  constexpr int kGroupsAll = ROWS / RL::kRowsPerGroup, kLaneShift = HD == 128 ? 5 : 4;
  static_assert(kGroupsAll % NW == 0, "every wave copies the same number of row groups");
  const int w = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), l = threadIdx.x & 63;
  const uint32_t tile_addr = (uint32_t)(uintptr_t)(__attribute__((address_space(3))) void*)tiles;
  const uint64_t base_bits = (uint64_t)(uintptr_t)base;
  const uint32_t base_hi = (uint32_t)__builtin_amdgcn_readfirstlane((int)(uint32_t)(base_bits >> 32));
  const uint32_t base_lo = (uint32_t)__builtin_amdgcn_readfirstlane((int)(uint32_t)base_bits);
  const uint64_t sbase = ((uint64_t)base_hi << 32) | (uint64_t)base_lo;
#pragma unroll
  for (int p = 0; p < kGroupsAll / NW; ++p) {
    const int grp = w + NW * p;
    const int row = min(RL::kRowsPerGroup * grp + (l >> kLaneShift), nvalid - 1);
    const uint32_t voff = (uint32_t)row * stride_bytes + (l & ((1 << kLaneShift) - 1)) * 16;
    const uint32_t lds_addr = __builtin_amdgcn_readfirstlane(tile_addr + grp * RL::kPitch * 4);
    asm volatile("s_mov_b32 m0, %2\n\tglobal_load_lds_dwordx4 %0, %1"
                 :
                 : "v"(voff), "s"(sbase), "s"(lds_addr)
                 : "memory");
  }
}

// The KS wave groups of a block each hold a partial sum of N float4 per lane;
// afterwards group 0 holds the total, added in group order.  `buf`: LDS of
// (KS - 1) * R * N * 1 KB that nobody reads any more.  Called by every thread.
template <int KS, int R, int N>
__device__ __forceinline__ void sum_over_groups(f32x4* buf, int rw, int kg, f32x4 (&acc)[N]) {
  const int l = threadIdx.x & 63;
  __syncthreads();
  if (kg > 0) {
#pragma unroll
    for (int i = 0; i < N; ++i) buf[(((kg - 1) * R + rw) * N + i) * 64 + l] = acc[i];
  }
  __syncthreads();
  if (kg == 0) {
#pragma unroll
    for (int s = 0; s < KS - 1; ++s)
#pragma unroll
      for (int i = 0; i < N; ++i) acc[i] += buf[((s * R + rw) * N + i) * 64 + l];
  }
}

// Block = NW waves = R row tiles (HB q heads of the group x 16-row blocks) x KS
// groups.  The keys of the tile's root path are streamed in chunks of 32 * KS
// keys, double-buffered in LDS; group kg of the block takes keys
// [32*kg, 32*kg + 32) of every chunk and the groups' results are merged at the
// end.  KS = 4 / 2 (head_dim 64 / 128): a fourth / half of the rows per block and of the
// steps per walk of blocks of 8 row tiles.  NW = 4: half the row
// tiles again, one wave per SIMD, for launches of so few blocks that a CU works on
// one of them: what a step takes is the SIMD's products, and two waves have twice as many.
template <int HD, int KS, int NW>
__global__ __launch_bounds__(64 * NW) void fwd_f32_kernel(
    const QTile* __restrict__ tiles, const KeySeg* __restrict__ segs, const int32_t* __restrict__ kend,
    const float* __restrict__ q, const float* __restrict__ k, const float* __restrict__ v,
    float* __restrict__ o, float* __restrict__ lse, int Hq, int Hkv, int HB, int hblocks, float scale) {
  using RL = Rows32<HD>;
  constexpr int NB = RL::NB, R = NW / KS, CH = 32 * KS;
  __shared__ __attribute__((aligned(1024))) float Ks[2][KS * RL::kTile];
  __shared__ __attribute__((aligned(1024))) float Vs[2][KS * RL::kTile];
  __shared__ __attribute__((aligned(16))) int32_t kendS[2][CH];
  __shared__ float mlS[2][KS][R][16];

  const int item = blockIdx.x / Hkv, g_kv = blockIdx.x % Hkv;
  const QTile tile = tiles[item / hblocks];
  const int w = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), l = threadIdx.x & 63;
  const int n16 = l & 15, lg = l >> 4;
  const int rw = w % R, kg = w / R;
  const int h = g_kv * (Hq / Hkv) + (item % hblocks) * HB + rw % HB;
  const int row_base = tile.t0 + 16 * (rw / HB);
  const int qrow = min(row_base + n16, tile.t1 - 1);

  f32x4 Qr[NB];
  {
    const float* qp = q + ((size_t)qrow * Hq + h) * HD + 4 * lg;
#pragma unroll
    for (int j = 0; j < NB; ++j) Qr[j] = *reinterpret_cast<const f32x4*>(qp + 16 * j);
  }
  f32x4 O[NB];
#pragma unroll
  for (int b = 0; b < NB; ++b) O[b] = f32x4{0.f, 0.f, 0.f, 0.f};
  float m = -INFINITY, lsum = 0.f;   // lsum: this lane's share of the row sum

  const size_t kv_stride = (size_t)Hkv * HD;
  const float* kbase = k + (size_t)g_kv * HD;
  const float* vbase = v + (size_t)g_kv * HD;
  const uint32_t kv_bytes = (uint32_t)kv_stride * 4;

  KeyChunksT<CH> it;
  it.init(segs, tile);
  int c0, n, full;
  bool have = it.next(c0, n, full);
  auto issue = [&](int b) {
    if ((!full || n < CH) && threadIdx.x < CH) {   // kendS is indexed by matrix position
      const int row = 32 * (threadIdx.x >> 5) + RL::row_of_pos(threadIdx.x & 31);
      kendS[b][threadIdx.x] = row >= n ? 0 : (full ? 0x7fffffff : kend[c0 + row]);
    }
    rows_async_load<HD, CH, NW>(Ks[b], kbase + (size_t)c0 * kv_stride, kv_bytes, n);
    rows_async_load<HD, CH, NW>(Vs[b], vbase + (size_t)c0 * kv_stride, kv_bytes, n);
  };
  issue(0);
  int buf = 0;
  const int rlo = kg * RL::kTile + RL::row_lane_off(), clo = kg * RL::kTile + RL::col_lane_off();

  while (have) {
    async_wait_all();
    __syncthreads();   // chunk `buf` has landed; everyone is done with the other buffer
    const int k0 = c0 + 32 * kg, nk = n - 32 * kg;   // this group's keys
    const bool need_mask = !full || nk < 32;
    have = it.next(c0, n, full);
    if (have) issue(buf ^ 1);
    // nothing here, or keys that come after every row of this wave (own range only)
    if (nk > 0 && !(need_mask && k0 > row_base + 15)) {
      const float* Kt = Ks[buf] + rlo;
      const float* Vt = Vs[buf] + clo;
      f32x4 Sh[2][2] = {};   // sums over each half of head_dim: shorter chains of roundings
#pragma unroll
      for (int j = 0; j < NB; ++j) {
        const f32x4 a0 = *reinterpret_cast<const f32x4*>(Kt + 16 * j);
        const f32x4 a1 = *reinterpret_cast<const f32x4*>(Kt + 128 + 16 * j);
        f32x4(&c)[2] = Sh[j / (NB / 2)];
#pragma unroll
        for (int e = 0; e < 4; ++e) {
          c[0] = mfma16_f32(a0[e], Qr[j][e], c[0]);
          c[1] = mfma16_f32(a1[e], Qr[j][e], c[1]);
        }
      }
      f32x4 S[2] = {Sh[0][0] + Sh[1][0], Sh[0][1] + Sh[1][1]};
      float mx = -INFINITY;
#pragma unroll
      for (int mb = 0; mb < 2; ++mb) {
        S[mb] *= scale;
        if (need_mask) {
          const int4 ke = *reinterpret_cast<const int4*>(&kendS[buf][32 * kg + 16 * mb + 4 * lg]);
          const int kev[4] = {ke.x, ke.y, ke.z, ke.w};
#pragma unroll
          for (int e = 0; e < 4; ++e)
            S[mb][e] = ((k0 + RL::row_of_acc(mb, lg, e) <= qrow) & (qrow < kev[e])) ? S[mb][e] : -INFINITY;
        }
#pragma unroll
        for (int e = 0; e < 4; ++e) mx = fmaxf(mx, S[mb][e]);
      }
      const float mnew = fmaxf(m, column_max(mx));
      const float mref = mnew == -INFINITY ? 0.f : mnew;
      const float alpha = expf(m - mref);
      m = mnew;
      float ps = 0.f;
#pragma unroll
      for (int mb = 0; mb < 2; ++mb)
#pragma unroll
        for (int e = 0; e < 4; ++e) {
          S[mb][e] = expf(S[mb][e] - mref);
          ps += S[mb][e];
        }
      lsum = fmaf(lsum, alpha, ps);
      if (__builtin_amdgcn_ballot_w64(alpha != 1.f) != 0) {
#pragma unroll
        for (int b = 0; b < NB; ++b) O[b] *= alpha;
      }
#pragma unroll
      for (int mb = 0; mb < 2; ++mb)
#pragma unroll
        for (int e = 0; e < 4; ++e) {
          f32x4 a[NB / 4];
#pragma unroll
          for (int x = 0; x < NB / 4; ++x)
            a[x] = *reinterpret_cast<const f32x4*>(Vt + 128 * mb + RL::kPitch * e + 4 * x);
#pragma unroll
          for (int b = 0; b < NB; ++b) O[b] = mfma16_f32(a[b >> 2][b & 3], S[mb][e], O[b]);
        }
    }
    buf ^= 1;
  }

  float lt = column_sum(lsum);
  // merge the groups: common maximum, then one sum
  if (lg == 0) {
    mlS[0][kg][rw][n16] = m;
    mlS[1][kg][rw][n16] = lt;
  }
  __syncthreads();
  float mall = mlS[0][0][rw][n16];
#pragma unroll
  for (int s = 1; s < KS; ++s) mall = fmaxf(mall, mlS[0][s][rw][n16]);
  const float mref = mall == -INFINITY ? 0.f : mall;   // (every score of the row may be -inf)
  lt = 0.f;
#pragma unroll
  for (int s = 0; s < KS; ++s) lt = fmaf(expf(mlS[0][s][rw][n16] - mref), mlS[1][s][rw][n16], lt);
  const float f = expf(m - mref);
#pragma unroll
  for (int b = 0; b < NB; ++b) O[b] *= f;
  m = mall;
  sum_over_groups<KS, R, NB>(reinterpret_cast<f32x4*>(&Ks[0][0]), rw, kg, O);
  if (kg != 0) return;
  const float inv = 1.f / lt;
  {
    // The products above multiply the V rows of masked keys by 0, which is NaN where such a
    // row is not finite: a row's output must not depend on keys it does not see.  Rows with a
    // finite sum and an output that is not finite are worked out again (row_by_keys).
    float t = 0.f;
#pragma unroll
    for (int b = 0; b < NB; ++b)
#pragma unroll
      for (int e = 0; e < 4; ++e) t = fmaf(O[b][e], 0.f, t);
    const bool spoilt = column_sum(t) != 0.f && lt - lt == 0.f;   // (NaN compares unequal)
    if (__builtin_amdgcn_ballot_w64(spoilt) != 0) {
      f32x4 acc[NB];
      row_by_keys<HD>(tile, segs, kend, qrow, q + ((size_t)qrow * Hq + h) * HD, kbase, vbase, kv_stride, scale, m, inv,
                      acc);
      if (spoilt && row_base + n16 < tile.t1) {
        float* op = o + ((size_t)qrow * Hq + h) * HD + 4 * lg;
#pragma unroll
        for (int j = 0; j < NB; ++j) *reinterpret_cast<f32x4*>(op + 16 * j) = acc[j];
        if (lg == 0) lse[(size_t)qrow * Hq + h] = m + logf(lt);
        return;
      }
    }
  }
  if (row_base + n16 < tile.t1) {
    float* op = o + ((size_t)qrow * Hq + h) * HD + NB * 4 * lg;
#pragma unroll
    for (int e = 0; e < 4; ++e)
#pragma unroll
      for (int x = 0; x < NB / 4; ++x) {
        f32x4 r;
#pragma unroll
        for (int b = 0; b < 4; ++b) r[b] = O[4 * x + b][e] * inv;
        *reinterpret_cast<f32x4*>(op + NB * e + 4 * x) = r;
      }
    if (lg == 0) lse[(size_t)qrow * Hq + h] = m + logf(lt);
  }
}

// D[t,h] = dO[t,h] . O[t,h], as a launch of its own: before a launch that does dQ and
// dK/dV together, and when the delta stage is asked for without dQ (otherwise the dQ
// launch computes it, in the same order).
template <int HD>
__global__ __launch_bounds__(256) void delta_f32_kernel(const float* __restrict__ o,
                                                        const float* __restrict__ d_o,
                                                        float* __restrict__ delta, size_t rows) {
  const size_t row = (size_t)blockIdx.x * 64 + threadIdx.x / 4;
  const int g = threadIdx.x % 4;   // plays lane group g of the dQ kernel
  float s = 0.f;
  if (row < rows) {
    const float* a = o + row * HD + 4 * g;
    const float* b = d_o + row * HD + 4 * g;
#pragma unroll
    for (int j = 0; j < HD / 16; ++j)
#pragma unroll
      for (int e = 0; e < 4; ++e) s = fmaf(a[16 * j + e], b[16 * j + e], s);
  }
  s += __shfl_xor(s, 1);
  s += __shfl_xor(s, 2);
  if (row < rows && g == 0) delta[row] = s;
}

template <int HD, int KS>
struct DqSmem {
  float K[2][KS * Rows32<HD>::kTile];
  float V[2][KS * Rows32<HD>::kTile];
  int32_t kendS[2][32 * KS];
};

// Same walk and block shapes as the forward kernel.  With o != nullptr the launch
// also computes D for its rows and leaves it in `delta` for dK/dV.
template <int HD, int KS, int NW>
__device__ __forceinline__ void dq_block(const F32BwdArgs& p, DqSmem<HD, KS>& sm, int block) {
  using RL = Rows32<HD>;
  constexpr int NB = RL::NB, R = NW / KS, CH = 32 * KS;
  auto& Ks = sm.K;
  auto& Vs = sm.V;
  auto& kendS = sm.kendS;
  const int32_t* __restrict__ kend = p.kend;
  const float *__restrict__ q = p.q, *__restrict__ k = p.k, *__restrict__ v = p.v, *__restrict__ d_o = p.d_o;
  const float *__restrict__ o = p.o, *__restrict__ lse = p.lse;
  const KeySeg* __restrict__ segs = p.segs;
  float *__restrict__ delta = p.delta, *__restrict__ dq = p.dq;
  const int Hq = p.Hq, Hkv = p.Hkv, HB = p.HB, hblocks = p.hblocks;
  const float scale = p.scale;

  const int item = block / Hkv, g_kv = block % Hkv;
  const QTile tile = p.tiles[item / hblocks];
  const int w = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), l = threadIdx.x & 63;
  const int n16 = l & 15, lg = l >> 4;
  const int rw = w % R, kg = w / R;
  const int h = g_kv * (Hq / Hkv) + (item % hblocks) * HB + rw % HB;
  const int row_base = tile.t0 + 16 * (rw / HB);
  const int qrow = min(row_base + n16, tile.t1 - 1);
  const size_t rh = (size_t)qrow * Hq + h;

  const size_t kv_stride = (size_t)Hkv * HD;
  const float* kbase = k + (size_t)g_kv * HD;
  const float* vbase = v + (size_t)g_kv * HD;
  const uint32_t kv_bytes = (uint32_t)kv_stride * 4;

  KeyChunksT<CH> it;
  it.init(segs, tile);
  int c0, n, full;
  bool have = it.next(c0, n, full);
  auto issue = [&](int b) {
    if ((!full || n < CH) && threadIdx.x < CH) {
      const int row = 32 * (threadIdx.x >> 5) + RL::row_of_pos(threadIdx.x & 31);
      kendS[b][threadIdx.x] = row >= n ? 0 : (full ? 0x7fffffff : kend[c0 + row]);
    }
    rows_async_load<HD, CH, NW>(Ks[b], kbase + (size_t)c0 * kv_stride, kv_bytes, n);
    rows_async_load<HD, CH, NW>(Vs[b], vbase + (size_t)c0 * kv_stride, kv_bytes, n);
  };
  issue(0);

  f32x4 Qr[NB], dOr[NB];
#pragma unroll
  for (int j = 0; j < NB; ++j) {
    Qr[j] = *reinterpret_cast<const f32x4*>(q + rh * HD + 4 * lg + 16 * j);
    dOr[j] = *reinterpret_cast<const f32x4*>(d_o + rh * HD + 4 * lg + 16 * j);
  }
  float dlt;
  if (o != nullptr) {
    dlt = 0.f;
#pragma unroll
    for (int j = 0; j < NB; ++j) {
      const f32x4 ox = *reinterpret_cast<const f32x4*>(o + rh * HD + 4 * lg + 16 * j);
#pragma unroll
      for (int e = 0; e < 4; ++e) dlt = fmaf(ox[e], dOr[j][e], dlt);
    }
    dlt = column_sum(dlt);
    if (kg == 0 && lg == 0 && row_base + n16 < tile.t1) delta[rh] = dlt;
  } else {
    dlt = delta[rh];
  }
  const float lse_t = lse[rh];
  f32x4 dQ[NB];
#pragma unroll
  for (int b = 0; b < NB; ++b) dQ[b] = f32x4{0.f, 0.f, 0.f, 0.f};

  int buf = 0;
  const int rlo = kg * RL::kTile + RL::row_lane_off(), clo = kg * RL::kTile + RL::col_lane_off();
  while (have) {
    async_wait_all();
    __syncthreads();
    const int k0 = c0 + 32 * kg, nk = n - 32 * kg;
    const bool need_mask = !full || nk < 32;
    have = it.next(c0, n, full);
    if (have) issue(buf ^ 1);
    if (nk > 0 && !(need_mask && k0 > row_base + 15)) {
      const float* Kt = Ks[buf] + rlo;
      const float* Vt = Vs[buf] + rlo;
      const float* Kc = Ks[buf] + clo;
      f32x4 Sh[2][2] = {}, dPh[2][2] = {};   // over each half of head_dim, as in the forward kernel
#pragma unroll
      for (int j = 0; j < NB; ++j)
#pragma unroll
        for (int mb = 0; mb < 2; ++mb) {
          const f32x4 ka = *reinterpret_cast<const f32x4*>(Kt + 128 * mb + 16 * j);
          const f32x4 va = *reinterpret_cast<const f32x4*>(Vt + 128 * mb + 16 * j);
#pragma unroll
          for (int e = 0; e < 4; ++e) {
            f32x4 &c = Sh[j / (NB / 2)][mb], &dc = dPh[j / (NB / 2)][mb];
            c = mfma16_f32(ka[e], Qr[j][e], c);
            dc = mfma16_f32(va[e], dOr[j][e], dc);
          }
        }
      f32x4 S[2] = {Sh[0][0] + Sh[1][0], Sh[0][1] + Sh[1][1]};
      const f32x4 dP[2] = {dPh[0][0] + dPh[1][0], dPh[0][1] + dPh[1][1]};
#pragma unroll
      for (int mb = 0; mb < 2; ++mb) {
#pragma unroll
        for (int e = 0; e < 4; ++e) S[mb][e] = expf(fmaf(S[mb][e], scale, -lse_t));
        if (need_mask) {
          const int4 ke = *reinterpret_cast<const int4*>(&kendS[buf][32 * kg + 16 * mb + 4 * lg]);
          const int kev[4] = {ke.x, ke.y, ke.z, ke.w};
#pragma unroll
          for (int e = 0; e < 4; ++e)
            S[mb][e] = ((k0 + RL::row_of_acc(mb, lg, e) <= qrow) & (qrow < kev[e])) ? S[mb][e] : 0.f;
        }
#pragma unroll
        for (int e = 0; e < 4; ++e) S[mb][e] *= dP[mb][e] - dlt;   // dS
      }
#pragma unroll
      for (int mb = 0; mb < 2; ++mb)
#pragma unroll
        for (int e = 0; e < 4; ++e) {
          f32x4 a[NB / 4];
#pragma unroll
          for (int x = 0; x < NB / 4; ++x)
            a[x] = *reinterpret_cast<const f32x4*>(Kc + 128 * mb + RL::kPitch * e + 4 * x);
#pragma unroll
          for (int b = 0; b < NB; ++b) dQ[b] = mfma16_f32(a[b >> 2][b & 3], S[mb][e], dQ[b]);
        }
    }
    buf ^= 1;
  }

  sum_over_groups<KS, R, NB>(reinterpret_cast<f32x4*>(&Ks[0][0]), rw, kg, dQ);
  if (kg == 0 && row_base + n16 < tile.t1) {
    float* op = dq + rh * HD + NB * 4 * lg;
#pragma unroll
    for (int e = 0; e < 4; ++e)
#pragma unroll
      for (int x = 0; x < NB / 4; ++x) {
        f32x4 r;
#pragma unroll
        for (int b = 0; b < 4; ++b) r[b] = dQ[4 * x + b][e] * scale;
        *reinterpret_cast<f32x4*>(op + NB * e + 4 * x) = r;
      }
  }
}

// Key-stationary: wave = 16 keys, K and V rows in registers; R key tiles x KS
// groups per block.  Q and dO of the rows that can see the keys are streamed in
// iterations of 32 rows of one q head, heads innermost, last chunk first, KS
// iterations per step, one per group.  KS and NW as in the forward kernel.
// Long walks are cut into items that write partial sums, as in bf16 mode.
template <int HD, int KS>
struct DkdvSmem {
  static constexpr int kStat = 32 * KS;
  float Q[2][KS * Rows32<HD>::kTile];
  float dO[2][KS * Rows32<HD>::kTile];
  __attribute__((aligned(256))) float stat[2][2][kStat];   // [buffer][lse | delta][position]
};

template <int HD, int KS, int NW>
__device__ __forceinline__ void dkdv_block(const F32BwdArgs& p, DkdvSmem<HD, KS>& sm, int block) {
  using RL = Rows32<HD>;
  constexpr int NB = RL::NB, R = NW / KS, kKeys = 16 * R, kStat = DkdvSmem<HD, KS>::kStat;
  auto& Qs = sm.Q;
  auto& dOs = sm.dO;
  auto& stat = sm.stat;
  const int32_t* __restrict__ kend = p.kend;
  const float *__restrict__ q = p.q, *__restrict__ k = p.k, *__restrict__ v = p.v, *__restrict__ d_o = p.d_o;
  const float *__restrict__ lse = p.lse, *__restrict__ delta = p.delta;
  float *__restrict__ dk = p.dk, *__restrict__ dv = p.dv, *__restrict__ partial = p.partial;
  const int accumulate = p.accumulate, Hq = p.Hq, Hkv = p.Hkv;
  const float scale = p.scale;

  const KvItem tile = p.items[block / Hkv];
  const int g = block % Hkv, G = Hq / Hkv;
  const int w = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), l = threadIdx.x & 63;
  const int n16 = l & 15, lg = l >> 4;
  const int kw = w % R, qg = w / R;
  const int kcol = tile.k0 + 16 * kw + n16;
  const int kc = min(kcol, tile.k1 - 1);
  const int my_kend = kcol < tile.k1 ? kend[kc] : 0;   // padded columns see nothing
  // rows [wave_lo, wave_hi) are the only ones any of this wave's keys can see
  int wave_hi = my_kend;
#pragma unroll
  for (int off = 8; off >= 1; off >>= 1) wave_hi = max(wave_hi, __shfl_xor(wave_hi, off));
  wave_hi = __builtin_amdgcn_readfirstlane(wave_hi);
  const int wave_lo = tile.k0 + 16 * kw;

  const size_t q_stride = (size_t)Hq * HD;
  const uint32_t q_bytes = (uint32_t)q_stride * 4;
  const int n_chunks = (tile.q_end - tile.q_begin + 31) / 32;
  const int total = tile.it_end;
  auto row_of_it = [&](int it) { return tile.q_begin + (n_chunks - 1 - it / G) * 32; };
  // copies iterations it .. it + KS-1 into buffer b (beyond the last one: the last again, never computed on)
  auto issue = [&](int it, int b) {
    if (w < kStat / 64) {   // stat is indexed by matrix position; a wave-wide copy covers two iterations
      const int r_base = row_of_it(min(it + 2 * w + 1, total - 1));
      const int i = min(it + 2 * w + (l >> 5), total - 1), r0 = row_of_it(i);
      const int row = min(RL::row_of_pos(l & 31), min(32, tile.q_end - r0) - 1);
      const uint32_t off = (uint32_t)(r0 - r_base + row) * (uint32_t)Hq + (uint32_t)(i % G);
      row_async_load(&stat[b][0][64 * w], lse + (size_t)r_base * Hq + g * G, off);
      row_async_load(&stat[b][1][64 * w], delta + (size_t)r_base * Hq + g * G, off);
    }
#pragma unroll
    for (int s = 0; s < KS; ++s) {
      const int i = min(it + s, total - 1), r0 = row_of_it(i), nv = min(32, tile.q_end - r0);
      const size_t at = (size_t)r0 * q_stride + (size_t)(g * G + i % G) * HD;
      rows_async_load<HD, 32, NW>(&Qs[b][s * RL::kTile], q + at, q_bytes, nv);
      rows_async_load<HD, 32, NW>(&dOs[b][s * RL::kTile], d_o + at, q_bytes, nv);
    }
  };
  if (tile.it_begin < total) issue(tile.it_begin, 0);

  f32x4 Kr[NB], Vr[NB];
#pragma unroll
  for (int j = 0; j < NB; ++j) {
    Kr[j] = *reinterpret_cast<const f32x4*>(k + ((size_t)kc * Hkv + g) * HD + 4 * lg + 16 * j);
    Vr[j] = *reinterpret_cast<const f32x4*>(v + ((size_t)kc * Hkv + g) * HD + 4 * lg + 16 * j);
  }
  f32x4 acc[2 * NB];   // dK, dV
#pragma unroll
  for (int b = 0; b < 2 * NB; ++b) acc[b] = f32x4{0.f, 0.f, 0.f, 0.f};

  const int rlo = qg * RL::kTile + RL::row_lane_off(), clo = qg * RL::kTile + RL::col_lane_off();
  int buf = 0;
  for (int it = tile.it_begin; it < total; it += KS) {
    async_wait_all();
    __syncthreads();
    if (it + KS < total) issue(it + KS, buf ^ 1);
    const int r0 = row_of_it(min(it + qg, total - 1));   // this group's rows
    const int nr = min(32, tile.q_end - r0);
    if (it + qg < total && r0 + nr > wave_lo && r0 < wave_hi) {
      const bool need_mask = !(r0 >= tile.k1 && r0 + 32 <= tile.q_full_end);
      const float* Qt = Qs[buf] + rlo;
      const float* dOt = dOs[buf] + rlo;
      const float* Qc = Qs[buf] + clo;
      const float* dOc = dOs[buf] + clo;
      // bounds of the visible rows of this lane's key, relative to r0
      const int lo = kcol - r0, hi = min(my_kend - r0, nr);
#pragma unroll
      for (int mb = 0; mb < 2; ++mb) {
        f32x4 Sh[2] = {}, dPh[2] = {};   // over each half of head_dim, as in the forward kernel
#pragma unroll
        for (int j = 0; j < NB; ++j) {
          const f32x4 qa = *reinterpret_cast<const f32x4*>(Qt + 128 * mb + 16 * j);
          const f32x4 da = *reinterpret_cast<const f32x4*>(dOt + 128 * mb + 16 * j);
#pragma unroll
          for (int e = 0; e < 4; ++e) {
            f32x4 &c = Sh[j / (NB / 2)], &dc = dPh[j / (NB / 2)];
            c = mfma16_f32(qa[e], Kr[j][e], c);
            dc = mfma16_f32(da[e], Vr[j][e], dc);
          }
        }
        f32x4 S = Sh[0] + Sh[1], dP = dPh[0] + dPh[1];
        const f32x4 ls = *reinterpret_cast<const f32x4*>(&stat[buf][0][32 * qg + 16 * mb + 4 * lg]);
        const f32x4 dl = *reinterpret_cast<const f32x4*>(&stat[buf][1][32 * qg + 16 * mb + 4 * lg]);
#pragma unroll
        for (int e = 0; e < 4; ++e) {
          float p = expf(fmaf(S[e], scale, -ls[e]));
          if (need_mask) {
            const int r = RL::row_of_acc(mb, lg, e);
            p = ((r >= lo) & (r < hi)) ? p : 0.f;
          }
          S[e] = p;
          dP[e] = p * (dP[e] - dl[e]);
        }
#pragma unroll
        for (int e = 0; e < 4; ++e) {
          f32x4 a[NB / 4], b[NB / 4];
#pragma unroll
          for (int x = 0; x < NB / 4; ++x) {
            a[x] = *reinterpret_cast<const f32x4*>(Qc + 128 * mb + RL::kPitch * e + 4 * x);
            b[x] = *reinterpret_cast<const f32x4*>(dOc + 128 * mb + RL::kPitch * e + 4 * x);
          }
#pragma unroll
          for (int i = 0; i < NB; ++i) {
            acc[i] = mfma16_f32(a[i >> 2][i & 3], dP[e], acc[i]);
            acc[NB + i] = mfma16_f32(b[i >> 2][i & 3], S[e], acc[NB + i]);
          }
        }
      }
    }
    buf ^= 1;
  }

  // (the LDS of both operands' buffers is one allocation only by declaration order: use each for its own half)
  f32x4(&a)[NB] = *reinterpret_cast<f32x4(*)[NB]>(&acc[0]);
  f32x4(&b)[NB] = *reinterpret_cast<f32x4(*)[NB]>(&acc[NB]);
  sum_over_groups<KS, R, NB>(reinterpret_cast<f32x4*>(&Qs[0][0]), kw, qg, a);
  sum_over_groups<KS, R, NB>(reinterpret_cast<f32x4*>(&dOs[0][0]), kw, qg, b);
  if (qg != 0) return;
  // lane (n16, lg) holds columns NB * (4*lg + e) + b of its key
  const int key = 16 * kw + n16;
#pragma unroll
  for (int half = 0; half < 2; ++half) {
    const float f = half == 0 ? scale : 1.f;
    float* out = half == 0 ? dk : dv;
    float* dst = tile.slot >= 0
                     ? partial + ((size_t)tile.slot * Hkv + g) * (2 * kKeys * HD) + (size_t)(half * kKeys + key) * HD
                     : out + ((size_t)kcol * Hkv + g) * HD;
    if (tile.slot < 0 && kcol >= tile.k1) continue;
#pragma unroll
    for (int e = 0; e < 4; ++e)
#pragma unroll
      for (int x = 0; x < NB / 4; ++x) {
        f32x4* at = reinterpret_cast<f32x4*>(dst + NB * (4 * lg + e) + 4 * x);
        f32x4 r;
#pragma unroll
        for (int b = 0; b < 4; ++b) r[b] = acc[half * NB + 4 * x + b][e];
        if (tile.slot < 0) {
          r *= f;
          // a segment call adds to the caller's accumulators (this block is the only
          // owner of the key in the launch)
          if (accumulate) r += *at;
        }
        *at = r;
      }
  }
}

template <int HD, int KS, int NW>
__global__ __launch_bounds__(64 * NW) void dq_f32_kernel(F32BwdArgs p) {
  __shared__ __attribute__((aligned(1024))) DqSmem<HD, KS> sm;
  dq_block<HD, KS, NW>(p, sm, blockIdx.x);
}

template <int HD, int KS, int NW>
__global__ __launch_bounds__(64 * NW, 1) void dkdv_f32_kernel(F32BwdArgs p) {
  __shared__ __attribute__((aligned(1024))) DkdvSmem<HD, KS> sm;
  dkdv_block<HD, KS, NW>(p, sm, blockIdx.x);
}

// Both in one launch, after one of the delta kernel: neither fills the chip by itself,
// and each is a few steps between a launch and its end.  Measured against dQ (which
// then computes D) and dK/dV after each other: 256 row tiles of 16, 32/8 heads of 128,
// 49 -> 35 us; 1000: 89 -> 85; 2000: 232 -> 208.
template <int HD, int KS, int NW>
__global__ __launch_bounds__(64 * NW, 1) void bwd_f32_kernel(F32BwdArgs p) {
  __shared__ __attribute__((aligned(1024))) union {
    DqSmem<HD, KS> dq;
    DkdvSmem<HD, KS> dkdv;
  } sm;
  if ((int)blockIdx.x < p.dkdv_blocks) dkdv_block<HD, KS, NW>(p, sm.dkdv, blockIdx.x);
  else dq_block<HD, KS, NW>(p, sm.dq, blockIdx.x - p.dkdv_blocks);
}

// Adds the partial sums of a split key tile in slot order and writes dK/dV.  One float4 of
// dK and dV per thread, and four slots in flight: a few split tiles of many parts are otherwise a chain of
// memory round trips.  Measured against four blocks per tile and head, one slot at a time: dK/dV stage of
// 1030 tokens with 32/1 heads of 128 215 -> 138 us, the launch alone for 4862 tokens with 32/8 heads 14.5 -> 9.
template <int HD>
__global__ __launch_bounds__(256) void dkdv_reduce_f32_kernel(const KvReduce* __restrict__ red,
                                                              const float* __restrict__ partial,
                                                              float* __restrict__ dk,
                                                              float* __restrict__ dv, int Hkv,
                                                              float scale, int keys) {
  const int blocks = (keys * (HD / 4) + 255) / 256;   // per (tile, kv head)
  const int tile_head = blockIdx.x / blocks;
  const KvReduce r = red[tile_head / Hkv];
  const int g = tile_head % Hkv, i = (blockIdx.x % blocks) * 256 + threadIdx.x;
  if (i >= (r.k1 - r.k0) * (HD / 4)) return;
  const size_t slot_stride = (size_t)Hkv * (2 * keys * HD);
  const float* src = partial + ((size_t)r.first_slot * Hkv + g) * (2 * keys * HD) + (size_t)4 * i;
  f32x4 sk = {0.f, 0.f, 0.f, 0.f}, sv = {0.f, 0.f, 0.f, 0.f};
  int p = 0;
  for (; p + 4 <= r.nparts; p += 4, src += 4 * slot_stride) {
    f32x4 a[4], b[4];
#pragma unroll
    for (int j = 0; j < 4; ++j) {
      a[j] = *reinterpret_cast<const f32x4*>(src + j * slot_stride);
      b[j] = *reinterpret_cast<const f32x4*>(src + j * slot_stride + keys * HD);
    }
#pragma unroll
    for (int j = 0; j < 4; ++j) {
      sk += a[j];
      sv += b[j];
    }
  }
  for (; p < r.nparts; ++p, src += slot_stride) {
    sk += *reinterpret_cast<const f32x4*>(src);
    sv += *reinterpret_cast<const f32x4*>(src + keys * HD);
  }
  const size_t o = ((size_t)(r.k0 + i / (HD / 4)) * Hkv + g) * HD + 4 * (i % (HD / 4));
  *reinterpret_cast<f32x4*>(dk + o) = sk * scale;
  *reinterpret_cast<f32x4*>(dv + o) = sv;
}

template <int HD>
int fwd_impl(const LaunchArgs& a) {
  clear_hip_error();
  const QueryTiles& qt = a.sched->forward_tiles();
  const size_t blocks = qt.q_tiles.size() * (size_t)a.p.n_kv_heads * (size_t)a.tc.hblocks;
  if (blocks == 0 || blocks > 0x7fffffffu) return DTA_ERR_UNSUPPORTED;
  if (a.tc.planes) return launch_fwd_f32_planes(a, blocks);
  constexpr int kSplit = HD == 64 ? 4 : 2;
  auto kernel = a.tc.tiny ? fwd_f32_kernel<HD, kSplit, 4> : fwd_f32_kernel<HD, kSplit, 8>;
  launch(a, true, kernel, blocks, a.tc.tiny ? 256 : 512,
      qt.d_q_tiles, qt.d_segs, a.d_kend, (const float*)a.q, (const float*)a.k,
      (const float*)a.v, (float*)a.o_out, a.lse_out, a.p.n_q_heads, a.p.n_kv_heads, a.tc.hb,
      a.tc.hblocks, a.p.softmax_scale);
  return launch_status(__func__);
}

template <int HD>
int bwd_impl(const LaunchArgs& a) {
  hipStream_t st = (hipStream_t)a.stream;
  clear_hip_error();
  const size_t row0 = (size_t)a.row_begin * a.p.n_q_heads;
  const size_t rows = (size_t)(a.row_end - a.row_begin) * a.p.n_q_heads;
  const size_t qblocks = a.sched->q_tiles.size() * (size_t)a.p.n_kv_heads * (size_t)a.tc.hblocks;
  const size_t kblocks = a.sched->kv_items.size() * (size_t)a.p.n_kv_heads;
  if (qblocks == 0 || qblocks > 0x7fffffffu || kblocks > 0x7fffffffu) return DTA_ERR_UNSUPPORTED;
  constexpr int kSplit = HD == 64 ? 4 : 2;
  const bool one_launch = a.tc.q_small && (a.stages & DTA_BWD_DQ) && (a.stages & DTA_BWD_DKDV) &&
                          qblocks + kblocks <= 0x7fffffffu;
  // otherwise the dQ launch computes D itself when both stages are asked for
  const bool fused_delta = (a.stages & DTA_BWD_DELTA) && (a.stages & DTA_BWD_DQ) && !one_launch;
  if ((a.stages & DTA_BWD_DELTA) && !fused_delta) {
    delta_f32_kernel<HD><<<(unsigned)((rows + 63) / 64), 256, 0, st>>>(
        (const float*)a.o + row0 * HD, (const float*)a.d_o + row0 * HD, a.delta + row0, rows);
    { int ls = launch_status(__func__); if (ls != DTA_OK) return ls; }
  }
  const F32BwdArgs args{a.sched->d_q_tiles, a.sched->d_segs, a.sched->d_kv_items, a.d_kend, (const float*)a.q,
                     (const float*)a.k, (const float*)a.v, (const float*)a.d_o,
                     fused_delta ? (const float*)a.o : nullptr, a.lse_in, a.delta, (float*)a.dq,
                     a.dk_acc ? a.dk_acc : (float*)a.dk, a.dk_acc ? a.dv_acc : (float*)a.dv, a.partial,
                     a.dk_acc != nullptr, a.p.n_q_heads, a.p.n_kv_heads, a.tc.hb, a.tc.hblocks,
                     a.p.softmax_scale, (int)kblocks};
  if (one_launch) {
    auto kernel = a.tc.tiny ? bwd_f32_kernel<HD, kSplit, 4> : bwd_f32_kernel<HD, kSplit, 8>;
    launch(a, a.sched->kv_reduce.empty(), kernel, qblocks + kblocks, a.tc.tiny ? 256 : 512, args);
    { int ls = launch_status(__func__); if (ls != DTA_OK) return ls; }
  } else if ((a.stages & DTA_BWD_DQ) && a.tc.planes) {
    const int ls = launch_dq_f32_planes(a, args, qblocks);
    if (ls != DTA_OK) return ls;
  } else if (a.stages & DTA_BWD_DQ) {
    auto kernel = a.tc.tiny ? dq_f32_kernel<HD, kSplit, 4> : dq_f32_kernel<HD, kSplit, 8>;
    kernel<<<(unsigned)qblocks, a.tc.tiny ? 256 : 512, 0, st>>>(args);
    { int ls = launch_status(__func__); if (ls != DTA_OK) return ls; }
  }
  if (a.stages & DTA_BWD_DKDV) {
    if (a.tc.planes) {
      const int ls = launch_dkdv_f32_planes(a, args, kblocks);
      if (ls != DTA_OK) return ls;
    } else if (!one_launch) {
      auto kernel = a.tc.tiny ? dkdv_f32_kernel<HD, kSplit, 4> : dkdv_f32_kernel<HD, kSplit, 8>;
      launch(a, a.sched->kv_reduce.empty(), kernel, kblocks, a.tc.tiny ? 256 : 512, args);
      { int ls = launch_status(__func__); if (ls != DTA_OK) return ls; }
    }
    if (!a.sched->kv_reduce.empty()) {
      const size_t per_tile = ((size_t)a.sched->kv_keys * (HD / 4) + 255) / 256;
      launch(a, true, dkdv_reduce_f32_kernel<HD>, a.sched->kv_reduce.size() * a.p.n_kv_heads * per_tile, 256,
          a.sched->d_kv_reduce, a.partial, (float*)a.dk, (float*)a.dv, a.p.n_kv_heads, a.p.softmax_scale,
          a.sched->kv_keys);
      { int ls = launch_status(__func__); if (ls != DTA_OK) return ls; }
    }
  }
  return DTA_OK;
}

}  // namespace

int launch_fwd_f32(const LaunchArgs& a) {
  return a.p.head_dim == 64 ? fwd_impl<64>(a) : fwd_impl<128>(a);
}
int launch_bwd_f32(const LaunchArgs& a) {
  return a.p.head_dim == 64 ? bwd_impl<64>(a) : bwd_impl<128>(a);
}

}  // namespace dta
