// bf16 tree attention for launches too small to fill the chip: segment calls of a
// few hundred rows, trees of a few hundred tokens.  Same arithmetic as the kernels
// of dta_bf16_fwd.hip / dta_bf16_bwd.hip (32x32x16 products, fp32 accumulation and
// softmax), other shape of the work.
//
// Such a launch is a handful of blocks, and its time is the longest block's chain
// of dependent steps.  A block here is 8 waves = 2 row (or key) tiles of 32 x 4
// groups: the groups share out the rows streamed through LDS, 32 each per step, and
// their results are added in LDS at the end.  Against the forms for large launches
// (8 row tiles, or 4 key tiles, walking 64 rows per step) a launch has 4 (dK/dV: 2)
// times as many blocks and each walks half as many steps, at the price of fewer
// tiles per copied row.
//
// The same launch does dQ and dK/dV: each alone is a few steps between a launch and
// its end, and together they fill the chip better.
//
// Measured on MI355X, head_dim 128, against the other forms (dta_tree.cpp has the
// rule that chooses and more figures): forward of 512 tokens, 32/8 heads, 18.3 -> 14.5 us,
// backward 100 -> 34; a 192-row segment under 2048 keys, 64/8 heads, forward 67 -> 35 us,
// backward 147 -> 75; under 8192 keys forward 204 -> 98, backward 401 -> 236.  With a step's first
// operands read before the next step's copies are issued, and a segment's accumulators read while the groups' sums
// are added, the calls of a leaf-order plan (short segments) take 11.0 us forward (11.3 before) and 14.6 us
// backward (17.1).  What is left
// is about 7 us from launch to store and 1.3 us per step of 128 streamed rows, a
// third of the matrix rate: one wave's chain of products, softmax, products, with
// only one other wave on its SIMD.
#include <hip/hip_runtime.h>

#include "dta_internal.h"
#include "dta_launch.h"
#include "dta_mfma.h"

namespace dta {
namespace {

constexpr int kThreads = 512;
constexpr int kGroupsOfWaves = 4, kTiles = 2;   // block = kTiles x kGroupsOfWaves waves
constexpr int kSub = 32;                        // streamed rows per group and step
constexpr int kStep = kSub * kGroupsOfWaves;

// The four 32-row sub-tiles of a step live in two 64-row LDS tiles (TileLayout):
// sub-tile s is half s & 1 of tile s >> 1, i.e. the matrix positions
// 32 * (s & 1) .. + 31 of that tile.  The two halves of a tile share every 1 KB
// group of rows, lanes 0-31 of the group's direct load filling one and lanes 32-63
// the other, so each half can come from its own rows of the tensor.
template <int HD>
struct SubLayout {
  using TL = TileLayout<HD>;
  static constexpr int kRowsPerHalfGroup = kSub / TL::kGroups;   // 2 or 4
  // row (0..31) of the sub-tile at matrix position x (0..31)
  __device__ __forceinline__ static int row_of_pos(int x) {
    const int s = sigma16(x & 15);
    return HD == 128 ? 2 * s + (x >> 4) : 4 * (s & 7) + (s >> 3) + 2 * (x >> 4);
  }
  // row behind accumulator value e of lane half hh
  __device__ __forceinline__ static constexpr int row_of_acc(int e, int hh) {
    return HD == 128 ? 8 * (e & 3) + 4 * ((e >> 2) & 1) + 2 * hh + (e >> 3)
                     : 16 * (e & 1) + 8 * ((e >> 2) & 1) + 4 * hh + ((e >> 1) & 1) + 2 * (e >> 3);
  }
};

// Starts the copy of the four sub-tiles of a step.  Sub-tile s: rows of HD bf16 at
// base + off[s] bytes, row pitch stride_bytes; rows >= nv[s] (>= 1) re-read row
// nv[s] - 1.  base and off are uniform over the block.
template <int HD>
__device__ __forceinline__ void subs_async_load(uint16_t* tiles, const uint16_t* base, uint32_t stride_bytes,
                                                const uint32_t (&off)[4], const int (&nv)[4]) {
  using TL = TileLayout<HD>;
  constexpr int kLaneShift = HD == 128 ? 4 : 3;
  const int w = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), l = threadIdx.x & 63;
  const uint32_t tile_addr = (uint32_t)(uintptr_t)(__attribute__((address_space(3))) void*)tiles;
  const uint64_t base_bits = (uint64_t)(uintptr_t)base;
  const uint32_t base_hi = (uint32_t)__builtin_amdgcn_readfirstlane((int)(uint32_t)(base_bits >> 32));
  const uint32_t base_lo = (uint32_t)__builtin_amdgcn_readfirstlane((int)(uint32_t)base_bits);
  const uint64_t sbase = ((uint64_t)base_hi << 32) | (uint64_t)base_lo;
  const int rr = (l >> kLaneShift) & (SubLayout<HD>::kRowsPerHalfGroup - 1);
  const uint32_t piece = (uint32_t)(l & ((1 << kLaneShift) - 1)) * 16;
#pragma unroll
  for (int p = 0; p < 2 * TL::kGroups / 8; ++p) {
    const int t = p * 8 / TL::kGroups, grp = (w + 8 * p) % TL::kGroups;
    const int row = SubLayout<HD>::kRowsPerHalfGroup * grp + rr;
    // (the elements are read on their own: a choice between them would put the arrays in memory)
    const int n0 = nv[2 * t], n1 = nv[2 * t + 1];
    const uint32_t o0 = off[2 * t], o1 = off[2 * t + 1];
    const uint32_t voff = (l < 32 ? o0 : o1) + (uint32_t)min(row, (l < 32 ? n0 : n1) - 1) * stride_bytes + piece;
    const uint32_t lds_addr =
        __builtin_amdgcn_readfirstlane(tile_addr + (t * TL::kTileElems + grp * kGroupPitch) * 2);
    asm volatile("s_mov_b32 m0, %2\n\tglobal_load_lds_dwordx4 %0, %1"
                 :
                 : "v"(voff), "s"(sbase), "s"(lds_addr)
                 : "memory");
  }
}

// Records of the schedule are read through the scalar cache, whatever the block
// stores in between.
typedef int i32x8 __attribute__((ext_vector_type(8)));
typedef int i32x16 __attribute__((ext_vector_type(16)));
template <typename V>
__device__ __forceinline__ V scalar_load(const void* p) {
  return *(const __attribute__((address_space(4))) V*)(uintptr_t)p;
}

// Adds the groups' accumulators of one row (key) tile: afterwards group b < DB holds
// the total of output block b in `out`, summed in group order.  buf: DB * 32 KB of
// LDS that nobody reads any more.  Called by every thread.
template <int DB>
__device__ __forceinline__ void sum_over_groups(float* buf, const f32x16 (&x)[DB], int tile, int grp, f32x16& out) {
  const int l = threadIdx.x & 63;
  auto slot = [&](int b, int src, int i) {
    return reinterpret_cast<f32x4*>(buf) + (((b * kGroupsOfWaves + src) * kTiles + tile) * 4 + i) * 64 + l;
  };
  __syncthreads();
#pragma unroll
  for (int b = 0; b < DB; ++b)
    if (b != grp) {
#pragma unroll
      for (int i = 0; i < 4; ++i)
        *slot(b, grp, i) = f32x4{x[b][4 * i], x[b][4 * i + 1], x[b][4 * i + 2], x[b][4 * i + 3]};
    }
  __syncthreads();
#pragma unroll
  for (int b = 0; b < DB; ++b)
    if (b == grp) {
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        f32x4 s = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
        for (int src = 0; src < kGroupsOfWaves; ++src)
          s += src == b ? f32x4{x[b][4 * i], x[b][4 * i + 1], x[b][4 * i + 2], x[b][4 * i + 3]} : *slot(b, src, i);
#pragma unroll
        for (int e = 0; e < 4; ++e) out[4 * i + e] = s[e];
      }
    }
}

// What the forward and dQ kernels share: the block's item and its walk over the keys.
// The host has cut the walk into steps (KeyStep: a piece of at most 32 keys for each
// group); working the pieces out here, between the barrier and the first product of
// every step, cost 6 % of a launch, more than the fuller steps give.  Measured over the
// 1034 forward and 446 backward calls of a leaf-order plan over 446 short segments:
// 13.4 -> 11.6 us a forward call, 18.7 -> 18.0 backward, against steps cut from one
// interval each.
template <int HD>
struct KeyWalk {
  using TL = TileLayout<HD>;
  const KeyStep* steps;
  int t1, at, end;    // next step to read ahead, end of the list
  int w, l, c, hh, rw, grp, g, h, row_base, qrow;
  i32x8 step, next;   // the step copied last, the one after it: c0[0..3], n[0..3]
  bool have;

  __device__ __forceinline__ void init(const StepTile* tiles, const KeyStep* list, int block, int Hq, int Hkv, int HB,
                                       int hblocks) {
    const int item = block / Hkv;
    steps = list;
    g = block % Hkv;
    const i32x16 rec = scalar_load<i32x16>(tiles + item / hblocks);
    const int t0 = rec[0];
    t1 = rec[1];
    at = rec[2];
    end = rec[3];
    step = i32x8{rec[8], rec[9], rec[10], rec[11], rec[12], rec[13], rec[14], rec[15]};
    have = true;
    read_ahead();
    w = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    l = threadIdx.x & 63;
    c = l & 31;
    hh = l >> 5;
    rw = w % kTiles;
    grp = w / kTiles;
    h = g * (Hq / Hkv) + (item % hblocks) * HB + rw % HB;
    row_base = t0 + 32 * (rw / HB);
    qrow = min(row_base + c, t1 - 1);
  }
  __device__ __forceinline__ void read_ahead() {
    if (at < end) next = scalar_load<i32x8>(steps + at);
  }
  // moves on to the next step; false at the end of the walk
  __device__ __forceinline__ bool advance() {
    if (at >= end) return false;
    step = next;
    ++at;
    read_ahead();
    return true;
  }
  // this group's piece of the step: first key, keys (may be none), every row sees every key
  __device__ __forceinline__ void mine(int& k0, int& nk, bool& full) const {
    k0 = grp == 0 ? step[0] : grp == 1 ? step[1] : grp == 2 ? step[2] : step[3];
    const int n = grp == 0 ? step[4] : grp == 1 ? step[5] : grp == 2 ? step[6] : step[7];
    nk = n & (kFullPiece - 1);
    full = (n & kFullPiece) != 0;
  }
  // copies the step's pieces of K and V into tile pair b
  __device__ __forceinline__ void issue(uint16_t* Kd, uint16_t* Vd, int32_t* kendS, const int32_t* kend,
                                        const uint16_t* kbase, const uint16_t* vbase, uint32_t kv_bytes) {
    uint32_t off[4];
    int nv[4];
#pragma unroll
    for (int s = 0; s < 4; ++s) {   // (no piece: the first one's first row again, which nobody uses)
      off[s] = (uint32_t)(step[s] - step[0]) * kv_bytes;
      nv[s] = max(1, step[4 + s] & (kFullPiece - 1));
    }
    if ((step[4] & step[5] & step[6] & step[7] & kFullPiece) == 0 && w < kStep / 64) {
      // kendS is indexed by matrix position; wave w fills sub-tiles 2w and 2w + 1
      const int f0 = w == 0 ? step[0] : step[2], f1 = w == 0 ? step[1] : step[3];
      const int n0 = w == 0 ? nv[0] : nv[2], n1 = w == 0 ? nv[1] : nv[3];
      const int row = min(SubLayout<HD>::row_of_pos(l & 31), (l < 32 ? n0 : n1) - 1);
      row_async_load(reinterpret_cast<float*>(kendS + 64 * w), reinterpret_cast<const float*>(kend + step[0]),
                     (uint32_t)((l < 32 ? f0 : f1) - step[0] + row));
    }
    const size_t at0 = (size_t)step[0] * (kv_bytes / 2);
    subs_async_load<HD>(Kd, kbase + at0, kv_bytes, off, nv);
    subs_async_load<HD>(Vd, vbase + at0, kv_bytes, off, nv);
  }
};

template <int HD>
__global__ __launch_bounds__(kThreads) __attribute__((amdgpu_waves_per_eu(2, 2))) void fwd_small_kernel(
    const StepTile* __restrict__ tiles, const KeyStep* __restrict__ steps, const int32_t* __restrict__ kend,
    const uint16_t* __restrict__ q, const uint16_t* __restrict__ k, const uint16_t* __restrict__ v,
    uint16_t* __restrict__ o, float* __restrict__ lse, int Hq, int Hkv, int HB, int hblocks, float scale) {
  using TL = TileLayout<HD>;
  constexpr int KS = TL::kSteps, DB = TL::kBlocks;
  struct Smem {
    uint16_t K[2][2 * TL::kTileElems];
    uint16_t V[2][2 * TL::kTileElems];
  };
  __shared__ __attribute__((aligned(1024))) Smem sm;
  __shared__ __attribute__((aligned(16))) int32_t kendS[2][kStep];
  __shared__ float mS[kGroupsOfWaves][kTiles][32], lS[kGroupsOfWaves][kTiles][32];

  KeyWalk<HD> wk;
  wk.init(tiles, steps, blockIdx.x, Hq, Hkv, HB, hblocks);
  const size_t kv_stride = (size_t)Hkv * HD;
  const uint16_t* kbase = k + (size_t)wk.g * HD;
  const uint16_t* vbase = v + (size_t)wk.g * HD;
  const uint32_t kv_bytes = (uint32_t)kv_stride * 2;
  wk.issue(sm.K[0], sm.V[0], kendS[0], kend, kbase, vbase, kv_bytes);
  const int c = wk.c, hh = wk.hh, grp = wk.grp, qrow = wk.qrow;
  // scores stay unscaled; a negative scale is moved into the sign of Q so that sc > 0
  const float sc = fabsf(scale) * kLog2e;
  bf16x8 Qr[KS];
  {
    const uint16_t* qp = q + ((size_t)qrow * Hq + wk.h) * HD + 8 * hh;
#pragma unroll
    for (int ks = 0; ks < KS; ++ks) {
      uint4 raw = *reinterpret_cast<const uint4*>(qp + 16 * ks);
      if (scale < 0.f) {
        raw.x ^= 0x80008000u; raw.y ^= 0x80008000u; raw.z ^= 0x80008000u; raw.w ^= 0x80008000u;
      }
      Qr[ks] = *reinterpret_cast<bf16x8*>(&raw);
    }
  }
  f32x16 O[DB];
#pragma unroll
  for (int a = 0; a < DB; ++a)
#pragma unroll
    for (int e = 0; e < 16; ++e) O[a][e] = 0.f;
  float m = -INFINITY, lsum = 0.f;
  int buf = 0;
  const int sub_off = (grp >> 1) * TL::kTileElems + 256 * (grp & 1);
  const int rlo = TL::row_lane_off() + sub_off, clo = TL::col_lane_off() + sub_off;

  while (wk.have) {
    async_wait_all();
    __syncthreads();   // step `buf` has landed; everyone is done with the other buffer
    int k0, nk;   // this group's keys
    bool full;
    wk.mine(k0, nk, full);
    const bool need_mask = !full || nk < kSub;
    const uint16_t* Kt = sm.K[buf] + rlo;
    const uint16_t* Vt = sm.V[buf] + clo;
    bf16x8 a[KS];   // (read before the copies are issued, whose addresses take a while to work out)
#pragma unroll
    for (int ks = 0; ks < KS; ++ks) a[ks] = tile_row8(Kt, 0, ks);
    wk.have = wk.advance();
    if (wk.have) wk.issue(sm.K[buf ^ 1], sm.V[buf ^ 1], kendS[buf ^ 1], kend, kbase, vbase, kv_bytes);
    if (nk > 0) {
      f32x16 S;
#pragma unroll
      for (int e = 0; e < 16; ++e) S[e] = 0.f;
#pragma unroll
      for (int ks = 0; ks < KS; ++ks) S = mfma32(a[ks], Qr[ks], S);
      if (need_mask) {   // (kendS is only filled if some piece of the step is not full)
        const int last = min(nk - 1, qrow - k0), no_end = full ? 0x7fffffff : 0;
#pragma unroll
        for (int e4 = 0; e4 < 4; ++e4) {
          const int4 ke = *reinterpret_cast<const int4*>(&kendS[buf][kSub * grp + 8 * e4 + 4 * hh]);
          const int kev[4] = {ke.x, ke.y, ke.z, ke.w};
#pragma unroll
          for (int j = 0; j < 4; ++j) {
            const bool ok = (SubLayout<HD>::row_of_acc(4 * e4 + j, hh) <= last) & (qrow < max(kev[j], no_end));
            S[4 * e4 + j] = ok ? S[4 * e4 + j] : -INFINITY;
          }
        }
      }
      float mx = -INFINITY;
#pragma unroll
      for (int e = 0; e < 16; ++e) mx = fmaxf(mx, S[e]);
      const float mnew = fmaxf(m, max_across_halves(mx));
      const float mref = mnew == -INFINITY ? 0.f : mnew;
      const float alpha = __builtin_amdgcn_exp2f((m - mref) * sc);
      m = mnew;
      const float msc = mref * sc;
      float ps = 0.f;
#pragma unroll
      for (int e = 0; e < 16; ++e) {
        S[e] = __builtin_amdgcn_exp2f(fmaf(S[e], sc, -msc));
        ps += S[e];
      }
      lsum = lsum * alpha + ps;
      if (__builtin_amdgcn_ballot_w64(alpha != 1.f) != 0) {
#pragma unroll
        for (int dmb = 0; dmb < DB; ++dmb)
#pragma unroll
          for (int e = 0; e < 16; ++e) O[dmb][e] *= alpha;
      }
#pragma unroll
      for (int kk = 0; kk < 2; ++kk) {
        const bf16x8 Pb = pack8(S, kk);
#pragma unroll
        for (int dmb = 0; dmb < DB; ++dmb) O[dmb] = mfma32(tile_col8(Vt, 16 * kk, 32 * dmb), Pb, O[dmb]);
      }
    }
    buf ^= 1;
  }

  // merge the groups: common maximum, row sum, then the accumulators block by block
  float lt = lsum + __shfl_xor(lsum, 32);
  if (hh == 0) {
    mS[grp][wk.rw][c] = m;
    lS[grp][wk.rw][c] = lt;
  }
  __syncthreads();
  float mall = mS[0][wk.rw][c];
#pragma unroll
  for (int s = 1; s < kGroupsOfWaves; ++s) mall = fmaxf(mall, mS[s][wk.rw][c]);
  const float mref = mall == -INFINITY ? 0.f : mall;   // (every score of the row may be -inf)
  lt = 0.f;
#pragma unroll
  for (int s = 0; s < kGroupsOfWaves; ++s)
    lt = fmaf(__builtin_amdgcn_exp2f((mS[s][wk.rw][c] - mref) * sc), lS[s][wk.rw][c], lt);
  const float f = __builtin_amdgcn_exp2f((m - mref) * sc);
#pragma unroll
  for (int dmb = 0; dmb < DB; ++dmb)
#pragma unroll
    for (int e = 0; e < 16; ++e) O[dmb][e] *= f;
  f32x16 out;
  sum_over_groups<DB>(reinterpret_cast<float*>(&sm), O, wk.rw, grp, out);
  const float inv = 1.f / lt;
  const int token = wk.row_base + c;
  if (token < wk.t1) {
    if (grp < DB) {
      uint16_t* op = o + ((size_t)token * Hq + wk.h) * HD + 32 * grp + 4 * hh;
#pragma unroll
      for (int v4 = 0; v4 < 4; ++v4) {
        bf16x4 r;
#pragma unroll
        for (int e = 0; e < 4; ++e) r[e] = (__bf16)(out[4 * v4 + e] * inv);
        *reinterpret_cast<bf16x4*>(op + 8 * v4) = r;
      }
    }
    if (grp == 0 && hh == 0) lse[(size_t)token * Hq + wk.h] = (mall * sc + log2f(lt)) * kLn2;
  }
}

// What a backward launch reads and writes.
struct BwdArgs {
  const StepTile* tiles;
  const KeyStep* steps;
  const KvItem* items;
  const int32_t* kend;
  const uint16_t *q, *k, *v, *d_o, *o;
  const float* lse;
  float *neg_delta, *neg_lse_s;
  uint16_t *dq, *dk, *dv;
  float *partial, *dk_acc, *dv_acc;
  int Hq, Hkv, HB, hblocks;
  float scale;
  int dkdv_blocks;   // blocks [0, dkdv_blocks) of the grid do dK/dV, the rest dQ
};

template <int HD>
struct DqSmem {
  uint16_t K[2][2 * TileLayout<HD>::kTileElems];
  uint16_t V[2][2 * TileLayout<HD>::kTileElems];
  int32_t kendS[2][kStep];
};

// With p.o != nullptr the block also computes the row statistics -D and -lse/scale
// and leaves them in the workspace, as dq_bf16_kernel does (same values to the bit).
template <int HD>
__device__ __forceinline__ void dq_block(const BwdArgs& p, DqSmem<HD>& sm, int block) {
  using TL = TileLayout<HD>;
  constexpr int KS = TL::kSteps, DB = TL::kBlocks;
  const int32_t* kend = p.kend;
  const uint16_t *q = p.q, *k = p.k, *v = p.v, *d_o = p.d_o, *o = p.o;
  const float* lse = p.lse;
  float *neg_delta = p.neg_delta, *neg_lse_s = p.neg_lse_s;
  uint16_t* dq = p.dq;
  const int Hq = p.Hq, Hkv = p.Hkv;
  const float scale = p.scale;
  auto& kendS = sm.kendS;

  KeyWalk<HD> wk;
  wk.init(p.tiles, p.steps, block, Hq, Hkv, p.HB, p.hblocks);
  const size_t kv_stride = (size_t)Hkv * HD;
  const uint16_t* kbase = k + (size_t)wk.g * HD;
  const uint16_t* vbase = v + (size_t)wk.g * HD;
  const uint32_t kv_bytes = (uint32_t)kv_stride * 2;
  wk.issue(sm.K[0], sm.V[0], kendS[0], kend, kbase, vbase, kv_bytes);
  const int c = wk.c, hh = wk.hh, grp = wk.grp, qrow = wk.qrow;
  const float sc = scale * kLog2e;
  const size_t rh = (size_t)qrow * Hq + wk.h;
  bf16x8 Qr[KS], dOr[KS];
  float dpart[KS];
#pragma unroll
  for (int ks = 0; ks < KS; ++ks) {
    Qr[ks] = *reinterpret_cast<const bf16x8*>(q + rh * HD + 8 * hh + 16 * ks);
    dOr[ks] = *reinterpret_cast<const bf16x8*>(d_o + rh * HD + 8 * hh + 16 * ks);
    if (o != nullptr) {
      const bf16x8 ox = *reinterpret_cast<const bf16x8*>(o + rh * HD + 8 * hh + 16 * ks);
      float s = 0.f;
#pragma unroll
      for (int e = 0; e < 8; ++e) s = fmaf((float)ox[e], (float)dOr[ks][e], s);
      dpart[ks] = s;
    }
  }
  const float nlse = -lse[rh] / scale;
  float ndlt;
  if (o != nullptr) {   // summation order of delta_bf16_kernel
#pragma unroll
    for (int ks = 0; ks < KS; ++ks) dpart[ks] += __shfl_xor(dpart[ks], 32);
    float d = (dpart[0] + dpart[1]) + (dpart[2] + dpart[3]);
    if constexpr (HD == 128) d += (dpart[KS - 4] + dpart[KS - 3]) + (dpart[KS - 2] + dpart[KS - 1]);
    ndlt = -d;
    if (grp == 0 && hh == 0 && wk.row_base + c < wk.t1) {
      neg_delta[rh] = ndlt;
      neg_lse_s[rh] = -lse[rh] * (1.f / scale);
    }
  } else {
    ndlt = neg_delta[rh];
  }
  f32x16 dQ[DB];
#pragma unroll
  for (int a = 0; a < DB; ++a)
#pragma unroll
    for (int e = 0; e < 16; ++e) dQ[a][e] = 0.f;
  int buf = 0;
  const int sub_off = (grp >> 1) * TL::kTileElems + 256 * (grp & 1);
  const int rlo = TL::row_lane_off() + sub_off, clo = TL::col_lane_off() + sub_off;

  while (wk.have) {
    async_wait_all();
    __syncthreads();
    int k0, nk;
    bool full;
    wk.mine(k0, nk, full);
    const bool need_mask = !full || nk < kSub;
    const uint16_t* Kt = sm.K[buf] + rlo;
    const uint16_t* Vt = sm.V[buf] + rlo;
    const uint16_t* Kc = sm.K[buf] + clo;
    bf16x8 a[KS];   // (read before the copies are issued, as in the forward kernel)
#pragma unroll
    for (int ks = 0; ks < KS; ++ks) a[ks] = tile_row8(Kt, 0, ks);
    wk.have = wk.advance();
    if (wk.have) wk.issue(sm.K[buf ^ 1], sm.V[buf ^ 1], kendS[buf ^ 1], kend, kbase, vbase, kv_bytes);
    if (nk > 0) {
      f32x16 S, dP;
#pragma unroll
      for (int e = 0; e < 16; ++e) { S[e] = nlse; dP[e] = ndlt; }
#pragma unroll
      for (int ks = 0; ks < KS; ++ks) S = mfma32(a[ks], Qr[ks], S);
#pragma unroll
      for (int ks = 0; ks < KS; ++ks) dP = mfma32(tile_row8(Vt, 0, ks), dOr[ks], dP);
#pragma unroll
      for (int e = 0; e < 16; ++e) S[e] = __builtin_amdgcn_exp2f(S[e] * sc);
      if (need_mask) {   // (kendS is only filled if some piece of the step is not full)
        const int last = min(nk - 1, qrow - k0), no_end = full ? 0x7fffffff : 0;
#pragma unroll
        for (int e4 = 0; e4 < 4; ++e4) {
          const int4 ke = *reinterpret_cast<const int4*>(&kendS[buf][kSub * grp + 8 * e4 + 4 * hh]);
          const int kev[4] = {ke.x, ke.y, ke.z, ke.w};
#pragma unroll
          for (int j = 0; j < 4; ++j) {
            const bool ok = (SubLayout<HD>::row_of_acc(4 * e4 + j, hh) <= last) & (qrow < max(kev[j], no_end));
            S[4 * e4 + j] = ok ? S[4 * e4 + j] : 0.f;
          }
        }
      }
#pragma unroll
      for (int e = 0; e < 16; ++e) S[e] *= dP[e];   // dS
#pragma unroll
      for (int kk = 0; kk < 2; ++kk) {
        const bf16x8 dSb = pack8(S, kk);
#pragma unroll
        for (int dmb = 0; dmb < DB; ++dmb) dQ[dmb] = mfma32(tile_col8(Kc, 16 * kk, 32 * dmb), dSb, dQ[dmb]);
      }
    }
    buf ^= 1;
  }

  f32x16 out;
  sum_over_groups<DB>(reinterpret_cast<float*>(&sm), dQ, wk.rw, grp, out);
  const int token = wk.row_base + c;
  if (grp < DB && token < wk.t1) {
    uint16_t* op = dq + ((size_t)token * Hq + wk.h) * HD + 32 * grp + 4 * hh;
#pragma unroll
    for (int v4 = 0; v4 < 4; ++v4) {
      bf16x4 r;
#pragma unroll
      for (int e = 0; e < 4; ++e) r[e] = (__bf16)(out[4 * v4 + e] * scale);
      *reinterpret_cast<bf16x4*>(op + 8 * v4) = r;
    }
  }
}

// dK/dV of 64 keys per block.  The walk is flattened over (32-row chunk, q head of
// the group), heads innermost, last chunk first; the four groups take four
// consecutive iterations per step, so short segments (one or two chunks) are split
// over the heads.
// (with head_dim 128 some k-steps of K and V live in LDS instead of registers, one
// copy for the four groups of a key tile: with all of them in registers the kernel
// needs more than 256)
template <int HD>
struct DkdvSmem {
  static constexpr int kStashK = HD == 128 ? 2 : 0, kStashV = HD == 128 ? 4 : 0;
  uint16_t Q[2][2 * TileLayout<HD>::kTileElems];
  uint16_t dO[2][2 * TileLayout<HD>::kTileElems];
  float stat[2][2][kStep];   // [buffer][-lse/scale | -delta][position]
  uint16_t stash[kTiles][kStashK + kStashV ? kStashK + kStashV : 1][64 * 8];
};

template <int HD>
__device__ __forceinline__ void dkdv_block(const BwdArgs& p, DkdvSmem<HD>& sm, int block) {
  using TL = TileLayout<HD>;
  constexpr int KS = TL::kSteps, DB = TL::kBlocks;
  constexpr int kKeys = 32 * kTiles;
  constexpr int kStashK = DkdvSmem<HD>::kStashK, kStashV = DkdvSmem<HD>::kStashV;
  constexpr int kRegK = KS - kStashK, kRegV = KS - kStashV;
  const int32_t* kend = p.kend;
  const uint16_t *q = p.q, *k = p.k, *v = p.v, *d_o = p.d_o;
  const float *neg_lse_s = p.neg_lse_s, *neg_delta = p.neg_delta;
  float *dk_acc = p.dk_acc, *dv_acc = p.dv_acc;
  const int Hq = p.Hq, Hkv = p.Hkv;
  const float scale = p.scale;

  KvItem tile;
  {
    const i32x8 r = scalar_load<i32x8>(p.items + block / Hkv);
    tile = KvItem{r[0], r[1], r[2], r[3], r[4], r[5], r[6], r[7]};
  }
  const int g = block % Hkv, G = Hq / Hkv;
  const int w = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), l = threadIdx.x & 63;
  const int c = l & 31, hh = l >> 5;
  const int kt = w % kTiles, grp = w / kTiles;
  const float sc = scale * kLog2e;
  const int kcol = tile.k0 + 32 * kt + c;
  const int kc = min(kcol, tile.k1 - 1);
  const int my_kend = kcol < tile.k1 ? kend[kc] : 0;   // padded columns see nothing
  const size_t q_stride = (size_t)Hq * HD;
  const uint32_t q_bytes = (uint32_t)q_stride * 2;
  const int n_chunks = (tile.q_end - tile.q_begin + kSub - 1) / kSub;
  const int total = tile.it_end;
  // Iterations it .. it+3 of a step, `it` = chunk * G + head: their first rows and heads;
  // iterations >= total repeat the last one (never computed on).  Kept up to date from
  // step to step, without divisions.
  int row[4], head[4];
  {
    const int chunk = tile.it_begin / G;
    head[0] = tile.it_begin - chunk * G;
    row[0] = tile.q_begin + (n_chunks - 1 - chunk) * kSub;
  }
  const int step_rows = kGroupsOfWaves / G * kSub, step_heads = kGroupsOfWaves % G;
  auto fill = [&](int it) {   // iterations it+1 .. it+3 from the one at `it`
#pragma unroll
    for (int s = 1; s < 4; ++s) {
      const bool wrap = head[s - 1] + 1 == G, stay = it + s >= total;
      head[s] = stay ? head[s - 1] : wrap ? 0 : head[s - 1] + 1;
      row[s] = stay || !wrap ? row[s - 1] : row[s - 1] - kSub;
    }
  };
  auto advance = [&](int it) {   // to the step that begins with iteration `it` < total
    head[0] += step_heads;
    row[0] -= step_rows;
    if (head[0] >= G) {
      head[0] -= G;
      row[0] -= kSub;
    }
    fill(it);
  };
  // copies the step's rows into buffer b
  auto issue = [&](int b) {
    // rows of the last of the four iterations are the lowest: offsets from there are not negative
    const int r_base = row[3];
    const uint16_t* qb = q + (size_t)r_base * q_stride + (size_t)(g * G) * HD;
    const uint16_t* db = d_o + (size_t)r_base * q_stride + (size_t)(g * G) * HD;
    uint32_t off[4];
    int nv[4];
#pragma unroll
    for (int s = 0; s < 4; ++s) {
      off[s] = (uint32_t)(row[s] - r_base) * q_bytes + (uint32_t)head[s] * (HD * 2);
      nv[s] = min(kSub, tile.q_end - row[s]);
    }
    if (w < kStep / 64) {   // stat is indexed by matrix position; wave w fills sub-tiles 2w and 2w + 1
      const int r0 = w == 0 ? row[0] : row[2], r1 = w == 0 ? row[1] : row[3];
      const int h0 = w == 0 ? head[0] : head[2], h1 = w == 0 ? head[1] : head[3];
      const int n0 = w == 0 ? nv[0] : nv[2], n1 = w == 0 ? nv[1] : nv[3];
      const int rr = min(SubLayout<HD>::row_of_pos(l & 31), (l < 32 ? n0 : n1) - 1);
      const uint32_t at = (uint32_t)((l < 32 ? r0 : r1) - r_base + rr) * (uint32_t)Hq + (uint32_t)(l < 32 ? h0 : h1);
      const size_t sb = (size_t)r_base * Hq + (size_t)(g * G);
      row_async_load(&sm.stat[b][0][64 * w], neg_lse_s + sb, at);
      row_async_load(&sm.stat[b][1][64 * w], neg_delta + sb, at);
    }
    subs_async_load<HD>(sm.Q[b], qb, q_bytes, off, nv);
    subs_async_load<HD>(sm.dO[b], db, q_bytes, off, nv);
  };
  fill(tile.it_begin);
  issue(0);

  bf16x8 Kr[kRegK], Vr[kRegV];
  uint16_t* stash = &sm.stash[kt][0][l * 8];
  {
    const uint16_t* kp = k + ((size_t)kc * Hkv + g) * HD + 8 * hh;
    const uint16_t* vp = v + ((size_t)kc * Hkv + g) * HD + 8 * hh;
#pragma unroll
    for (int ks = 0; ks < KS; ++ks) {
      const bf16x8 kx = *reinterpret_cast<const bf16x8*>(kp + 16 * ks);
      const bf16x8 vx = *reinterpret_cast<const bf16x8*>(vp + 16 * ks);
      if (ks < kRegK) Kr[ks < kRegK ? ks : 0] = kx;
      else if (grp == 0) *reinterpret_cast<bf16x8*>(stash + (ks - kRegK) * 512) = kx;
      if (ks < kRegV) Vr[ks < kRegV ? ks : 0] = vx;
      else if (grp == 0) *reinterpret_cast<bf16x8*>(stash + (kStashK + ks - kRegV) * 512) = vx;
    }
  }
  auto k_op = [&](int ks) {
    return ks < kRegK ? Kr[ks < kRegK ? ks : 0] : *reinterpret_cast<const bf16x8*>(stash + (ks - kRegK) * 512);
  };
  auto v_op = [&](int ks) {
    return ks < kRegV ? Vr[ks < kRegV ? ks : 0]
                      : *reinterpret_cast<const bf16x8*>(stash + (kStashK + ks - kRegV) * 512);
  };
  f32x16 dK[DB], dV[DB];
#pragma unroll
  for (int a = 0; a < DB; ++a)
#pragma unroll
    for (int e = 0; e < 16; ++e) { dK[a][e] = 0.f; dV[a][e] = 0.f; }
  const int sub_off = (grp >> 1) * TL::kTileElems + 256 * (grp & 1);
  const int rlo = TL::row_lane_off() + sub_off, clo = TL::col_lane_off() + sub_off;

  int wave_hi = my_kend;   // rows [wave_lo, wave_hi) are the only ones this wave's keys can see
#pragma unroll
  for (int off = 16; off >= 1; off >>= 1) wave_hi = max(wave_hi, __shfl_xor(wave_hi, off));
  wave_hi = __builtin_amdgcn_readfirstlane(wave_hi);
  const int wave_lo = tile.k0 + 32 * kt;

  int buf = 0;
  for (int it = tile.it_begin; it < total; it += kGroupsOfWaves) {
    async_wait_all();
    __syncthreads();   // step `buf` has landed (and, first time, the stash); everyone is done with the other buffer
    const int my_it = it + grp;
    const int r0 = grp == 0 ? row[0] : grp == 1 ? row[1] : grp == 2 ? row[2] : row[3];
    const int nv = min(kSub, tile.q_end - r0);
    const uint16_t* Qt = sm.Q[buf] + rlo;
    const uint16_t* dOt = sm.dO[buf] + rlo;
    const uint16_t* Qc = sm.Q[buf] + clo;
    const uint16_t* dOc = sm.dO[buf] + clo;
    const float* stat = &sm.stat[buf][0][kSub * grp + 4 * hh];
    // operand reads run two products ahead (the first ones before the copies are issued, as in the forward
    // kernel); the barriers bound their registers
    constexpr int kAhead = 2;
    bf16x8 a[KS];
#pragma unroll
    for (int ks = 0; ks < kAhead; ++ks) a[ks] = tile_row8(Qt, 0, ks);
    f32x16 S, dP;
#pragma unroll
    for (int e4 = 0; e4 < 4; ++e4) {
      const f32x4 ls = *reinterpret_cast<const f32x4*>(stat + 8 * e4);
#pragma unroll
      for (int j = 0; j < 4; ++j) S[4 * e4 + j] = ls[j];
    }
    if (it + kGroupsOfWaves < total) {
      advance(it + kGroupsOfWaves);
      issue(buf ^ 1);
    }
    if (my_it < total && r0 + nv > wave_lo && r0 < wave_hi) {
      const bool need_mask = !(r0 >= tile.k1 && r0 + kSub <= tile.q_full_end);
#pragma unroll
      for (int e4 = 0; e4 < 4; ++e4) {
        const f32x4 dl = *reinterpret_cast<const f32x4*>(stat + kStep + 8 * e4);
#pragma unroll
        for (int j = 0; j < 4; ++j) dP[4 * e4 + j] = dl[j];
      }
#pragma unroll
      for (int ks = 0; ks < KS; ++ks) {
        if (ks + kAhead < KS) a[ks + kAhead] = tile_row8(Qt, 0, ks + kAhead);
        S = mfma32(a[ks], k_op(ks), S);
        __builtin_amdgcn_sched_barrier(0);
      }
      constexpr int VP = 16 / KS;
#pragma unroll
      for (int ks = 0; ks < kAhead; ++ks) a[ks] = tile_row8(dOt, 0, ks);
      __builtin_amdgcn_sched_barrier(0);
#pragma unroll
      for (int ks = 0; ks < KS; ++ks) {
        if (ks + kAhead < KS) a[ks + kAhead] = tile_row8(dOt, 0, ks + kAhead);
        dP = mfma32(a[ks], v_op(ks), dP);
#pragma unroll
        for (int t = 0; t < VP; ++t) S[VP * ks + t] = __builtin_amdgcn_exp2f(S[VP * ks + t] * sc);
        __builtin_amdgcn_sched_barrier(0);
      }
      if (need_mask) {   // query row t sees this lane's key iff kcol <= t < kend[kcol]
        constexpr int kHalf = SubLayout<HD>::row_of_acc(0, 1) - SubLayout<HD>::row_of_acc(0, 0);
        const int lo = kcol - r0 - kHalf * hh, hi = min(my_kend - r0, nv) - kHalf * hh;
#pragma unroll
        for (int e = 0; e < 16; ++e) {
          const int rc = SubLayout<HD>::row_of_acc(e, 0);
          S[e] = ((rc >= lo) & (rc < hi)) ? S[e] : 0.f;
        }
      }
      const bf16x8 Pb[2] = {pack8(S, 0), pack8(S, 1)};
      bf16x8 dSb[2];
#pragma unroll
      for (int i = 0; i < kAhead; ++i) a[i] = tile_col8(dOc, 16 * (i & 1), 32 * (i >> 1));
      __builtin_amdgcn_sched_barrier(0);
#pragma unroll
      for (int i = 0; i < KS; ++i) {
        if (i + kAhead < KS) a[i + kAhead] = tile_col8(dOc, 16 * ((i + kAhead) & 1), 32 * ((i + kAhead) >> 1));
        dV[i >> 1] = mfma32(a[i], Pb[i & 1], dV[i >> 1]);
#pragma unroll
        for (int t = 0; t < VP; ++t) {
          const int e = VP * i + t;
          dSb[e >> 3][e & 7] = (__bf16)(dP[e] * S[e]);
        }
        __builtin_amdgcn_sched_barrier(0);
      }
#pragma unroll
      for (int i = 0; i < kAhead; ++i) a[i] = tile_col8(Qc, 16 * (i & 1), 32 * (i >> 1));
      __builtin_amdgcn_sched_barrier(0);
#pragma unroll
      for (int i = 0; i < KS; ++i) {
        if (i + kAhead < KS) a[i + kAhead] = tile_col8(Qc, 16 * ((i + kAhead) & 1), 32 * ((i + kAhead) >> 1));
        dK[i >> 1] = mfma32(a[i], dSb[i & 1], dK[i >> 1]);
        __builtin_amdgcn_sched_barrier(0);
      }
    }
    buf ^= 1;
  }

  // A segment call adds to the caller's accumulators (this block is the only owner of these keys in the
  // launch): what they hold is read while the groups' sums are added.  Read after each sum it is 2 us
  // of the 4 between a walk and its end, of 13 us a block lives on short segments.
  const int col0 = 32 * grp + 4 * hh;
  const size_t base = ((size_t)kcol * Hkv + g) * HD + col0;
  const bool adds = dk_acc != nullptr && tile.slot < 0 && grp < DB && kcol < tile.k1;
  f32x4 old[2][4];
  if (adds) {
#pragma unroll
    for (int half = 0; half < 2; ++half)
#pragma unroll
      for (int v4 = 0; v4 < 4; ++v4)
        old[half][v4] = *reinterpret_cast<const f32x4*>((half == 0 ? dk_acc : dv_acc) + base + 8 * v4);
  }
#pragma unroll
  for (int half = 0; half < 2; ++half) {
    f32x16 out;
    sum_over_groups<DB>(reinterpret_cast<float*>(&sm), half == 0 ? dK : dV, kt, grp, out);
    if (grp >= DB) continue;
    const float f = half == 0 ? scale : 1.f;
    if (tile.slot >= 0) {   // one of several items of this key tile: fp32 partial sums
      float* dst = p.partial + ((size_t)tile.slot * Hkv + g) * (2 * kKeys * HD) +
                 (size_t)(half * kKeys + 32 * kt + c) * HD + col0;
#pragma unroll
      for (int v4 = 0; v4 < 4; ++v4)
        *reinterpret_cast<f32x4*>(dst + 8 * v4) =
            f32x4{out[4 * v4], out[4 * v4 + 1], out[4 * v4 + 2], out[4 * v4 + 3]};
    } else if (kcol < tile.k1) {
      if (adds) {
        float* dst = (half == 0 ? dk_acc : dv_acc) + base;
#pragma unroll
        for (int v4 = 0; v4 < 4; ++v4) {
          f32x4 r = old[half][v4];
#pragma unroll
          for (int e = 0; e < 4; ++e) r[e] = fmaf(out[4 * v4 + e], f, r[e]);   // (one rounding)
          *reinterpret_cast<f32x4*>(dst + 8 * v4) = r;
        }
      } else {
        uint16_t* dst = (half == 0 ? p.dk : p.dv) + base;
#pragma unroll
        for (int v4 = 0; v4 < 4; ++v4) {
          bf16x4 r;
#pragma unroll
          for (int e = 0; e < 4; ++e) r[e] = (__bf16)(out[4 * v4 + e] * f);
          *reinterpret_cast<bf16x4*>(dst + 8 * v4) = r;
        }
      }
    }
  }
}

// dQ and dK/dV in one launch: neither fills the chip by itself, and each is a few
// steps between a launch and its end.
template <int HD>
__global__ __launch_bounds__(kThreads) __attribute__((amdgpu_waves_per_eu(2, 2))) void bwd_small_kernel(BwdArgs p) {
  __shared__ __attribute__((aligned(1024))) union {
    DqSmem<HD> dq;
    DkdvSmem<HD> dkdv;
  } sm;
  if ((int)blockIdx.x < p.dkdv_blocks) dkdv_block<HD>(p, sm.dkdv, blockIdx.x);
  else dq_block<HD>(p, sm.dq, blockIdx.x - p.dkdv_blocks);
}

}  // namespace

int launch_fwd_bf16_small(const LaunchArgs& a) {
  const size_t blocks = a.sched->q_tiles.size() * (size_t)a.p.n_kv_heads * (size_t)a.tc.hblocks;
  if (blocks == 0 || blocks > 0x7fffffffu) return DTA_ERR_UNSUPPORTED;
  auto kernel = a.p.head_dim == 128 ? fwd_small_kernel<128> : fwd_small_kernel<64>;
  launch(a, true, kernel, blocks, kThreads,
      a.sched->d_step_tiles, a.sched->d_steps, a.d_kend, (const uint16_t*)a.q, (const uint16_t*)a.k,
      (const uint16_t*)a.v, (uint16_t*)a.o_out, a.lse_out, a.p.n_q_heads, a.p.n_kv_heads, a.tc.hb,
      a.tc.hblocks, a.p.softmax_scale);
  return launch_status(__func__);
}

// The stages DTA_BWD_DQ and DTA_BWD_DKDV of `stages` in one launch.  Both read the
// row statistics of the delta stage from the workspace, unless fused_delta (dQ
// alone), which computes them.
int launch_bwd_bf16_small(const LaunchArgs& a, uint32_t stages, bool fused_delta) {
  const size_t dkdv = stages & DTA_BWD_DKDV ? a.sched->kv_items.size() * (size_t)a.p.n_kv_heads : 0;
  const size_t dq =
      stages & DTA_BWD_DQ ? a.sched->q_tiles.size() * (size_t)a.p.n_kv_heads * (size_t)a.tc.hblocks : 0;
  if (dq + dkdv == 0 || dq + dkdv > 0x7fffffffu) return DTA_ERR_UNSUPPORTED;
  const BwdArgs p{a.sched->d_step_tiles, a.sched->d_steps, a.sched->d_kv_items, a.d_kend, (const uint16_t*)a.q,
                  (const uint16_t*)a.k, (const uint16_t*)a.v, (const uint16_t*)a.d_o,
                  fused_delta ? (const uint16_t*)a.o : nullptr, a.lse_in, a.delta, a.lse2, (uint16_t*)a.dq,
                  (uint16_t*)a.dk, (uint16_t*)a.dv, a.partial, a.dk_acc, a.dv_acc, a.p.n_q_heads,
                  a.p.n_kv_heads, a.tc.hb, a.tc.hblocks, a.p.softmax_scale, (int)dkdv};
  auto kernel = a.p.head_dim == 128 ? bwd_small_kernel<128> : bwd_small_kernel<64>;
  launch(a, dkdv != 0 && a.sched->kv_reduce.empty(), kernel, dq + dkdv, kThreads, p);
  return launch_status(__func__);
}

}  // namespace dta
