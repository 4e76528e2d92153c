// bf16 forward tree attention for gfx950 (the attention inside the paper's FWD
// primitive, pseudocode appendix, for every segment of the tree in one launch).
//
// One block = 8 waves works on one query tile of the DFS-packed tree and one kv
// head.  Each wave owns 32 query rows of one q head of the group, so a K/V tile
// staged in LDS is shared by the whole GQA group, and everything a wave keeps
// fits in 256 registers: two waves per SIMD let the hardware overlap one
// wave's softmax arithmetic with the other's matrix products.  The block
// streams the key intervals of the tile's root path (full rectangles), then the
// tile's own keys (visibility mask k <= t < kend[k]), 64 keys at a time:
//   S^T = K Q^T  (32x32x16 bf16 MFMA, K rows from LDS, Q^T held in registers)
//   online softmax in fp32; in the transposed product every lane owns one
//   query column, so max / sum / rescale need one cross-lane exchange only
//   O^T += V^T P^T  (V columns via the transposing LDS read, P^T straight from
//   the S^T accumulators)
#include <hip/hip_runtime.h>

#include "dta_internal.h"
#include "dta_launch.h"
#include "dta_mfma.h"
#include "dta_queue.h"
#include "dta_tile_walk.h"

namespace dta {
namespace {

constexpr int kThreads = 512;

// kCh = keys per streamed chunk (one or two 64-row LDS tiles per operand): one
// barrier, one round of bookkeeping and one online-softmax step per chunk, so
// long key intervals run faster with 128, while every interval is padded to a
// multiple of the chunk, so forests of short segments want 64.
//
// kGroups = 2 (with kCh = 64): a block is 4 row tiles x 2 groups of waves, which take
// every other chunk of the walk and are merged in LDS at the end: twice the blocks, each
// half as long, for launches of so few rounds of blocks that the last one decides.
//
// kSkip: a wave leaves out masked chunks of which none of its 32 rows sees a key (what comes after
// them, or belongs to a neighbouring node that shares the tile).  For tiles of 128 tokens and more (at most two q heads
// of a group per block), whose row blocks see different keys, where masked chunks are many; the branch itself
// costs the schedule of the loop 1 to 3 %.
template <int kCh, int HD, int kGroups = 1, bool kSkip = false>
__global__ __launch_bounds__(kThreads) __attribute__((amdgpu_waves_per_eu(2, 2))) void fwd_bf16_kernel(
    const QTile* __restrict__ tiles, const KeySeg* __restrict__ segs,
    const int32_t* __restrict__ kend, const uint16_t* __restrict__ q,
    const uint16_t* __restrict__ k, const uint16_t* __restrict__ v, uint16_t* __restrict__ o,
    float* __restrict__ lse, int Hq, int Hkv, int HB, int hblocks, float scale,
    int* __restrict__ tickets, int n_items) {
  using TL = TileLayout<HD>;
  static_assert(kGroups == 1 || kCh == 64, "a group takes one 64-row tile per step");
  static_assert(kGroups == 1 || !kSkip, "kSkip: for blocks of 8 row tiles");
  constexpr int kSub = kCh / 64, kTileElems = TL::kTileElems, kHeadDim = HD;   // kSub: LDS tiles per group
  constexpr int KS = TL::kSteps, DB = TL::kBlocks;   // k-steps over head_dim, 32-wide output blocks
  __shared__ __attribute__((aligned(1024))) uint16_t Ks[2][kGroups * kSub][kTileElems];
  __shared__ __attribute__((aligned(1024))) uint16_t Vs[2][kGroups * kSub][kTileElems];
  __shared__ __attribute__((aligned(16))) int32_t kendS[2][kGroups * kCh];
  __shared__ int next_item[2];

  // tickets == nullptr: one (tile, kv head, head block) per block, from the block
  // index.  Otherwise resident blocks that draw (tile, head block) items from one
  // queue per kv head.
  ItemQueues queues;
  queues.init(tickets, n_items, Hkv);
  int item_idx = blockIdx.x / (Hkv * hblocks) * hblocks + (blockIdx.x % (Hkv * hblocks)) / Hkv;
  int g_idx = blockIdx.x % Hkv;
  if (tickets != nullptr && !queues.draw(next_item, item_idx, g_idx, false)) return;
  for (;;) {
  const QTile tile = tiles[item_idx / hblocks];
  const int g = g_idx, hblk = item_idx % hblocks;
  const int G = Hq / Hkv;
  const int w = threadIdx.x >> 6, l = threadIdx.x & 63;
  const int c = l & 31, hh = l >> 5;
  const int rw = w % (8 / kGroups), grp = kGroups == 1 ? 0 : __builtin_amdgcn_readfirstlane(w / (8 / kGroups));
  const int h = g * G + hblk * HB + (rw % HB);
  const int row_base = tile.t0 + 32 * (rw / HB);
  // scores stay unscaled; the softmax scale (times log2 e) is folded into the
  // exponent.  A negative scale is moved into the sign of Q so that sc > 0.
  const float sc = fabsf(scale) * kLog2e;

  const int qrow = min(row_base + c, tile.t1 - 1);
  bf16x8 Qr[KS];
  {
    const uint16_t* qp = q + ((size_t)qrow * Hq + h) * kHeadDim + 8 * hh;
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
  float m = -INFINITY, lsum = 0.f;   // running max of unscaled scores, partial row sum

  const size_t kv_stride = (size_t)Hkv * kHeadDim;
  const uint16_t* kbase = k + (size_t)g * kHeadDim;
  const uint16_t* vbase = v + (size_t)g * kHeadDim;
  const uint32_t kv_bytes = (uint32_t)kv_stride * 2;

  // Chunk i lives in buffer i & 1 and is copied global -> LDS one iteration ahead
  // of its use, so one barrier per chunk is enough.
  KeyChunksT<kCh> it;
  it.init(segs, tile);
  int c0[kGroups], n[kGroups], full[kGroups];   // of the chunk(s) copied last; n = 0: none
  auto next = [&] {
    const bool some = it.next(c0[0], n[0], full[0]);
    if constexpr (kGroups == 2)
      if (!it.next(c0[1], n[1], full[1])) n[1] = 0;
    return some;
  };
  bool have = next();
  auto issue = [&](int b) {
#pragma unroll
    for (int gi = 0; gi < kGroups; ++gi) {
      if (n[gi] == 0) continue;
      if (!full[gi] || n[gi] < kCh) {   // rare: a chunk that needs the visibility mask
        const unsigned x = threadIdx.x - gi * kCh;
        if (x < kCh) {   // kendS is indexed by matrix position within each 64-key half
          const int row = 64 * (x >> 6) + TL::row_of_pos(x & 63);
          kendS[b][threadIdx.x] = row >= n[gi] ? 0 : (full[gi] ? 0x7fffffff : kend[c0[gi] + row]);
        }
      }
#pragma unroll
      for (int sub = 0; sub < kSub; ++sub) {
        // a half with no valid key re-reads the chunk's first row (finite data the mask hides)
        const int nv = n[gi] - 64 * sub;
        const int r0 = nv > 0 ? c0[gi] + 64 * sub : c0[gi];
        const int nvalid = nv > 0 ? min(nv, 64) : 1;
        tile_async_load<kThreads, HD>(Ks[b][gi * kSub + sub], kbase + (size_t)r0 * kv_stride, kv_bytes, nvalid);
        tile_async_load<kThreads, HD>(Vs[b][gi * kSub + sub], vbase + (size_t)r0 * kv_stride, kv_bytes, nvalid);
      }
    }
  };
  issue(0);
  int buf = 0;
  const int rlo = TL::row_lane_off(), clo = TL::col_lane_off();

  while (have) {
    async_wait_all();
    __syncthreads();   // chunk `buf` has landed; everyone is done with the other buffer
    const int cc0 = kGroups == 1 || grp == 0 ? c0[0] : c0[kGroups - 1];
    const int nn = kGroups == 1 || grp == 0 ? n[0] : n[kGroups - 1];
    const bool need_mask = !(kGroups == 1 || grp == 0 ? full[0] : full[kGroups - 1]) || nn < kCh;
    have = next();
    if (have) issue(buf ^ 1);
    if (kGroups == 2 && nn == 0) break;   // the walk's last step has a chunk for the first group only
    if constexpr (kSkip) {
      if (need_mask && !wave_sees<kSub, HD>(kendS[buf], cc0, row_base)) {
        buf ^= 1;
        continue;
      }
    }
    const uint16_t* Kt = Ks[buf][grp * kSub] + rlo;
    const uint16_t* Vt = Vs[buf][grp * kSub] + clo;

    // ---- S^T = K Q^T : 64 keys x 32 queries
    f32x16 S[2 * kSub];
#pragma unroll
    for (int a = 0; a < 2 * kSub; ++a)
#pragma unroll
      for (int e = 0; e < 16; ++e) S[a][e] = 0.f;
#pragma unroll
    for (int sub = 0; sub < kSub; ++sub)
#pragma unroll
      for (int ks = 0; ks < KS; ++ks) {
        const bf16x8 a0 = tile_row8(Kt + sub * kTileElems, 0, ks);
        const bf16x8 a1 = tile_row8(Kt + sub * kTileElems, 1, ks);
        S[2 * sub] = mfma32(a0, Qr[ks], S[2 * sub]);
        S[2 * sub + 1] = mfma32(a1, Qr[ks], S[2 * sub + 1]);
      }

    // ---- mask: key kv is visible to row t iff kv <= t < kend[kv]; kendS holds
    // 0 for padding keys and INT_MAX for keys every row of the tile sees (those
    // lie before the tile, so the causal test is true for them anyway)
    if (need_mask) {
#pragma unroll
      for (int mb = 0; mb < 2 * kSub; ++mb)
#pragma unroll
        for (int e4 = 0; e4 < 4; ++e4) {
          const int kvl0 = 32 * mb + 8 * e4 + 4 * hh;
          const int4 ke = *reinterpret_cast<const int4*>(&kendS[buf][grp * kCh + kvl0]);
          const int kev[4] = {ke.x, ke.y, ke.z, ke.w};
#pragma unroll
          for (int j = 0; j < 4; ++j) {
            const bool ok = (cc0 + 64 * (mb >> 1) + TL::row_of_acc(mb & 1, 4 * e4 + j, hh) <= qrow) & (qrow < kev[j]);
            S[mb][4 * e4 + j] = ok ? S[mb][4 * e4 + j] : -INFINITY;
          }
        }
    }

    // ---- online softmax, one query column per lane
    float mx = -INFINITY;
#pragma unroll
    for (int mb = 0; mb < 2 * kSub; ++mb)
#pragma unroll
      for (int e = 0; e < 16; ++e) mx = fmaxf(mx, S[mb][e]);
    mx = max_across_halves(mx);
    const float mnew = fmaxf(m, mx);
    const float mref = mnew == -INFINITY ? 0.f : mnew;
    const float alpha = __builtin_amdgcn_exp2f((m - mref) * sc);
    m = mnew;
    const float msc = mref * sc;
    float ps = 0.f;
    bf16x8 Pb[4 * kSub];
#pragma unroll
    for (int mb = 0; mb < 2 * kSub; ++mb) {
#pragma unroll
      for (int e = 0; e < 16; ++e) {
        const float p = __builtin_amdgcn_exp2f(fmaf(S[mb][e], sc, -msc));
        S[mb][e] = p;
        ps += p;
      }
      Pb[2 * mb] = pack8(S[mb], 0);
      Pb[2 * mb + 1] = pack8(S[mb], 1);
    }
    lsum = lsum * alpha + ps;
    // the accumulators are rescaled only when some row's running max moved
    if (__builtin_amdgcn_ballot_w64(alpha != 1.f) != 0) {
#pragma unroll
      for (int dmb = 0; dmb < DB; ++dmb)
#pragma unroll
        for (int e = 0; e < 16; ++e) O[dmb][e] *= alpha;
    }

    // ---- O^T += V^T P^T
#pragma unroll
    for (int sub = 0; sub < kSub; ++sub)
#pragma unroll
      for (int kk = 0; kk < 4; ++kk) {
#pragma unroll
        for (int dmb = 0; dmb < DB; ++dmb) {
          const bf16x8 va = tile_col8(Vt + sub * kTileElems, 16 * kk, 32 * dmb);
          O[dmb] = mfma32(va, Pb[4 * sub + kk], O[dmb]);
        }
      }
    buf ^= 1;
  }

  // ---- normalise and store
  if (tickets != nullptr) queues.prefetch();
  float lt = lsum + __shfl_xor(lsum, 32);
  constexpr int kOut = DB / kGroups;   // 32-wide output blocks this wave stores, from block kOut * grp
  if constexpr (kGroups == 2) {
    // common maximum and row sum, then every group hands the other one its half of the output blocks
    __shared__ float mS[8][32], lS[8][32];
    f32x4* xs = reinterpret_cast<f32x4*>(&Ks[0][0][0]);
    static_assert(sizeof(Ks) >= 8 * kOut * 4 * 64 * sizeof(f32x4), "room for the exchange");
    if (hh == 0) {
      mS[w][c] = m;
      lS[w][c] = lt;
    }
    __syncthreads();   // everyone is done with the tiles, too
    const float m2 = mS[w ^ 4][c], l2 = lS[w ^ 4][c], own = m;
    m = fmaxf(own, m2);
    const float mref = m == -INFINITY ? 0.f : m;   // (every score of the row may be -inf)
    const float f = __builtin_amdgcn_exp2f((own - mref) * sc);
    lt = lt * f + l2 * __builtin_amdgcn_exp2f((m2 - mref) * sc);
#pragma unroll
    for (int dmb = 0; dmb < DB; ++dmb)
#pragma unroll
      for (int e = 0; e < 16; ++e) O[dmb][e] *= f;
#pragma unroll
    for (int b = 0; b < kOut; ++b)
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        const f32x16& x0 = O[b];
        const f32x16& x1 = O[kOut + b];
        xs[((w * kOut + b) * 4 + i) * 64 + l] =
              grp == 0 ? f32x4{x1[4 * i], x1[4 * i + 1], x1[4 * i + 2], x1[4 * i + 3]}
                       : f32x4{x0[4 * i], x0[4 * i + 1], x0[4 * i + 2], x0[4 * i + 3]};
      }
    __syncthreads();
#pragma unroll
    for (int b = 0; b < kOut; ++b)
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        const f32x4 x = xs[(((w ^ 4) * kOut + b) * 4 + i) * 64 + l];
#pragma unroll
        for (int e = 0; e < 4; ++e) O[b][4 * i + e] = (grp == 0 ? O[b][4 * i + e] : O[kOut + b][4 * i + e]) + x[e];
      }
  }
  const float inv = 1.f / lt;
  const int token = row_base + c;
  if (token < tile.t1) {
    uint16_t* op = o + ((size_t)token * Hq + h) * kHeadDim + 32 * kOut * grp + 4 * hh;
#pragma unroll
    for (int dmb = 0; dmb < kOut; ++dmb)
#pragma unroll
      for (int v4 = 0; v4 < 4; ++v4) {
        bf16x4 r;
#pragma unroll
        for (int e = 0; e < 4; ++e) r[e] = (__bf16)(O[dmb][4 * v4 + e] * inv);
        *reinterpret_cast<bf16x4*>(op + 32 * dmb + 8 * v4) = r;
      }
    if (hh == 0 && grp == 0) lse[(size_t)token * Hq + h] = (m * sc + log2f(lt)) * kLn2;
  }
  if (tickets == nullptr || !queues.draw(next_item, item_idx, g_idx, true)) break;
  }   // next item
}

// Sets n ints to zero (the ticket counters; a fill kernel rather than a memset
// so that the launch sequence can be captured in a graph).
__global__ void zero_i32_kernel(int* __restrict__ p, int n) {
  for (int i = threadIdx.x; i < n; i += blockDim.x) p[i] = 0;
}

}  // namespace

int launch_fwd_bf16(const LaunchArgs& a) {
  hipStream_t st = (hipStream_t)a.stream;
  clear_hip_error();
  if (a.tc.q_small) return launch_fwd_bf16_small(a);
  const bool split = a.tc.q_split;
  const QueryTiles& qt = a.sched->forward_tiles();
  const size_t blocks = qt.q_tiles.size() * (size_t)a.p.n_kv_heads * (size_t)a.tc.hblocks;
  if (blocks == 0 || blocks > 0x7fffffffu) return DTA_ERR_UNSUPPORTED;
  // With a workspace for the counters and enough items, resident blocks draw the
  // items from per-head queues (see dta_queue.h); otherwise one block per item.
  const bool queues = !split && a.tickets != nullptr && blocks >= 8 * (size_t)kNumCUs;
  if (queues) {
    zero_i32_kernel<<<1, 256, 0, st>>>(a.tickets, a.p.n_kv_heads);
    { int ls = launch_status(__func__); if (ls != DTA_OK) return ls; }
  }
  // chunk size: 128 keys when padding every key interval to 128 instead of 64 adds
  // at most 6 % to the keys streamed (measured: 5 % faster at +0.5 %, 1.4 % faster
  // at +5.6 %, 2 % slower at +9.6 %)
  const bool wide = 2 * qt.fwd_chunks128 * 100 <= qt.fwd_chunks64 * 106;
  // kSkip where more than 30 % of the chunks are masked.  Measured, without / with, by share of masked chunks: 16/16
  // heads of 128, 79 % 319 / 295 us (short answers), 40 % 333 / 319 (pairs), 36 % 1476 / 1402, 15 % 80.0 / 81.4, 6 %
  // 344 / 348; 8/4 heads, 61 % 129 / 117, 23 % 154.5 / 156.3, 20 % 650.5 / 651.2, 3 % 203 / 208
  const bool skip = a.tc.hb <= 2 && 10 * qt.fwd_masked64 > 3 * qt.fwd_chunks64;
  auto kernel = split ? (a.p.head_dim == 128 ? fwd_bf16_kernel<64, 128, 2> : fwd_bf16_kernel<64, 64, 2>)
                : a.p.head_dim == 128
                    ? (skip ? (wide ? fwd_bf16_kernel<128, 128, 1, true> : fwd_bf16_kernel<64, 128, 1, true>)
                            : (wide ? fwd_bf16_kernel<128, 128> : fwd_bf16_kernel<64, 128>))
                    : (skip ? (wide ? fwd_bf16_kernel<128, 64, 1, true> : fwd_bf16_kernel<64, 64, 1, true>)
                            : (wide ? fwd_bf16_kernel<128, 64> : fwd_bf16_kernel<64, 64>));
  launch(a, true, kernel, queues ? (size_t)kNumCUs : blocks, kThreads,
      qt.d_q_tiles, qt.d_segs, a.d_kend, (const uint16_t*)a.q, (const uint16_t*)a.k,
      (const uint16_t*)a.v, (uint16_t*)a.o_out, a.lse_out, a.p.n_q_heads, a.p.n_kv_heads, a.tc.hb,
      a.tc.hblocks, a.p.softmax_scale, queues ? a.tickets : nullptr,
      (int)(qt.q_tiles.size() * (size_t)a.tc.hblocks));
  return launch_status(__func__);
}

}  // namespace dta
