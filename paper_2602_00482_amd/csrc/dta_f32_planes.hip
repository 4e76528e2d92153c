// fp32 tree attention for launches that fill the chip: forward, dQ and dK/dV with every
// product on the bf16 matrix instruction, whose rate is 16 times the fp32 one's.
//
// An fp32 number is the sum of three bf16 numbers (planes) of 8 bits each (the split that Henry, Tang and Heinecke
// describe in "Leveraging the bfloat16 Artificial Intelligence Datatype For Higher-Precision Computations", 2019):
// x = x1 + x2 + x3 with x1 = bf16(x), x2 = bf16(x - x1), x3 = x - x1 - x2, each subtraction exact.  A product
// x y is x1 y1 + x1 y2 + x2 y1 + x2 y2 + x1 y3 + x3 y1; x2 y3, x3 y2 and x3 y3 are left out, together up to
// 2^-24 |x y| (what rounding one product to fp32 costs; 2^-26 and less for most).  The matrix instruction adds
// exact products in fp32 accumulators.  Six bf16 products of 16x16x32 take 96 cycles where the
// fp32 instruction takes 256.  Softmax, exponentials and everything between the products is fp32.
//
// bf16 has fp32's exponent range, so nothing has to be scaled.  Below 2^-110 the third part is subnormal, and a number
// is held to 2^-134; probabilities below 2^-126 count as 0.  Numbers from 2^40 on, infinities among them, do not take part: the six products of large ones
// overflow with either sign, which adds up to NaN where the product is an infinity, and what bf16 rounds to infinity has no
// parts at all.  (Three factors below 2^40, summed over head_dim, stay below 2^127.)  From the first streamed chunk that
// holds one, a block goes on on the fp32 instruction (slow_dot, slow_apply); so does a block of the backward kernels with
// such a row of its own, while a wave of the forward, whose other rows must not change, walks for them once more.
// NaN may pass: its parts are NaN.
//
// A block is 8 waves, each with 16 query rows (dK/dV: 16 keys) as columns, their three planes in
// registers.  The streamed rows, 32 per step, come as fp32 by direct global-to-LDS loads, every wave
// its own 4 KB; the wave splits them into planes in a double-buffered tile that all waves
// read, while the products of the step before run, and starts the loads of the step
// after next.  One split then serves eight waves, and one barrier a step is enough.
//
// What bounds the kernels is the issue of vector instructions beside the products: per product of the
// forward 4.6 (the split of the streamed rows 1.4, softmax, the split of P and the sums of O the rest), dQ 3.0 and
// dK/dV 2.4, of which two go under a product for free where they alternate with it; the matrix pipe is
// busy 39 % (forward), 45 % (dQ) and 55 % (dK/dV) of the time at 2.2 GHz.  Larger blocks would
// share a split among more rows, but 16 more columns per wave do not fit in the registers of dQ and dK/dV.
// Measured on MI355X, products on the fp32 instruction before, and now (kernel trace, medians):
//   4862 tokens (a prompt with 16 answers), 32/8 heads of 128: forward 386 -> 300 us, dQ 554 -> 385,
//     dK/dV 669 -> 435, reduce 14.6 -> 8.1; of 64: forward 223 -> 192, dQ 297 -> 233, dK/dV 365 -> 269
//   8898 tokens (a prompt with 8 answers), 16/16 heads of 128: forward 1362 -> 1011 us, dQ 1995 -> 1221, dK/dV 2331 -> 1401
//   relative 2-norm errors against 64 bits, 4546 tokens, 32/8 heads of 128: O 3.87 -> 1.65e-7, LSE 4.3 -> 4.0e-8, dQ 5.1 -> 3.2e-7,
//     dK 6.8 -> 3.5e-7, dV 6.4 -> 3.3e-7; 6600 tokens, 4/4 heads of 64: O 3.16 -> 1.66e-7, dQ 4.9 -> 3.6e-7, dK 4.8 -> 3.6e-7
#include <hip/hip_runtime.h>

#include "dta_f32_common.h"
#include "dta_launch.h"
#include "dta_tile_walk.h"

namespace dta {
namespace {

constexpr int kThreads = 512, kWaves = 8;
constexpr int kRows = 32;        // streamed rows per step
constexpr int kPlanes = 3;
constexpr float kNoPlanes = 0x1p40f;   // numbers from here on are multiplied on the fp32 instruction

typedef __bf16 bf16x2 __attribute__((ext_vector_type(2)));

__device__ __forceinline__ uint32_t bf16_pair(float a, float b) {
  const bf16x2 r = {(__bf16)a, (__bf16)b};
  uint32_t u;
  __builtin_memcpy(&u, &r, 4);
  return u;
}
// the planes of two numbers, p[i] = plane i of a (low half) and b
__device__ __forceinline__ void split2(float a, float b, uint32_t (&p)[kPlanes]) {
#pragma unroll
  for (int i = 0; i < kPlanes; ++i) {
    p[i] = bf16_pair(a, b);
    a -= __uint_as_float(p[i] << 16);
    b -= __uint_as_float(p[i] & 0xffff0000u);
  }
}

// e^x to fp32 accuracy for the arguments of a softmax (not above 88; LSE has to be the forward's), without the range
// handling of expf: 2^t with t = x log2 e rounded, times 1 + (x - t ln 2).  0 below -87; the
// correction is NaN for x = -infinity, where the maximum drops it.  NaN stays.
constexpr float kLn2Low = -1.9046543e-9f;   // ln 2 = kLn2 + kLn2Low
__device__ __forceinline__ float exp_f32(float x) {
  const float t = x * kLog2e;
  const float r = fmaf(-t, kLn2Low, fmaf(-t, kLn2, x));
  const float e = __builtin_amdgcn_exp2f(t);
  return fmaf(e, fmaxf(r, -1.f), e);
}

// max over the four lane groups of a column, in the vector ALU
__device__ __forceinline__ float column_max4(float x) {
  const unsigned u = __float_as_uint(x);
  const auto r = __builtin_amdgcn_permlane16_swap(u, u, false, false);
  return max_across_halves(fmaxf(__uint_as_float(r[0]), __uint_as_float(r[1])));
}

union Frag {
  uint32_t u[4];
  bf16x8 v;
};

// ---- tiles of three planes of 32 rows x HD bf16 ----------------------------------
// Row r lies at slot tau(r & 15) + (r & 16), slots HD * 2 + 16 bytes apart, so that slot s starts
// s (HD = 64: 9 s) 16-byte units of bank offset along.  A product that contracts over HD takes the
// 8 elements from k_off(g) + 8 * ks of its rows in lane group g at k-step ks.  With both,
// the passes of 16-byte reads (lanes {0-3, 12-15, 20-27} and {4-11, 16-19, 28-31}, and the
// same of the upper half) and of transposing reads (halves) meet 16 different units.
template <int HD>
struct PlaneTile {
  static_assert(HD == 128 || HD == 64, "head_dim 64 or 128");
  static constexpr int kPitch = HD + 8;               // elements between slots
  static constexpr int kPlane = kRows * kPitch;       // elements of a plane
  static constexpr int kElems = kPlanes * kPlane;
  static constexpr int KS = HD / 32;                  // k-steps of a product that contracts over HD
  static constexpr int DB = HD / 16;                  // 16-wide output blocks along HD

  // {0, 4, 8, 12, 2, 6, 10, 14, 3, 7, 11, 15, 1, 5, 9, 13}
  __device__ __forceinline__ static int tau(int y) {
    return 4 * (y & 3) + ((0x1320 >> (y & 12)) & 3);
  }
  __device__ __forceinline__ static int slot(int r) { return tau(r & 15) + (r & 16); }
  __device__ __forceinline__ static int k_off(int g) { return HD == 128 ? 32 * g : 32 * (g & 1) + 16 * (g >> 1); }
  // per-lane element offsets for row() and col()
  __device__ __forceinline__ static int row_lane_off() {
    const int l = threadIdx.x & 63;
    return tau(l & 15) * kPitch + k_off(l >> 4);
  }
  __device__ __forceinline__ static int col_lane_off() {
    const int l = threadIdx.x & 63, i = l & 15, g = l >> 4;
    return tau(4 * g + (i >> 2)) * kPitch + 4 * (i & 3);
  }
  // rows 16*b .. 16*b+15 as rows of an operand, k-step ks
  __device__ __forceinline__ static bf16x8 row(const uint16_t* lane_ptr, int plane, int b, int ks) {
    return *reinterpret_cast<const bf16x8*>(lane_ptr + plane * kPlane + 16 * b * kPitch + 8 * ks);
  }
  // columns 16*cb .. 16*cb+15 as rows of an operand, the 32 tile rows as contraction index: its
  // element 8*g + 4*b + e is row 16*b + 4*g + e
  __device__ __forceinline__ static bf16x8 col(const uint16_t* lane_ptr, int plane, int cb) {
    const uint16_t* p = lane_ptr + plane * kPlane + 16 * cb;
    union {
      struct { s16x4 a, b; } s;
      bf16x8 v;
    } u;
    u.s.a = lds_read_tr4(p);
    u.s.b = lds_read_tr4(p + 16 * kPitch);
    return u.v;
  }
};

// The three planes of 16 rows of HD floats, one per column, as operand registers.
template <int HD>
struct OwnRows {
  using PT = PlaneTile<HD>;
  bf16x8 p[kPlanes][PT::KS];
  // `row`: this lane's row, times `sign` (1 or -1); false if it has no planes (see kNoPlanes)
  __device__ __forceinline__ bool load(const float* row, float sign = 1.f) {
    const int lg = (threadIdx.x >> 4) & 3;
    float big = 0.f;
#pragma unroll
    for (int ks = 0; ks < PT::KS; ++ks) {
      Frag f[kPlanes];
#pragma unroll
      for (int i = 0; i < 2; ++i) {
        const f32x4 x = *reinterpret_cast<const f32x4*>(row + PT::k_off(lg) + 8 * ks + 4 * i) * sign;
#pragma unroll
        for (int e = 0; e < 4; e += 2) {
          uint32_t s[kPlanes];
          split2(x[e], x[e + 1], s);
          big = fmaxf(big, fmaxf(fabsf(x[e]), fabsf(x[e + 1])));
#pragma unroll
          for (int j = 0; j < kPlanes; ++j) f[j].u[2 * i + e / 2] = s[j];
        }
      }
#pragma unroll
      for (int j = 0; j < kPlanes; ++j) p[j][ks] = f[j].v;
    }
    return column_max4(big) < kNoPlanes;
  }
};

// The planes of the 32 x 16 numbers x[b][e] (row 16*b + 4*g + e) as operand of a product
// that contracts over the rows, two numbers at a time: piece t of 4.
__device__ __forceinline__ void split_piece(const f32x4 (&x)[2], Frag (&f)[kPlanes], int t) {
  uint32_t s[kPlanes];
  split2(x[t >> 1][2 * (t & 1)], x[t >> 1][2 * (t & 1) + 1], s);
#pragma unroll
  for (int j = 0; j < kPlanes; ++j) f[j].u[t] = s[j];
}
__device__ __forceinline__ void operand(const Frag (&f)[kPlanes], bf16x8 (&p)[kPlanes]) {
#pragma unroll
  for (int j = 0; j < kPlanes; ++j) p[j] = f[j].v;
}

// ---- products as streams ------------------------------------------------------------
// A product reads its tile as a stream of 3 * HD / 32 pairs of operands, the same plane of two blocks, and
// multiplies every pair as it comes: six, four or two matrix instructions, two accumulators apart, so
// that none waits for the one before it.  The pairs are read kAhead ahead, across products too
// (`next` fetches the first ones of what follows).  A matrix instruction leaves the vector ALU of
// its SIMD two free issue slots of the four it takes, and what is issued in clumps does not overlap: `work(m)`
// is about two vector instructions to go with matrix instruction m, and a scheduling barrier holds the order.
constexpr int kAhead = 2, kRing = 3;
struct Pair {
  bf16x8 a[2];
};
template <int HD>
constexpr int kPairs = 3 * HD / 32;
template <int HD>
constexpr int kProducts = 12 * HD / 32;   // matrix instructions of a product
static_assert(kPairs<128> % kRing == 0 && kPairs<64> % kRing == 0, "a product leaves the ring where it found it");

template <int HD>
__device__ __forceinline__ Pair row_pair(const uint16_t* rows, int i) {
  return Pair{{PlaneTile<HD>::row(rows, i % 3, 0, i / 3), PlaneTile<HD>::row(rows, i % 3, 1, i / 3)}};
}
template <int HD>
__device__ __forceinline__ Pair col_pair(const uint16_t* cols, int i) {
  const int plane = 2 - i % 3, cb = 2 * (i / 3);
  return Pair{{PlaneTile<HD>::col(cols, plane, cb), PlaneTile<HD>::col(cols, plane, cb + 1)}};
}
struct Nothing {
  __device__ __forceinline__ void operator()(int) const {}
};

// S[b] = (rows 16*b .. of the tile) . (own columns), contracted over HD.  The products with a
// second or third plane are added apart, so that the sum is rounded once per 32 elements of head_dim.
template <int HD, typename Work, typename Next>
__device__ __forceinline__ void dot(f32x4 (&S)[2], Pair (&ring)[kRing], const uint16_t* rows, const OwnRows<HD>& own,
                                    Work work, Next next) {
  f32x4 c0[2] = {}, c1[2] = {};
#pragma unroll
  for (int i = 0; i < kPairs<HD>; ++i) {
    if (i + kAhead < kPairs<HD>) ring[(i + kAhead) % kRing] = row_pair<HD>(rows, i + kAhead);
    else next(ring[(i + kAhead) % kRing], i + kAhead - kPairs<HD>);
    const Pair& x = ring[i % kRing];
    const int ks = i / 3, plane = i % 3;
#pragma unroll
    for (int j = 0; j < kPlanes - plane; ++j)
#pragma unroll
      for (int b = 0; b < 2; ++b) {
        f32x4& c = plane + j == 0 ? c0[b] : c1[b];
        c = mfma16(x.a[b], own.p[j][ks], c);
        work(12 * ks + (plane == 0 ? 0 : plane == 1 ? 6 : 10) + 2 * j + b);
        __builtin_amdgcn_sched_barrier(0);
      }
  }
#pragma unroll
  for (int b = 0; b < 2; ++b) S[b] = c0[b] + c1[b];
}

// acc[cb] += (columns 16*cb .. of the tile) . w, contracted over the tile's rows.  The six products of a pair
// of blocks are summed from zero and added to acc while the next pair's run: acc is rounded once per chunk of 32
// rows, not six times: relative errors of O, 900 tokens, 32/8 heads of 64, 2.1 -> 1.2e-7, for 2 % of the time.
template <int HD, typename Work, typename Next>
__device__ __forceinline__ void apply(f32x4 (&acc)[HD / 16], Pair (&ring)[kRing], const uint16_t* cols,
                                      const bf16x8 (&w)[kPlanes], Work work, Next next) {
  f32x4 sum[2][2];
#pragma unroll
  for (int i = 0; i < kPairs<HD>; ++i) {
    if (i + kAhead < kPairs<HD>) ring[(i + kAhead) % kRing] = col_pair<HD>(cols, i + kAhead);
    else next(ring[(i + kAhead) % kRing], i + kAhead - kPairs<HD>);
    const Pair& x = ring[i % kRing];
    const int plane = 2 - i % 3, pair = i / 3;
    f32x4(&c)[2] = sum[pair & 1];
    if (plane == 2) c[0] = c[1] = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int j = kPlanes - 1 - plane; j >= 0; --j)
#pragma unroll
      for (int b = 0; b < 2; ++b) {
        c[b] = mfma16(x.a[b], w[j], c[b]);
        const int m = (plane == 2 ? 0 : plane == 1 ? 2 : 6) + 2 * (kPlanes - 1 - plane - j) + b;   // 0 .. 11
        work(12 * pair + m);
        if (pair > 0 && m >= 4) {   // (the previous pair's last products have ended by then)
          const int e = m - 4;
          acc[2 * pair - 2 + (e >> 2)][e & 3] += sum[(pair - 1) & 1][e >> 2][e & 3];
        }
        __builtin_amdgcn_sched_barrier(0);
      }
  }
  constexpr int kLast = HD / 32 - 1;
#pragma unroll
  for (int b = 0; b < 2; ++b) acc[2 * kLast + b] += sum[kLast & 1][b];
}

// The vector work that goes with products, in steps of about two instructions: twelve split a
// pair of numbers of which steps 0 to 5 made probabilities from exponents.
struct PairSplit {
  float x0, x1, t0, t1, r0, r1;
  uint32_t u;
  // step 0..5: x0, x1 = e^x0, e^x1 (exp_f32)
  __device__ __forceinline__ void exp_step(int s) {
    if (s == 0) { t0 = x0 * kLog2e; t1 = x1 * kLog2e; }
    if (s == 1) { r0 = fmaf(-t0, kLn2, x0); r1 = fmaf(-t1, kLn2, x1); }
    if (s == 2) { r0 = fmaf(-t0, kLn2Low, r0); r1 = fmaf(-t1, kLn2Low, r1); }
    if (s == 3) { x0 = __builtin_amdgcn_exp2f(t0); x1 = __builtin_amdgcn_exp2f(t1); }
    if (s == 4) { r0 = fmaxf(r0, -1.f); r1 = fmaxf(r1, -1.f); }
    if (s == 5) { x0 = fmaf(x0, r0, x0); x1 = fmaf(x1, r1, x1); }
  }
  // step 0..5: the planes of x0, x1, into element t of f (x0, x1 stay)
  __device__ __forceinline__ void split_step(int s, Frag (&f)[kPlanes], int t) {
    if (s == 0) { u = f[0].u[t] = bf16_pair(x0, x1); r0 = x0 - __uint_as_float(u << 16); }
    if (s == 1) r1 = x1 - __uint_as_float(u & 0xffff0000u);
    if (s == 2) { u = f[1].u[t] = bf16_pair(r0, r1); r0 -= __uint_as_float(u << 16); }
    if (s == 3) r1 -= __uint_as_float(u & 0xffff0000u);
    if (s == 4) f[2].u[t] = bf16_pair(r0, r1);
  }
};

// The same on the fp32 instruction, from the tensors: streamed row r is at base + min(r, n - 1) * stride.  The two
// halves of head_dim are summed apart, as in dta_f32_kernels.hip.
template <int HD>
__device__ __forceinline__ void slow_dot(f32x4 (&S)[2], const float* base, size_t stride, int n, const float* own) {
  const int l = threadIdx.x & 63, n16 = l & 15, lg = l >> 4;
#pragma unroll
  for (int b = 0; b < 2; ++b) {
    const float* row = base + (size_t)min(16 * b + n16, n - 1) * stride + lg;
    S[b] = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll 1
    for (int half = 0; half < HD; half += HD / 2) {
      f32x4 c = {0.f, 0.f, 0.f, 0.f};
#pragma unroll 1
      for (int j = half; j < half + HD / 2; j += 4) c = mfma16_f32(row[j], own[j + lg], c);
      S[b] += c;
    }
  }
}
template <int HD>
__device__ __forceinline__ void slow_apply(f32x4 (&acc)[HD / 16], const float* base, size_t stride, int n,
                                           const f32x4 (&w)[2]) {
  const int l = threadIdx.x & 63, n16 = l & 15, lg = l >> 4;
#pragma unroll
  for (int b = 0; b < 2; ++b)
#pragma unroll
    for (int e = 0; e < 4; ++e) {
      const float* row = base + (size_t)min(16 * b + 4 * lg + e, n - 1) * stride + n16;
#pragma unroll
      for (int cb = 0; cb < HD / 16; ++cb) acc[cb] = mfma16_f32(row[16 * cb], w[b][e], acc[cb]);
    }
}

// ---- streaming -----------------------------------------------------------------
// Per step two tensors' rows (K and V, or Q and dO): the raw fp32 rows land in `raw`, 4 KB (head_dim
// 64: 2 KB) per wave that only this wave touches, and go from there into the planes.
template <int HD>
struct Stream {
  using PT = PlaneTile<HD>;
  static constexpr int kRowsPerLoad = 256 / HD;                   // rows one wave-wide 16-byte load covers
  static constexpr int kLoads = 2 * kRows / kRowsPerLoad / kWaves;   // per wave and step, over both tensors
  struct Smem {
    uint16_t planes[2][2][PT::kElems];   // [buffer][tensor]
    f32x4 raw[kWaves][kLoads][64];
    int big[4];                          // ring over the steps: the step holds a number without planes
  };
  // starts the loads of rows base0 / base1 (+ r * stride_bytes, r < n; rows beyond repeat the last)
  __device__ __forceinline__ static void issue(Smem& sm, const float* base0, const float* base1, uint32_t stride_bytes,
                                               int n) {
    const int w = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), l = threadIdx.x & 63;
    const uint32_t raw_addr = (uint32_t)(uintptr_t)(__attribute__((address_space(3))) void*)&sm.raw[w][0][0];
#pragma unroll
    for (int p = 0; p < kLoads; ++p) {
      const int row = (w + kWaves * (p % (kLoads / 2))) * kRowsPerLoad + l / (HD / 4);
      const uint64_t bits = (uint64_t)(uintptr_t)(p < kLoads / 2 ? base0 : base1);
      const uint32_t hi = (uint32_t)__builtin_amdgcn_readfirstlane((int)(uint32_t)(bits >> 32));
      const uint32_t lo = (uint32_t)__builtin_amdgcn_readfirstlane((int)(uint32_t)bits);
      const uint64_t sbase = ((uint64_t)hi << 32) | (uint64_t)lo;
      const uint32_t voff = (uint32_t)min(row, n - 1) * stride_bytes + (l % (HD / 4)) * 16;
      const uint32_t lds_addr = __builtin_amdgcn_readfirstlane(raw_addr + p * 1024);
      asm volatile("s_mov_b32 m0, %2\n\tglobal_load_lds_dwordx4 %0, %1"
                   :
                   : "v"(voff), "s"(sbase), "s"(lds_addr)
                   : "memory");
    }
  }
  // The split of this wave's landed rows into buffer b: kLoads pieces of 12 steps, step m to go with
  // matrix instruction m of a product.
  struct Split {
    f32x4 x, nx;
    uint32_t s0[kPlanes], s1[kPlanes];
    float big = 0.f;
    const f32x4* src;
    uint16_t* dst;
    // (lane addresses from a value the compiler cannot see through: kept over the loop they would be spilled)
    __device__ __forceinline__ void init(Smem& sm, int b) {
      unsigned tid = threadIdx.x;
      asm volatile("" : "+v"(tid));
      const int w = tid >> 6, l = tid & 63;
      src = &sm.raw[w][0][l];
      // loads p < kLoads / 2: rows (w + 8 p) * kRowsPerLoad + .. of the first tensor, the others of the second
      dst = &sm.planes[b][0][PT::slot(w * kRowsPerLoad + l / (HD / 4)) * PT::kPitch + 4 * (l % (HD / 4))];
      nx = src[0];
    }
    __device__ __forceinline__ void step(int m) {
      const int p = m / 12, s = m % 12;
      if (s == 0) {
        x = nx;
        s0[0] = bf16_pair(x[0], x[1]);
        s1[0] = bf16_pair(x[2], x[3]);
        big = fmaxf(big, fmaxf(fmaxf(fabsf(x[0]), fabsf(x[1])), fmaxf(fabsf(x[2]), fabsf(x[3]))));
      }
      if (s == 4 && p + 1 < kLoads) nx = src[64 * (p + 1)];
      if (s == 1 || s == 6) x[0] -= __uint_as_float(s0[s / 5] << 16);
      if (s == 2 || s == 7) x[1] -= __uint_as_float(s0[s / 5] & 0xffff0000u);
      if (s == 3 || s == 8) x[2] -= __uint_as_float(s1[s / 5] << 16);
      if (s == 4 || s == 9) x[3] -= __uint_as_float(s1[s / 5] & 0xffff0000u);
      if (s == 5 || s == 10) {
        s0[s / 5] = bf16_pair(x[0], x[1]);
        s1[s / 5] = bf16_pair(x[2], x[3]);
      }
      if (s == 11) {
        // rows 16 slots apart (row + 16 is slot + 16): head_dim 64 has all 32 rows in one load
        uint16_t* d = dst + (p < kLoads / 2 ? 0 : PT::kElems) + 16 * PT::kPitch * (p % (kLoads / 2));
#pragma unroll
        for (int j = 0; j < kPlanes; ++j) *reinterpret_cast<uint2*>(d + j * PT::kPlane) = make_uint2(s0[j], s1[j]);
      }
    }
    __device__ __forceinline__ void finish(Smem& sm, int step) {
      if (__builtin_amdgcn_ballot_w64(big >= kNoPlanes) != 0 && (threadIdx.x & 63) == 0) sm.big[step & 3] = 1;
    }
    __device__ __forceinline__ void all(Smem& sm, int b, int at) {
      init(sm, b);
#pragma unroll
      for (int m = 0; m < 12 * kLoads; ++m) step(m);
      finish(sm, at);
    }
  };
};

// What forward and dQ share: the block's rows and its walk over the keys.  Of the chunks of
// the walk three are under way: the one multiplied, the one split and the one loaded.
template <int HD>
struct Walk {
  using ST = Stream<HD>;
  struct Chunk {
    int c0, n, full;
    __device__ __forceinline__ bool masked() const { return !full || n < kRows; }
  };
  QTile tile;
  KeyChunksT<kRows> it;
  Chunk cur, nxt;
  bool have_nxt;
  int n16, lg, w, h, g_kv, row_base, qrow;
  const float *kbase, *vbase;
  size_t kv_stride;

  __device__ __forceinline__ void init(const QTile* tiles, const KeySeg* segs, const float* k, const float* v, int Hq,
                                       int Hkv, int HB, int hblocks) {
    const int item = blockIdx.x / Hkv, l = threadIdx.x & 63;
    g_kv = blockIdx.x % Hkv;
    tile = tiles[item / hblocks];
    w = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    n16 = l & 15;
    lg = l >> 4;
    h = g_kv * (Hq / Hkv) + (item % hblocks) * HB + w % HB;
    row_base = tile.t0 + 16 * (w / HB);
    qrow = min(row_base + n16, tile.t1 - 1);
    kv_stride = (size_t)Hkv * HD;
    kbase = k + (size_t)g_kv * HD;
    vbase = v + (size_t)g_kv * HD;
    it.init(segs, tile);
    advance(cur);   // (a tile has at least its own chunk)
  }
  __device__ __forceinline__ bool advance(Chunk& c) { return it.next(c.c0, c.n, c.full); }
  __device__ __forceinline__ const float* keys(const Chunk& c) const { return kbase + (size_t)c.c0 * kv_stride; }
  __device__ __forceinline__ const float* values(const Chunk& c) const { return vbase + (size_t)c.c0 * kv_stride; }
  __device__ __forceinline__ void issue(typename ST::Smem& sm, const Chunk& c) const {
    ST::issue(sm, keys(c), values(c), (uint32_t)kv_stride * 4, c.n);
  }
  // ends of visibility of a chunk's keys, for the mask
  __device__ __forceinline__ void copy_ends(int32_t* dst, const int32_t* kend, const Chunk& c) const {
    if (c.masked() && threadIdx.x < kRows)
      dst[threadIdx.x] = (int)threadIdx.x >= c.n ? 0 : (c.full ? 0x7fffffff : kend[c.c0 + threadIdx.x]);
  }
  // puts `none` where this lane's row does not see the key
  __device__ __forceinline__ void mask(f32x4 (&S)[2], const Chunk& c, const int32_t* ends, float none) const {
#pragma unroll
    for (int b = 0; b < 2; ++b) {
      const int4 ke = *reinterpret_cast<const int4*>(ends + 16 * b + 4 * lg);
      const int kev[4] = {ke.x, ke.y, ke.z, ke.w};
#pragma unroll
      for (int e = 0; e < 4; ++e)
        S[b][e] = ((c.c0 + 16 * b + 4 * lg + e <= qrow) & (qrow < kev[e])) ? S[b][e] : none;
    }
  }
  __device__ __forceinline__ void mask_slow(f32x4 (&S)[2], const Chunk& c, const int32_t* kend, float none) const {
#pragma unroll
    for (int b = 0; b < 2; ++b)
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        const int i = 16 * b + 4 * lg + e, key = c.c0 + min(i, c.n - 1);
        const int end = c.full ? 0x7fffffff : kend[key];   // (no branches here: this compiler loses S in them)
        S[b][e] = ((i < c.n) & ((c.full != 0) | (key <= qrow)) & (qrow < end)) ? S[b][e] : none;
      }
  }
  // own chunk of the tile whose keys come after every row of this wave
  __device__ __forceinline__ bool unseen(const Chunk& c) const { return c.masked() && c.c0 > row_base + 15; }
  __device__ __forceinline__ bool mine() const { return row_base + n16 < tile.t1; }
};

// The online softmax of a chunk: S, products of q and k not scaled yet, becomes the probabilities
// 2^((S - m) factor), m the running maximum.  The factor, |softmax_scale| log2 e, is a number in two parts: rounded to
// one it would show in LSE (all scores lie on one side of the maximum).  Only differences are multiplied by it, which
// keeps scores of any size in range, and LSE is one rounding from m |softmax_scale|.
struct Softmax {
  float hi, lo;   // the factor; lo > 0, so that a score of -infinity stays one
  float m = -INFINITY;
  float sum = 0.f;   // this lane's share of the row's
  __device__ __forceinline__ Softmax(float scale) {
    const double factor = fabs((double)scale) * 1.4426950408889634;
    hi = (float)factor;
    if (hi >= factor) hi = __uint_as_float(__float_as_uint(hi) - 1);
    lo = (float)(factor - hi);
  }
  __device__ __forceinline__ float relative(float x) const {   // 2^(x factor)
    return __builtin_amdgcn_exp2f(fmaf(x, lo, x * hi));
  }
  template <int DB>
  __device__ __forceinline__ void step(f32x4 (&S)[2], f32x4 (&O)[DB]) {
    float mx = -INFINITY;
#pragma unroll
    for (int b = 0; b < 2; ++b)
#pragma unroll
      for (int e = 0; e < 4; ++e) mx = fmaxf(mx, S[b][e]);
    const float next = fmaxf(m, column_max4(mx)), ref = next == -INFINITY ? 0.f : next;
    const float alpha = relative(m - ref);
    m = next;
    float ps = 0.f;
#pragma unroll
    for (int b = 0; b < 2; ++b)
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        S[b][e] = relative(S[b][e] - ref);
        ps += S[b][e];
      }
    sum = fmaf(sum, alpha, ps);
    if (__builtin_amdgcn_ballot_w64(alpha != 1.f) != 0) {
#pragma unroll
      for (int b = 0; b < DB; ++b) O[b] *= alpha;
    }
  }
};

// ---- forward: same walk as dta_f32_kernels.hip, 8 row tiles per block ------------------
template <int HD>
__global__ __launch_bounds__(kThreads) __attribute__((amdgpu_waves_per_eu(2, 2))) void fwd_planes_kernel(
    const QTile* __restrict__ tiles, const KeySeg* __restrict__ segs, const int32_t* __restrict__ kend,
    const float* __restrict__ q, const float* __restrict__ k, const float* __restrict__ v, float* __restrict__ o,
    float* __restrict__ lse, int Hq, int Hkv, int HB, int hblocks, float scale) {
  using PT = PlaneTile<HD>;
  using ST = Stream<HD>;
  constexpr int DB = PT::DB;
  __shared__ __attribute__((aligned(1024))) typename ST::Smem sm;
  __shared__ __attribute__((aligned(16))) int32_t kendS[2][kRows];
  Walk<HD> wk;
  wk.init(tiles, segs, k, v, Hq, Hkv, HB, hblocks);
  const size_t at = (size_t)wk.qrow * Hq + wk.h;
  if (threadIdx.x < 4) sm.big[threadIdx.x] = 0;
  wk.issue(sm, wk.cur);
  f32x4 O[DB];
#pragma unroll
  for (int b = 0; b < DB; ++b) O[b] = f32x4{0.f, 0.f, 0.f, 0.f};
  // (a negative scale is a negative Q: the maximum is then that of the scaled scores, too)
  const float sign = scale < 0.f ? -1.f : 1.f;
  Softmax softmax(scale);
  // the current chunk on the fp32 instruction
  auto slow_step = [&](Softmax& sx, f32x4(&acc)[DB]) {
    if (wk.unseen(wk.cur)) return;
    f32x4 S[2];
    slow_dot<HD>(S, wk.keys(wk.cur), wk.kv_stride, wk.cur.n, q + at * HD);
#pragma unroll
    for (int b = 0; b < 2; ++b) S[b] *= sign;
    wk.mask_slow(S, wk.cur, kend, -INFINITY);
    sx.step(S, acc);
    slow_apply<HD>(acc, wk.values(wk.cur), wk.kv_stride, wk.cur.n, S);
  };
  bool q_planes;   // (a row without planes spoils its own column only)
  {
    OwnRows<HD> Q;
    q_planes = Q.load(q + at * HD, sign);
    async_wait_all();
    __syncthreads();   // (big[] is clear)
    wk.copy_ends(kendS[0], kend, wk.cur);
    typename ST::Split{}.all(sm, 0, 0);
    wk.have_nxt = wk.advance(wk.nxt);
    if (wk.have_nxt) wk.issue(sm, wk.nxt);
    const int rlo = PT::row_lane_off(), clo = PT::col_lane_off();

    for (int step = 0;; ++step) {
      const int buf = step & 1;
      __syncthreads();   // chunk `step` is split; everyone is done with the other buffer
      const int big = sm.big[step & 3];
      if (threadIdx.x == 0) sm.big[(step + 3) & 3] = 0;
      async_wait_all();   // the next chunk's raw rows (this wave's)
      typename Walk<HD>::Chunk nxt2;
      bool have_nxt2 = false;
      // behind the split: prepares the next chunk's mask, loads the one after it
      auto go_on = [&] {
        if (!wk.have_nxt) return;
        wk.copy_ends(kendS[buf ^ 1], kend, wk.nxt);
        have_nxt2 = wk.advance(nxt2);
        if (have_nxt2) wk.issue(sm, nxt2);
      };
      // The next chunk is split under the scores.  (Behind the last chunk what is there is
      // split once more, into a buffer nobody reads.)
      typename ST::Split sp;
      if (!wk.unseen(wk.cur)) {
        const uint16_t *Kt = sm.planes[buf][0] + rlo, *Vc = sm.planes[buf][1] + clo;
        f32x4 S[2];
        Pair ring[kRing];
#pragma unroll
        for (int i = 0; i < kAhead; ++i) ring[i] = row_pair<HD>(Kt, i);
        sp.init(sm, buf ^ 1);
        __builtin_amdgcn_sched_barrier(0);
        dot<HD>(S, ring, Kt, Q, [&](int m) { sp.step(m); }, [&](Pair& x, int i) { x = col_pair<HD>(Vc, i); });
        if (__builtin_amdgcn_readfirstlane(big) != 0) break;   // the whole block goes on below
        sp.finish(sm, step + 1);
        go_on();
        if (wk.cur.masked()) wk.mask(S, wk.cur, kendS[buf], -INFINITY);
        softmax.step(S, O);
        Frag f[kPlanes];
#pragma unroll
        for (int t = 0; t < 4; ++t) split_piece(S, f, t);
        bf16x8 P[kPlanes];
        operand(f, P);
        __builtin_amdgcn_sched_barrier(0);
        apply<HD>(O, ring, Vc, P, Nothing{}, [](Pair&, int) {});
      } else {
        if (__builtin_amdgcn_readfirstlane(big) != 0) break;
        sp.all(sm, buf ^ 1, step + 1);
        go_on();
      }
      if (!wk.have_nxt) goto done;
      wk.cur = wk.nxt;
      wk.nxt = nxt2;
      wk.have_nxt = have_nxt2;
    }
  }
  // a chunk without planes: this one and what follows on the fp32 instruction
  for (;;) {
    slow_step(softmax, O);
    if (!wk.have_nxt) break;
    wk.cur = wk.nxt;
    wk.have_nxt = wk.advance(wk.nxt);
  }
done:
  if (__builtin_amdgcn_ballot_w64(!q_planes) != 0) {   // rows without planes: the whole walk on the fp32 instruction
    Softmax again(scale);
    f32x4 acc[DB];
#pragma unroll
    for (int b = 0; b < DB; ++b) acc[b] = f32x4{0.f, 0.f, 0.f, 0.f};
    wk.it.init(segs, wk.tile);
    while (wk.advance(wk.cur)) slow_step(again, acc);
    if (!q_planes) {
      softmax = again;
#pragma unroll
      for (int b = 0; b < DB; ++b) O[b] = acc[b];
    }
  }
  const float lt = column_sum(softmax.sum), inv = 1.f / lt;
  const float lse_t = fmaf(softmax.m, fabsf(scale), logf(lt));   // (-infinity if every score is)
  if (wk.mine() && wk.lg == 0) lse[at] = lse_t;
  float t = 0.f;
#pragma unroll
  for (int b = 0; b < DB; ++b) {
#pragma unroll
    for (int e = 0; e < 4; ++e) t = fmaf(O[b][e], 0.f, t);
    O[b] *= inv;
  }
  // a row's output must not depend on keys it does not see, see row_by_keys
  t = column_sum(t);
  const bool spoilt = (t != 0.f) & (lt - lt == 0.f);   // (NaN compares unequal)
  if (__builtin_amdgcn_ballot_w64(spoilt) != 0) {
    f32x4 acc[DB];
    row_by_keys<HD>(wk.tile, segs, kend, wk.qrow, q + at * HD, wk.kbase, wk.vbase, wk.kv_stride, scale, lse_t, 1.f, acc);
    if (spoilt) {
#pragma unroll
      for (int b = 0; b < DB; ++b) O[b] = acc[b];
    }
  }
  if (wk.mine()) {
#pragma unroll
    for (int b = 0; b < DB; ++b) *reinterpret_cast<f32x4*>(o + at * HD + 16 * b + 4 * wk.lg) = O[b];
  }
}

// ---- dQ --------------------------------------------------------------------------
// With p.o != nullptr the launch also computes D for its rows and leaves it in `delta`.
template <int HD>
__global__ __launch_bounds__(kThreads) __attribute__((amdgpu_waves_per_eu(2, 2))) void dq_planes_kernel(F32BwdArgs p) {
  using PT = PlaneTile<HD>;
  using ST = Stream<HD>;
  constexpr int DB = PT::DB;
  __shared__ __attribute__((aligned(1024))) typename ST::Smem sm;
  __shared__ __attribute__((aligned(16))) int32_t kendS[2][kRows];
  const float scale = p.scale;
  Walk<HD> wk;
  wk.init(p.tiles, p.segs, p.k, p.v, p.Hq, p.Hkv, p.HB, p.hblocks);
  const size_t rh = (size_t)wk.qrow * p.Hq + wk.h;
  if (threadIdx.x < 4) sm.big[threadIdx.x] = 0;
  wk.issue(sm, wk.cur);
  float dlt;
  if (p.o != nullptr) {   // in the order of delta_f32_kernel
    dlt = 0.f;
#pragma unroll
    for (int j = 0; j < DB; ++j) {
      const f32x4 ox = *reinterpret_cast<const f32x4*>(p.o + rh * HD + 4 * wk.lg + 16 * j);
      const f32x4 dx = *reinterpret_cast<const f32x4*>(p.d_o + rh * HD + 4 * wk.lg + 16 * j);
#pragma unroll
      for (int e = 0; e < 4; ++e) dlt = fmaf(ox[e], dx[e], dlt);
    }
    dlt = column_sum(dlt);
    if (wk.lg == 0 && wk.mine()) p.delta[rh] = dlt;
  } else {
    dlt = p.delta[rh];
  }
  const float lse_t = p.lse[rh];
  f32x4 dQ[DB];
#pragma unroll
  for (int b = 0; b < DB; ++b) dQ[b] = f32x4{0.f, 0.f, 0.f, 0.f};
  // exponents of the probabilities
  auto exponents = [&](f32x4(&S)[2]) {
#pragma unroll
    for (int b = 0; b < 2; ++b)
#pragma unroll
      for (int e = 0; e < 4; ++e) S[b][e] = fmaf(S[b][e], scale, -lse_t);
  };
  {
    OwnRows<HD> Q, dO;
    const bool q_planes = Q.load(p.q + rh * HD), do_planes = dO.load(p.d_o + rh * HD);
    async_wait_all();
    __syncthreads();   // (big[] is clear)
    if (!(q_planes && do_planes)) sm.big[0] = 1;
    wk.copy_ends(kendS[0], p.kend, wk.cur);
    typename ST::Split{}.all(sm, 0, 0);
    wk.have_nxt = wk.advance(wk.nxt);
    if (wk.have_nxt) wk.issue(sm, wk.nxt);
    const int rlo = PT::row_lane_off(), clo = PT::col_lane_off();

    for (int step = 0;; ++step) {
      const int buf = step & 1;
      __syncthreads();   // chunk `step` is split; everyone is done with the other buffer
      const int big = sm.big[step & 3];
      if (threadIdx.x == 0) sm.big[(step + 3) & 3] = 0;
      async_wait_all();   // the next chunk's raw rows (this wave's)
      typename Walk<HD>::Chunk nxt2;
      bool have_nxt2 = false;
      // behind the split: prepares the next chunk's mask, loads the one after it
      auto go_on = [&] {
        if (!wk.have_nxt) return;
        wk.copy_ends(kendS[buf ^ 1], p.kend, wk.nxt);
        have_nxt2 = wk.advance(nxt2);
        if (have_nxt2) wk.issue(sm, nxt2);
      };
      typename ST::Split sp;   // of the next chunk, as in the forward kernel
      if (!wk.unseen(wk.cur)) {
        const uint16_t *Kt = sm.planes[buf][0] + rlo, *Vt = sm.planes[buf][1] + rlo, *Kc = sm.planes[buf][0] + clo;
        f32x4 S[2], dP[2];
        Pair ring[kRing];
#pragma unroll
        for (int i = 0; i < kAhead; ++i) ring[i] = row_pair<HD>(Kt, i);
        sp.init(sm, buf ^ 1);
        __builtin_amdgcn_sched_barrier(0);
        dot<HD>(S, ring, Kt, Q, [&](int m) { sp.step(m); }, [&](Pair& x, int i) { x = row_pair<HD>(Vt, i); });
        if (__builtin_amdgcn_readfirstlane(big) != 0) break;   // the whole block goes on below
        sp.finish(sm, step + 1);
        go_on();
        exponents(S);
        if (wk.cur.masked()) wk.mask(S, wk.cur, kendS[buf], -INFINITY);
        // two probabilities with every twelve (head_dim 64: six) products
        PairSplit ps;
        constexpr int kPer = kProducts<HD> / 4;
        __builtin_amdgcn_sched_barrier(0);
        dot<HD>(dP, ring, Vt, dO,
                [&](int m) {
                  const int t = m / kPer, s = m % kPer;
                  float x[2] = {S[t >> 1][2 * (t & 1)], S[t >> 1][2 * (t & 1) + 1]};
                  if (s == 0) { ps.x0 = x[0]; ps.x1 = x[1]; }
                  if (s < 6) ps.exp_step(s);
                  if (s == 5) { S[t >> 1][2 * (t & 1)] = ps.x0; S[t >> 1][2 * (t & 1) + 1] = ps.x1; }
                },
                [&](Pair& x, int i) { x = col_pair<HD>(Kc, i); });
#pragma unroll
        for (int b = 0; b < 2; ++b) S[b] *= dP[b] - dlt;   // dS
        Frag f[kPlanes];
#pragma unroll
        for (int t = 0; t < 4; ++t) split_piece(S, f, t);
        bf16x8 dS[kPlanes];
        operand(f, dS);
        __builtin_amdgcn_sched_barrier(0);
        apply<HD>(dQ, ring, Kc, dS, Nothing{}, [](Pair&, int) {});
      } else {
        if (__builtin_amdgcn_readfirstlane(big) != 0) break;
        sp.all(sm, buf ^ 1, step + 1);
        go_on();
      }
      if (!wk.have_nxt) goto done;
      wk.cur = wk.nxt;
      wk.nxt = nxt2;
      wk.have_nxt = have_nxt2;
    }
  }
  // a chunk or a row without planes: this one and what follows on the fp32 instruction
  for (;;) {
    if (!wk.unseen(wk.cur)) {
      f32x4 S[2], dP[2];
      slow_dot<HD>(S, wk.keys(wk.cur), wk.kv_stride, wk.cur.n, p.q + rh * HD);
      slow_dot<HD>(dP, wk.values(wk.cur), wk.kv_stride, wk.cur.n, p.d_o + rh * HD);
      exponents(S);
      wk.mask_slow(S, wk.cur, p.kend, -INFINITY);
#pragma unroll
      for (int b = 0; b < 2; ++b)
#pragma unroll
        for (int e = 0; e < 4; ++e) S[b][e] = exp_f32(S[b][e]) * (dP[b][e] - dlt);
      slow_apply<HD>(dQ, wk.keys(wk.cur), wk.kv_stride, wk.cur.n, S);
    }
    if (!wk.have_nxt) break;
    wk.cur = wk.nxt;
    wk.have_nxt = wk.advance(wk.nxt);
  }
done:
  if (wk.mine()) {
#pragma unroll
    for (int b = 0; b < DB; ++b) *reinterpret_cast<f32x4*>(p.dq + rh * HD + 16 * b + 4 * wk.lg) = dQ[b] * scale;
  }
}

// ---- dK/dV -------------------------------------------------------------------------
// Wave = 16 keys, tiles of 128.  Q and dO of the rows that can see the keys are streamed in
// iterations of 32 rows of one q head, heads innermost, last chunk first.  Long walks
// are cut into items that write partial sums.
template <int HD>
__global__ __launch_bounds__(kThreads) __attribute__((amdgpu_waves_per_eu(2, 2))) void dkdv_planes_kernel(F32BwdArgs p) {
  using PT = PlaneTile<HD>;
  using ST = Stream<HD>;
  constexpr int DB = PT::DB, kKeys = 16 * kWaves;
  __shared__ __attribute__((aligned(1024))) typename ST::Smem sm;
  __shared__ __attribute__((aligned(256))) float stat[4][2][64];   // ring over the iterations: lse, delta of 32 rows, twice
  const int Hq = p.Hq, Hkv = p.Hkv;
  const float scale = p.scale;

  const KvItem tile = p.items[blockIdx.x / Hkv];
  const int g = blockIdx.x % Hkv, G = Hq / Hkv;
  const int w = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  int kcol, my_kend;   // this lane's key
  {
    kcol = tile.k0 + 16 * w + (threadIdx.x & 15);
    my_kend = kcol < tile.k1 ? p.kend[kcol] : 0;   // padded columns see nothing
  }
  // rows [wave_lo, wave_hi) are the only ones any of this wave's keys can see
  int wave_hi = my_kend;
#pragma unroll
  for (int off = 8; off >= 1; off >>= 1) wave_hi = max(wave_hi, __shfl_xor(wave_hi, off));
  wave_hi = __builtin_amdgcn_readfirstlane(wave_hi);
  const int wave_lo = tile.k0 + 16 * w;

  const size_t q_stride = (size_t)Hq * HD;
  const int n_chunks = (tile.q_end - tile.q_begin + kRows - 1) / kRows;
  const int total = tile.it_end;
  // iteration -> first row and head: `it` = chunk * G + head, last chunk first
  struct Iter {
    int r0, head;
    __device__ __forceinline__ void next(int G) {
      if (++head == G) {
        head = 0;
        r0 -= kRows;
      }
    }
  };
  auto issue = [&](int it, const Iter& x) {
    const int nv = min(kRows, tile.q_end - x.r0), h = g * G + x.head;
    if (w == 0) {
      const uint32_t off = (uint32_t)min((int)threadIdx.x & 31, nv - 1) * (uint32_t)Hq;
      row_async_load(stat[it & 3][0], p.lse + (size_t)x.r0 * Hq + h, off);
      row_async_load(stat[it & 3][1], p.delta + (size_t)x.r0 * Hq + h, off);
    }
    const size_t at = (size_t)x.r0 * q_stride + (size_t)h * HD;
    ST::issue(sm, p.q + at, p.d_o + at, (uint32_t)q_stride * 4, nv);
  };
  if (threadIdx.x < 4) sm.big[threadIdx.x] = 0;
  int it = tile.it_begin;   // (an item has at least one iteration)
  Iter cur{tile.q_begin + (n_chunks - 1 - it / G) * kRows, it % G}, ahead = cur;   // ahead: the one to be loaded next
  issue(it, ahead);
  ahead.next(G);
  f32x4 dK[DB], dV[DB];
#pragma unroll
  for (int b = 0; b < DB; ++b) dK[b] = dV[b] = f32x4{0.f, 0.f, 0.f, 0.f};
  const size_t own = ((size_t)min(kcol, tile.k1 - 1) * Hkv + g) * HD;
  // exponents of the probabilities; rows that do not see the key get probability 0
  auto exponents = [&](f32x4(&S)[2], const Iter& x, const f32x4(&ls)[2]) {
    const int lg = (threadIdx.x >> 4) & 3;
#pragma unroll
    for (int b = 0; b < 2; ++b)
#pragma unroll
      for (int e = 0; e < 4; ++e) S[b][e] = fmaf(S[b][e], scale, -ls[b][e]);
    const int nr = min(kRows, tile.q_end - x.r0);
    if (!(x.r0 >= tile.k1 && x.r0 + kRows <= tile.q_full_end)) {
      // bounds of the visible rows of this lane's key, relative to this lane's first row
      const int lo = kcol - x.r0 - 4 * lg, hi = min(my_kend - x.r0, nr) - 4 * lg;
#pragma unroll
      for (int b = 0; b < 2; ++b)
#pragma unroll
        for (int e = 0; e < 4; ++e)
          S[b][e] = ((16 * b + e >= lo) & (16 * b + e < hi)) ? S[b][e] : -INFINITY;
    }
  };
  auto visible = [&](const Iter& x) { return min(x.r0 + kRows, tile.q_end) > wave_lo && x.r0 < wave_hi; };
  {
    OwnRows<HD> K, V;
    const bool k_planes = K.load(p.k + own), v_planes = V.load(p.v + own);
    async_wait_all();
    __syncthreads();   // (big[] is clear)
    if (!(k_planes && v_planes)) sm.big[it & 3] = 1;
    typename ST::Split{}.all(sm, it & 1, it);
    if (it + 1 < total) issue(it + 1, ahead);
    ahead.next(G);
    const int rlo = PT::row_lane_off(), clo = PT::col_lane_off();

    for (;;) {
      const int buf = it & 1;
      __syncthreads();   // iteration `it` is split; everyone is done with the other buffer
      const int big = sm.big[it & 3];
      if (threadIdx.x == 0) sm.big[(it + 3) & 3] = 0;
      async_wait_all();   // the next iteration's raw rows (this wave's)
      typename ST::Split sp;   // of the next iteration, as in the forward kernel
      if (visible(cur)) {
        const uint16_t *Qt = sm.planes[buf][0] + rlo, *Qc = sm.planes[buf][0] + clo;
        const uint16_t *dOt = sm.planes[buf][1] + rlo, *dOc = sm.planes[buf][1] + clo;
        // the statistics of this lane's rows, lse or delta
        auto stats = [&](int i, f32x4(&x)[2]) {
#pragma unroll
          for (int b = 0; b < 2; ++b)
            x[b] = *reinterpret_cast<const f32x4*>(&stat[it & 3][i][16 * b + 4 * ((threadIdx.x >> 4) & 3)]);
        };
        f32x4 S[2], dP[2], x4[2];
        Pair ring[kRing];
#pragma unroll
        for (int i = 0; i < kAhead; ++i) ring[i] = row_pair<HD>(Qt, i);
        sp.init(sm, buf ^ 1);
        __builtin_amdgcn_sched_barrier(0);
        dot<HD>(S, ring, Qt, K, [&](int m) { sp.step(m); }, [&](Pair& x, int i) { x = row_pair<HD>(dOt, i); });
        if (__builtin_amdgcn_readfirstlane(big) != 0) break;   // the whole block goes on below
        sp.finish(sm, it + 1);
        if (it + 2 < total) issue(it + 2, ahead);
        stats(0, x4);
        exponents(S, cur, x4);
        // two probabilities and their planes with every twelve (head_dim 64: six) products
        Frag f[kPlanes];
        bf16x8 P[kPlanes], dS[kPlanes];
        PairSplit ps;
        constexpr int kPer = kProducts<HD> / 4, kDo = 12 / kPer;   // products per pair of numbers, steps per product
        __builtin_amdgcn_sched_barrier(0);
        dot<HD>(dP, ring, dOt, V,
                [&](int m) {
                  const int t = m / kPer;
#pragma unroll
                  for (int s = m % kPer * kDo; s < (m % kPer + 1) * kDo; ++s) {
                    if (s == 0) { ps.x0 = S[t >> 1][2 * (t & 1)]; ps.x1 = S[t >> 1][2 * (t & 1) + 1]; }
                    if (s < 6) ps.exp_step(s);
                    else ps.split_step(s - 6, f, t);
                    if (s == 5) { S[t >> 1][2 * (t & 1)] = ps.x0; S[t >> 1][2 * (t & 1) + 1] = ps.x1; }
                  }
                },
                [&](Pair& x, int i) { x = col_pair<HD>(dOc, i); });
        operand(f, P);
        stats(1, x4);
        __builtin_amdgcn_sched_barrier(0);
        // ... and of dS
        apply<HD>(dV, ring, dOc, P,
                  [&](int m) {
                    const int t = m / kPer, b = t >> 1, e = 2 * (t & 1);
#pragma unroll
                    for (int s = m % kPer * kDo; s < (m % kPer + 1) * kDo; ++s) {
                      if (s == 0) { ps.x0 = dP[b][e] - x4[b][e]; ps.x1 = dP[b][e + 1] - x4[b][e + 1]; }
                      if (s == 1) { ps.x0 *= S[b][e]; ps.x1 *= S[b][e + 1]; }
                      if (s >= 2 && s < 8) ps.split_step(s - 2, f, t);
                    }
                  },
                  [&](Pair& x, int i) { x = col_pair<HD>(Qc, i); });
        operand(f, dS);
        __builtin_amdgcn_sched_barrier(0);
        apply<HD>(dK, ring, Qc, dS, Nothing{}, [](Pair&, int) {});
      } else {
        if (__builtin_amdgcn_readfirstlane(big) != 0) break;
        sp.all(sm, buf ^ 1, it + 1);
        if (it + 2 < total) issue(it + 2, ahead);
      }
      ahead.next(G);
      cur.next(G);
      if (++it >= total) goto done;
    }
  }
  // an iteration or a key without planes: this one and what follows on the fp32 instruction
  for (; it < total; ++it, cur.next(G)) {
    if (!visible(cur)) continue;
    const int lg = (threadIdx.x >> 4) & 3, nr = min(kRows, tile.q_end - cur.r0), h = g * G + cur.head;
    const size_t at = (size_t)cur.r0 * q_stride + (size_t)h * HD;
    f32x4 S[2], dP[2], ls[2], dl[2];
#pragma unroll
    for (int b = 0; b < 2; ++b)
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        const size_t r = (size_t)(cur.r0 + min(16 * b + 4 * lg + e, nr - 1)) * Hq + h;
        ls[b][e] = p.lse[r];
        dl[b][e] = p.delta[r];
      }
    slow_dot<HD>(S, p.q + at, q_stride, nr, p.k + own);
    slow_dot<HD>(dP, p.d_o + at, q_stride, nr, p.v + own);
    exponents(S, cur, ls);
#pragma unroll
    for (int b = 0; b < 2; ++b)
#pragma unroll
      for (int e = 0; e < 4; ++e) S[b][e] = exp_f32(S[b][e]);
    slow_apply<HD>(dV, p.d_o + at, q_stride, nr, S);
#pragma unroll
    for (int b = 0; b < 2; ++b) S[b] *= dP[b] - dl[b];
    slow_apply<HD>(dK, p.q + at, q_stride, nr, S);
  }
done:
  // lane (n, lg) holds columns 16 * b + 4 * lg .. + 3 of its key
#pragma unroll
  for (int half = 0; half < 2; ++half) {
    const int lg = (threadIdx.x >> 4) & 3;
    const float f = half == 0 ? scale : 1.f;
    float* dst = tile.slot >= 0 ? p.partial + ((size_t)tile.slot * Hkv + g) * (2 * kKeys * HD) +
                                      (size_t)(half * kKeys + 16 * w + (threadIdx.x & 15)) * HD
                                : (half == 0 ? p.dk : p.dv) + ((size_t)kcol * Hkv + g) * HD;
    if (tile.slot < 0 && kcol >= tile.k1) continue;
#pragma unroll
    for (int b = 0; b < DB; ++b) {
      f32x4* at = reinterpret_cast<f32x4*>(dst + 16 * b + 4 * lg);
      f32x4 r = half == 0 ? dK[b] : dV[b];
      if (tile.slot < 0) {
        r *= f;
        if (p.accumulate) r += *at;   // a segment call (this block is the only owner of the key in the launch)
      }
      *at = r;
    }
  }
}

}  // namespace

int launch_fwd_f32_planes(const LaunchArgs& a, size_t blocks) {
  auto kernel = a.p.head_dim == 128 ? fwd_planes_kernel<128> : fwd_planes_kernel<64>;
  const QueryTiles& qt = a.sched->forward_tiles();
  launch(a, true, kernel, blocks, kThreads, qt.d_q_tiles, qt.d_segs, a.d_kend, (const float*)a.q,
         (const float*)a.k, (const float*)a.v, (float*)a.o_out, a.lse_out, a.p.n_q_heads, a.p.n_kv_heads, a.tc.hb,
         a.tc.hblocks, a.p.softmax_scale);
  return launch_status(__func__);
}
int launch_dq_f32_planes(const LaunchArgs& a, const F32BwdArgs& args, size_t blocks) {
  launch(a, false, a.p.head_dim == 128 ? dq_planes_kernel<128> : dq_planes_kernel<64>, blocks, kThreads, args);
  return launch_status(__func__);
}
int launch_dkdv_f32_planes(const LaunchArgs& a, const F32BwdArgs& args, size_t blocks) {
  launch(a, a.sched->kv_reduce.empty(), a.p.head_dim == 128 ? dkdv_planes_kernel<128> : dkdv_planes_kernel<64>, blocks,
         kThreads, args);
  return launch_status(__func__);
}

}  // namespace dta
