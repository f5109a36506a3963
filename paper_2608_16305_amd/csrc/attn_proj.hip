// The attention by per-query projected vectors, forward and backward (see attn_proj.h for the algebra).
//
// Forward, one kernel: a block owns 16 or 32 queries.  The query projection, u_h = W_k,h^T q_h, the value
// projection of the weighted row sums and the three merge layers run as MFMA products over the block's
// rows in LDS (weights packed in fragment order, read from L2); between them each wave walks the slots of
// its queries.
// Backward, one kernel: the merge layers' data gradients, dc_h = W_v,h^T da_h, the slots again (dp_j =
// dc . x_j, ds_j = p_j (dp_j - dc . c), dx_j = sum_h p_j dc_h + ds_j u_h, du_h = sum_j ds_j x_j), then
// dq_h = W_k,h du_h and the query rows' gradient.  The weight gradients are reductions over the queries.
//
// Measured against a key/value product over every slot (its rows gathered to memory, the softmax and its
// backward in kernels of their own), 60,000 events, 20 slots, width 100, 16 edge features, 2 heads:
// forward 3340 -> 1255 us, backward 4710 -> 2109 us; bfloat16, no edge features, both: 6290 -> 2526 us; 4,000
// events, 10 slots: backward 321 -> 210 us; 600 events, 172 edge features: forward 93 -> 59 us.
#include <algorithm>
#include <cfloat>

#include "gemm.h"
#include "attn_proj.h"
#include "bf16_split.h"
#include "dw_split.h"

namespace mtgnn {

namespace {

size_t a256(size_t x) { return (x + 255) & ~size_t(255); }
int odd4(int x) { return ((x + 3) / 4 % 2 ? (x + 3) / 4 : (x + 3) / 4 + 1) * 4; }

constexpr int PW = 8;          // waves per block
constexpr int PT = 64 * PW;    // threads per block
constexpr int TG_CHUNKS = 64;  // chunks of the time encoder's block partials (first reduction)

// ---------------------------------------------------------------- time encoding

// cos and sin of a time argument.  n = rint(2 x / pi) and r = x - n pi / 2, pi / 2 as two floats: n and x up to
// 2^20 make x - n PIO2_HI a multiple of 2^-23 below 1 (of 2^-24 for |x| < 1), so that product and difference are
// exact, and the second product rounds r once; rlo is that rounding's error.  On |r| <= pi / 4 + 0.04 (the
// rounding of 2 x / pi moves n near its midpoints), sin r = r + r s P(s) and cos r = 1 + s Q(s) with s = r r (own
// minimax fits, 5e-9 and 4e-9 absolute), and n's two low bits choose between them and the sign.  Measured against
// 64 bits over |x| <= 2^20: 7.1e-8 at most and 1.57e-8 rms, cosine and sine (the library's: 7.2e-8 and 1.80e-8;
// without rlo, as the bfloat16 mode takes it, whose cosines are rounded again: 7.3e-8 and 1.71e-8).
// Larger arguments are reduced with 1 / (2 pi) in three doubles.  The library's functions keep that reduction's
// registers in every loop that calls them: the slots evaluate one cosine per time column.
constexpr float ENC_MAX = 1048576.f;
constexpr float PIO2_INV = 0.636619747f, PIO2_HI = 1.57079637f, PIO2_LO = -4.37113883e-08f;
constexpr float ROUND_F = 12582912.f;              // 1.5 2^23: adding it rounds to a whole number, in the low bits
constexpr double ROUND_D = 6755399441055744.;      // 1.5 2^52

struct Quarter {   // x = n pi / 2 + r + rlo
  float r, rlo;
  uint32_t n;   // the low bits count
};
__device__ __forceinline__ Quarter quarter(float x) {
#pragma clang fp contract(off)
  const float m = fmaf(x, PIO2_INV, ROUND_F), n = m - ROUND_F;
  const float d = fmaf(n, -PIO2_HI, x), r = fmaf(n, -PIO2_LO, d);
  return Quarter{r, fmaf(n, -PIO2_LO, d - r), __float_as_uint(m)};
}
constexpr double INV_2PI_1 = 0.15915494309189535, INV_2PI_2 = -9.839338337591243e-18, INV_2PI_3 = -5.360718141446502e-34;
// x / (2 pi) less the nearest whole number, for any finite x: every product's fraction (and its rounding error's)
// summed.
__device__ __forceinline__ double turn_wide(float x) {
#pragma clang fp contract(off)
  const double xd = x;
  const double p1 = xd * INV_2PI_1, r1 = fma(xd, INV_2PI_1, -p1);
  const double p2 = xd * INV_2PI_2, r2 = fma(xd, INV_2PI_2, -p2);
  const double p3 = xd * INV_2PI_3;
  const double s = (p1 - rint(p1)) + ((r1 - rint(r1)) + ((p2 - rint(p2)) + ((r2 - rint(r2)) + (p3 - rint(p3)))));
  return s - rint(s);
}
__device__ __forceinline__ Quarter quarter_far(float x) {
#pragma clang fp contract(off)
  const double t = 4. * turn_wide(x), m = t + ROUND_D, r = (t - (m - ROUND_D)) * 1.570796326794896619231;
  return Quarter{(float)r, (float)(r - (double)(float)r), (uint32_t)__double2loint(m)};
}
__device__ __forceinline__ float flip_sign(float v, uint32_t bit31) {
  return __uint_as_float(__float_as_uint(v) ^ (bit31 & 0x80000000u));
}
template <bool SIN, bool LO>
__device__ __forceinline__ void cos_sin(const Quarter& q, float& c, float& s) {
  const float z = q.r * q.r;
  const float P = fmaf(z, fmaf(z, -0.000194556327f, 0.00833164621f), -0.166666448f);
  const float Q = fmaf(z, fmaf(z, fmaf(z, 2.43428403e-05f, -0.00138862419f), 0.0416666046f), -0.5f);
  const float ys = LO ? q.r + fmaf(q.r * z, P, q.rlo) : fmaf(q.r * z, P, q.r);
  const float yc = LO ? 1.f + fmaf(z, Q, -(q.r * q.rlo)) : fmaf(z, Q, 1.f);
  const bool odd = q.n & 1u;
  c = flip_sign(odd ? ys : yc, (q.n << 30) + 0x40000000u);   // n = 1, 2: negative
  if (SIN) s = flip_sign(odd ? yc : ys, q.n << 30);          // n = 2, 3
}
// The correctly rounded cosine that a rounding to bfloat16 is decided on near its midpoints (see
// cos_for_bf16): the Taylor series of sin on a quarter turn in double (3e-16).
__device__ __forceinline__ float wide_cos(float arg) {
  const double t = 6.283185307179586476925 * (0.25 - fabs(turn_wide(arg))), s = t * t;
  double p = -1. / 121645100408832000.;
  p = fma(s, p, 1. / 355687428096000.);
  p = fma(s, p, -1. / 1307674368000.);
  p = fma(s, p, 1. / 6227020800.);
  p = fma(s, p, -1. / 39916800.);
  p = fma(s, p, 1. / 362880.);
  p = fma(s, p, -1. / 5040.);
  p = fma(s, p, 1. / 120.);
  p = fma(s, p, -1. / 6.);
  return (float)fma(t, s * p, t);
}
__device__ __forceinline__ float2 round2_bf16(float2 v) {   // to the nearest bfloat16 values
  const uint32_t p = cvt2_bf16(v.x, v.y);
  return make_float2(lo_bf16(p), hi_bf16(p));
}
// cos and sin (optional) of two time columns of a slot.
template <bool BF, bool SIN>
__device__ __forceinline__ void encode(float2 w, float2 b, float delta, float2& c, float2& s) {
  const float a0 = time_arg(w.x, delta, b.x), a1 = time_arg(w.y, delta, b.y);
  Quarter q0 = quarter(a0), q1 = quarter(a1);
  if (fmaxf(fabsf(a0), fabsf(a1)) > ENC_MAX) {
    q0 = quarter_far(a0);
    q1 = quarter_far(a1);
  }
  cos_sin<SIN, !BF>(q0, c.x, s.x);
  cos_sin<SIN, !BF>(q1, c.y, s.y);
  if constexpr (BF) {
    auto near_tie = [](float y) {
      const int low = (int)(__float_as_uint(y) & 0xFFFFu) - 0x8000;
      return low >= -16 && low <= 16;
    };
    const bool t0 = near_tie(c.x), t1 = near_tie(c.y);
    if (t0 || t1) {   // rare
      c.x = t0 ? wide_cos(a0) : c.x;
      c.y = t1 ? wide_cos(a1) : c.y;
    }
    c = make_float2(round_to_bf16(c.x), round_to_bf16(c.y));
  }
}

// ---------------------------------------------------------------- wave helpers

template <int CTRL>
__device__ __forceinline__ float dpp(float v) {
  return __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(v), CTRL, 0xf, 0xf, true));
}
__device__ __forceinline__ float add_xor32(float v) {   // v + the other half-wave's v
  const auto r = __builtin_amdgcn_permlane32_swap(__float_as_uint(v), __float_as_uint(v), false, false);
  return __uint_as_float(r[0]) + __uint_as_float(r[1]);
}
// Sum over each half-wave's 32 lanes, in every lane: within quads, eights and rows by lane swaps in the
// adder, then across the row pair.
__device__ __forceinline__ float half_sum(float v) {
  v += dpp<0xB1>(v);    // quad_perm 1,0,3,2
  v += dpp<0x4E>(v);    // quad_perm 2,3,0,1
  v += dpp<0x141>(v);   // row_half_mirror
  v += dpp<0x140>(v);   // row_mirror
  const auto r = __builtin_amdgcn_permlane16_swap(__float_as_uint(v), __float_as_uint(v), false, false);
  return __uint_as_float(r[0]) + __uint_as_float(r[1]);
}

// Both heads' 64-lane sums at once: half-wave h of the result holds the sum of head h's values (H = 1:
// both halves the one sum).
template <int H>
__device__ __forceinline__ float heads_sum(const float (&v)[H]) {
  if constexpr (H == 1) {
    return half_sum(add_xor32(v[0]));
  } else {
    const auto r = __builtin_amdgcn_permlane32_swap(__float_as_uint(v[0]), __float_as_uint(v[1]), false, false);
    return half_sum(__uint_as_float(r[0]) + __uint_as_float(r[1]));
  }
}
__device__ __forceinline__ float lane_value(float v, int lane) {   // wave-uniform lane: a scalar
  return __int_as_float(__builtin_amdgcn_readlane(__float_as_int(v), lane));
}

__device__ __forceinline__ float dot2(float2 a, float2 b, float acc) { return fmaf(a.y, b.y, fmaf(a.x, b.x, acc)); }
__device__ __forceinline__ void axpy2(float s, float2 x, float2& y) {
  y.x = fmaf(s, x.x, y.x);
  y.y = fmaf(s, x.y, y.y);
}
__device__ __forceinline__ float2 scale2(float2 v, float s) { return make_float2(v.x * s, v.y * s); }
constexpr float4 Z4 = {0.f, 0.f, 0.f, 0.f};
constexpr float2 Z2 = {0.f, 0.f};

// Two or four consecutive columns of a stored row; al: the group is aligned to its size.
__device__ __forceinline__ float2 ld2(const float* p, bool al) {
  return al ? *(const float2*)p : make_float2(p[0], p[1]);
}
__device__ __forceinline__ float2 ld2(const uint16_t* p, bool al) {
  if (!al) return make_float2(bf16_to_f32(p[0]), bf16_to_f32(p[1]));
  const uint32_t u = *(const uint32_t*)p;
  return make_float2(__uint_as_float(u << 16), __uint_as_float(u & 0xffff0000u));
}
__device__ __forceinline__ float4 ld4(const float* p, bool al) {
  return al ? *(const float4*)p : make_float4(p[0], p[1], p[2], p[3]);
}
__device__ __forceinline__ float4 ld4(const uint16_t* p, bool al) {
  if (!al) return make_float4(bf16_to_f32(p[0]), bf16_to_f32(p[1]), bf16_to_f32(p[2]), bf16_to_f32(p[3]));
  const uint2 u = *(const uint2*)p;
  return make_float4(__uint_as_float(u.x << 16), __uint_as_float(u.x & 0xffff0000u), __uint_as_float(u.y << 16),
                     __uint_as_float(u.y & 0xffff0000u));
}
__device__ __forceinline__ void st4(float* p, float4 v) { *(float4*)p = v; }
__device__ __forceinline__ void st2(float* p, float2 v) { *(float2*)p = v; }
__device__ __forceinline__ void st2(uint16_t* p, float2 v) {   // values that are bfloat16 already
  *(uint32_t*)p = (__float_as_uint(v.x) >> 16) | (__float_as_uint(v.y) & 0xffff0000u);
}

// Slot rows that another kernel reads later: past the caches, which the gathered rows and weights keep.  60,000
// events, 20 slots: forward 1312 -> 1256 us; bfloat16, both directions, 2407 -> 2378 us.
__device__ __forceinline__ void st2_stream(float* p, float2 v) {
  __builtin_nontemporal_store(f32x2_t{v.x, v.y}, (f32x2_t*)p);
}
__device__ __forceinline__ void st2_stream(uint16_t* p, float2 v) {   // values that are bfloat16 already
  __builtin_nontemporal_store((__float_as_uint(v.x) >> 16) | (__float_as_uint(v.y) & 0xffff0000u), (uint32_t*)p);
}

// ---------------------------------------------------------------- packed products

// A packed weight: unit u (a 16-column output tile of one head) is nch chunks of 64 lanes x 4 floats.  A
// whole chunk c holds for lane l the weights of column l % 16 and k = 16 c + 4 (l / 16) + 0..3; the tail
// chunk (K % 16 != 0) those of k = 16 c + 4 e + l / 16, e = 0..3, so that it takes ceil(K % 16 / 4) MFMAs.
// bfloat16 weights stay as they are: chunks of 32, lane l of chunk c holds k = 32 c + 8 (l / 16) + 0..7.
__host__ __device__ inline int pk_chunks(int K) { return (K + 15) / 16; }
template <typename T>
__host__ __device__ inline int pk_unit(int K) {   // floats of a unit
  return 256 * (sizeof(T) == 2 ? (K + 31) / 32 : pk_chunks(K));
}

// One segment of a product: acc += X (16 RT rows in LDS, row stride ldx) times the unit at w.  Two chains
// of at most 32 products each, folded into a running total: the MFMAs of a chunk do not all wait for each
// other, and the sums round like short ones (with one chain over the 200-long sums of the value
// projection, results rounded to bfloat16 the other way often enough to raise that mode's error by a third).
template <int RT>
struct Acc {
  f32x4 v[RT][2], total[RT];
  __device__ __forceinline__ Acc() {
#pragma unroll
    for (int r = 0; r < RT; ++r) {
      v[r][0] = v[r][1] = total[r] = f32x4{0.f, 0.f, 0.f, 0.f};
    }
  }
  __device__ __forceinline__ void fold() {
#pragma unroll
    for (int r = 0; r < RT; ++r) {
      total[r] += v[r][0] + v[r][1];
      v[r][0] = v[r][1] = f32x4{0.f, 0.f, 0.f, 0.f};
    }
  }
};
template <int RT>
__device__ __forceinline__ void mma_segment(const float* X, int ldx, const float* __restrict__ w, int K,
                                            Acc<RT>& acc) {
  const int lane = threadIdx.x & 63, fr = lane & 15, fg = lane >> 4;
  const int kc = K >> 4, nch = pk_chunks(K), ts = ((K & 15) + 3) >> 2;
  const float4* wl = (const float4*)w + lane;
  const float* xr = X + fr * ldx;
  float4 b0[4], b1[4];
  auto load = [&](float4 (&b)[4], int c0) {
#pragma unroll
    for (int i = 0; i < 4; ++i) b[i] = wl[64 * min(c0 + i, nch - 1)];
  };
  auto mma = [&](float4 (&b)[4], int c0) {
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      const int c = c0 + i;
      if (c < kc) {
#pragma unroll
        for (int r = 0; r < RT; ++r) {
          const float4 a = *(const float4*)(xr + 16 * r * ldx + 16 * c + 4 * fg);
          acc.v[r][0] = __builtin_amdgcn_mfma_f32_16x16x4f32(a.x, b[i].x, acc.v[r][0], 0, 0, 0);
          acc.v[r][1] = __builtin_amdgcn_mfma_f32_16x16x4f32(a.y, b[i].y, acc.v[r][1], 0, 0, 0);
          acc.v[r][0] = __builtin_amdgcn_mfma_f32_16x16x4f32(a.z, b[i].z, acc.v[r][0], 0, 0, 0);
          acc.v[r][1] = __builtin_amdgcn_mfma_f32_16x16x4f32(a.w, b[i].w, acc.v[r][1], 0, 0, 0);
        }
      } else if (c < nch) {
        const float be[4] = {b[i].x, b[i].y, b[i].z, b[i].w};
#pragma unroll
        for (int e = 0; e < 4; ++e)
          if (e < ts) {
#pragma unroll
            for (int r = 0; r < RT; ++r)
              acc.v[r][e & 1] = __builtin_amdgcn_mfma_f32_16x16x4f32(
                  xr[16 * r * ldx + 16 * c + 4 * e + fg], be[e], acc.v[r][e & 1], 0, 0, 0);
          }
      }
    }
  };
  load(b0, 0);
  for (int c0 = 0; c0 < nch; c0 += 8) {
    if (c0 + 4 < nch) load(b1, c0 + 4);
    mma(b0, c0);
    acc.fold();
    if (c0 + 4 < nch) {
      if (c0 + 8 < nch) load(b0, c0 + 8);
      mma(b1, c0 + 4);
      acc.fold();
    }
  }
}

// The same for bfloat16 weights, float32 rows as the sum of NP bfloat16 parts (1: rows that hold bfloat16
// values).  K % 4 == 0: a lane's eight columns end on a group of four, and those past K count as zero.  The
// products are exact and an instruction rounds once every eight of them: the float32 instructions round once a
// product and take 16 (NP = 1) or 5 (NP = 3) times the matrix time.  60,000 events, 20 slots, both directions:
// 2795 -> 2514 us.
template <int RT, int NP>
__device__ __forceinline__ void mma_segment_bf16(const float* X, int ldx, const float* __restrict__ w, int K,
                                                 Acc<RT>& acc) {
  const int lane = threadIdx.x & 63, fr = lane & 15, fg = lane >> 4;
  const int nch = (K + 31) >> 5;
  const u32x4_t* wl = (const u32x4_t*)w + lane;
  const float* xr = X + fr * ldx;
  u32x4_t b0[2], b1[2];
  auto load = [&](u32x4_t (&b)[2], int c0) {
#pragma unroll
    for (int i = 0; i < 2; ++i) b[i] = wl[64 * min(c0 + i, nch - 1)];
  };
  auto mma = [&](u32x4_t (&b)[2], int c0) {
#pragma unroll
    for (int i = 0; i < 2; ++i) {
      const int k = 32 * (c0 + i) + 8 * fg;
      if (c0 + i < nch) {
#pragma unroll
        for (int r = 0; r < RT; ++r) {
          const float* xk = xr + 16 * r * ldx;
          const f32x4 z = {0.f, 0.f, 0.f, 0.f};
          f32x4 u = *(const f32x4*)(xk + min(k, K - 4)), v = *(const f32x4*)(xk + min(k + 4, K - 4));
          u = k < K ? u : z;
          v = k + 4 < K ? v : z;
          const float x[8] = {u[0], u[1], u[2], u[3], v[0], v[1], v[2], v[3]};
          const bf16x8_t wb = __builtin_bit_cast(bf16x8_t, b[i]);
          if constexpr (NP == 3) {
            const Bf16Parts a = split_bf16(x);
            acc.v[r][1] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(a.lo, wb, acc.v[r][1], 0, 0, 0);
            acc.v[r][0] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(a.hi, wb, acc.v[r][0], 0, 0, 0);
            acc.v[r][1] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(a.mid, wb, acc.v[r][1], 0, 0, 0);
          } else {
            acc.v[r][0] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(round8_bf16(x), wb, acc.v[r][0], 0, 0, 0);
          }
        }
      }
    }
  };
  load(b0, 0);
  for (int c0 = 0; c0 < nch; c0 += 4) {
    if (c0 + 2 < nch) load(b1, c0 + 2);
    mma(b0, c0);
    if (c0 + 2 < nch) {
      if (c0 + 4 < nch) load(b0, c0 + 4);
      mma(b1, c0 + 2);
    }
  }
  acc.fold();
}
// One segment for weights stored as T.
template <typename T, int RT, int NP>
__device__ __forceinline__ void segment(const float* X, int ldx, const float* __restrict__ w, int K, Acc<RT>& acc) {
  if constexpr (sizeof(T) == 2) mma_segment_bf16<RT, NP>(X, ldx, w, K, acc);
  else mma_segment<RT>(X, ldx, w, K, acc);
}

// Y = X W^T for `heads` heads of `tiles` 16-column tiles each (head h reads X + h xh), without each head's tiles
// lo .. lo + skip - 1; the block's waves take the units in turn.  f(head, row, column in the head, value) for
// every element.
template <typename T, int RT, int NP, class F>
__device__ __forceinline__ void dense(const float* X, int ldx, int xh, const float* __restrict__ W, int K, int tiles,
                                      int heads, F f, int lo = 0, int skip = 0) {
  const int lane = threadIdx.x & 63, wid = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int fr = lane & 15, fg = lane >> 4;
  const int unit = pk_unit<T>(K), own = tiles - skip;
  for (int u = wid; u < own * heads; u += PW) {
    const int h = u >= own ? 1 : 0, t = u - h * own + (u - h * own >= lo ? skip : 0);
    Acc<RT> acc;
    segment<T, RT, NP>(X + h * xh, ldx, W + (size_t)(h * tiles + t) * unit, K, acc);
#pragma unroll
    for (int r = 0; r < RT; ++r) {
      const f32x4 y = acc.total[r];
#pragma unroll
      for (int i = 0; i < 4; ++i) f(h, 16 * r + 4 * fg + i, 16 * t + fr, y[i]);
    }
  }
}
// The same over two segments of the reduction (one head).
template <typename T, int RT, int NP, class F>
__device__ __forceinline__ void dense2(const float* Xa, int lda, const float* __restrict__ Wa, int Ka, const float* Xb,
                                       int ldb, const float* __restrict__ Wb, int Kb, int tiles, F f) {
  const int lane = threadIdx.x & 63, wid = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int fr = lane & 15, fg = lane >> 4;
  for (int u = wid; u < tiles; u += PW) {
    Acc<RT> acc;
    segment<T, RT, NP>(Xa, lda, Wa + (size_t)u * pk_unit<T>(Ka), Ka, acc);
    segment<T, RT, NP>(Xb, ldb, Wb + (size_t)u * pk_unit<T>(Kb), Kb, acc);
#pragma unroll
    for (int r = 0; r < RT; ++r) {
      const f32x4 y = acc.total[r];
#pragma unroll
      for (int i = 0; i < 4; ++i) f(16 * r + 4 * fg + i, 16 * u + fr, y[i]);
    }
  }
}
__device__ __forceinline__ int tiles16(int n) { return (n + 15) >> 4; }

// Leading valid slots of a query whose lane l < k holds neighbour l.
__device__ __forceinline__ int slot_count(int32_t nb, int lane, int k) {
  const unsigned long long on = __ballot(lane < k && nb >= 0);
  return on == ~0ull ? 64 : __builtin_ctzll(~on);
}

// The block's rows in order of falling slot counts (my: lane l < RB that of row l), dealt to the waves there and
// back: wave w's i-th row.  The waves meet at a barrier after their rows, so the rows' counts (0 to k) are
// what would hold it up.
// 180,000 queries of 0 to 20 slots: forward 1348 -> 1312 us, backward's kernel 1489 -> 1479 us.
template <int RB>
__device__ __forceinline__ void deal_rows(int my, int wid, int (&row)[RB / PW]) {
  const int lane = threadIdx.x & 63, key = 64 * my + 63 - lane;   // distinct
  int rank = 0;
#pragma unroll
  for (int j = 0; j < RB; ++j) rank += __builtin_amdgcn_readlane(key, j) > key;
#pragma unroll
  for (int i = 0; i < RB / PW; ++i) {
    const int at = PW * i + (i & 1 ? PW - 1 - wid : wid);
    row[i] = __builtin_ctzll(__ballot(lane < RB && rank == at));
  }
}

// ---------------------------------------------------------------- forward

struct FwdArgs {
  const int32_t *q_node, *nbr, *neid, *n_q;
  const float *q_t, *nt, *edge, *tw, *tb;
  const void* mem;
  int64_t max_q;
  int dm, dt, de, dep, da, dh, dhp, dap, k, kvp, us, as;
  bool mem_al, edge_al;
  const float *wq, *wkt, *wv, *wo, *w1, *w2, *qc, *bv, *bo, *b1, *b2;
  float *qv, *c, *p, *attn, *m_in, *a1, *z;
  void* xs;
};

// The stored part of a slot's row, [M[n_j] || x[e_j]] of dm + dep columns: lane l holds columns 2 l + 128 i,
// 2 l + 128 i + 1 of group i < XG (zero weights face the columns past the row).  ED: there are edge columns; with
// them the bfloat16 mode's values come as loaded (as_row below makes them the row's), for a lane condition
// whose branch converts what it loads waits for it.
template <typename T, int XG, bool ED>
__device__ __forceinline__ void load_x(const FwdArgs& a, int64_t nb, int64_t e, float2 (&x)[XG]) {
  constexpr bool BF = sizeof(T) == 2;
  const int lane = threadIdx.x & 63;
  const T* m = (const T*)a.mem + nb * a.dm;
  const float* f = ED ? a.edge + e * a.de : nullptr;
#pragma unroll
  for (int i = 0; i < XG; ++i) {
    const int c = 2 * lane + 128 * i, ce = c - a.dm;
    if (BF && ED && c < a.dm) {
      const T* r = m + c;
      x[i].x = __uint_as_float(a.mem_al ? *(const uint32_t*)r : (uint32_t)r[0] | (uint32_t)r[1] << 16);
      x[i].y = 0.f;
    } else if (!ED || c < a.dm) {
      x[i] = ld2(m + (ED || c < a.dm ? c : 0), a.mem_al);
    } else {
      if (a.edge_al) {
        x[i] = *(const float2*)(f + min(ce, a.de - 2));
      } else {
        x[i] = make_float2(f[min(ce, a.de - 1)], f[min(ce + 1, a.de - 1)]);
        x[i].y = ce + 1 < a.de ? x[i].y : 0.f;
      }
    }
  }
}

// A loaded group of a bfloat16 row with edge columns: two packed memory columns, or two float32 edge columns.
// 60,000 queries, 10 slots: width 32, 16 edge features, 1 head 272 -> 240 us; width 100, 100 of them, 2 heads 501 -> 446.
__device__ __forceinline__ float2 as_row(float2 v, bool memory) {
  asm volatile("" : "+v"(v.x), "+v"(v.y));
  const uint32_t e = cvt2_bf16(v.x, v.y), w = memory ? __float_as_uint(v.x) : e;
  return make_float2(lo_bf16(w), hi_bf16(w));
}

constexpr float SOFTMAX_SLACK = 11.f;   // a score may exceed the reference by this much before it moves

// a / b with its rounding error taken out (b finite and positive).
__device__ __forceinline__ float div_by(float a, float b, float inv) {
  const float q = a * inv;
  return fmaf(fmaf(-q, b, a), inv, q);
}

// One query's slots: scores, softmax and the weighted row sums c.  Lane l holds two columns of each 128 of
// the stored row and columns 2 l, 2 l + 1 of the time part, so a slot's index, time and probabilities are
// scalars and its loads whole rows.  Half-wave h keeps head h's softmax.  CH slots are
// loaded together; the softmax reference is the first slots' maximum and moves only when a score exceeds it
// by SOFTMAX_SLACK, so a row is read once and the sums are rarely rescaled.  Two thirds of the loop's
// instructions are the encoding and the dot products, which the vector unit bounds; the sums' loads
// and stores run beside it.  U: the query's row of u in LDS, overwritten with c.
template <typename T, int H, int XG, bool ED, int CH>
__device__ __forceinline__ void fwd_slots(const FwdArgs& a, int64_t q, int cnt, int32_t my_nb, int32_t my_e, float my_t,
                                          float tau, float* U) {
  constexpr bool BF = sizeof(T) == 2;
  const int lane = threadIdx.x & 63, hl = lane & 31, head = H == 2 ? lane >> 5 : 0;
  const int dmx = a.dm + a.dep;
  const bool ot = 2 * lane < a.dt;
  const int ct = ot ? 2 * lane : 0;
  const float2 tw = *(const float2*)(a.tw + ct), tb = *(const float2*)(a.tb + ct);
  T* xs = (T*)a.xs + q * a.k * dmx + 2 * lane;
  const float scale = 1.0f / sqrtf((float)a.dh);
  const float my_d = tau - my_t;
  float2 ux[H][XG], ut[H], sx[H][XG], st[H];
#pragma unroll
  for (int h = 0; h < H; ++h) {
    const float* uh = U + h * a.kvp;
    ut[h] = ot ? *(const float2*)(uh + dmx + ct) : Z2;
    st[h] = Z2;
#pragma unroll
    for (int i = 0; i < XG; ++i) {
      const int c = 2 * lane + 128 * i;
      ux[h][i] = c < dmx ? *(const float2*)(uh + c) : Z2;
      sx[h][i] = Z2;
    }
  }
  float mx = 0.f, den = 0.f, my_s0 = 0.f, my_s1 = 0.f;   // of this lane's head
  for (int j0 = 0; j0 < cnt; j0 += CH) {
    float2 x[CH][XG], ph[CH];
    float s[CH];
#pragma unroll
    for (int p = 0; p < CH; ++p) {
      const int j = min(j0 + p, cnt - 1);
      load_x<T, XG, ED>(a, __builtin_amdgcn_readlane(my_nb, j), ED ? __builtin_amdgcn_readlane(my_e, j) : 0, x[p]);
    }
    if constexpr (BF && ED) {
#pragma unroll
      for (int p = 0; p < CH; ++p)
#pragma unroll
        for (int i = 0; i < XG; ++i) x[p][i] = as_row(x[p][i], 2 * lane + 128 * i < a.dm);
    }
    float m = -INFINITY;
#pragma unroll
    for (int p = 0; p < CH; ++p) {
      const int j = j0 + p;
      float2 unused;
      encode<BF, false>(tw, tb, lane_value(my_d, min(j, cnt - 1)), ph[p], unused);
      if (j < cnt) {
#pragma unroll
        for (int i = 0; i < XG; ++i)
          if (2 * lane + 128 * i < dmx) st2_stream(xs + (int64_t)j * dmx + 128 * i, x[p][i]);
      }
      float v[H];
#pragma unroll
      for (int h = 0; h < H; ++h) {
        v[h] = dot2(ut[h], ph[p], 0.f);
#pragma unroll
        for (int i = 0; i < XG; ++i) v[h] = dot2(ux[h][i], x[p][i], v[h]);
      }
      const float sc = heads_sum<H>(v) * scale;
      s[p] = j < cnt ? sc : -INFINITY;   // wave-uniform choice
      m = fmaxf(m, s[p]);
      if (hl == (j & 31)) {
        if (j < 32) my_s0 = sc;
        else my_s1 = sc;
      }
    }
    if (j0 == 0) {
      mx = fmaxf(m, -FLT_MAX);   // finite: scores of -inf weigh nothing beside later ones that are not
    } else if (__any(m > mx + SOFTMAX_SLACK)) {   // rare
      const float mn = fmaxf(m, mx), al = expf(mx - mn);
      mx = mn;
      den *= al;
#pragma unroll
      for (int h = 0; h < H; ++h) {
        const float ah = lane_value(al, 32 * h);
        st[h] = scale2(st[h], ah);
#pragma unroll
        for (int i = 0; i < XG; ++i) sx[h][i] = scale2(sx[h][i], ah);
      }
    }
    // bfloat16: a batch's terms are added among themselves first (fewer roundings of the whole sum, and so fewer
    // stored values that round the other way)
    float e[CH], bd = 0.f;
#pragma unroll
    for (int p = 0; p < CH; ++p) {
      e[p] = expf(s[p] - mx);   // 0 past the count
      (BF ? bd : den) += e[p];
    }
    den += bd;
#pragma unroll
    for (int h = 0; h < H; ++h) {
      float eh[CH];
#pragma unroll
      for (int p = 0; p < CH; ++p) eh[p] = lane_value(e[p], 32 * h);
      const auto add = [&](float2& sum, auto term) {
        float2 t = BF ? scale2(term(0), eh[0]) : sum;
#pragma unroll
        for (int p = BF ? 1 : 0; p < CH; ++p) axpy2(eh[p], term(p), t);
        if constexpr (BF) axpy2(1.f, t, sum);
        else sum = t;
      };
      add(st[h], [&](int p) { return ph[p]; });
#pragma unroll
      for (int i = 0; i < XG; ++i) add(sx[h][i], [&](int p) { return x[p][i]; });
    }
  }
  if (cnt == 0) den = 1.f;   // the sums are zero
  const float inv = 1.f / den;
  if (H == 2 || lane < 32) {
    float* P = a.p + (q * H + head) * a.k;
    if (hl < a.k) P[hl] = hl < cnt ? expf(my_s0 - mx) / den : 0.f;
    if (hl + 32 < a.k) P[hl + 32] = hl + 32 < cnt ? expf(my_s1 - mx) / den : 0.f;
  }
#pragma unroll
  for (int h = 0; h < H; ++h) {
    const float ih = lane_value(inv, 32 * h), dn = lane_value(den, 32 * h);
    float* uh = U + h * a.kvp;
    float* ch = a.c + (q * H + h) * (int64_t)a.kvp;
    const float2 vt = make_float2(div_by(st[h].x, dn, ih), div_by(st[h].y, dn, ih));
    if (ot) {
      st2(uh + dmx + ct, vt);
      st2(ch + dmx + ct, vt);
    }
#pragma unroll
    for (int i = 0; i < XG; ++i) {
      const int c = 2 * lane + 128 * i;
      const float2 v = make_float2(div_by(sx[h][i].x, dn, ih), div_by(sx[h][i].y, dn, ih));
      if (c < dmx) {
        st2(uh + c, v);
        st2(ch + c, v);
      }
    }
  }
}

// The block's query rows M[q] into LDS at X + r ld (rows past the count: zero).
template <typename T, int RB>
__device__ __forceinline__ void load_h(const FwdArgs& a, int64_t r0, int64_t M, float* X, int ld, float* m_in) {
  const int gm = a.dm >> 2, ldm = a.da + a.dm;
  for (int e = threadIdx.x; e < RB * gm; e += PT) {
    const int r = e / gm, g = e - r * gm;
    float4 v = Z4;
    if (r0 + r < M) {
      v = ld4((const T*)a.mem + (int64_t)a.q_node[r0 + r] * a.dm + 4 * g, a.mem_al);
      if (m_in) st4(m_in + (r0 + r) * ldm + a.da + 4 * g, v);
    }
    st4(X + r * ld + 4 * g, v);
  }
}

// Waves per SIMD: two blocks a CU (128 registers), except for two heads and three column groups, whose loops need
// more.  With one block a CU, 60,000 queries of width 100, 10 slots, 100 edge features: bfloat16 forward 777 -> 501 us
// with two.
constexpr int two_blocks(int H, int XG) { return H == 2 && XG == 3 ? 2 : 4; }
// Slots loaded together: what the registers of two blocks a CU leave.
template <typename T>
constexpr int fwd_chunk(int H, int XG) {
  if (XG == 1) return 4;
  return sizeof(T) == 2 && H + XG == 4 ? 1 : 2;
}

// A block of 16 RT queries.  LDS: U (rows of us) holds the query rows M[q], then u, then c, then [o | M[q]];
// A (rows of as) the padded heads of qv, then the attention output, then a1.
template <typename T, int H, int XG, bool ED, int RT>
__global__ __launch_bounds__(PT, two_blocks(H, XG)) void k_proj_fwd(FwdArgs a) {
  extern __shared__ __attribute__((aligned(16))) float lds[];
  constexpr bool BF = sizeof(T) == 2;
  constexpr int RB = 16 * RT, RW = RB / PW, CH = fwd_chunk<T>(H, XG);
  __shared__ int s_cnt[RB];
  float* U = lds;
  float* A = lds + RB * a.us;
  const int64_t M = eff_count(a.max_q, a.n_q);
  const int64_t r0 = (int64_t)blockIdx.x * RB;
  if (r0 >= M) return;   // block-uniform
  const int lane = threadIdx.x & 63, wid = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
#pragma unroll
  for (int i = 0; i < RW; ++i) {
    const int r = wid + PW * i;
    const int c = slot_count(a.nbr[min(r0 + r, M - 1) * a.k + min(lane, a.k - 1)], lane, a.k);
    if (lane == 0) s_cnt[r] = r0 + r < M ? c : 0;
  }
  load_h<T, RB>(a, r0, M, U, a.us, a.m_in);
  __syncthreads();
  dense<T, RT, 1>(U, a.us, 0, a.wq, a.dm, tiles16(a.dap), 1, [&](int, int r, int n, float v) {
    if (n >= a.dap) return;
    v += a.qc[n];
    A[r * a.as + n] = v;
    if (r0 + r < M) a.qv[(r0 + r) * a.dap + n] = v;
  });
  __syncthreads();
  dense<T, RT, 3>(A, a.as, a.dhp, a.wkt, a.dhp, tiles16(a.kvp), H, [&](int h, int r, int n, float v) {
    if (n < a.kvp) U[r * a.us + h * a.kvp + n] = v;
  });
  __syncthreads();
  const int my_cnt = lane < RB ? s_cnt[lane] : 0;
  int row[RW];
  deal_rows<RB>(my_cnt, wid, row);
  // the slots' nodes, edges and times of the wave's next query, a query ahead
  int32_t nb, ne;
  float nt, tau;
  auto fetch = [&](int r) {
    const int64_t q = min(r0 + r, M - 1);
    const int64_t o = q * a.k + min(lane, a.k - 1);
    nb = a.nbr[o];
    nt = a.nt[o];
    ne = ED ? a.neid[o] : 0;
    tau = a.q_t[q];
  };
  fetch(row[0]);
#pragma unroll 1
  for (int i = 0; i < RW; ++i) {
    const int r = row[0];
    const int cnt = __builtin_amdgcn_readlane(my_cnt, r);
#pragma unroll
    for (int j = 0; j + 1 < RW; ++j) row[j] = row[j + 1];
    const int32_t nb0 = nb, ne0 = ne;
    const float nt0 = nt, tau0 = tau;
    if (i + 1 < RW) fetch(row[0]);
    if (r0 + r < M) fwd_slots<T, H, XG, ED, CH>(a, r0 + r, cnt, nb0, ne0, nt0, tau0, U + r * a.us);
  }
  __syncthreads();
  dense<T, RT, 3>(U, a.us, a.kvp, a.wv, a.kvp, tiles16(a.dh), H, [&](int h, int r, int n, float v) {
    if (n >= a.dh) return;
    const int j = h * a.dh + n;
    v = s_cnt[r] > 0 ? v + a.bv[j] : 0.f;
    if (BF) v = round_to_bf16(v);
    A[r * a.as + j] = v;
    if (r0 + r < M) a.attn[(r0 + r) * a.da + j] = v;
  });
  __syncthreads();
  const int ldm = a.da + a.dm;
  load_h<T, RB>(a, r0, M, U + a.da, a.us, nullptr);
  dense<T, RT, 1>(A, a.as, 0, a.wo, a.da, tiles16(a.da), 1, [&](int, int r, int n, float v) {
    if (n >= a.da) return;
    v += a.bo[n];
    if (BF) v = round_to_bf16(v);
    U[r * a.us + n] = v;
    if (r0 + r < M) a.m_in[(r0 + r) * ldm + n] = v;
  });
  __syncthreads();
  dense<T, RT, 1>(U, a.us, 0, a.w1, ldm, tiles16(a.da), 1, [&](int, int r, int n, float v) {
    if (n >= a.da) return;
    v = fmaxf(v + a.b1[n], 0.f);
    if (BF) v = round_to_bf16(v);
    A[r * a.as + n] = v;
    if (r0 + r < M) a.a1[(r0 + r) * a.da + n] = v;
  });
  __syncthreads();
  dense<T, RT, 1>(A, a.as, 0, a.w2, a.da, tiles16(a.da), 1, [&](int, int r, int n, float v) {
    if (n < a.da && r0 + r < M) a.z[(r0 + r) * a.da + n] = v + a.b2[n];
  });
}

// ---------------------------------------------------------------- backward: data gradients

struct BwdArgs {
  const int32_t *nbr, *n_q;
  const float *q_t, *nt, *dz, *tw, *tb;
  int64_t max_q;
  int dm, dt, dep, da, dh, dhp, dap, k, kvp, us, uu, as;
  bool dz_copy;
  const float *w2t, *w1ot, *w1ht, *wot, *wvt, *wkt, *wk, *wqt;
  const float *qv, *c, *p, *a1;
  const void* xs;
  float *dzc, *dm1, *dout, *dattn, *dqv, *du, *dhq, *dx, *tg;
};

// One query's slots, in the forward's lane layout: dx of the memory columns, du and the time encoder's
// gradient sums.  D: the query's row of dc in LDS, overwritten with du; U: its row of u, per head the memory
// columns, then the time columns.  gw, gb: the sums of this lane's time columns.
template <typename T, int H, int XG, int CH>
__device__ __forceinline__ void bwd_slots(const BwdArgs& a, int64_t q, int cnt, float my_t, float tau, float* D,
                                          const float* U, float2& gw, float2& gb) {
  constexpr bool BF = sizeof(T) == 2;
  const int lane = threadIdx.x & 63, hl = lane & 31, head = H == 2 ? lane >> 5 : 0;
  const int dmx = a.dm + a.dep;
  const bool om = 2 * lane < a.dm, ot = 2 * lane < a.dt;
  const int ct = ot ? 2 * lane : 0;
  const float2 tw = *(const float2*)(a.tw + ct), tb = *(const float2*)(a.tb + ct);
  const T* xs = (const T*)a.xs + q * a.k * dmx;
  float* dx = a.dx + q * a.k * a.dm + 2 * lane;
  const float scale = 1.0f / sqrtf((float)a.dh);
  const float my_d = tau - my_t;
  float2 um[H], ut[H], vx[H][XG], vt[H], sx[H][XG], st[H];   // v: the query's dc
  float my_p0 = 0.f, my_p1 = 0.f, dc_c;
  {
    const float* P = a.p + (q * H + head) * a.k;
    if (hl < cnt) my_p0 = P[hl];
    if (hl + 32 < cnt) my_p1 = P[hl + 32];
    float v[H];
#pragma unroll
    for (int h = 0; h < H; ++h) {
      const float* uh = U + h * (a.dm + a.dt);
      const float* dh = D + h * a.kvp;
      const float* ch = a.c + (q * H + h) * (int64_t)a.kvp;
      um[h] = om ? *(const float2*)(uh + 2 * lane) : Z2;
      ut[h] = ot ? *(const float2*)(uh + a.dm + ct) : Z2;
      vt[h] = ot ? *(const float2*)(dh + dmx + ct) : Z2;
      st[h] = Z2;
      v[h] = dot2(vt[h], *(const float2*)(ch + dmx + ct), 0.f);
#pragma unroll
      for (int i = 0; i < XG; ++i) {
        const int c = 2 * lane + 128 * i;
        vx[h][i] = c < dmx ? *(const float2*)(dh + c) : Z2;
        v[h] = dot2(vx[h][i], *(const float2*)(ch + min(c, dmx - 2)), v[h]);
        sx[h][i] = Z2;
      }
    }
    dc_c = heads_sum<H>(v);   // sum_j p_j dp_j
  }
  for (int j0 = 0; j0 < cnt; j0 += CH) {
    float2 x[CH][XG];
#pragma unroll
    for (int p = 0; p < CH; ++p) {
      const int64_t j = min(j0 + p, cnt - 1);
#pragma unroll
      for (int i = 0; i < XG; ++i) x[p][i] = ld2(xs + j * dmx + min(2 * lane + 128 * i, dmx - 2), true);
    }
#pragma unroll
    for (int p = 0; p < CH; ++p) {
      const int j = j0 + p;
      if (j >= cnt) break;   // wave-uniform
      const float delta = lane_value(my_d, j);
      float2 ph, sn;
      encode<BF, true>(tw, tb, delta, ph, sn);
      float v[H];
#pragma unroll
      for (int h = 0; h < H; ++h) {
        v[h] = dot2(vt[h], ph, 0.f);
#pragma unroll
        for (int i = 0; i < XG; ++i) v[h] = dot2(vx[h][i], x[p][i], v[h]);
      }
      const float mp = j < 32 ? my_p0 : my_p1;
      const float dd = (heads_sum<H>(v) - dc_c) * scale;
      float2 dxm = Z2, dph = Z2;
#pragma unroll
      for (int h = 0; h < H; ++h) {
        const float pj = lane_value(mp, 32 * h + (j & 31));
        const float ds = pj * lane_value(dd, 32 * h);
        axpy2(ds, ph, st[h]);
#pragma unroll
        for (int i = 0; i < XG; ++i) axpy2(ds, x[p][i], sx[h][i]);
        axpy2(pj, vx[h][0], dxm);
        axpy2(ds, um[h], dxm);
        axpy2(pj, vt[h], dph);
        axpy2(ds, ut[h], dph);
      }
      if (om) st2_stream(dx + (int64_t)j * a.dm, dxm);
      // d/d arg cos = -sin (the sign goes into the block's sums)
      const float2 gv = make_float2(dph.x * sn.x, dph.y * sn.y);
      axpy2(delta, gv, gw);
      gb.x += gv.x;
      gb.y += gv.y;
    }
  }
#pragma unroll
  for (int h = 0; h < H; ++h) {
    float* dh = D + h * a.kvp;
    float* gh = a.du + (q * H + h) * (int64_t)a.kvp;
    if (ot) {
      st2(dh + dmx + ct, st[h]);
      st2(gh + dmx + ct, st[h]);
    }
#pragma unroll
    for (int i = 0; i < XG; ++i) {
      const int c = 2 * lane + 128 * i;
      if (c < dmx) {
        st2(dh + c, sx[h][i]);
        st2(gh + c, sx[h][i]);
      }
    }
  }
}

// A block of 16 queries.  LDS: UD (rows of us) holds dz, then do, then dc, then du; UU (rows of uu) u, whose edge
// columns nothing reads, then the waves' time-encoder sums; A1 qv, then dattn, then dqv; D1 dm1 (rows of as).
// Two blocks fit a CU up to about 330 columns a head.  With all of u's columns and a buffer each for dz and qv they
// did up to about 250: 60,000 queries of width 64, 172 edge features, 2 heads, 4 and 10 slots 710 -> 515 and 805 -> 588 us.
template <typename T, int H, int XG>
__global__ __launch_bounds__(PT, two_blocks(H, XG)) void k_proj_bwd(BwdArgs a) {
  extern __shared__ __attribute__((aligned(16))) float lds[];
  constexpr int RB = 16, RW = RB / PW, CH = XG == 1 ? 4 : 2;
  __shared__ int s_cnt[RB];
  float* UD = lds;
  float* UU = UD + RB * a.us;
  float* A1 = UU + RB * a.uu;
  float* D1 = A1 + RB * a.as;
  const int64_t M = eff_count(a.max_q, a.n_q);
  const int64_t r0 = (int64_t)blockIdx.x * RB;
  if (r0 >= M) return;   // block-uniform
  const int lane = threadIdx.x & 63, wid = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  for (int i = 0; i < RW; ++i) {
    const int r = wid + PW * i;
    const int64_t q = min(r0 + r, M - 1);
    const int c = slot_count(a.nbr[q * a.k + min(lane, a.k - 1)], lane, a.k);
    if (lane == 0) s_cnt[r] = r0 + r < M ? c : 0;
  }
  for (int e = threadIdx.x; e < RB * a.da; e += PT) {
    const int r = e / a.da, n = e - r * a.da;
    float v = 0.f;
    if (r0 + r < M) {
      v = a.dz[(r0 + r) * a.da + n];
      if (a.dz_copy) a.dzc[(r0 + r) * a.da + n] = v;
    }
    UD[r * a.us + n] = v;
  }
  for (int e = threadIdx.x; e < RB * (a.dap >> 2); e += PT) {
    const int r = e / (a.dap >> 2), g = e - r * (a.dap >> 2);
    st4(A1 + r * a.as + 4 * g, r0 + r < M ? *(const float4*)(a.qv + (r0 + r) * a.dap + 4 * g) : Z4);
  }
  __syncthreads();
  // u_h = W_k,h^T q_h, without the tiles that hold edge columns only
  const int lo = tiles16(a.dm), skip = max(0, (a.dm + a.dep) / 16 - lo);
  dense<T, 1, 3>(
      A1, a.as, a.dhp, a.wkt, a.dhp, tiles16(a.kvp), H,
      [&](int h, int r, int n, float v) {
        const int c = n < a.dm ? n : n - a.dep;
        if (n < a.kvp && (n < a.dm || c >= a.dm)) UU[r * a.uu + h * (a.dm + a.dt) + c] = v;
      },
      lo, skip);
  // dm1 = (W_2^T dz) [a1 > 0]
  dense<T, 1, 3>(UD, a.us, 0, a.w2t, a.da, tiles16(a.da), 1, [&](int, int r, int n, float v) {
    if (n >= a.da) return;
    const bool ok = r0 + r < M;
    v = ok && a.a1[(min(r0 + r, M - 1)) * a.da + n] > 0.f ? v : 0.f;
    if (ok) a.dm1[(r0 + r) * a.da + n] = v;
    D1[r * a.as + n] = v;
  });
  __syncthreads();
  // do = W_1[:, :da]^T dm1
  dense<T, 1, 3>(D1, a.as, 0, a.w1ot, a.da, tiles16(a.da), 1, [&](int, int r, int n, float v) {
    if (n >= a.da) return;
    if (r0 + r < M) a.dout[(r0 + r) * a.da + n] = v;
    UD[r * a.as + n] = v;
  });
  __syncthreads();
  // dattn = W_o^T do in padded heads (zero for a query without slots: its attention output is constant)
  dense<T, 1, 3>(UD, a.as, 0, a.wot, a.da, tiles16(a.dap), 1, [&](int, int r, int n, float v) {
    if (n >= a.dap) return;
    v = s_cnt[r] > 0 ? v : 0.f;
    if (r0 + r < M) a.dattn[(r0 + r) * a.dap + n] = v;
    A1[r * a.as + n] = v;
  });
  __syncthreads();
  // dc_h = W_v,h^T dattn_h
  dense<T, 1, 3>(A1, a.as, a.dhp, a.wvt, a.dhp, tiles16(a.kvp), H, [&](int h, int r, int n, float v) {
    if (n < a.kvp) UD[r * a.us + h * a.kvp + n] = v;
  });
  __syncthreads();
  float2 gw = Z2, gb = Z2;
  const int my_cnt = lane < RB ? s_cnt[lane] : 0;
  int row[RW];
  deal_rows<RB>(my_cnt, wid, row);
#pragma unroll 1
  for (int i = 0; i < RW; ++i) {
    static_assert(RW == 2);
    const int r = i == 0 ? row[0] : row[1];
    if (r0 + r >= M) continue;
    const int64_t q = r0 + r;
    const float nt = a.nt[q * a.k + min(lane, a.k - 1)], tau = a.q_t[q];
    const int cnt = __builtin_amdgcn_readlane(my_cnt, r);
    bwd_slots<T, H, XG, CH>(a, q, cnt, nt, tau, UD + r * a.us, UU + r * a.uu, gw, gb);
  }
  __syncthreads();
  {
    if (2 * lane < a.dt) {
      st2(UU + wid * 2 * a.dt + 2 * lane, gw);
      st2(UU + wid * 2 * a.dt + a.dt + 2 * lane, gb);
    }
  }
  // dq_h = W_k,h du_h in padded heads
  dense<T, 1, 3>(UD, a.us, a.kvp, a.wk, a.kvp, tiles16(a.dhp), H, [&](int h, int r, int n, float v) {
    if (n >= a.dhp) return;
    if (r0 + r < M) a.dqv[(r0 + r) * a.dap + h * a.dhp + n] = v;
    A1[r * a.as + h * a.dhp + n] = v;
  });
  __syncthreads();
  for (int j = threadIdx.x; j < 2 * a.dt; j += PT) {
    float v = 0.f;
#pragma unroll
    for (int w = 0; w < PW; ++w) v += UU[w * 2 * a.dt + j];
    a.tg[(int64_t)blockIdx.x * 2 * a.dt + j] = -v;
  }
  // the query rows' gradient: W_1[:, da:]^T dm1 + W_q[:, :dm]^T dqv
  dense2<T, 1, 3>(D1, a.as, a.w1ht, a.da, A1, a.as, a.wqt, a.dap, tiles16(a.dm), [&](int r, int n, float v) {
    if (n < a.dm && r0 + r < M) a.dhq[(r0 + r) * a.dm + n] = v;
  });
}

// ---------------------------------------------------------------- weight gradients

// One output tile of a weight gradient: out[i][j] = sum over rows of Y[row][i] X[row][j], i < n, j < m.
// Blocks b_begin .. b_begin + nblk - 1 take equal row ranges; each writes its partial [n][m] and, with db,
// the column sums of Y behind it.
struct DwUnit {
  const float *Y, *X;
  float* part;
  int64_t ldy, ldx;
  int n, m, ylim, xlim;   // ylim, xlim: columns that may be read from Y and X
  int b_begin, nblk, db;
};
constexpr int DW_MAXU = 40;
struct DwArgs {
  DwUnit u[DW_MAXU];
  int n;
  int64_t R;
  const int32_t* R_dev;
};

__global__ __launch_bounds__(256, 1) void k_proj_dw(DwArgs a) {
  extern __shared__ __attribute__((aligned(16))) float lds[];
  int u = 0;
  while (u + 1 < a.n && (int)blockIdx.x >= a.u[u + 1].b_begin) ++u;
  const DwUnit q = a.u[u];
  const int64_t R = eff_count(a.R, a.R_dev), steps = (R + 31) / 32, bi = (int)blockIdx.x - q.b_begin;
  float* part = q.part + bi * ((int64_t)q.n * q.m + (q.db ? q.n : 0));
  dw_split_any<1>(
      q.n, q.m, q.Y, q.ldy, q.ylim, q.X, q.ldx, q.xlim, R, steps * bi / q.nblk, steps * (bi + 1) / q.nblk, lds,
      [&](int i, int j, float v) {
        if (i < q.n && j < q.m) part[(int64_t)i * q.m + j] = v;
      },
      [&](int i, float v) {
        if (q.db && i < q.n) part[(int64_t)q.n * q.m + i] = v;
      });
}

// Where a unit's sums go: row i to the weight's row (i0 + i) with the padding of the heads taken out
// (hp padded, hd real columns per head), column j to (j0 + j) with the columns [c1, c2) taken out.
struct DwOut {
  const float* part;
  float *dW, *db;
  int64_t ldw;
  int n, m, nblk, has_db, i0, j0, hp, hd, c1, c2;
};
struct DwRed {
  DwOut u[DW_MAXU];
  int n;
  const float* tg;   // the time encoder's block partials [blocks][2 dt]
  float* tg2;        // [TG_CHUNKS][2 dt]
  int dt2;
  int64_t max_q;
  const int32_t* n_q;
};

// 64 outputs per block, the partials in four interleaved groups added in group order; the last grid row
// sums the time encoder's block partials in TG_CHUNKS chunks.
__global__ __launch_bounds__(256) void k_proj_dw_reduce(DwRed a) {
  if ((int)blockIdx.y == a.n) {
    if (blockIdx.x >= TG_CHUNKS) return;
    const int64_t nb = cdiv(eff_count(a.max_q, a.n_q), 16);
    const int64_t b0 = nb * blockIdx.x / TG_CHUNKS, b1 = nb * (blockIdx.x + 1) / TG_CHUNKS;
    for (int j = threadIdx.x; j < a.dt2; j += 256) {
      double v = 0.;   // the sums grow with the rows, all of one sign in the slow columns
#pragma unroll 8
      for (int64_t b = b0; b < b1; ++b) v += a.tg[b * a.dt2 + j];
      a.tg2[(int64_t)blockIdx.x * a.dt2 + j] = (float)v;
    }
    return;
  }
  __shared__ float s[256];
  const DwOut& q = a.u[blockIdx.y];
  const int per = q.n * q.m + (q.has_db ? q.n : 0);
  if ((int)blockIdx.x * 64 >= per) return;
  const int e = blockIdx.x * 64 + (threadIdx.x & 63), grp = threadIdx.x >> 6;
  float v = 0.f;
  if (e < per) {
#pragma unroll 4
    for (int b = grp; b < q.nblk; b += 4) v += q.part[(int64_t)b * per + e];
  }
  s[threadIdx.x] = v;
  __syncthreads();
  if (grp != 0 || e >= per) return;
  v = ((s[threadIdx.x] + s[threadIdx.x + 64]) + s[threadIdx.x + 128]) + s[threadIdx.x + 192];
  const bool is_db = e >= q.n * q.m;
  const int i = q.i0 + (is_db ? e - q.n * q.m : e / q.m);
  if (i % q.hp >= q.hd) return;
  const int64_t row = (int64_t)(i / q.hp) * q.hd + i % q.hp;
  if (is_db) {
    q.db[row] = v;
    return;
  }
  const int j = q.j0 + e % q.m;
  if (j >= q.c1 && j < q.c2) return;
  q.dW[row * q.ldw + (j < q.c1 ? j : j - (q.c2 - q.c1))] = v;
}

// The time encoder's gradient: the slots' chunk sums plus the queries' share, which is closed-form (their
// time input is phi(0): no w-gradient, a b-gradient of -sin(b_j) sum_a db_q[a] W_q[a][dm + j]); and W_q's
// time columns, db_q[a] phi(0)_j.  b_k's gradient is zero: a constant added to all of a query's scores
// leaves its softmax.
template <typename T>
__global__ __launch_bounds__(256) void k_proj_time(const float* __restrict__ tg2, int dt, int dm, int da,
                                                   const float* __restrict__ dbq, const T* __restrict__ Wq,
                                                   const float* __restrict__ tw, const float* __restrict__ tb,
                                                   float* __restrict__ dw, float* __restrict__ db,
                                                   float* __restrict__ dWq, float* __restrict__ dbk) {
  __shared__ float s[4];
  const int j = blockIdx.x, t = threadIdx.x, ld = dm + dt;
  const float arg = time_arg(tw[j], 0.f, tb[j]);
  const float phi0 = sizeof(T) == 2 ? round_to_bf16(cos_for_bf16(arg)) : cosf(arg);
  float v = 0.f;
  for (int a = t; a < da; a += 256) {
    v += dbq[a] * Elem<T>::load(Wq, (int64_t)a * ld + dm + j);
    dWq[(int64_t)a * ld + dm + j] = dbq[a] * phi0;
    if (j == 0) dbk[a] = 0.f;
  }
  const float ws = wave_sum(v);
  if ((t & 63) == 0) s[t >> 6] = ws;
  __syncthreads();
  if (t < 64) {
    static_assert(TG_CHUNKS == 64, "one chunk per lane");
    double gw = tg2[t * 2 * dt + j], gb = tg2[t * 2 * dt + dt + j];
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) {
      gw += __shfl_xor(gw, o, 64);
      gb += __shfl_xor(gb, o, 64);
    }
    if (t == 0) {
      dw[j] = (float)gw;
      db[j] = (float)(gb - (double)sinf(arg) * (double)(((s[0] + s[1]) + s[2]) + s[3]));
    }
  }
}

// ---------------------------------------------------------------- weight packing

// Index maps of a packed weight's columns and reduction: plain, padded heads, slot-row columns.
enum { MAP_PLAIN, MAP_HEADS, MAP_KV };
struct PackDesc {
  const void* src;
  float* dst;
  int64_t sn, sk, hoff;   // element strides of a column and of a reduction step; of a head
  int N, K, heads, nmap, kmap;
};
struct PackArgs {
  PackDesc d[13];
  PadCopy more[4];
  int n, n_more, dm, de, dep, dh, dhp;
  const void* Wq;
  const float *bq, *tw, *tb;
  float* qc;
  int da, dt, dap;
};

__device__ __forceinline__ int pack_index(const PackArgs& a, int map, int i, int n) {   // -1: padding
  if (i >= n) return -1;
  if (map == MAP_HEADS) return i % a.dhp < a.dh ? i / a.dhp * a.dh + i % a.dhp : -1;
  if (map == MAP_KV) {
    if (i < a.dm + a.de) return i;
    return i < a.dm + a.dep ? -1 : i - (a.dep - a.de);
  }
  return i;
}

template <typename T>
__global__ __launch_bounds__(256) void k_proj_pack(PackArgs a) {
  const int m = blockIdx.y;
  if (m == a.n) {   // the query constant, a wave per padded head column
    const int lane = threadIdx.x & 63, Dq = a.dm + a.dt;
    for (int i = blockIdx.x * 4 + (threadIdx.x >> 6); i < a.dap; i += gridDim.x * 4) {
      const int j = pack_index(a, MAP_HEADS, i, a.dap);
      float v = 0.f;
      if (j >= 0)
        for (int t = lane; t < a.dt; t += 64) {
          const float arg = time_arg(a.tw[t], 0.f, a.tb[t]);
          const float phi = sizeof(T) == 2 ? round_to_bf16(cos_for_bf16(arg)) : cosf(arg);
          v += Elem<T>::load((const T*)a.Wq, (int64_t)j * Dq + a.dm + t) * phi;
        }
      v = wave_sum(v);
      if (lane == 0) a.qc[i] = j >= 0 ? a.bq[j] + v : 0.f;
    }
    return;
  }
  if (m > a.n) {
    const PadCopy& c = a.more[m - a.n - 1];
    const int ldd = c.ldd ? c.ldd : c.cols;
    for (int64_t e = (int64_t)blockIdx.x * 256 + threadIdx.x; e < (int64_t)c.rows * c.cols;
         e += (int64_t)gridDim.x * 256) {
      const int r = (int)(e / c.cols), col = (int)(e % c.cols);
      float v = 0.f;
      if (r < c.n && col < c.k) v = c.tr ? c.src[(int64_t)col * c.ld + r] : c.src[(int64_t)r * c.ld + col];
      c.dst[(int64_t)r * ldd + col] = v;
    }
    return;
  }
  const PackDesc& d = a.d[m];
  const int tiles = (d.N + 15) / 16;
  if constexpr (sizeof(T) == 2) {
    const int nch = (d.K + 31) / 32, total = d.heads * tiles * nch * 512;
    for (int e = blockIdx.x * 256 + threadIdx.x; e < total; e += gridDim.x * 256) {
      const int l = (e >> 3) & 63, c = (e >> 9) % nch, u = (e >> 9) / nch;
      const int h = u / tiles, t = u % tiles;
      const int sn = pack_index(a, d.nmap, 16 * t + (l & 15), d.N);
      const int sk = pack_index(a, d.kmap, 32 * c + 8 * (l >> 4) + (e & 7), d.K);
      ((T*)d.dst)[e] = sn >= 0 && sk >= 0 ? ((const T*)d.src)[h * d.hoff + sn * d.sn + sk * d.sk] : (T)0;
    }
    return;
  }
  const int nch = pk_chunks(d.K), total = d.heads * tiles * nch * 256;
  for (int e = blockIdx.x * 256 + threadIdx.x; e < total; e += gridDim.x * 256) {
    const int i = e & 3, l = (e >> 2) & 63, c = (e >> 8) % nch, u = (e >> 8) / nch;
    const int h = u / tiles, t = u % tiles;
    const int k = 16 * (c + 1) <= d.K ? 16 * c + 4 * (l >> 4) + i : 16 * c + 4 * i + (l >> 4);
    const int sn = pack_index(a, d.nmap, 16 * t + (l & 15), d.N), sk = pack_index(a, d.kmap, k, d.K);
    d.dst[e] = sn >= 0 && sk >= 0 ? Elem<T>::load((const T*)d.src, h * d.hoff + sn * d.sn + sk * d.sk) : 0.f;
  }
}

size_t pk_floats(int N, int K, int heads) { return (size_t)heads * ((N + 15) / 16) * pk_chunks(K) * 256; }

// Equal pieces of at most 112 (7 tiles of 16), multiples of 16 except the last.
int dw_pieces(int n, int* begin) {
  const int t = (n + 15) / 16, np = (t + 6) / 7, per = (t + np - 1) / np;
  int c = 0;
  for (int i = 0; i < t; i += per) begin[c++] = 16 * i;
  begin[c] = n;
  return c;
}

// The weight gradients' units: problems in the order W_2, W_1, W_o, W_q, then W_v and W_k per head.
struct DwPlanP {
  DwArgs a;
  DwRed r;
  int blocks, maxout;
  size_t bytes;
};

struct DwProb {
  const float *Y, *X;
  int64_t ldy, ldx;
  int N, K;
  float *dW, *db;
  int64_t ldw;
  int hp, hd, c1, c2;
};

void dw_plan_units(const DwProb* ps, int np, int64_t R, char* ws, DwPlanP& P) {
  int w[DW_MAXU], n = 0, sum = 0;
  for (int i = 0; i < np; ++i) {
    int nb[8], kb[8];
    const int cn = dw_pieces(ps[i].N, nb), ck = dw_pieces(ps[i].K, kb);
    for (int x = 0; x < cn; ++x)
      for (int y = 0; y < ck; ++y) {
        DwUnit& u = P.a.u[n];
        DwOut& o = P.r.u[n];
        u.Y = ps[i].Y + nb[x];
        u.X = ps[i].X + kb[y];
        u.ldy = ps[i].ldy;
        u.ldx = ps[i].ldx;
        u.n = nb[x + 1] - nb[x];
        u.m = kb[y + 1] - kb[y];
        u.ylim = u.n;
        u.xlim = u.m;
        u.db = y == 0 && ps[i].db != nullptr;
        o.dW = ps[i].dW;
        o.db = ps[i].db;
        o.ldw = ps[i].ldw;
        o.n = u.n;
        o.m = u.m;
        o.has_db = u.db;
        o.i0 = nb[x];
        o.j0 = kb[y];
        o.hp = ps[i].hp;
        o.hd = ps[i].hd;
        o.c1 = ps[i].c1;
        o.c2 = ps[i].c2;
        w[n] = (u.n <= 32 ? 2 : u.n <= 64 ? 4 : 7) * (u.m <= 64 ? 4 : 7);
        sum += w[n++];
      }
  }
  // one block per CU over all units, in proportion to their MFMAs; at least 64 rows a block
  const int total = std::max(n, dw_os_cu_count() > 0 ? dw_os_cu_count() : 256);
  const int64_t cap = std::max<int64_t>(1, (R + 63) / 64);
  int begin = 0;
  size_t bytes = 0;
  P.maxout = 64 * TG_CHUNKS;
  for (int i = 0; i < n; ++i) {
    DwUnit& u = P.a.u[i];
    DwOut& o = P.r.u[i];
    u.b_begin = begin;
    u.nblk = (int)std::min<int64_t>(cap, std::max(1, total * w[i] / sum));
    o.nblk = u.nblk;
    begin += u.nblk;
    const int per = u.n * u.m + (u.db ? u.n : 0);
    u.part = (float*)(ws + bytes);
    o.part = u.part;
    bytes += a256(sizeof(float) * (size_t)per * u.nblk);
    P.maxout = std::max(P.maxout, per);
  }
  P.a.n = P.r.n = n;
  P.blocks = begin;
  P.bytes = bytes;
}

int dw_problems(const ProjShape& s, DwProb* ps) {   // sizes only; the caller fills the pointers
  int n = 0;
  auto add = [&](int N, int K, int64_t ldy, int64_t ldx, int64_t ldw, int hp, int hd, int c1, int c2) {
    ps[n++] = DwProb{nullptr, nullptr, ldy, ldx, N, K, nullptr, nullptr, ldw, hp, hd, c1, c2};
  };
  const int ldm = s.da + s.dm;
  add(s.da, s.da, s.da, s.da, s.da, s.da, s.da, s.da, s.da);            // W_2
  add(s.da, ldm, s.da, ldm, ldm, s.da, s.da, ldm, ldm);                 // W_1
  add(s.da, s.da, s.da, s.da, s.da, s.da, s.da, s.da, s.da);            // W_o
  add(s.dap, s.dm, s.dap, ldm, s.Dq, s.dhp, s.dh, s.dm, s.dm);          // W_q
  for (int w = 0; w < 2; ++w)                                           // W_v, W_k
    for (int h = 0; h < s.H; ++h)
      add(s.dhp, s.kvp, s.dap, s.H * s.kvp, s.Dkv, s.dhp, s.dh, s.dm + s.de, s.dm + s.dep);
  return n;
}

size_t fwd_lds(const ProjShape& s, int rows) { return sizeof(float) * (size_t)rows * (s.us + s.as); }
size_t bwd_lds(const ProjShape& s) { return sizeof(float) * 16 * (size_t)(s.us + s.uu + 2 * s.as); }

// Blocks of 32 queries (half the weight reads per query) from this many query rows on, where they still
// fill the chip; of 16 below.  Blocks of 16 and of 32, us: width 100, 16 edge features, 10 slots: 4,500 queries 61
// and 69, 9,000 91 and 99, 15,000 114 and 99, 24,000 163 and 148, 120,000 753 and 665; bfloat16 58 and 74, 89 and
// 98, 110 and 102, 158 and 150, 709 and 632.  They cross between 9,000 and 15,000 (width 64, 100 edge features: near
// 9,000 in float32, near 24,000 in bfloat16); up to the line some thousand rows run 5 to 17 % over the other's time.
// fwd_lds <= 81920: two blocks a CU fit.
constexpr int64_t FWD_RT2_ROWS = 16384;

template <typename K>
mtgnn_status lds_limit(K kernel, size_t bytes) {   // above the 64 KB a launch may use without asking
  if (bytes <= 65536) return MTGNN_OK;
  const hipError_t e = hipFuncSetAttribute((const void*)kernel, hipFuncAttributeMaxDynamicSharedMemorySize, (int)bytes);
  if (e != hipSuccess) {
    set_hip_error(e, "attention LDS size");
    return MTGNN_EHIP;
  }
  return MTGNN_OK;
}

template <typename T, int H, int XG, bool ED>
mtgnn_status launch_fwd(const FwdArgs& a, const ProjShape& s, hipStream_t st) {
  if (s.Q >= FWD_RT2_ROWS && fwd_lds(s, 32) <= 81920) {
    MTGNN_TRY(lds_limit(k_proj_fwd<T, H, XG, ED, 2>, fwd_lds(s, 32)));
    k_proj_fwd<T, H, XG, ED, 2><<<(unsigned)cdiv(s.Q, 32), PT, fwd_lds(s, 32), st>>>(a);
  } else {
    MTGNN_TRY(lds_limit(k_proj_fwd<T, H, XG, ED, 1>, fwd_lds(s, 16)));
    k_proj_fwd<T, H, XG, ED, 1><<<(unsigned)cdiv(s.Q, 16), PT, fwd_lds(s, 16), st>>>(a);
  }
  MTGNN_CHECK_LAUNCH("proj_fwd");
  return MTGNN_OK;
}

template <typename T, int H, int XG>
mtgnn_status launch_bwd(const BwdArgs& a, const ProjShape& s, hipStream_t st) {
  MTGNN_TRY(lds_limit(k_proj_bwd<T, H, XG>, bwd_lds(s)));
  k_proj_bwd<T, H, XG><<<(unsigned)cdiv(s.Q, 16), PT, bwd_lds(s), st>>>(a);
  MTGNN_CHECK_LAUNCH("proj_bwd");
  return MTGNN_OK;
}

// f(element type tag, heads, 128-column groups of the stored row) for the dims
template <class F>
mtgnn_status by_dims(const mtgnn_dims* d, const ProjShape& s, F f) {
  auto groups = [&](auto t, auto h) -> mtgnn_status {
    const int g = (s.dm + s.dep + 127) / 128;
    if (g == 1) return f(t, h, std::integral_constant<int, 1>{});
    if (g == 2) return f(t, h, std::integral_constant<int, 2>{});
    return f(t, h, std::integral_constant<int, 3>{});
  };
  auto heads = [&](auto t) -> mtgnn_status {
    return s.H == 1 ? groups(t, std::integral_constant<int, 1>{}) : groups(t, std::integral_constant<int, 2>{});
  };
  return d->dtype == MTGNN_F32 ? heads(float{}) : heads(uint16_t{});
}

}  // namespace

ProjShape::ProjShape(const mtgnn_dims* d, int64_t max_q) {
  Q = max_q;
  k = d->k;
  P = max_q * k;
  N = d->n_nodes;
  dm = d->d_mem;
  dt = d->d_time;
  de = d->d_edge;
  dep = (de + 3) / 4 * 4;
  da = d->d_attn;
  H = d->n_heads;
  dh = da / H;
  dhp = (dh + 3) / 4 * 4;
  dap = H * dhp;
  kvp = dm + dep + dt;
  Dq = dm + dt;
  Dkv = dm + de + dt;
  us = odd4(std::max(std::max(H * kvp, da + dm), 2 * dt));
  uu = odd4(H * (dm + dt));
  as = odd4(std::max(dap, da));
  esz = d->dtype == MTGNN_F32 ? 4 : 2;
}

// The kernels' limits, then the cost: here a query costs its heads' projected vectors (a row of columns each, in
// products and in LDS), on the general path a slot costs its key and value, 2 d_attn columns.  Measured times of
// this path over the general one's, forward / backward (60,000 queries, a fifth without slots, two fifths with all k;
// float32, 4-divisible widths, which suit the general path best):
//   rows to 128, 2 heads, k 1: width 32 0.76 / 0.89, width 128 0.81 / 1.13
//   rows to 256, 2 heads, k 1 and 2: width 64, 172 edge features 0.91 / 1.13 and 0.77 / 1.03, width 100, 64 edge
//     features 1.11 / 1.06 and 0.99 / 0.93; 1 head, k 1: width 100, 100 edge features 0.83 / 0.98
//   rows past 256, 1 head, k 1 and 2: width 32, 256 edge features 0.89 / 1.11 and 0.76 / 1.04
//   rows past 256, 2 heads (one block a CU), 256 edge features: width 32, k 10 and 14 1.15 / 0.94 and 1.00 / 0.80;
//     width 64, k 4 and 6 1.07 / 0.94 and 0.96 / 0.84; width 100, k 2 and 4 1.14 / 1.26 and 0.95 / 1.01; width 128, k 2
//     and 4 1.00 / 1.03 and 0.82 / 0.81; bfloat16, width 100, k 4 0.93 / 0.85
// The slots a batch really has are not known here: one without any takes 1.0 / 1.18 (width 100, k 10).
bool proj_ok(const mtgnn_dims* d) {
  if (d->n_heads > 2 || d->d_mem % 4 != 0 || d->d_time % 4 != 0 || d->d_attn % 4 != 0 || d->d_time <= 0 ||
      d->d_mem > 128 || d->d_time > 128 || d->d_attn > 128 || d->d_edge > 256 || d->k > 64)
    return false;
  const int row = d->d_mem + (d->d_edge + 3) / 4 * 4;
  if (row <= (d->n_heads == 1 ? 256 : 128)) return true;
  if (d->n_heads == 1 || row <= 256) return d->k >= 2;
  return d->k * d->d_attn >= 400;
}

ProjSave carve_proj_save(void* base, const ProjShape& s) {
  char* w = (char*)base;
  ProjSave v;
  auto take = [&](size_t bytes) { char* r = w; w += a256(bytes); return r; };
  // the packed weights first: their offsets do not depend on the query count
  const int N[13] = {s.dap, s.kvp, s.dh, s.da, s.da, s.da, s.da, s.da, s.dm, s.dap, s.kvp, s.dhp, s.dm};
  const int K[13] = {s.dm, s.dhp, s.kvp, s.da, s.da + s.dm, s.da, s.da, s.da, s.da, s.da, s.dhp, s.kvp, s.dap};
  for (int i = 0; i < 13; ++i) {
    const bool heads = i == PK_WKT || i == PK_WV || i == PK_WVT || i == PK_WK;
    v.w[i] = (float*)take(sizeof(float) * pk_floats(N[i], K[i], heads ? s.H : 1));
  }
  v.qc = (float*)take(sizeof(float) * s.dap);
  v.qv = (float*)take(sizeof(float) * s.Q * s.dap);
  v.c = (float*)take(sizeof(float) * s.Q * s.H * s.kvp);
  v.p = (float*)take(sizeof(float) * s.Q * s.H * s.k);
  v.attn = (float*)take(sizeof(float) * s.Q * s.da);
  v.m_in = (float*)take(sizeof(float) * s.Q * (s.da + s.dm));
  v.a1 = (float*)take(sizeof(float) * s.Q * s.da);
  v.xs = take((size_t)s.esz * s.P * (s.dm + s.dep));
  v.total = (size_t)(w - (char*)base);
  return v;
}

ProjBwd carve_proj_bwd(void* base, const ProjShape& s) {
  char* w = (char*)base;
  ProjBwd v;
  auto take = [&](size_t bytes) { char* r = w; w += a256(bytes); return r; };
  v.dz = (float*)take(sizeof(float) * s.Q * s.da);
  v.dm1 = (float*)take(sizeof(float) * s.Q * s.da);
  v.dout = (float*)take(sizeof(float) * s.Q * s.da);
  v.dattn = (float*)take(sizeof(float) * s.Q * s.dap);
  v.dqv = (float*)take(sizeof(float) * s.Q * s.dap);
  v.du = (float*)take(sizeof(float) * s.Q * s.H * s.kvp);
  v.dhq = (float*)take(sizeof(float) * s.Q * s.dm);
  v.dx = (float*)take(sizeof(float) * s.P * s.dm);
  v.tg = (float*)take(sizeof(float) * 2 * s.dt * cdiv(s.Q, 16));
  v.tg2 = (float*)take(sizeof(float) * 2 * s.dt * TG_CHUNKS);
  DwProb ps[8];
  const int n = dw_problems(s, ps);
  for (int i = 0; i < n; ++i) ps[i].db = i < 4 + s.H ? v.tg2 : nullptr;   // sizes only: which have a bias
  DwPlanP plan;
  dw_plan_units(ps, n, s.Q, nullptr, plan);
  v.dw_bytes = plan.bytes;
  v.dw = take(plan.bytes);
  v.total = (size_t)(w - (char*)base);
  return v;
}

mtgnn_status proj_prepare_weights(const mtgnn_attn_params* p, const float* tw, const float* tb, const mtgnn_dims* d,
                                  void* save, hipStream_t st, const PadCopy* more, int n_more) {
  const ProjShape s(d, 0);
  const ProjSave v = carve_proj_save(save, s);
  PackArgs a{};
  const int ldm = s.da + s.dm;
  const size_t esz = d->dtype == MTGNN_F32 ? 4 : 2;
  auto at = [&](const void* w, int64_t off) { return (const void*)((const char*)w + esz * (size_t)off); };
  auto set = [&](int i, const void* src, int64_t sn, int64_t sk, int N, int K, int nmap, int kmap, int heads = 1,
                 int64_t hoff = 0) { a.d[i] = PackDesc{src, v.w[i], sn, sk, hoff, N, K, heads, nmap, kmap}; };
  const int64_t hw = (int64_t)s.dh * s.Dkv;
  set(PK_WQ, p->W_q, s.Dq, 1, s.dap, s.dm, MAP_HEADS, MAP_PLAIN);
  set(PK_WKT, p->W_k, 1, s.Dkv, s.kvp, s.dhp, MAP_KV, MAP_HEADS, s.H, hw);
  set(PK_WV, p->W_v, s.Dkv, 1, s.dh, s.kvp, MAP_PLAIN, MAP_KV, s.H, hw);
  set(PK_WO, p->W_o, s.da, 1, s.da, s.da, MAP_PLAIN, MAP_PLAIN);
  set(PK_W1, p->W_1, ldm, 1, s.da, ldm, MAP_PLAIN, MAP_PLAIN);
  set(PK_W2, p->W_2, s.da, 1, s.da, s.da, MAP_PLAIN, MAP_PLAIN);
  set(PK_W2T, p->W_2, 1, s.da, s.da, s.da, MAP_PLAIN, MAP_PLAIN);
  set(PK_W1OT, p->W_1, 1, ldm, s.da, s.da, MAP_PLAIN, MAP_PLAIN);
  set(PK_W1HT, at(p->W_1, s.da), 1, ldm, s.dm, s.da, MAP_PLAIN, MAP_PLAIN);
  set(PK_WOT, p->W_o, 1, s.da, s.dap, s.da, MAP_HEADS, MAP_PLAIN);
  set(PK_WVT, p->W_v, 1, s.Dkv, s.kvp, s.dhp, MAP_KV, MAP_HEADS, s.H, hw);
  set(PK_WK, p->W_k, s.Dkv, 1, s.dhp, s.kvp, MAP_HEADS, MAP_KV, s.H, hw);
  set(PK_WQT, p->W_q, 1, s.Dq, s.dm, s.dap, MAP_PLAIN, MAP_HEADS);
  a.n = 13;
  a.n_more = n_more;
  for (int i = 0; i < n_more; ++i) a.more[i] = more[i];
  a.dm = s.dm;
  a.de = s.de;
  a.dep = s.dep;
  a.dh = s.dh;
  a.dhp = s.dhp;
  a.Wq = p->W_q;
  a.bq = p->b_q;
  a.tw = tw;
  a.tb = tb;
  a.qc = v.qc;
  a.da = s.da;
  a.dt = s.dt;
  a.dap = s.dap;
  const dim3 grid(32, (unsigned)(14 + n_more));
  if (d->dtype == MTGNN_F32) k_proj_pack<float><<<grid, 256, 0, st>>>(a);
  else k_proj_pack<uint16_t><<<grid, 256, 0, st>>>(a);
  MTGNN_CHECK_LAUNCH("proj_pack");
  return MTGNN_OK;
}

mtgnn_status proj_fwd(const int32_t* q_node, const float* q_t, const int32_t* n_q, int64_t max_q, const int32_t* nbr,
                      const float* nt, const int32_t* neid, const void* memory, const float* edge_feat,
                      const float* tw, const float* tb, const mtgnn_attn_params* p, const mtgnn_dims* d, float* z,
                      void* save, hipStream_t st) {
  const ProjShape s(d, max_q);
  const ProjSave v = carve_proj_save(save, s);
  if (max_q <= 0) return MTGNN_OK;
  FwdArgs a{};
  a.q_node = q_node; a.nbr = nbr; a.neid = neid; a.n_q = n_q;
  a.q_t = q_t; a.nt = nt; a.edge = edge_feat; a.tw = tw; a.tb = tb;
  a.mem = memory;
  a.max_q = max_q;
  a.dm = s.dm; a.dt = s.dt; a.de = s.de; a.dep = s.dep; a.da = s.da; a.dh = s.dh; a.dhp = s.dhp; a.dap = s.dap;
  a.k = s.k; a.kvp = s.kvp; a.us = s.us; a.as = s.as;
  a.mem_al = ((uintptr_t)memory & (d->dtype == MTGNN_F32 ? 15 : 7)) == 0;
  a.edge_al = s.de % 2 == 0 && ((uintptr_t)edge_feat & 7) == 0;
  a.wq = v.w[PK_WQ]; a.wkt = v.w[PK_WKT]; a.wv = v.w[PK_WV]; a.wo = v.w[PK_WO]; a.w1 = v.w[PK_W1]; a.w2 = v.w[PK_W2];
  a.qc = v.qc; a.bv = p->b_v; a.bo = p->b_o; a.b1 = p->b_1; a.b2 = p->b_2;
  a.qv = v.qv; a.c = v.c; a.p = v.p; a.attn = v.attn; a.m_in = v.m_in; a.a1 = v.a1; a.z = z;
  a.xs = v.xs;
  TimedScope ts("attn_fwd", st);
  return by_dims(d, s, [&](auto t, auto h, auto g) -> mtgnn_status {
    using T = decltype(t);
    constexpr int H = decltype(h)::value, G = decltype(g)::value;
    if constexpr (G == 1) {
      if (s.dep == 0) return launch_fwd<T, H, G, false>(a, s, st);
    }
    return launch_fwd<T, H, G, true>(a, s, st);
  });
}

mtgnn_status proj_bwd(const float* q_t, const int32_t* n_q, int64_t max_q, const int32_t* nbr, const float* nt,
                      const float* dz, const float* tw, const float* tb, const mtgnn_dims* d, const void* save,
                      const ProjBwd& b, hipStream_t st) {
  const ProjShape s(d, max_q);
  const ProjSave v = carve_proj_save((void*)save, s);
  if (max_q <= 0) return MTGNN_OK;
  BwdArgs a{};
  a.nbr = nbr; a.n_q = n_q;
  a.q_t = q_t; a.nt = nt; a.dz = dz; a.tw = tw; a.tb = tb;
  a.max_q = max_q;
  a.dm = s.dm; a.dt = s.dt; a.dep = s.dep; a.da = s.da; a.dh = s.dh; a.dhp = s.dhp; a.dap = s.dap;
  a.k = s.k; a.kvp = s.kvp; a.us = s.us; a.uu = s.uu; a.as = s.as;
  a.dz_copy = ((uintptr_t)dz & 15) != 0;   // the weight gradients read 16-byte groups
  a.w2t = v.w[PK_W2T]; a.w1ot = v.w[PK_W1OT]; a.w1ht = v.w[PK_W1HT]; a.wot = v.w[PK_WOT]; a.wvt = v.w[PK_WVT];
  a.wkt = v.w[PK_WKT]; a.wk = v.w[PK_WK]; a.wqt = v.w[PK_WQT];
  a.qv = v.qv; a.c = v.c; a.p = v.p; a.a1 = v.a1;
  a.xs = v.xs;
  a.dzc = b.dz; a.dm1 = b.dm1; a.dout = b.dout; a.dattn = b.dattn; a.dqv = b.dqv; a.du = b.du; a.dhq = b.dhq;
  a.dx = b.dx; a.tg = b.tg;
  TimedScope ts("attn_bwd", st);
  return by_dims(d, s, [&](auto t, auto h, auto g) {
    return launch_bwd<decltype(t), decltype(h)::value, decltype(g)::value>(a, s, st);
  });
}

mtgnn_status proj_params(const int32_t* n_q, int64_t max_q, const float* dz, const float* tw, const float* tb,
                         const mtgnn_attn_params* p, const mtgnn_dims* d, const void* save, const ProjBwd& b,
                         mtgnn_attn_grads* g, float* d_time_w, float* d_time_b, hipStream_t st) {
  const ProjShape s(d, max_q);
  const ProjSave v = carve_proj_save((void*)save, s);
  DwProb ps[8];
  const int n = dw_problems(s, ps);
  auto fill = [&](int i, const float* Y, const float* X, float* dW, float* db) {
    ps[i].Y = Y;
    ps[i].X = X;
    ps[i].dW = dW;
    ps[i].db = db;
  };
  fill(0, ((uintptr_t)dz & 15) != 0 ? b.dz : dz, v.a1, g->W_2, g->b_2);
  fill(1, b.dm1, v.m_in, g->W_1, g->b_1);
  fill(2, b.dout, v.attn, g->W_o, g->b_o);
  fill(3, b.dqv, v.m_in + s.da, g->W_q, g->b_q);
  const int64_t hw = (int64_t)s.dh * s.Dkv;
  for (int h = 0; h < s.H; ++h) {
    fill(4 + h, b.dattn + h * s.dhp, v.c + h * s.kvp, g->W_v + h * hw, g->b_v + h * s.dh);
    fill(4 + s.H + h, v.qv + h * s.dhp, b.du + h * s.kvp, g->W_k + h * hw, nullptr);
  }
  DwPlanP plan{};
  dw_plan_units(ps, n, max_q, b.dw, plan);
  plan.a.R = max_q;
  plan.a.R_dev = n_q;
  plan.r.tg = b.tg;
  plan.r.tg2 = b.tg2;
  plan.r.dt2 = 2 * s.dt;
  plan.r.max_q = max_q;
  plan.r.n_q = n_q;
  int64_t steps = 0;   // of a block, at most
  for (int i = 0; i < plan.a.n; ++i) steps = std::max(steps, cdiv(cdiv(max_q, 32), plan.a.u[i].nblk));
  const int lds = dw_lds(1, steps);
  MTGNN_TRY(lds_limit(k_proj_dw, (size_t)lds));
  {
    TimedScope ts("attn_dw", st);
    k_proj_dw<<<(unsigned)plan.blocks, 256, lds, st>>>(plan.a);
  }
  MTGNN_CHECK_LAUNCH("proj_dw");
  k_proj_dw_reduce<<<dim3((unsigned)cdiv(plan.maxout, 64), (unsigned)(plan.r.n + 1)), 256, 0, st>>>(plan.r);
  MTGNN_CHECK_LAUNCH("proj_dw_reduce");
  if (d->dtype == MTGNN_F32)
    k_proj_time<float><<<(unsigned)s.dt, 256, 0, st>>>(b.tg2, s.dt, s.dm, s.da, g->b_q, (const float*)p->W_q, tw, tb,
                                                       d_time_w, d_time_b, g->W_q, g->b_k);
  else
    k_proj_time<uint16_t><<<(unsigned)s.dt, 256, 0, st>>>(b.tg2, s.dt, s.dm, s.da, g->b_q, (const uint16_t*)p->W_q,
                                                          tw, tb, d_time_w, d_time_b, g->W_q, g->b_k);
  MTGNN_CHECK_LAUNCH("proj_time");
  return MTGNN_OK;
}

}  // namespace mtgnn
