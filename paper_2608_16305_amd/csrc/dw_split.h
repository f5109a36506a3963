// Weight gradients (sums over rows of products of two rows' columns) on the bfloat16 matrix instructions, float32
// operands split into three parts each (bf16_split.h).
#pragma once

#include "bf16_split.h"
#include "gemm.h"

namespace mtgnn {

// A row's columns as NT column tiles of 16: the lane's 16-byte group 4 fr + t for the first four, 64 + 3 fr + t - 4
// for the other three; NT = 2: the 8-byte group 2 fr + t.  One load a row and group.
template <int NT>
__device__ __forceinline__ int dw_col(int t, int i) {
  if (NT == 2) return 2 * i + t;
  return t < 4 ? 4 * i + t : 64 + 3 * i + t - 4;
}
// Groups 0 (tiles 0..3, or both of NT = 2) and 1 (tiles 4..6) of rows r .. r + 7 (those < R; zero past them), the
// columns clamped to the first lim (what lies past a unit's columns is never stored).
template <int NT, int G>
__device__ __forceinline__ void dw_load(const float* p, int64_t ld, int64_t r, int64_t R, int fr, int lim,
                                        float (&v)[NT][8]) {
  constexpr int T0 = G ? 4 : 0, T1 = G ? 7 : NT < 4 ? NT : 4;
  if constexpr (T0 < NT) {
    const int c = G ? min(64 + 3 * fr, lim - 3) : min(T1 * fr, lim - T1);
#pragma unroll
    for (int e = 0; e < 8; ++e) {
      const float* row = p + min(r + e, R - 1) * ld + c;
#pragma unroll
      for (int t = T0; t < T1; ++t) v[t][e] = row[t - T0];
    }
  }
}
template <int NT, int G>
__device__ __forceinline__ void dw_zero(int64_t r, int64_t R, float (&v)[NT][8]) {   // rows past R, as loaded
  constexpr int T0 = G ? 4 : 0, T1 = G ? 7 : NT < 4 ? NT : 4;
  if constexpr (T0 < NT) {
#pragma unroll
    for (int e = 0; e < 8; ++e)
#pragma unroll
      for (int t = T0; t < T1; ++t) v[t][e] = r + e < R ? v[t][e] : 0.f;
  }
}

// The lane whose group 1 straddles the last column has loaded the columns that end there: its values move to their
// places.  dw_ragged: whether there is such a lane.
template <int NT>
__device__ __forceinline__ bool dw_ragged(int lim) { return NT > 4 && lim > 64 && (lim - 64) % 3 != 0; }
template <int NT>
__device__ __forceinline__ void dw_shift(int fr, int lim, float (&v)[NT][8]) {
  if constexpr (NT > 4) {
    const int sh = 64 + 3 * fr + 3 - lim;   // 1 or 2 where it matters
#pragma unroll
    for (int e = 0; e < 8; ++e) {
      const float a = v[4][e], b = v[5][e], c = v[6][e];
      v[4][e] = sh == 1 ? b : sh == 2 ? c : a;
      v[5][e] = sh == 1 ? c : b;
    }
  }
}

// One output's sum over rows [r0, r1) with float32 products, four sums in turn.
__device__ __forceinline__ float dw_plain(const float* y, int64_t ldy, const float* x, int64_t ldx, int64_t r0,
                                          int64_t r1) {
  float v[4] = {0.f, 0.f, 0.f, 0.f};
  for (int64_t r = r0; r < r1; r += 4) {
#pragma unroll
    for (int e = 0; e < 4; ++e)
      if (r + e < r1) v[e] = fmaf(y[(r + e) * ldy], x[(r + e) * ldx], v[e]);
  }
  return (v[0] + v[1]) + (v[2] + v[3]);
}

// The block's waves take its rows 32 at a time in turn, operands straight from memory: lane (fr, fg) holds rows
// 8 fg .. 8 fg + 7 of a step, each column of Y and X split into three bfloat16 parts, and a pair of tiles takes
// six 16x16x32 products (bf16_split.h) where float32 instructions take eight of twice the time.  A group's
// next rows are requested as soon as its parts are made.  G column groups (the caller passes each wave its
// group's X): wave w works for group w % G, 4 / G waves share a group's steps and their sums are added in
// wave order.
// An operand past the largest bfloat16, or infinite, meets the others' zero parts (NaN): a lane that stores a sum
// which is not finite goes over its sums again with float32 products.
// Matrix time and the operands' reads bound it about equally.  Against 16x16x4 float32 instructions: the
// attention's eight products of 180,000 rows (1.35 GB) 500 -> 352 us (before the segments
// below, which add 55), of 12,000 rows 46 -> 35 us.
//
// An instruction rounds its accumulator every eight products (16x16x4: every one), so a long sum's error is of those
// roundings at its full size: a sum of DW_SEGMENT steps joins the total by one addition.  The attention's value
// gradient over 60,000 rows against 64 bits: 1.4e-7 with one chain a block, 7.9e-8 with segments of 16, 5.6e-8 with 8
// (float32 products over its 700,000 slots: 7.6e-8).  180,000 rows: backward 2058 us, 2081 with 16, 2116 with 8.
constexpr int DW_SEGMENT = 8;
template <int NI, int NJ, int G, class Out, class Bias>
__device__ __forceinline__ void dw_split(const float* Y, int64_t ldy, int ylim, const float* X, int64_t ldx, int xlim,
                                         int64_t R, int64_t s0, int64_t s1, float* lds, Out out, Bias bias) {
  constexpr int NW = 4 / G;   // waves of a group
  const int lane = threadIdx.x & 63, wid = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int grp = wid % G, mine = wid / G;
  const int fr = lane & 15, fg = lane >> 4;
  float bad = 0.f;   // NaN once a stored sum is not finite
  const auto store = [&](int i, int j, float v) {
    bad = fmaf(v, 0.f, bad);
    out(i, j, v);
  };
  // the lane's sums again, of every tile row and of columns b0, b0 + db, ..
  const auto again = [&](int b0, int db) {
    const int64_t r0 = 32 * s0, r1 = min(32 * s1, R);
    for (int a = 0; a < NI; ++a)
      for (int b = b0; b < NJ; b += db)
        for (int r = 0; r < 4; ++r) {
          const int i = dw_col<NI>(a, 4 * fg + r), j = dw_col<NJ>(b, fr);
          if (i < ylim && j < xlim) out(i, j, dw_plain(Y + i, ldy, X + j, ldx, r0, r1));
        }
  };
  f32x4 acc[NI][NJ];
  float cs[NI];
#pragma unroll
  for (int i = 0; i < NI; ++i) cs[i] = 0.f;
  const auto steps = [&](int64_t begin, int64_t end) {   // the wave's steps of [begin, end), begin + mine the first
#pragma unroll
    for (int i = 0; i < NI; ++i)
#pragma unroll
      for (int j = 0; j < NJ; ++j) acc[i][j] = f32x4{0.f, 0.f, 0.f, 0.f};
  float y[NI][8], x[NJ][8];
  if (begin + mine < end) {
    const int64_t r = 32 * (begin + mine) + 8 * fg;
    dw_load<NJ, 0>(X, ldx, r, R, fr, xlim, x);
    dw_load<NJ, 1>(X, ldx, r, R, fr, xlim, x);
    dw_load<NI, 0>(Y, ldy, r, R, fr, ylim, y);
    dw_load<NI, 1>(Y, ldy, r, R, fr, ylim, y);
  }
    for (int64_t s = begin + mine; s < end; s += NW) {
      const int64_t r = 32 * s + 8 * fg, rn = min(32 * (s + NW), R - 1) + 8 * fg;   // the next step's (in range) rows
      if (32 * s + 32 > R) {   // the last, ragged step
        dw_zero<NJ, 0>(r, R, x);
        dw_zero<NJ, 1>(r, R, x);
        dw_zero<NI, 0>(r, R, y);
        dw_zero<NI, 1>(r, R, y);
      }
      if (dw_ragged<NJ>(xlim)) dw_shift<NJ>(fr, xlim, x);
      if (dw_ragged<NI>(ylim)) dw_shift<NI>(fr, ylim, y);
      Bf16Right xp[NJ];
#pragma unroll
      for (int j = 0; j < NJ; ++j) xp[j] = split_right(x[j]);
      dw_load<NJ, 0>(X, ldx, rn, R, fr, xlim, x);
      dw_load<NJ, 1>(X, ldx, rn, R, fr, xlim, x);
      auto tile = [&](int i) {
        const Bf16Left yp = split_left(y[i]);
        float c = 0.f;
#pragma unroll
        for (int e = 0; e < 8; ++e) c += y[i][e];
        cs[i] += c;
        // the small products first; a pair of terms of all tiles before the next of one (the chains don't wait)
#pragma unroll
        for (int j = 0; j < NJ; ++j)
          acc[i][j] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(yp.hm, xp[j].mm, acc[i][j], 0, 0, 0);
#pragma unroll
        for (int j = 0; j < NJ; ++j)
          acc[i][j] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(yp.mh, xp[j].mm, acc[i][j], 0, 0, 0);
#pragma unroll
        for (int j = 0; j < NJ; ++j)
          acc[i][j] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(yp.mh, xp[j].hl, acc[i][j], 0, 0, 0);
#pragma unroll
        for (int j = 0; j < NJ; ++j)
          acc[i][j] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(yp.hm, xp[j].lh, acc[i][j], 0, 0, 0);
#pragma unroll
        for (int j = 0; j < NJ; ++j)
          acc[i][j] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(yp.hl, xp[j].hh, acc[i][j], 0, 0, 0);
#pragma unroll
        for (int j = 0; j < NJ; ++j)
          acc[i][j] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(yp.lh, xp[j].hh, acc[i][j], 0, 0, 0);
      };
#pragma unroll
      for (int i = 0; i < (NI < 4 ? NI : 4); ++i) tile(i);
      dw_load<NI, 0>(Y, ldy, rn, R, fr, ylim, y);
      if constexpr (NI > 4) {
#pragma unroll
        for (int i = 4; i < NI; ++i) tile(i);
        dw_load<NI, 1>(Y, ldy, rn, R, fr, ylim, y);
      }
    }
  };
  if constexpr (NW == 1) {
    steps(s0, s1);
#pragma unroll
    for (int a = 0; a < NI; ++a) {
#pragma unroll
      for (int b = 0; b < NJ; ++b)
#pragma unroll
        for (int r = 0; r < 4; ++r) store(dw_col<NI>(a, 4 * fg + r), dw_col<NJ>(b, fr), acc[a][b][r]);
      float v = cs[a];
      v += __shfl_xor(v, 16, 64);
      v += __shfl_xor(v, 32, 64);
      if (fg == 0 && grp == 0) bias(dw_col<NI>(a, fr), v);
    }
    if (bad != 0.f) again(0, 1);
    return;
  }
  // The waves' sums meet in LDS a tile row at a time (two buffers, so that one barrier a row is enough; one where the
  // totals leave no room), and a group's waves add its tiles in turn: every DW_SEGMENT steps of a wave to the
  // totals of the steps before, in LDS too, and store them after the last.
  constexpr int BUFS = G == 2 ? 1 : 2;
  float* lsum = lds + BUFS * 4 * 7 * 256;
  float* total = lsum + 7 * 4 * 64;
#pragma unroll 1
  for (int64_t begin = s0;; begin += NW * DW_SEGMENT) {
    const bool last = begin + NW * DW_SEGMENT >= s1;
    steps(begin, last ? s1 : begin + NW * DW_SEGMENT);
    int ln = lane;
    asm volatile("" : "+v"(ln));   // no address of what follows is kept through the steps' loop
    const int lr = ln & 15, lg = ln >> 4;
#pragma unroll
    for (int a = 0; a < NI; ++a) {
      float* buf = lds + a % BUFS * 4 * 7 * 256;
#pragma unroll
      for (int b = 0; b < NJ; ++b) *(f32x4*)(buf + ((wid * NJ + b) * 64 + ln) * 4) = acc[a][b];
      if (last) lsum[(a * 4 + wid) * 64 + ln] = cs[a];
      __syncthreads();
      for (int b = mine; b < NJ; b += NW) {
        f32x4 v = *(const f32x4*)(buf + ((grp * NJ + b) * 64 + ln) * 4);
#pragma unroll
        for (int l = 1; l < NW; ++l) v += *(const f32x4*)(buf + (((grp + G * l) * NJ + b) * 64 + ln) * 4);
        f32x4* t = (f32x4*)(total + (((a * G + grp) * NJ + b) * 64 + ln) * 4);   // this lane's alone
        if (begin > s0) v += *t;
        if (last) {
#pragma unroll
          for (int r = 0; r < 4; ++r) store(dw_col<NI>(a, 4 * lg + r), dw_col<NJ>(b, lr), v[r]);
        } else {
          *t = v;
        }
      }
      if (last && wid == 3) {   // the last wave: it has the fewest tiles; group 0's sums
        float v = lsum[a * 4 * 64 + ln];
#pragma unroll
        for (int l = 1; l < NW; ++l) v += lsum[(a * 4 + G * l) * 64 + ln];
        v += __shfl_xor(v, 16, 64);
        v += __shfl_xor(v, 32, 64);
        if (lg == 0) bias(dw_col<NI>(a, lr), v);
      }
      if (BUFS == 1) __syncthreads();
    }
    if (last) break;
    __syncthreads();   // the buffers are free for the next segment
  }
  if (bad != 0.f) again(mine, NW);
}

// Bytes of LDS for blocks of at most `steps` steps: buffers, the columns' sums and, past one segment, the totals
// (G column groups).  Without the totals a block finds room beside another kernel's: the link decoder's gradient beside
// the attention's backward, 4,000 events, 13 us, with them 29.
inline int dw_lds(int G, int64_t steps) {
  const bool totals = steps > 4 / G * DW_SEGMENT;
  return (int)sizeof(float) * ((totals && G == 2 ? 1 : 2) * 4 * 7 * 256 + 7 * 4 * 64 + (totals ? G * 7 * 7 * 256 : 0));
}

// The body for the tiles that n by m outputs take (n and m at most 112; m at most 64 with G = 4).
template <int G, class Out, class Bias>
__device__ __forceinline__ void dw_split_any(int n, int m, const float* Y, int64_t ldy, int ylim, const float* X,
                                             int64_t ldx, int xlim, int64_t R, int64_t s0, int64_t s1, float* lds,
                                             Out out, Bias bias) {
  auto run = [&](auto ni, auto nj) {
    dw_split<decltype(ni)::value, decltype(nj)::value, G>(Y, ldy, ylim, X, ldx, xlim, R, s0, s1, lds, out, bias);
  };
  auto cols = [&](auto ni) {
    if (m <= 32) run(ni, std::integral_constant<int, 2>{});
    else if (m <= 64) run(ni, std::integral_constant<int, 4>{});
    else if constexpr (G < 4) run(ni, std::integral_constant<int, 7>{});
  };
  if (n <= 32) cols(std::integral_constant<int, 2>{});
  else if (n <= 64) cols(std::integral_constant<int, 4>{});
  else cols(std::integral_constant<int, 7>{});
}

}  // namespace mtgnn
