// Wavefront Top-k primitives shared by the routing kernels (Eq. 10 and the
// prefix re-route of Sec. 3.3): a total order on (value, index) pairs, DPP
// arg-max and sum over a wavefront, and the selection of the k best of one
// token's first Klim logits with their softmax weights.
#pragma once

#include <float.h>

#include "common.hpp"

namespace decomoe {
namespace {

// A candidate (value, expert) as one 64-bit key whose unsigned order is the
// selection's order -- value descending, index ascending on ties -- so that a
// comparison is one instruction without mask arithmetic between the scalar and
// vector units.  High word: the float's bits mapped to unsigned order (-0 as
// +0); low word: 0x7fffffff - e.  Key 0: taken, absent or NaN (never chosen
// while a candidate is left; reads back as -inf, 0x7fffffff).
// (Top-k of 64 tokens, E 128, k 8, one wavefront per token: 4.4 -> 3.6 us.)
typedef unsigned long long tkey;
__device__ __forceinline__ tkey topk_key(float v, int e) {
  uint32_t u = __float_as_uint(v + 0.f);
  u ^= static_cast<uint32_t>(static_cast<int32_t>(u) >> 31) | 0x80000000u;
  const tkey q = (static_cast<tkey>(u) << 32) | static_cast<uint32_t>(0x7fffffff - e);
  return v == v ? q : 0ull;
}
__device__ __forceinline__ int key_index(tkey q) { return 0x7fffffff - static_cast<int>(static_cast<uint32_t>(q)); }
__device__ __forceinline__ float key_value(tkey q) {
  const uint32_t u = static_cast<uint32_t>(q >> 32);
  const float v = __uint_as_float(u & 0x80000000u ? u ^ 0x80000000u : ~u);
  return q ? v : -INFINITY;
}
__device__ __forceinline__ tkey key_max(tkey a, tkey b) { return a > b ? a : b; }

// The same order for more than TOPK_KEYS values per lane, where the selection is
// bound by its instructions and 64-bit compares are slow: the float mapped to a
// signed int, its maximum first and then the lowest index that holds it.
// TOPK_NONE: taken, absent or NaN.  (8192 tokens on given logits, one row of 16
// lanes per token, against keys: E 128, k 8 5.1 -> 4.3 us; E 256, k 16 20.4 ->
// 8.6; one wavefront per token, E 512, k 8: 19.4 -> 14.7.  Up to TOPK_KEYS
// values a round is one chain of DPP moves instead of two.)
constexpr int TOPK_KEYS = 4;
constexpr int TOPK_NONE = -0x7fffffff - 1;
__device__ __forceinline__ int topk_ord(float v) {
  int s = __float_as_int(v + 0.f);
  s ^= (s >> 31) & 0x7fffffff;
  return v == v ? s : TOPK_NONE;
}
__device__ __forceinline__ tkey ord_key(int s, int e) {  // as topk_key
  return s == TOPK_NONE ? 0ull
                        : (static_cast<tkey>(static_cast<uint32_t>(s) ^ 0x80000000u) << 32) |
                              static_cast<uint32_t>(0x7fffffff - e);
}

// the best key of a row of 16 lanes in all its lanes, by DPP moves (quad
// swaps, then the half-row and row mirrors pair the groups); the wavefront's
// best: the four row results read with v_readlane (the same in every lane)
template <int CTRL>
__device__ __forceinline__ float dpp_f(float v) {
  return __builtin_bit_cast(float, __builtin_amdgcn_mov_dpp(__builtin_bit_cast(int, v), CTRL, 0xF, 0xF, false));
}
template <int CTRL>
__device__ __forceinline__ tkey dpp_max(tkey q) {
  const int lo = __builtin_amdgcn_mov_dpp(static_cast<int>(q), CTRL, 0xF, 0xF, false);
  const int hi = __builtin_amdgcn_mov_dpp(static_cast<int>(q >> 32), CTRL, 0xF, 0xF, false);
  return key_max(q, (static_cast<tkey>(static_cast<uint32_t>(hi)) << 32) | static_cast<uint32_t>(lo));
}
__device__ __forceinline__ float lane_f(float v, int l) {
  return __builtin_bit_cast(float, __builtin_amdgcn_readlane(__builtin_bit_cast(int, v), l));
}
__device__ __forceinline__ tkey row_best(tkey q) {
  q = dpp_max<0xB1>(q);   // quad_perm [1, 0, 3, 2]
  q = dpp_max<0x4E>(q);   // quad_perm [2, 3, 0, 1]
  q = dpp_max<0x141>(q);  // row_half_mirror
  return dpp_max<0x140>(q);  // row_mirror
}
__device__ __forceinline__ tkey wave_best(tkey q) {
  q = row_best(q);
  tkey best = 0;
#pragma unroll
  for (int r = 0; r < 4; ++r) {
    const uint32_t lo = __builtin_amdgcn_readlane(static_cast<int>(q), 16 * r);
    const uint32_t hi = __builtin_amdgcn_readlane(static_cast<int>(q >> 32), 16 * r);
    best = key_max(best, (static_cast<tkey>(hi) << 32) | lo);
  }
  return best;
}
template <int CTRL>
__device__ __forceinline__ int dpp_i(int v) {
  return __builtin_amdgcn_mov_dpp(v, CTRL, 0xF, 0xF, false);
}
__device__ __forceinline__ int row_max(int v) {
  v = max(v, dpp_i<0xB1>(v));
  v = max(v, dpp_i<0x4E>(v));
  v = max(v, dpp_i<0x141>(v));
  return max(v, dpp_i<0x140>(v));
}
__device__ __forceinline__ int row_min(int v) {
  v = min(v, dpp_i<0xB1>(v));
  v = min(v, dpp_i<0x4E>(v));
  v = min(v, dpp_i<0x141>(v));
  return min(v, dpp_i<0x140>(v));
}

// One lane's candidates (value c is expert j + STRIDE c) and their rounds: best()
// returns the best one of the row of 16 lanes (STRIDE 16) or of the wavefront
// (STRIDE 64) and takes it out.
template <int MAXC, int STRIDE, bool KEYS = (MAXC <= TOPK_KEYS)>
struct Candidates {
  tkey q[MAXC];
  __device__ __forceinline__ void set(int c, float v, int e, bool in) { q[c] = in ? topk_key(v, e) : 0ull; }
  __device__ __forceinline__ tkey best(int) {
    tkey b = q[0];
#pragma unroll
    for (int c = 1; c < MAXC; ++c) b = key_max(b, q[c]);
    b = STRIDE == 16 ? row_best(b) : wave_best(b);
#pragma unroll
    for (int c = 0; c < MAXC; ++c) q[c] = q[c] == b ? 0ull : q[c];
    return b;
  }
};
template <int MAXC, int STRIDE>
struct Candidates<MAXC, STRIDE, false> {
  int s[MAXC];
  __device__ __forceinline__ void set(int c, float v, int, bool in) { s[c] = in ? topk_ord(v) : TOPK_NONE; }
  __device__ __forceinline__ tkey best(int j) {
    int b = s[0];
#pragma unroll
    for (int c = 1; c < MAXC; ++c) b = max(b, s[c]);
    b = row_max(b);
    if (STRIDE == 64)
      b = max(max(__builtin_amdgcn_readlane(b, 0), __builtin_amdgcn_readlane(b, 16)),
              max(__builtin_amdgcn_readlane(b, 32), __builtin_amdgcn_readlane(b, 48)));
    int lo = 0x7fffffff, hi = 0x7fffffff;  // two chains
#pragma unroll
    for (int c = MAXC / 2 - 1; c >= 0; --c) {
      lo = s[c] == b ? j + STRIDE * c : lo;
      hi = s[c + MAXC / 2] == b ? j + STRIDE * (c + MAXC / 2) : hi;
    }
    int e = row_min(min(lo, hi));
    if (STRIDE == 64)
      e = min(min(__builtin_amdgcn_readlane(e, 0), __builtin_amdgcn_readlane(e, 16)),
              min(__builtin_amdgcn_readlane(e, 32), __builtin_amdgcn_readlane(e, 48)));
#pragma unroll
    for (int c = 0; c < MAXC; ++c) s[c] = j + STRIDE * c == e ? TOPK_NONE : s[c];
    return ord_key(b, e);
  }
};

// sum over the wavefront: row sums by DPP, then the four rows in order
__device__ __forceinline__ float wave_sum(float v) {
  v += dpp_f<0xB1>(v);
  v += dpp_f<0x4E>(v);
  v += dpp_f<0x141>(v);
  v += dpp_f<0x140>(v);
  return ((lane_f(v, 0) + lane_f(v, 16)) + lane_f(v, 32)) + lane_f(v, 48);
}

// The k largest of one token's logits [0, Klim), one wavefront: lane l
// holds experts l, l + 64, ... in vals[c] (expert l + 64 c); k rounds of a
// wavefront arg-max (value descending, index ascending on ties) pick the
// slots in order; the weights are the softmax of the k selected logits.
// Lane r < k writes slot r.  Values at experts >= Klim are never selected.
template <int MAXC>  // values per lane: E <= 64 MAXC
__device__ __forceinline__ void topk_select_vals(const float (&vals)[MAXC], int E, int k, int Klim, int lane,
                                                 int32_t* idx_t, float* w_t) {
  Candidates<MAXC, 64> cand;
#pragma unroll
  for (int c = 0; c < MAXC; ++c) cand.set(c, vals[c], lane + c * 64, lane + c * 64 < Klim);
  tkey mine = 0;
  for (int r = 0; r < k; ++r) {
    const tkey best = cand.best(lane);
    if (lane == r) mine = best;
  }
  const float my_v = key_value(mine);
  const int my_i = key_index(mine);
  const float v0 = __builtin_bit_cast(float, __builtin_amdgcn_readlane(__builtin_bit_cast(int, my_v), 0));
  float ex = lane < k ? expf(my_v - v0) : 0.f;
  float sum = ex;
  sum = wave_sum(sum);
  if (lane < k) {
    idx_t[lane] = my_i;
    w_t[lane] = ex / sum;
  }
}

// the same on row[0, Klim) in memory
template <int MAXC>
__device__ __forceinline__ void topk_select(const float* row, int E, int k, int Klim, int lane,
                                            int32_t* idx_t, float* w_t) {
  float v[MAXC];
#pragma unroll
  for (int c = 0; c < MAXC; ++c) {
    const int e = lane + c * 64;
    v[c] = e < Klim ? row[e] : 0.f;
  }
  topk_select_vals<MAXC>(v, E, k, Klim, lane, idx_t, w_t);
}

// ---- one token per row of 16 lanes (four tokens per wavefront) ---------
__device__ __forceinline__ float row_sum(float v) {
  v += dpp_f<0xB1>(v);
  v += dpp_f<0x4E>(v);
  v += dpp_f<0x141>(v);
  v += dpp_f<0x140>(v);
  return v;
}

// The k best of one token's logits [0, Klim) held by the 16 lanes of a row:
// lane j holds experts j, j + 16, ... in v[c] (expert j + 16 c).  Each
// round's arg-max is a lane-local scan plus DPP moves within the row; round r's winner is
// kept by lane r % 16 in slot r / 16 (k <= 32).  Same selection order, tie
// rule and weights as topk_select_vals: the slots' exponentials are summed
// by the same butterfly, so for k <= 16 the weights are bitwise equal.
template <int MAXC>
__device__ __forceinline__ void row_topk_select(const float (&v)[MAXC], int j, int E, int k, int Klim,
                                                int32_t* idx_t, float* w_t) {
  Candidates<MAXC, 16> cand;
#pragma unroll
  for (int c = 0; c < MAXC; ++c) cand.set(c, v[c], j + 16 * c, j + 16 * c < Klim);
  tkey mine[2] = {0, 0};
  float v0 = 0.f;
  for (int r = 0; r < k; ++r) {
    const tkey best = cand.best(j);
    if (r == 0) v0 = key_value(best);
    if ((r & 15) == j) mine[r >> 4] = best;
  }
  const float my_v[2] = {key_value(mine[0]), key_value(mine[1])};
  const int my_i[2] = {key_index(mine[0]), key_index(mine[1])};
  float ex[2];
#pragma unroll
  for (int q = 0; q < 2; ++q) ex[q] = j + 16 * q < k ? expf(my_v[q] - v0) : 0.f;
  // slots in order r = 0..k-1: lanes hold r = j and r = j + 16; the row sum
  // adds the k exponentials (the same total in every lane of the row)
  const float sum = row_sum(ex[0] + ex[1]);
#pragma unroll
  for (int q = 0; q < 2; ++q) {
    const int r = j + 16 * q;
    if (r < k) {
      idx_t[r] = my_i[q];
      w_t[r] = ex[q] / sum;
    }
  }
}

}  // namespace
}  // namespace decomoe
