// Stable counting sort of up to DS_MAX routing entries by expert in one
// workgroup of DS_THREADS threads (Algorithm 2's dispatch: the rows of one
// expert keep ascending (token, slot) order).  Device code shared by the
// dispatch kernel and the one-launch calibration of moe_route_rcep.
#pragma once

#include "common.hpp"

#include <type_traits>

namespace decomoe {
namespace {

constexpr int DS_THREADS = 1024;
constexpr int DS_WAVES = DS_THREADS / kWave;
constexpr int DS_R = 16;                      // rounds of 64 entries per wavefront
constexpr int DS_MAX = DS_THREADS * DS_R;     // entries it can hold

// The wavefronts take contiguous slices in entry order, in rounds of W <= 64:
// rounds per wavefront (the same for all) for A entries, and the first entry
// of this thread's wavefront.
__device__ __forceinline__ int slice_rounds(int A, int W = kWave) {
  return ((A + DS_WAVES - 1) / DS_WAVES + W - 1) / W;
}
__device__ __forceinline__ int slice_lo(int A, int nr, int W = kWave) {
  return min(A, (int)(threadIdx.x >> 6) * nr * W);
}

// Ranks of this wavefront's entries, in order: lanes with the same key are
// found with ballots over the key bits, a popcount gives each its rank, and
// `run` (this wavefront's next position per expert, in LDS) advances from
// round to round.  The ballots of up to four rounds are formed together, ahead
// of the chain through `run` (8192 entries: the whole sort 10.3 -> 8.6 us);
// a last one or two rounds are not filled up to four (2048 entries, two rounds, the
// whole sort with 1024 experts: 7.3 -> 6.4 us; forms for one and for three rounds
// too grow the code and were 1-4 % slower in the calibration).
// emit(round, position, key, lanes of this round with the same key) is called
// with position -1 for keys outside [0, E).
template <int R0, int Q, int R, class Emit>
__device__ __forceinline__ void rank_group(const int (&key)[R], int E, int key_bits, int* run, Emit& emit) {
  const int lane = threadIdx.x & 63;
  const uint64_t lt_mask = lane == 0 ? 0ull : (~0ull >> (64 - lane));
  uint64_t peers[Q];
#pragma unroll
  for (int q = 0; q < Q; ++q) peers[q] = __ballot(key[R0 + q] >= 0 && key[R0 + q] < E);
#pragma unroll 1
  for (int b = 0; b < key_bits; ++b)
#pragma unroll
    for (int q = 0; q < Q; ++q) {
      const bool bit = (key[R0 + q] >> b) & 1;
      const uint64_t m = __ballot(bit);
      peers[q] &= bit ? m : ~m;
    }
#pragma unroll
  for (int q = 0; q < Q; ++q) {
    const int e = key[R0 + q];
    int pos = -1;
    if (e >= 0 && e < E) {
      const int at = run[e];
      pos = at + __popcll(peers[q] & lt_mask);
      // the highest lane of the group advances the expert's counter
      if ((63 - __clzll(peers[q])) == lane) run[e] = at + __popcll(peers[q]);
    }
    __builtin_amdgcn_wave_barrier();
    emit(R0 + q, pos, e, peers[q]);
  }
}
template <int R, int R0 = 0, class Emit>
__device__ __forceinline__ void rank_rounds(const int (&key)[R], int nr, int E, int key_bits, int* run, Emit emit) {
  if constexpr (R0 < R) {
    const int left = nr - R0;
    if (left <= 0) return;
    if constexpr (R - R0 < 4) {
      rank_group<R0, 1>(key, E, key_bits, run, emit);
      rank_rounds<R, R0 + 1>(key, nr, E, key_bits, run, emit);
    } else {
      if (left <= 2)
        rank_group<R0, 2>(key, E, key_bits, run, emit);
      else
        rank_group<R0, 4>(key, E, key_bits, run, emit);
      rank_rounds<R, R0 + 4>(key, nr, E, key_bits, run, emit);
    }
  }
}

// Per-wavefront counts of the keys in wh (DS_WAVES rows of ld >= E ints),
// turned into each wavefront's first position per expert by one scan over the
// experts; thread e < E gets its expert's count and first position.
template <int R>
__device__ __forceinline__ void slice_scan(const int (&key)[R], int nr, int E, int* wh, int ld, int* part, int& cnt,
                                           int& first) {
  const int tid = threadIdx.x, lane = tid & 63, wv = tid >> 6;
  for (int i = tid; i < DS_WAVES * ld; i += DS_THREADS) wh[i] = 0;
  __syncthreads();
#pragma unroll
  for (int r = 0; r < R; ++r)
    if (r < nr && key[r] >= 0 && key[r] < E) atomicAdd(&wh[wv * ld + key[r]], 1);
  __syncthreads();
  int c[DS_WAVES];
  cnt = 0;
  if (tid < E) {
#pragma unroll
    for (int w = 0; w < DS_WAVES; ++w) c[w] = wh[w * ld + tid];
#pragma unroll
    for (int w = 0; w < DS_WAVES; ++w) cnt += c[w];
  }
  int incl = cnt;
#pragma unroll
  for (int off = 1; off < kWave; off <<= 1) {
    const int y = __shfl_up(incl, off, kWave);
    if (lane >= off) incl += y;
  }
  if (lane == kWave - 1) part[wv] = incl;
  __syncthreads();
  first = incl - cnt;
  for (int w = 0; w < wv; ++w) first += part[w];
  if (tid < E) {
    int r = first;
#pragma unroll
    for (int w = 0; w < DS_WAVES; ++w) {
      wh[w * ld + tid] = r;
      r += c[w];
    }
  }
  __syncthreads();
}

// f(R) with R = the smallest of 1, 4 and MAX rounds that hold nr: short slices
// pay for no rounds that they do not have (256 entries: sort 3.9 -> 2.0 us)
template <int MAX, class F>
__device__ __forceinline__ void with_rounds(int nr, F f) {
  if (nr <= 1)
    f(std::integral_constant<int, 1>{});
  else if (nr <= 4)
    f(std::integral_constant<int, 4>{});
  else
    f(std::integral_constant<int, MAX>{});
}

// All DS_THREADS threads call it.  keys[a] is the expert of entry a (global
// or LDS memory); entries outside [0, E) are dropped (row_of_slot = -1).
// R: rounds per wavefront that the slices of A entries fit.
template <int R>
__device__ __forceinline__ void sort_rounds(const int32_t* keys, int A, int E, int key_bits, int* wh, int* part,
                                            int32_t* __restrict__ counts, int32_t* __restrict__ offsets,
                                            int32_t* __restrict__ src_of_row, int32_t* __restrict__ row_of_slot) {
  const int tid = threadIdx.x, lane = tid & 63, wv = tid >> 6;
  const int nr = slice_rounds(A), lo = slice_lo(A, nr), hi = min(A, lo + nr * kWave);
  int key[R];
#pragma unroll
  for (int r = 0; r < R; ++r) {
    const int a = lo + r * kWave + lane;
    key[r] = r < nr && a < hi ? keys[a] : -1;
  }
  int cnt, first;
  slice_scan<R>(key, nr, E, wh, E, part, cnt, first);
  if (tid < E) {
    counts[tid] = cnt;
    offsets[tid] = first;
    if (tid == E - 1) offsets[E] = first + cnt;
  }
  rank_rounds<R>(key, nr, E, key_bits, wh + wv * E, [&](int r, int pos, int, uint64_t) {
    const int a = lo + r * kWave + lane;
    if (a >= hi) return;
    row_of_slot[a] = pos;
    if (pos >= 0) src_of_row[pos] = a;
  });
}
// wh: DS_WAVES rows of E ints
__device__ __forceinline__ void sort_small(const int32_t* keys, int A, int E, int key_bits, int* wh, int* part,
                           int32_t* __restrict__ counts, int32_t* __restrict__ offsets,
                           int32_t* __restrict__ src_of_row, int32_t* __restrict__ row_of_slot) {
  with_rounds<DS_R>(slice_rounds(A), [&](auto RC) {
    sort_rounds<decltype(RC)::value>(keys, A, E, key_bits, wh, part, counts, offsets, src_of_row, row_of_slot);
  });
}

}  // namespace
}  // namespace decomoe
