// Activated mass of one invocation and its prefix length (Eqs. 11, 12):
// device code shared by the calibration kernel and the fused calibration +
// prefix re-route kernel.  Every function here is called by all
// CAL_THREADS threads of the workgroup (they synchronise it).
//
//   mass_sorted   where cal_sorted() holds (up to CAL_SORT_A routing entries and
//                 E <= CAL_SORT_E): the entries are loaded into registers and
//                 their weights grouped by expert with a stable counting sort
//                 in LDS (token order kept within an expert); thread e adds its
//                 expert's weights in that order
//   mass_chunked  larger invocations: chunks of tokens are scattered into a
//                 dense LDS table [token][expert] (float64) and thread e
//                 adds column e in ascending token order
// Either way one float64 running sum per expert over the tokens: the
// sequence of additions of the plain definition (unrouted tokens add zeros,
// which change nothing).  An expert repeated within a token: up to CAL_STAGE
// entries its weights are added one by one, beyond they are summed within the
// token first, on either path.
//   prefix_K      the running sum c_K over the experts by one wavefront, then
//                 the first K with c_K >= p * c_E by a ballot; K = max(k, K)
#pragma once

#include "common.hpp"
#include "sort_dev.hpp"

namespace decomoe {
namespace {

constexpr int CAL_THREADS = 1024;
constexpr int CAL_TABLE = 8192;  // doubles in the LDS table (64 KB)
constexpr int CAL_STAGE = 8192;  // routing entries staged per bulk load (64 KB)
constexpr int CAL_ENT = 1024;    // routing entries scattered per chunk (one per thread)
constexpr int CAL_WAVES = CAL_THREADS / kWave;
constexpr int CAL_SORT_A = DS_MAX;  // routing entries of the sorted path
constexpr int CAL_SORT_E = 512;  // the sorted path keeps [waves][E] counts in the table

// Whether n_all = tokens * k entries take the sorted path.  Beyond CAL_STAGE
// entries its rounds hold whole tokens.  The dense table has one addition per
// token where the sorted path has one per entry of an expert, so it stays ahead
// where few tokens make many entries (calibration + re-route of 262 tokens, k 32:
// E 32 24.7 us against 26.6, E 256 31.5 against 34.1, E 512 51.9 against 43.9;
// 525 tokens, k 16: E 32 25.3 against 24.1, E 256 32.6 against 32.3).
// (Rounds for all CAL_SORT_A entries where k does not divide 64, up to 24, spill.)
__host__ __device__ inline bool cal_sorted(size_t n_all, int E, int k) {
  if (E > CAL_SORT_E) return false;
  if (n_all <= (size_t)CAL_STAGE) return true;
  return (k <= 16 || E > 256) && n_all <= (size_t)(CAL_SORT_A / kWave) * (kWave / k * k);
}

// Tokens per chunk: the table holds ch x E doubles and a chunk holds at most
// CAL_ENT routing entries.
__host__ __device__ inline int cal_chunk(int E, int k) {
  int c = CAL_TABLE / E;
  if (c * k > CAL_ENT) c = CAL_ENT / k;
  return c < 64 ? c : 64;
}

static_assert(CAL_THREADS == DS_THREADS && CAL_SORT_A <= 2 * CAL_STAGE && CAL_WAVES * CAL_SORT_E <= 2 * CAL_TABLE &&
                  CAL_STAGE == DS_MAX / 2,
              "the sorted path's arrays fit");
struct CalLds {
  double table[CAL_TABLE];
  double smass[1024 + 32];  // zero past E (the c_K loop reads whole batches)
  int st_e[CAL_STAGE];  // mass_sorted: with st_w the CAL_SORT_A grouped weights
  float st_w[CAL_STAGE];
  int part[CAL_WAVES];
  int repeats;  // mass_sorted: a token names an expert twice
  int s_K;
};

// The masses of the tokens [lo, hi), any size: sets L.smass[e] = the mass of
// expert e (zero past E) and returns it in thread e < E.
__device__ double mass_chunked(const int32_t* __restrict__ idx, const float* __restrict__ w, int lo, int hi,
                               int E, int k, CalLds& L) {
  const int tid = threadIdx.x;
  const int ch = cal_chunk(E, k);
  const int super_t = (CAL_STAGE / k) / ch * ch;  // tokens staged per bulk load
  for (int i = tid; i < ch * E; i += CAL_THREADS) L.table[i] = 0.0;
  double acc = 0.0;
  for (int s0 = lo; s0 < hi; s0 += super_t) {
    // stage the routing entries of up to super_t tokens with one bulk load
    const int n_ent = min(super_t, hi - s0) * k;
    __syncthreads();  // previous stage fully consumed
    {
      constexpr int SPT = CAL_STAGE / CAL_THREADS;  // all loads in flight together
      int re[SPT];
      float rw[SPT];
#pragma unroll
      for (int q = 0; q < SPT; ++q) {
        const int i = tid + q * CAL_THREADS;
        re[q] = i < n_ent ? idx[(size_t)s0 * k + i] : -1;
        rw[q] = i < n_ent ? w[(size_t)s0 * k + i] : 0.f;
      }
#pragma unroll
      for (int q = 0; q < SPT; ++q) {
        L.st_e[tid + q * CAL_THREADS] = re[q];
        L.st_w[tid + q * CAL_THREADS] = rw[q];
      }
    }
    __syncthreads();
    for (int t0 = s0; t0 < min(s0 + super_t, hi); t0 += ch) {
      const int nt = min(ch, hi - t0);
      // scatter: a token's experts are distinct (Top-k), so each cell gets
      // one addition onto 0.0 and holds the weight exactly; a repeated
      // expert adds its weights into the cell
#pragma unroll
      for (int q = 0; q < CAL_ENT / CAL_THREADS; ++q) {
        const int j = tid + q * CAL_THREADS;
        if (j < nt * k) {
          const int i = (t0 - s0) * k + j;
          const int e = L.st_e[i];
          if (e >= 0 && e < E) atomicAdd(&L.table[(j / k) * E + e], static_cast<double>(L.st_w[i]));
        }
      }
      __syncthreads();
      // column sums: thread e adds column e in ascending token order, then
      // clears it for the next chunk
      if (tid < E) {
        double a = acc;
#pragma unroll 8
        for (int r = 0; r < nt; ++r) {
          a += L.table[r * E + tid];
          L.table[r * E + tid] = 0.0;
        }
        acc = a;
      }
      __syncthreads();
    }
  }
  if (tid < E) {
    L.smass[tid] = acc;
  } else {
    L.smass[tid] = 0.0;
  }
  if (tid < 32) L.smass[1024 + tid] = 0.0;
  __syncthreads();
  return acc;
}

// The same from this thread's entries (key, weight) in the slices of
// sort_dev.hpp; `sorted` (LDS) holds the weights grouped by expert.
// REPEATS: rounds hold whole tokens and repeated experts are looked for, token_mask
// being the earlier lanes of this lane's token (L.repeats is then set if a token
// names an expert twice, and the masses are not what is wanted).
template <int R, bool REPEATS = false>
__device__ __forceinline__ double mass_of_entries(const int (&key)[R], const float (&rw)[R], int nr, int E,
                                                  int key_bits, float* sorted, CalLds& L, uint64_t token_mask = 0) {
  const int tid = threadIdx.x, wv = tid >> 6;
  int* wh = reinterpret_cast<int*>(L.table);  // [waves][E]
  uint64_t again = 0;
  int cnt, first;
  slice_scan<R>(key, nr, E, wh, E, L.part, cnt, first);
  rank_rounds<R>(key, nr, E, key_bits, wh + wv * E, [&](int r, int pos, int, uint64_t peers) {
    if (pos >= 0) sorted[pos] = rw[r];
    if constexpr (REPEATS) again |= pos >= 0 ? peers & token_mask : 0;
  });
  if (REPEATS && again) L.repeats = 1;
  __syncthreads();
  double a = 0.0;
  if (tid < E) {
    // one dependent float64 chain per expert (the latency of the
    // additions, not of the LDS reads, bounds it)
#pragma unroll 8
    for (int j = first; j < first + cnt; ++j) a += static_cast<double>(sorted[j]);
    L.smass[tid] = a;
  } else {
    L.smass[tid] = 0.0;
  }
  if (tid < 32) L.smass[1024 + tid] = 0.0;
  __syncthreads();
  return a;
}

// The masses of the n_all routing entries of the tokens from lo_t on (where
// cal_sorted() holds), each wavefront loading its own slice into registers.
__device__ __forceinline__ double mass_sorted(const int32_t* __restrict__ idx, const float* __restrict__ w, int lo_t,
                                              int n_all, int E, int k, int key_bits, CalLds& L) {
  const int lane = threadIdx.x & 63;
  const size_t base = (size_t)lo_t * k;
  double mass = 0.0;
  auto run = [&](auto RC, auto REP, int W, int nr, uint64_t token_mask) {
    constexpr int R = decltype(RC)::value;
    const int lo = slice_lo(n_all, nr, W), hi = lane < W ? min(n_all, lo + nr * W) : 0;
    int key[R];
    float rw[R];
#pragma unroll
    for (int r = 0; r < R; ++r) {
      const int a = lo + r * W + lane;
      const bool in = r < nr && a < hi;
      key[r] = in ? idx[base + a] : -1;
      rw[r] = in ? w[base + a] : 0.f;
    }
    mass = mass_of_entries<R, decltype(REP)::value>(key, rw, nr, E, key_bits, reinterpret_cast<float*>(L.st_e), L,
                                                    token_mask);
  };
  if (n_all <= CAL_STAGE) {
    const int nr = slice_rounds(n_all);
    with_rounds<DS_R / 2>(nr, [&](auto RC) { run(RC, std::false_type{}, kWave, nr, 0); });
  } else {
    // beyond CAL_STAGE entries: rounds of whole tokens (64 entries where k
    // divides 64), so that a token's repeated experts meet in one round
    if (threadIdx.x == 0) L.repeats = 0;  // (slice_scan's barriers order it before the ranks)
    const int W = kWave / k * k;
    run(std::integral_constant<int, DS_R>{}, std::true_type{}, W, slice_rounds(n_all, W),
        ((1ull << lane) - 1) & ~((1ull << (lane - lane % k)) - 1));
    if (L.repeats) mass = mass_chunked(idx, w, lo_t, lo_t + n_all / k, E, k, L);
  }
  return mass;
}

// K = max(k, the first K with c_K >= p * c_E) from L.smass, in every thread.
// c_K is one running sum in expert order (the definition's sequence of
// float64 additions): in wavefront 0, lane l of a block of 64 experts adds the
// masses of the experts up to its own, the others adding +0.0, which changes
// no bit of a non-negative sum -- so all 64 c_K come out of one chain with no
// store between its additions (128 experts: 2.1 -> 1.7 us), and a ballot finds
// the first with c_K >= p * c_E.
__device__ int prefix_K(int E, int k, double p, CalLds& L) {
  const int tid = threadIdx.x;
  double* cbuf = L.table;  // free once the masses are formed
  if (tid < kWave) {
    constexpr int B = 16;
    double base = 0.0;
    for (int e0 = 0; e0 < E; e0 += kWave) {
      double c = base, v[B], nv[B];
#pragma unroll
      for (int u = 0; u < B; ++u) v[u] = L.smass[e0 + u];
#pragma unroll
      for (int j0 = 0; j0 < kWave; j0 += B) {
#pragma unroll
        for (int u = 0; u < B; ++u) nv[u] = L.smass[e0 + j0 + B + u];  // (zero past E, padded by 32)
#pragma unroll
        for (int u = 0; u < B; ++u) c += j0 + u <= tid ? v[u] : 0.0;
#pragma unroll
        for (int u = 0; u < B; ++u) v[u] = nv[u];
      }
      cbuf[e0 + tid] = c;
      base = __shfl(c, kWave - 1, kWave);
    }
    // the masses past E are zero: base = c_E
    const double thr = p * base;
    int k_hat = E;
    for (int e0 = 0; e0 < E; e0 += kWave) {
      const unsigned long long hit = __ballot(e0 + tid < E && cbuf[e0 + tid] >= thr);
      if (hit) {
        k_hat = e0 + __ffsll((long long)hit);  // K = index + 1
        break;
      }
    }
    if (tid == 0) L.s_K = k_hat > k ? k_hat : k;
  }
  __syncthreads();
  return L.s_K;
}

}  // namespace
}  // namespace decomoe
