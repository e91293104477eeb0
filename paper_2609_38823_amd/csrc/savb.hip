// SAVB exit gate (Sec. 3.2, Eqs. 2 and 3) and the flag-driven visual-block
// removal.
//
//   pool     the n - 1 preceding text rows are summed per column in float32,
//            rows split over blockIdx.y (each split sums its rows in order)
//   mlp      every workgroup forms the feature x = [sum / (n - 1); row n - 1]
//            in LDS (the splits added in order, then one scaling) while its
//            first weights are on their way, and each wavefront hidden units
//            relu(W1[u] . x + b1[u]); the last workgroup to finish forms
//            the two class logits, p_exit = softmax(z)_1 and the exit flag
//            p_exit >= theta (compared in float64)
// Every sum has a fixed order, so the gate is deterministic.  The gate is
// bound by its launches and their dependent loads: two launches instead of
// four (feature and decision on their own): gate over 512 rows, d 2048, 512
// hidden units, and the drop behind it: 32.5 -> 21.4 us.
#include "common.hpp"

#include <algorithm>

namespace decomoe {
namespace {

constexpr int SG_ROWS = 32;  // rows per pooling split until there are 16 splits
// Workgroups of savb_mlp_kernel: each forms the feature and adds one count at
// the one address, so beyond a few hundred hidden units the wavefronts take
// several units each (512 rows, d 256, 8192 units: 62 us with one unit per
// wavefront, 30 with 256 workgroups; four launches with the feature formed
// once took 40.  d 2048, 2048 units: 23.0, 21.4 and 28.2; d 8192, 8192 units:
// 161, 126 and 211.  128 or 512 workgroups: d 2048, 2048 units 23.8, 23.0).
constexpr unsigned SG_WGS = 256;

int savb_splits(int n) {
  const int rows = n - 1;
  if (rows <= 0) return 0;
  int s = (rows + SG_ROWS - 1) / SG_ROWS;
  return s > 16 ? 16 : s;
}

// partial[s][c] = sum of rows [s*per, (s+1)*per) of column c (rows < n - 1)
template <bool BF16>
__global__ __launch_bounds__(256) void savb_pool_kernel(const void* __restrict__ rows, int n, int d,
                                                        int per, float* __restrict__ partial, int* __restrict__ ctr, const Guard g) {
  if (guard_skip(g)) return;
  if (blockIdx.x == 0 && blockIdx.y == 0 && threadIdx.x == 0) *ctr = 0;  // the workgroups the next launch finishes
  if (n < 2) return;  // no preceding rows
  const int c = blockIdx.x * 256 + threadIdx.x;
  if (c >= d) return;
  const int r0 = blockIdx.y * per, r1 = min(n - 1, r0 + per);
  float acc = 0.f;
  int r = r0;
  for (; r + 8 <= r1; r += 8) {  // eight loads in flight, added in row order
    float v[8];
#pragma unroll
    for (int u = 0; u < 8; ++u)
      v[u] = BF16 ? bf16_to_f32(static_cast<const uint16_t*>(rows)[(size_t)(r + u) * d + c])
                  : static_cast<const float*>(rows)[(size_t)(r + u) * d + c];
#pragma unroll
    for (int u = 0; u < 8; ++u) acc += v[u];
  }
  for (; r < r1; ++r)
    acc += BF16 ? bf16_to_f32(static_cast<const uint16_t*>(rows)[(size_t)r * d + c])
                : static_cast<const float*>(rows)[(size_t)r * d + c];
  partial[(size_t)blockIdx.y * d + c] = acc;
}

// the value of text row n - 1 at column c
template <bool BF16>
__device__ __forceinline__ float last_row(const void* rows, int n, int d, int c) {
  return BF16 ? bf16_to_f32(static_cast<const uint16_t*>(rows)[(size_t)(n - 1) * d + c])
              : static_cast<const float*>(rows)[(size_t)(n - 1) * d + c];
}

// PRE: 16-byte weight loads per lane that are in flight ahead of a unit; MULTI:
// several units per wavefront
template <bool BF16, int PRE, bool MULTI>
__global__ __launch_bounds__(256) void savb_mlp_kernel(
    const void* __restrict__ rows, int n, int d, int splits, const float* __restrict__ partial,
    float* __restrict__ feature, const float* __restrict__ w1, const float* __restrict__ b1, int hid,
    float* __restrict__ hidden, const float* __restrict__ w2, const float* __restrict__ b2, double theta,
    float* __restrict__ p_exit, int32_t* __restrict__ exit_flag, int32_t* __restrict__ exit_layer, int layer,
    int* __restrict__ ctr, const Guard g) {
  if (guard_skip(g)) return;
  extern __shared__ __attribute__((aligned(16))) float xs[];  // [2d], 64 KB at d = 8192: the last steps reuse it
  const int tid = threadIdx.x, lane = tid & 63, wv = tid >> 6;
  // 16-byte weight loads: lane l takes columns 4 (l + 64 j) .. + 4 for j = 0,
  // 1, ...; the first PRE of a unit (and its bias) are issued before x is
  // formed, or before the previous unit's are used
  const bool vec = (d & 127) == 0 && (reinterpret_cast<uintptr_t>(w1) & 15) == 0;
  const int n4 = (2 * d) >> 2;
  float4 v[PRE];
  float bu = 0.f;
  auto first_weights = [&](int u) {
    u = min(u, hid - 1);
    const float4* w4 = reinterpret_cast<const float4*>(w1 + (size_t)u * 2 * d);
    if (b1) bu = b1[u];
#pragma unroll
    for (int q = 0; q < PRE; ++q) {
      const int j = lane + 64 * q;
      v[q] = vec && j < n4 ? w4[j] : make_float4(0.f, 0.f, 0.f, 0.f);
    }
  };
  first_weights(blockIdx.x * 4 + wv);
  const float bz = b2 ? b2[wv & 1] : 0.f;
  const float inv = n > 1 ? 1.f / static_cast<float>(n - 1) : 0.f;
  if ((d & 3) == 0) {  // the partials' rows are whole 16-byte vectors (the workspace is 16-byte aligned)
    for (int c = 4 * tid; c < d; c += 1024) {
      float4 pv[16];
#pragma unroll
      for (int q = 0; q < 16; ++q)
        pv[q] = q < splits ? *reinterpret_cast<const float4*>(partial + (size_t)q * d + c)
                           : make_float4(0.f, 0.f, 0.f, 0.f);
      float4 s = make_float4(0.f, 0.f, 0.f, 0.f);
#pragma unroll
      for (int q = 0; q < 16; ++q)
        if (q < splits) {
          s.x += pv[q].x;
          s.y += pv[q].y;
          s.z += pv[q].z;
          s.w += pv[q].w;
        }
      *reinterpret_cast<float4*>(xs + c) = n > 1 ? make_float4(s.x * inv, s.y * inv, s.z * inv, s.w * inv)
                                                 : make_float4(0.f, 0.f, 0.f, 0.f);
#pragma unroll
      for (int e = 0; e < 4; ++e) xs[d + c + e] = last_row<BF16>(rows, n, d, c + e);
    }
  } else {
    for (int c = tid; c < d; c += 256) {
      float s = 0.f;
      for (int q = 0; q < splits; ++q) s += partial[(size_t)q * d + c];
      xs[c] = n > 1 ? s * inv : 0.f;
      xs[d + c] = last_row<BF16>(rows, n, d, c);
    }
  }
  __syncthreads();
  if (feature && blockIdx.x == 0)
    for (int c = tid; c < 2 * d; c += 256) feature[c] = xs[c];
  auto unit = [&](int u, const float4 (&c)[PRE], float b) {
    const float* wr = w1 + (size_t)u * 2 * d;
    float acc = 0.f;
    auto add4 = [&](const float4& w, int j) {
      const float4 x = *reinterpret_cast<const float4*>(xs + 4 * j);
      acc = fmaf(w.x, x.x, acc);
      acc = fmaf(w.y, x.y, acc);
      acc = fmaf(w.z, x.z, acc);
      acc = fmaf(w.w, x.w, acc);
    };
    if (vec) {
      const float4* w4 = reinterpret_cast<const float4*>(wr);
#pragma unroll
      for (int q = 0; q < PRE; ++q)
        if (lane + 64 * q < n4) add4(c[q], lane + 64 * q);
      for (int j0 = lane + 64 * PRE; j0 < n4; j0 += 64 * 8) {  // eight loads in flight
        float4 r[8];
#pragma unroll
        for (int q = 0; q < 8; ++q) r[q] = j0 + 64 * q < n4 ? w4[j0 + 64 * q] : make_float4(0.f, 0.f, 0.f, 0.f);
#pragma unroll
        for (int q = 0; q < 8; ++q)
          if (j0 + 64 * q < n4) add4(r[q], j0 + 64 * q);
      }
    } else {
      for (int c0 = lane; c0 < 2 * d; c0 += 64 * 16) {  // sixteen loads in flight
        float r[16];
#pragma unroll
        for (int q = 0; q < 16; ++q) r[q] = wr[min(c0 + 64 * q, 2 * d - 1)];
#pragma unroll
        for (int q = 0; q < 16; ++q)
          if (c0 + 64 * q < 2 * d) acc = fmaf(r[q], xs[c0 + 64 * q], acc);
      }
    }
    // lanes in order: the sum of lane partials is formed by lane 0
    for (int off = 32; off >= 1; off >>= 1) acc += __shfl_down(acc, off, 64);
    // agent scope: the deciding workgroup may run on another XCD
    if (lane == 0)
      __hip_atomic_store(hidden + u, fmaxf(acc + b, 0.f), __ATOMIC_RELAXED,
                         __HIP_MEMORY_SCOPE_AGENT);
  };
  int u = blockIdx.x * 4 + wv;
  if constexpr (MULTI) {
    for (; u < hid; u += gridDim.x * 4) {
      const float b = bu;
      float4 c[PRE];
#pragma unroll
      for (int q = 0; q < PRE; ++q) c[q] = v[q];
      if (u + (int)gridDim.x * 4 < hid) first_weights(u + gridDim.x * 4);
      unit(u, c, b);
    }
  } else if (u < hid) {
    unit(u, v, bu);
  }
  // every unit of the workgroup is stored (vmcnt 0), then it counts itself;
  // the last one decides
  __builtin_amdgcn_s_waitcnt(0);
  __syncthreads();
  if (tid == 0)
    xs[0] = __hip_atomic_fetch_add(ctr, 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) == (int)gridDim.x - 1;
  __syncthreads();
  if (xs[0] == 0.f) return;
  __syncthreads();
  float* z = xs;
  if (wv < 2) {  // class = wavefront
    float acc = 0.f;
    for (int h0 = 0; h0 < hid; h0 += 64 * 8) {  // eight loads in flight, added in order
      float hv[8], wq[8];
#pragma unroll
      for (int q = 0; q < 8; ++q)
        if (h0 + 64 * q < hid) {  // (the same for all lanes)
          const int h = min(h0 + 64 * q + lane, hid - 1);
          hv[q] = __hip_atomic_load(hidden + h, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
          wq[q] = w2[(size_t)wv * hid + h];
        }
#pragma unroll
      for (int q = 0; q < 8; ++q)
        if (h0 + 64 * q + lane < hid) acc = fmaf(wq[q], hv[q], acc);
    }
    for (int off = 32; off >= 1; off >>= 1) acc += __shfl_down(acc, off, 64);
    if (lane == 0) z[wv] = acc + bz;
  }
  __syncthreads();
  if (tid == 0) {
    const float mx = fmaxf(z[0], z[1]);
    const float e0 = expf(z[0] - mx), e1 = expf(z[1] - mx);
    const float p = e1 / (e0 + e1);
    *p_exit = p;
    const bool fire = static_cast<double>(p) >= theta;
    *exit_flag = fire ? 1 : 0;
    if (fire && exit_layer) *exit_layer = layer;  // the exit layer of a predicated gate
  }
}

// the rows outside [v0, v1) when *flag != 0; nothing otherwise
template <typename VEC>
__global__ __launch_bounds__(256) void drop_rows_if_kernel(const VEC* __restrict__ h, int rows_out,
                                                           int chunks, int v0, int nv,
                                                           const int32_t* __restrict__ flag,
                                                           VEC* __restrict__ out) {
  if (*flag == 0) return;
  const size_t n = (size_t)rows_out * chunks;
  for (size_t i = (size_t)blockIdx.x * 256 + threadIdx.x; i < n; i += (size_t)gridDim.x * 256) {
    const int r = (int)(i / chunks), c = (int)(i % chunks);
    const int src = r < v0 ? r : r + nv;
    out[i] = h[(size_t)src * chunks + c];
  }
}
template <typename VEC>
hipError_t drop_if_launch(const void* h, int rows_out, int chunks, int v0, int nv, const int32_t* flag,
                          void* out, hipStream_t s) {
  const size_t n = (size_t)rows_out * chunks;
  size_t blocks = (n + 255) / 256;
  if (blocks > 65536) blocks = 65536;
  drop_rows_if_kernel<VEC><<<(unsigned)blocks, 256, 0, s>>>(static_cast<const VEC*>(h), rows_out, chunks,
                                                             v0, nv, flag, static_cast<VEC*>(out));
  return hipGetLastError();
}
}  // namespace

size_t savb_ws_bytes(int n, int d, int hid) {
  const int splits = savb_splits(n);
  return ((size_t)splits * d + (size_t)hid + (size_t)2 * d) * sizeof(float);
}

hipError_t launch_savb_gate(const void* rows, bool bf16, int n, int d, const float* w1,
                            const float* b1, int hid, const float* w2, const float* b2, double theta,
                            float* feature, float* p_exit, int32_t* exit_flag, void* ws,
                            hipStream_t s, Guard g, int32_t* exit_layer, int layer) {
  const int splits = savb_splits(n);
  float* partial = static_cast<float*>(ws);
  float* hidden = partial + (size_t)splits * d;
  int* ctr = reinterpret_cast<int*>(hidden + hid);
  const dim3 grid(splits > 0 ? (d + 255) / 256 : 1, splits > 0 ? splits : 1);
  const int per = splits > 0 ? (n - 1 + splits - 1) / splits : 0;  // rows per split (splits * per >= n - 1)
  if (bf16)
    savb_pool_kernel<true><<<grid, 256, 0, s>>>(rows, n, d, per, partial, ctr, g);
  else
    savb_pool_kernel<false><<<grid, 256, 0, s>>>(rows, n, d, per, partial, ctr, g);
  hipError_t e = hipGetLastError();
  if (e != hipSuccess) return e;
  const unsigned hb = std::min(SG_WGS, (unsigned)((hid + 3) / 4));
  const size_t lds = (size_t)2 * d * sizeof(float);
  const bool multi = hid > 4 * (int)hb;
#define SAVB_MLP(BF16, PRE, MULTI)                                                                                  \
  savb_mlp_kernel<BF16, PRE, MULTI><<<hb, 256, lds, s>>>(rows, n, d, splits, partial, feature, w1, b1, hid, hidden, \
                                                         w2, b2, theta, p_exit, exit_flag, exit_layer, layer, ctr, g)
  if (multi) {
    if (bf16) SAVB_MLP(true, 16, true); else SAVB_MLP(false, 16, true);
  } else if (d <= 512) {
    if (bf16) SAVB_MLP(true, 4, false); else SAVB_MLP(false, 4, false);
  } else {
    if (bf16) SAVB_MLP(true, 16, false); else SAVB_MLP(false, 16, false);
  }
#undef SAVB_MLP
  return hipGetLastError();
}

hipError_t launch_drop_rows_if(const void* h, int elt, int S, int d, int v0, int v1,
                               const int32_t* flag, void* out, hipStream_t s) {
  const int rows_out = S - (v1 - v0), nv = v1 - v0;
  const size_t row_bytes = (size_t)d * elt;
  const uintptr_t al = reinterpret_cast<uintptr_t>(h) | reinterpret_cast<uintptr_t>(out);
  if (row_bytes % 16 == 0 && al % 16 == 0)
    return drop_if_launch<uint4>(h, rows_out, (int)(row_bytes / 16), v0, nv, flag, out, s);
  if (row_bytes % 4 == 0 && al % 4 == 0)
    return drop_if_launch<uint32_t>(h, rows_out, (int)(row_bytes / 4), v0, nv, flag, out, s);
  return drop_if_launch<uint16_t>(h, rows_out, (int)(row_bytes / 2), v0, nv, flag, out, s);
}

}  // namespace decomoe
