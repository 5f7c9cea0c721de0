// Exchanges between the lanes of a wavefront and the gate's row functions, shared by the router and the permutes.
#pragma once
#include "common.hpp"

namespace bigmac {

// The value of lane ^ J, without the LDS: moves inside rows of 16 lanes (DPP), swaps between them.
template <int J>
__device__ __forceinline__ unsigned from_lane_xor(unsigned v, int lane) {
  static_assert(J == 1 || J == 2 || J == 4 || J == 8 || J == 16 || J == 32, "a power of two");
  if constexpr (J == 1) return (unsigned)__builtin_amdgcn_mov_dpp((int)v, 0xB1, 0xF, 0xF, true);        // quad [1,0,3,2]
  else if constexpr (J == 2) return (unsigned)__builtin_amdgcn_mov_dpp((int)v, 0x4E, 0xF, 0xF, true);   // quad [2,3,0,1]
  else if constexpr (J == 4)    // mirror of 8 lanes, then of each quad
    return (unsigned)__builtin_amdgcn_mov_dpp(__builtin_amdgcn_mov_dpp((int)v, 0x141, 0xF, 0xF, true), 0x1B, 0xF, 0xF, true);
  else if constexpr (J == 8) return (unsigned)__builtin_amdgcn_mov_dpp((int)v, 0x128, 0xF, 0xF, true);  // row rotated by 8
  else if constexpr (J == 16) {
    const auto r = __builtin_amdgcn_permlane16_swap(v, v, false, false);
    return (lane & 16) ? r[0] : r[1];
  } else {
    const auto r = __builtin_amdgcn_permlane32_swap(v, v, false, false);
    return (lane & 32) ? r[0] : r[1];
  }
}
// sum over the wavefront, in every lane: pairs 32, 16, 8, 4, 2, 1 apart
__device__ __forceinline__ float wave_sum(float v, int lane) {
  v += __uint_as_float(from_lane_xor<32>(__float_as_uint(v), lane));
  v += __uint_as_float(from_lane_xor<16>(__float_as_uint(v), lane));
  v += __uint_as_float(from_lane_xor<8>(__float_as_uint(v), lane));
  v += __uint_as_float(from_lane_xor<4>(__float_as_uint(v), lane));
  v += __uint_as_float(from_lane_xor<2>(__float_as_uint(v), lane));
  v += __uint_as_float(from_lane_xor<1>(__float_as_uint(v), lane));
  return v;
}
__device__ __forceinline__ float read_lane(float v, int lane) { return __uint_as_float(__builtin_amdgcn_readlane(__float_as_uint(v), lane)); }

// softmax over all N logits of one token by one wavefront: lane l holds experts l, l + 64, ...
template <int PER>
__device__ __forceinline__ void softmax_row(const float* __restrict__ row, int N, int lane, float (&p)[PER]) {
  float m = -INFINITY;
#pragma unroll
  for (int i = 0; i < PER; ++i) {
    const int n = i * 64 + lane;
    p[i] = n < N ? row[n] : -INFINITY;
    m = fmaxf(m, p[i]);
  }
#pragma unroll
  for (int off = 32; off >= 1; off >>= 1) m = fmaxf(m, __shfl_xor(m, off, 64));
  float sum = 0.0f;
#pragma unroll
  for (int i = 0; i < PER; ++i) {
    p[i] = i * 64 + lane < N ? expf(p[i] - m) : 0.0f;
    sum += p[i];
  }
#pragma unroll
  for (int off = 32; off >= 1; off >>= 1) sum += __shfl_xor(sum, off, 64);
  const float inv = 1.0f / sum;
#pragma unroll
  for (int i = 0; i < PER; ++i) p[i] *= inv;
}

// Gradient of the load-balance loss  alpha N sum_e f_e P_e  with respect to one token's logits,
// the pair shares f held fixed:  scale p_n (f_n - sum_e f_e p_e),  scale = alpha N / T.
template <int PER>
__device__ __forceinline__ void aux_grad_row(const float* __restrict__ row, const float* __restrict__ share, int N, int lane,
                                             float scale, float (&g)[PER]) {
  float f[PER];
  softmax_row<PER>(row, N, lane, g);
  float mix = 0.0f;
#pragma unroll
  for (int i = 0; i < PER; ++i) {
    const int n = i * 64 + lane;
    f[i] = n < N ? share[n] : 0.0f;
    mix = fmaf(f[i], g[i], mix);
  }
#pragma unroll
  for (int off = 32; off >= 1; off >>= 1) mix += __shfl_xor(mix, off, 64);
#pragma unroll
  for (int i = 0; i < PER; ++i) g[i] = scale * g[i] * (f[i] - mix);
}

// Backward of one token's gate (softmax over the k picked logits) by one wavefront.  Lane j < k holds pick j: its
// weight w, the gradient g of that weight and its expert e.
//   dl_j = w_j (g_j - sum_m w_m g_m)
// goes to dl_picked[j] (optional) and, among zeros, to the dense row dL; with the load-balance loss
// (logits != NULL) the loss's gradient joins every entry of the row.  entry[i]: what the row holds at expert i * 64 + lane.
template <typename DT, int PER>
__device__ __forceinline__ void gate_backward_row(float w, float g, int e, const float* __restrict__ logits, const float* __restrict__ share,
                                                  float aux_scale, int N, int k, int lane, DT* __restrict__ dL, float* __restrict__ dl_picked,
                                                  float (&entry)[PER], float& dl) {
#pragma unroll
  for (int i = 0; i < PER; ++i) entry[i] = 0.0f;
  if (logits) aux_grad_row<PER>(logits, share, N, lane, aux_scale, entry);
  float mix = 0.0f;
  for (int j = 0; j < k; ++j) mix = fmaf(read_lane(w, j), read_lane(g, j), mix);
  dl = w * (g - mix);
  if (dl_picked && lane < k) dl_picked[lane] = dl;
#pragma unroll
  for (int i = 0; i < PER; ++i) {
    if (i * 64 >= N) break;
    const int n = i * 64 + lane;
    float val = 0.0f;
    for (int j = 0; j < k; ++j) {
      const float dj = read_lane(dl, j);
      if (__builtin_amdgcn_readlane(e, j) == n) val = dj;
    }
    entry[i] += val;
    if (n < N) Elem<DT>::store(dL + n, logits ? entry[i] : val);
  }
}

// A workgroup's piece of a SliceSum: four neighbouring elements per thread, eight slices on their way at a time.
template <int THREADS>
__device__ __forceinline__ void slice_sum_block(const SliceSum& job, int block) {
  const size_t i = ((size_t)block * THREADS + threadIdx.x) * 4;
  if (i >= job.n) return;
  float4 s = make_float4(0.f, 0.f, 0.f, 0.f);
  for (int z = 0; z < job.nslices; z += 8) {
    float4 v[8];
#pragma unroll
    for (int u = 0; u < 8; ++u) v[u] = *(const float4*)(job.part + (size_t)min(z + u, job.nslices - 1) * job.n + i);
#pragma unroll
    for (int u = 0; u < 8; ++u)
      if (z + u < job.nslices) { s.x += v[u].x; s.y += v[u].y; s.z += v[u].z; s.w += v[u].w; }
  }
  *(uint2*)((bf16_t*)job.out + i) = make_uint2(f2bf_pair(s.x, s.y), f2bf_pair(s.z, s.w));
}

}  // namespace bigmac
