// Top-k and gate of tokens whose logits are there: a workgroup's work, for the kernel of its own (route.hip) and for workgroups beside
// a matrix product (gemm.hip).
#pragma once
#include "wave.hpp"

namespace bigmac {

// (logit, expert) as one number: the greater key comes first, equal logits (-0 counts as 0) by lower index.  NaN logits
// have a place in that order too (by their sign, past the infinities), and a lane past the N experts comes after every
// expert, so that whatever the logits are the k <= N picks are k different experts: the sort writes to slots counted by them.
__device__ __forceinline__ unsigned long long logit_key(float logit, int expert) {
  const unsigned u = __float_as_uint(logit + 0.0f);
  return ((unsigned long long)((u & 0x80000000u) ? ~u : u | 0x80000000u) << 32) | (unsigned)~expert;
}
__device__ __forceinline__ unsigned long long pick_key(const float* row, int expert, int N) {
  return expert >= N ? (unsigned)~expert : logit_key(row[expert], expert);
}
__device__ __forceinline__ float key_logit(unsigned long long key) {
  const unsigned u = (unsigned)(key >> 32);
  return __uint_as_float((u & 0x80000000u) ? u & 0x7FFFFFFFu : ~u);
}
// One compare-exchange step of a bitonic network over the wavefront, for U independent networks: partner lane
// ^ J, the greater key of the pair goes to the lane for which greater_here holds.
template <int J, int U>
__device__ __forceinline__ void exchange_keys(unsigned long long (&key)[U], int lane, bool greater_here) {
#pragma unroll
  for (int u = 0; u < U; ++u) {
    const unsigned long long other = ((unsigned long long)from_lane_xor<J>((unsigned)(key[u] >> 32), lane) << 32) | from_lane_xor<J>((unsigned)key[u], lane);
    if ((key[u] > other) != greater_here) key[u] = other;
  }
}
template <int SIZE, int J, int U>
__device__ __forceinline__ void merge_keys(unsigned long long (&key)[U], int lane) {
  exchange_keys<J>(key, lane, ((lane & J) == 0) == ((lane & SIZE) == 0));   // lower lane of a descending block
  if constexpr (J > 1) merge_keys<SIZE, J / 2>(key, lane);
}
template <int SIZE, int U>
__device__ __forceinline__ void sort_keys(unsigned long long (&key)[U], int lane) {   // lane 0 ends with the greatest
  if constexpr (SIZE > 2) sort_keys<SIZE / 2>(key, lane);
  merge_keys<SIZE, SIZE / 2>(key, lane);
}

// The k picks of each token in pick order (greater logit first, ties to the lower index) and the softmax over
// their logits, summed in pick order.  One wavefront per token; a workgroup walks the `tokens` tokens of
// its share and, if counts is given (up to 128 experts), counts their pairs per expert on the way (the sort's counters,
// see launch_build_permutation).  PER = logits per lane.  Up to 64 experts: one key per lane, sorted across the wavefront by a
// bitonic network (the order is strict and total, so the result is the unique sorted sequence);
// lanes 0 .. k-1 then hold the picks.  Up to 128: two keys per lane, both halves sorted the same way;
// the first 64 of their union are, lane by lane, the first of (half 0 at lane l, half 1 at lane
// 63 - l), a bitonic sequence that six more steps sort: k <= 64 picks are all there.  More: every lane
// ranks its logits against all N by broadcast (rank = how many logits come first); ranks below k
// are the selection.  That one is bound by its comparisons, which take no branches (1024 tokens, 512 experts: 106 us with, 52 without).
// The network is a serial chain of 21 (27) exchanges and bound by its latency: keys of 64 bits cost one
// comparison, partners are read by DPP moves and row swaps instead of through the LDS, and a
// wavefront takes U tokens at a time: two where the grid follows the sort's chunks (8192 tokens, 64 experts, counting included: 15.0 us by wavefronts
// that take eight one by one, 6.3 us so).
// (hist: room for 128 counters in the LDS, with counts only; block: the workgroup's number)
template <int PER, int U>
__device__ __forceinline__ void topk_gate_block(const float* __restrict__ logits, int T, int N, int k, int tokens, int block,
                                                int32_t* __restrict__ topk_idx, float* __restrict__ topk_w, int32_t* __restrict__ counts, int* hist) {
  const int lane = threadIdx.x & 63;
  if (PER <= 2 && counts) {
    for (int e = threadIdx.x; e < N; e += blockDim.x) hist[e] = 0;
    __syncthreads();
  }
  auto finish = [&](int t, float logit, int expert) {   // lane j < k holds pick j
    const float m = __uint_as_float(__builtin_amdgcn_readlane(__float_as_uint(logit), 0));
    const float e = lane < k ? expf(logit - m) : 0.0f;
    float s = 0.0f;
    for (int j = 0; j < k; ++j) s += __uint_as_float(__builtin_amdgcn_readlane(__float_as_uint(e), j));
    if (lane < k) {
      topk_idx[(size_t)t * k + lane] = expert;
      topk_w[(size_t)t * k + lane] = e / s;
      if (PER <= 2 && counts) atomicAdd(&hist[expert], 1);
    }
  };
  const int t_end = min(T, (block + 1) * tokens), step = blockDim.x >> 6;
  for (int t = block * tokens + (threadIdx.x >> 6); t < t_end; t += U * step) {
    if constexpr (PER <= 2) {
      unsigned long long key[U];
#pragma unroll
      for (int u = 0; u < U; ++u) {     // (tokens past the chunk repeat the last one's loads and are not finished)
        const float* row = logits + (size_t)min(t + u * step, t_end - 1) * N;
        key[u] = pick_key(row, lane, N);
      }
      if constexpr (PER == 1) {
        sort_keys<64>(key, lane);
      } else {
        unsigned long long upper[U];
#pragma unroll
        for (int u = 0; u < U; ++u) {
          const float* row = logits + (size_t)min(t + u * step, t_end - 1) * N;
          upper[u] = pick_key(row, 64 + lane, N);
        }
        sort_keys<64>(key, lane);
        sort_keys<64>(upper, lane);
#pragma unroll
        for (int u = 0; u < U; ++u) {
          const unsigned hi = __shfl((unsigned)(upper[u] >> 32), 63 - lane, 64), lo = __shfl((unsigned)upper[u], 63 - lane, 64);
          const unsigned long long mirrored = ((unsigned long long)hi << 32) | lo;
          if (mirrored > key[u]) key[u] = mirrored;
        }
        merge_keys<64, 32>(key, lane);
      }
#pragma unroll
      for (int u = 0; u < U; ++u)
        if (t + u * step < t_end) finish(t + u * step, key_logit(key[u]), (int)~(unsigned)key[u]);
    } else {
      const float* row = logits + (size_t)t * N;
      float v[PER];
      int rank[PER];
#pragma unroll
      for (int i = 0; i < PER; ++i) {
        const int n = i * 64 + lane;
        v[i] = n < N ? row[n] : -INFINITY;
        rank[i] = 0;
      }
#pragma unroll
      for (int io = 0; io < PER; ++io) {
        const int live = min(64, N - io * 64);        // lanes of this register that hold a logit
        for (int l = 0; l < live; ++l) {
          const float o = __int_as_float(__builtin_amdgcn_readlane(__float_as_int(v[io]), l));
          const int on = io * 64 + l;
#pragma unroll
          for (int i = 0; i < PER; ++i) rank[i] += (int)(o > v[i]) | ((int)(o == v[i]) & (int)(on < i * 64 + lane));   // (no branches)
        }
      }
      // lane j < k collects the j-th pick: its index and logit
      float selv = 0.0f;
      int seli = 0;
      for (int j = 0; j < k; ++j) {
#pragma unroll
        for (int i = 0; i < PER; ++i) {
          const unsigned long long hit = __ballot(rank[i] == j && i * 64 + lane < N);
          if (hit) {                                  // wave-uniform: exactly one (i, lane) has rank j
            const int src = __ffsll((long long)hit) - 1;
            const float pv = __int_as_float(__builtin_amdgcn_readlane(__float_as_int(v[i]), src));
            if (lane == j) { selv = pv; seli = i * 64 + src; }
          }
        }
      }
      finish(t, selv, seli);
    }
  }
  if (PER <= 2 && counts) {
    __syncthreads();
    for (int e = threadIdx.x; e < N; e += blockDim.x) counts[(size_t)block * N + e] = hist[e];
  }
}

}  // namespace bigmac
