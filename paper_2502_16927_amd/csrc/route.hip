// Gating of the BigMac layer (Section 3.1: the router reads the full-width token x; T is the
// set of top_k experts, p_i the gate value).  The logits decide integers, so their fp32
// summation order is fixed and every product is a fused multiply-add:
//   p_l  = fma(x[t, 64q + l], W_g[64q + l, n], p_l),  q ascending, l = 0..63   (one lane each)
//   tree = p_l + p_{l+off} for off = 32, 16, 8, 4, 2, 1;  logit = tree (+ bias[n], added last)
// The tree is evaluated as a reduce-scatter over the wavefront: same pairs, 1/6 of the adds.
#include "gemm_core.hpp"
#include "topk.hpp"

namespace bigmac {

namespace {

constexpr int R_TB = 8;     // tokens per wave
constexpr int R_NB = 16;    // experts per pass
constexpr int R_QT = 4;     // 64-row blocks of W_g staged per LDS tile
constexpr int ROUTER_DX_PICKS = 1024;   // (token, pick) pairs a workgroup of the router's dx kernel stages
#ifndef ROUTER_DX_CPL
#define ROUTER_DX_CPL 4                 // output columns per lane of that kernel
#endif
#ifndef ROUTER_DX_THREADS
#define ROUTER_DX_THREADS 1024
#endif
#ifndef ROUTER_DX_TOKENS
#define ROUTER_DX_TOKENS 128
#endif
constexpr int R_PAD = 20;   // floats per staged row (16 + 4: conflict-free 16-byte reads)

// Block = 4 wavefronts x 8 tokens, one pass of 16 experts (blockIdx.y); the 16 router columns are
// staged through LDS in tiles of 256 rows and shared by the four wavefronts.
template <typename XT>
__global__ __launch_bounds__(256) void router_logits_kernel(const XT* __restrict__ x, const float* __restrict__ wg,
                                                            const float* __restrict__ bias, float* __restrict__ logits,
                                                            int T, int d, int N) {
  __shared__ float sw[R_QT * 64 * R_PAD];
  const int wave = threadIdx.x >> 6, lane = threadIdx.x & 63;
  const int t0 = blockIdx.x * (4 * R_TB) + wave * R_TB;
  const int n0 = blockIdx.y * R_NB;
  const int nq = d / 64;
  const bool vec = (N % 4) == 0;
  float acc[R_TB * R_NB];
#pragma unroll
  for (int v = 0; v < R_TB * R_NB; ++v) acc[v] = 0.0f;
  for (int q0 = 0; q0 < nq; q0 += R_QT) {
    // this tile's tokens first: R_QT x R_TB independent loads in flight
    float xv[R_QT][R_TB];
#pragma unroll
    for (int qq = 0; qq < R_QT; ++qq)
#pragma unroll
      for (int i = 0; i < R_TB; ++i) {
        const int t = t0 + i;
        xv[qq][i] = (t < T && q0 + qq < nq) ? Elem<XT>::load(x + (size_t)t * d + (size_t)(q0 + qq) * 64 + lane) : 0.0f;
      }
    __syncthreads();
    if (vec) {
      for (int e = threadIdx.x; e < R_QT * 64 * (R_NB / 4); e += 256) {
        const int row = e / (R_NB / 4), c = (e % (R_NB / 4)) * 4;
        const int gi = q0 * 64 + row, gn = n0 + c;
        float4 w = make_float4(0.f, 0.f, 0.f, 0.f);
        if (gi < d && gn < N) w = *(const float4*)(wg + (size_t)gi * N + gn);
        *(float4*)(sw + row * R_PAD + c) = w;
      }
    } else {
      for (int e = threadIdx.x; e < R_QT * 64 * R_NB; e += 256) {
        const int row = e / R_NB, c = e % R_NB;
        const int gi = q0 * 64 + row, gn = n0 + c;
        sw[row * R_PAD + c] = (gi < d && gn < N) ? wg[(size_t)gi * N + gn] : 0.0f;
      }
    }
    __syncthreads();
#pragma unroll
    for (int qq = 0; qq < R_QT; ++qq) {
      if (q0 + qq >= nq) break;
      const float4* wrow = (const float4*)(sw + (qq * 64 + lane) * R_PAD);
      float wv[R_NB];
#pragma unroll
      for (int c4 = 0; c4 < R_NB / 4; ++c4) {
        float4 w = wrow[c4];
        wv[c4 * 4 + 0] = w.x; wv[c4 * 4 + 1] = w.y; wv[c4 * 4 + 2] = w.z; wv[c4 * 4 + 3] = w.w;
      }
#pragma unroll
      for (int i = 0; i < R_TB; ++i)
#pragma unroll
        for (int c = 0; c < R_NB; ++c) acc[i * R_NB + c] = fmaf(xv[qq][i], wv[c], acc[i * R_NB + c]);
    }
  }
  // halving tree as a reduce-scatter: at distance off the lanes with that bit set keep the
  // upper half of the values, the others the lower half; value 2*lane + {0,1} ends on lane.
#pragma unroll
  for (int off = 32, half = R_TB * R_NB / 2; off >= 1; off >>= 1, half >>= 1) {
    const bool hi = (lane & off) != 0;
#pragma unroll
    for (int v = 0; v < half; ++v) {
      const float send = hi ? acc[v] : acc[v + half];
      const float keep = hi ? acc[v + half] : acc[v];
      acc[v] = keep + __shfl_xor(send, off, 64);
    }
  }
#pragma unroll
  for (int u = 0; u < 2; ++u) {
    const int v = 2 * lane + u;
    const int t = t0 + v / R_NB, n = n0 + v % R_NB;
    if (t < T && n < N) {
      float val = acc[u];
      if (bias) val = val + bias[n];
      logits[(size_t)t * N + n] = val;
    }
  }
}

// The same sums on the matrix cores, for N % 4 == 0.  v_mfma_f32_16x16x1_4b_f32 has a contraction of one: every output
// element takes part in exactly one fused multiply-add per instruction (bit for bit that of fmaf, subnormals, infinities
// and NaN included), so 64 accumulators per logit, each fed in ascending q, are the partial sums p_l in their order.
// The four blocks of an instruction hold residues l of the four runs 16 b .. 16 b + 15.  With c = l % 16 = 8 h + 2 q + p, a
// wavefront holds RR of the c's for a tile of 16 tokens x 16 ET experts: one (h, p) with all four q, or one (h, p, q % 2).  Block b of an
// instruction takes another q, that is another word of a 16-byte chunk, in each block: with the rows' chunks swizzled by the token
// the 64 lanes of an operand read fall on the 64 banks.  The tree's distances 32 and 16 stay inside a lane's registers; the rest goes
// through the LDS, with (h, p) wavefronts as two exchanges (8; 4 and 2 in registers; 1).
// What bounds it: the matrix rate of fp32, 157 TFLOP/s by the clock and 140 in a register-only loop on all CUs.  These instructions
// run on the vector ALU's multipliers: a vector instruction among them costs some 9 cycles of theirs, and a stretch of other
// instructions that both wavefronts of a SIMD run at once leaves the multipliers idle.  So the loop has no vector instruction but the
// ring's address steps, and everything else stands between the matrix instructions, one or two at a time.  Operands travel
// global -> LDS directly (16 bytes per lane) through a ring of S stages of QQT 64-row blocks, the next tile's behind this one's
// reduction.  Token rows past T and columns past N arrive as zeros and are never used.
template <typename XT, int TT, int ET, int QQT>
struct RouterTile {
  static constexpr int THREADS = 512;
  static constexpr int WPT = 8 / TT, RR = 16 / WPT, M = RR * ET;          // wavefronts per token tile, c's of each, instructions per block
  static constexpr int TOKENS = 16 * TT, EXPERTS = 16 * ET;
  static constexpr int XROW = 64 * (int)sizeof(XT) / 16;                  // 16-byte chunks of a token's 64-element block: 8, 16
  static constexpr int XCH = TOKENS * XROW * QQT, WCH = 64 * QQT * 4 * ET;  // chunks of a stage: tokens, router rows
  static constexpr int XL = XCH / THREADS, WL = WCH / THREADS, LPT = XL + WL;
  static_assert((TT == 1 || (TT == 2 && ET == 2)) && XCH % THREADS == 0 && WCH % THREADS == 0, "whole passes");
  static_assert(QQT % 2 == 0, "a stage starts with the first register set");
  static constexpr int STAGE = (XCH + WCH) * 16;
  static constexpr int S = 5 * 24576 / STAGE > 6 ? 6 : 5 * 24576 / STAGE; // ring stages
  static constexpr int SUMS_AT = S * STAGE, BIAS_AT = SUMS_AT + (TT == 2 ? 36864 : ET * 16384), LDS = BIAS_AT + 4096;
  static_assert(S >= 3 && LDS <= 160 * 1024, "LDS of a CU");
};
template <int OFFSET>
__device__ __forceinline__ void lds_read_b32(unsigned addr, unsigned& v) {
  asm volatile("ds_read_b32 %0, %1 offset:%2" : "=v"(v) : "v"(addr), "n"(OFFSET) : "memory");
}
template <int OFFSET>
__device__ __forceinline__ void lds_read_high_u16(unsigned addr, unsigned& v) {   // to the upper half; the lower one stays as it is
  asm volatile("ds_read_u16_d16_hi %0, %1 offset:%2" : "+v"(v) : "v"(addr), "n"(OFFSET) : "memory");
}
template <int OFFSET>
__device__ __forceinline__ void lds_read_b64(unsigned addr, u32x2_t& v) {
  asm volatile("ds_read_b64 %0, %1 offset:%2" : "=v"(v) : "v"(addr), "n"(OFFSET) : "memory");
}
template <int FIRST, int SECOND>   // bytes
__device__ __forceinline__ void lds_read_two_b32(unsigned addr, u32x2_t& v) {
  static_assert(FIRST % 256 == 0 && SECOND % 256 == 0 && SECOND < 65536, "instruction offsets");
  asm volatile("ds_read2st64_b32 %0, %1 offset0:%2 offset1:%3" : "=v"(v) : "v"(addr), "n"(FIRST / 256), "n"(SECOND / 256) : "memory");
}
template <int OFFSET>
__device__ __forceinline__ void lds_write_b64(unsigned addr, u32x2_t v) {
  asm volatile("ds_write_b64 %0, %1 offset:%2" ::"v"(addr), "v"(v), "n"(OFFSET) : "memory");
}
// The same sums for few tokens of few elements, or few experts (N % 4 == 0; see launch_router_logits), on the vector ALU: TB tokens per wavefront, 16 experts
// per workgroup of four.  Bound by latency: what counts is the chain from the launch over the first loads to the logits, which is shorter here than
// in the matrix kernel below (no rounding up to stages of 256 elements, the tree in registers instead of through the LDS).  Tiles of 128 elements of the
// tokens and of the router's columns travel global -> LDS directly (16 bytes per lane) through a ring of three, two in flight while one is
// consumed.  Token rows past T and router rows past d lie outside the buffer ranges and arrive as zeros; they are never used anyway.
template <typename XT, int TB>
__global__ __launch_bounds__(256) void router_logits_few_kernel(const XT* __restrict__ x, const float* __restrict__ wg, const float* __restrict__ bias,
                                                                float* __restrict__ logits, int T, int d, int N) {
  constexpr int S = 3, QQT = 2, TROWS = 64 * QQT;   // ring stages; 64-element blocks of a tile
  constexpr int ES = (int)sizeof(XT), TOKENS = 4 * TB, ACCS = TB * R_NB;
  constexpr int XROW = TROWS * ES / 16;             // 16-byte chunks per token row of a tile
  constexpr int XCH = TOKENS * XROW;                // chunks of a token tile: at most one per thread, or whole passes
  constexpr int XL = (XCH + 255) / 256, WL = TROWS * 4 / 256, LPT = XL + WL;
  __shared__ uint4 xring[S * XL * 256], wring[S * WL * 256];
  const int wave = threadIdx.x >> 6, lane = threadIdx.x & 63;
  // The workgroups of a token block lie 8 apart, that is on one XCD: its token rows come from memory once.
  const int slices = (N + R_NB - 1) / R_NB, lin = (int)(blockIdx.x >> 3);
  const int tb = ((lin / slices) * 8 + (int)(blockIdx.x & 7)) * TOKENS, n0 = (lin % slices) * R_NB;
  if (tb >= T) return;
  const int nq = d / 64, ntiles = (nq + QQT - 1) / QQT;
  const __amdgpu_buffer_rsrc_t rx = __builtin_amdgcn_make_buffer_rsrc((void*)(x + (size_t)tb * d), 0, (int)((size_t)min(TOKENS, T - tb) * d * ES), 0x00020000);
  const __amdgpu_buffer_rsrc_t rw = __builtin_amdgcn_make_buffer_rsrc((void*)(wg + n0), 0, (int)(((size_t)(d - 1) * N + min(R_NB, N - n0)) * 4), 0x00020000);
  unsigned xoff[XL], woff[WL];
#pragma unroll
  for (int i = 0; i < XL; ++i) {
    const int q = i * 256 + (int)threadIdx.x;
    xoff[i] = q < XCH ? (unsigned)((q / XROW) * d * ES + (q % XROW) * 16) : 0x80000000u;
  }
  // LDS position q holds column chunk (q & 3) ^ ((row >> 2) & 3) of row q >> 2: the 16 rows of one pass of a 16-byte read fall on 16
  // different bank groups
#pragma unroll
  for (int i = 0; i < WL; ++i) {
    const int q = i * 256 + (int)threadIdx.x, row = q >> 2;
    woff[i] = (unsigned)((row * N + (((q & 3) ^ ((row >> 2) & 3)) << 2)) * 4);
  }
  const int wave_chunk = __builtin_amdgcn_readfirstlane((int)(threadIdx.x & ~63u));
  auto issue = [&](int tile) {
    uint4* xs = xring + (tile % S) * (XL * 256) + wave_chunk;
    uint4* ws = wring + (tile % S) * (WL * 256) + wave_chunk;
#if defined(__HIP_DEVICE_COMPILE__)
#pragma unroll
    for (int i = 0; i < XL; ++i)
      __builtin_amdgcn_raw_ptr_buffer_load_lds(rx, (__attribute__((address_space(3))) void*)(xs + i * 256), 16, xoff[i] + (unsigned)(tile * TROWS * ES), 0, 0, 0);
#pragma unroll
    for (int i = 0; i < WL; ++i)
      __builtin_amdgcn_raw_ptr_buffer_load_lds(rw, (__attribute__((address_space(3))) void*)(ws + i * 256), 16, woff[i] + (unsigned)(tile * TROWS * N * 4), 0, 0, 0);
#else
    (void)xs; (void)ws;
#endif
  };
  float acc[ACCS];
#pragma unroll
  for (int v = 0; v < ACCS; ++v) acc[v] = 0.0f;
  // The tile reads are assembly: the compiler would make an LDS access that it can see wait for every direct-to-LDS load in flight, the
  // next tiles' included.  No branch lies between a read and the wait for it (the compiler may copy a register there).
  const unsigned xring_at = lds_address(xring) + (unsigned)((wave * TB * TROWS + lane) * ES), wring_at = lds_address(wring) + (unsigned)(lane * 64);
  unsigned xraw[QQT][TB];                           // (a bf16 element arrives in the upper half; the lower one is zero for good)
  u32x4_t wraw[QQT][4];
#pragma unroll
  for (int i = 0; i < QQT * TB; ++i) xraw[i % QQT][i / QQT] = 0u;
  auto request = [&](int tile, auto block) {
    constexpr int QQ = decltype(block)::value;
    const unsigned stage = (unsigned)(tile % S), xat = xring_at + stage * (XL * 256 * 16), wat = wring_at + stage * (WL * 256 * 16);
    auto& xs = xraw[QQ];
    auto& ws = wraw[QQ];
    static_for<0, TB>([&](auto token) {
      constexpr int I = decltype(token)::value;
      if constexpr (ES == 2) lds_read_high_u16<(I * TROWS + QQ * 64) * 2>(xat, xs[I]);
      else lds_read_b32<(I * TROWS + QQ * 64) * 4>(xat, xs[I]);
    });
#pragma unroll
    for (int c = 0; c < 4; ++c) lds_read_b128<QQ * 64 * 64>(wat + (unsigned)((c ^ ((lane >> 2) & 3)) * 16), ws[c]);
  };
  auto arrive = [&](auto block, auto younger) {      // (reads requested behind this block's)
    constexpr int QQ = decltype(block)::value;
    lds_wait_for<decltype(younger)::value>();
    auto& xs = xraw[QQ];
    auto& ws = wraw[QQ];
#pragma unroll
    for (int i = 0; i < TB; ++i) asm volatile("" : "+v"(xs[i]));
#pragma unroll
    for (int c = 0; c < 4; ++c) asm volatile("" : "+v"(ws[c]));
  };
  auto add = [&](auto block) {
    constexpr int QQ = decltype(block)::value;
#pragma unroll
    for (int i = 0; i < TB; ++i)
#pragma unroll
      for (int c = 0; c < R_NB; ++c) acc[i * R_NB + c] = fmaf(__uint_as_float(xraw[QQ][i]), __uint_as_float(wraw[QQ][c >> 2][c & 3]), acc[i * R_NB + c]);
  };
  constexpr StaticIndex<0> I0{};
  constexpr StaticIndex<1> I1{};
  // At tile t a wavefront waits until only the tiles requested after t are in flight; the barrier makes that true for everyone's part of t
  // and says that everyone has left tile t - 1, whose stage then takes tile t + S - 1.
  for (int tile = 0; tile < S - 1 && tile < ntiles; ++tile) issue(tile);
  for (int tile = 0; tile < ntiles; ++tile) {
    if (tile + 1 < ntiles) BIGMAC_WAIT_VMCNT(LPT);
    else BIGMAC_WAIT_VMCNT(0);
    __builtin_amdgcn_s_barrier();
    if (tile + S - 1 < ntiles) issue(tile + S - 1);
    if (tile * QQT + 1 < nq) {
      request(tile, I0);
      request(tile, I1);
      arrive(I0, StaticIndex<TB + 4>{});
      add(I0);
      arrive(I1, I0);
      add(I1);
    } else {
      request(tile, I0);
      arrive(I0, I0);
      add(I0);
    }
  }
  // Halving tree (lane l with lane l ^ off).  While a lane holds two or more sums a step is a reduce-scatter (see router_logits_kernel): at
  // distances 32 and 16 one swap exchanges the upper half (odd 16-lane rows) of one sum with the lower half (even rows) of another, and
  // every lane then holds what it keeps and what its partner sent; once a lane is down to one sum both lanes of a pair add the
  // other's.  The sum of accumulator v ends on the lanes whose top bits spell v.
  constexpr int SCATTER_STEPS = TB == 1 ? 4 : TB == 2 ? 5 : 6;
  static_assert(ACCS == 1 << SCATTER_STEPS, "1, 2 or 4 tokens per wavefront");
  static_for<0, 6>([&](auto n) {
    constexpr int step = decltype(n)::value, off = 32 >> step, half = ACCS >> (step + 1);
    if constexpr (off >= 16) {
#pragma unroll
      for (int v = 0; v < half; ++v) {
        const unsigned a = __float_as_uint(acc[v]), b = __float_as_uint(acc[v + half]);
        if constexpr (off == 32) {
          const auto r = __builtin_amdgcn_permlane32_swap(a, b, false, false);
          acc[v] = __uint_as_float(r[0]) + __uint_as_float(r[1]);
        } else {
          const auto r = __builtin_amdgcn_permlane16_swap(a, b, false, false);
          acc[v] = __uint_as_float(r[0]) + __uint_as_float(r[1]);
        }
      }
    } else if constexpr (step < SCATTER_STEPS) {
      const bool hi = (lane & off) != 0;
#pragma unroll
      for (int v = 0; v < half; ++v) {
        const float send = hi ? acc[v] : acc[v + half], keep = hi ? acc[v + half] : acc[v];
        acc[v] = keep + __uint_as_float(from_lane_xor<off>(__float_as_uint(send), lane));
      }
    } else {
      acc[0] = acc[0] + __uint_as_float(from_lane_xor<off>(__float_as_uint(acc[0]), lane));
    }
  });
  constexpr int SHARE = 6 - SCATTER_STEPS;          // low lane bits that hold copies of the same sum
  if ((lane & ((1 << SHARE) - 1)) == 0) {
    const int v = lane >> SHARE, t = tb + wave * TB + v / R_NB, n = n0 + v % R_NB;
    if (t < T && n < N) logits[(size_t)t * N + n] = bias ? acc[0] + bias[n] : acc[0];
  }
}

struct RouterJob {
  const void* x;
  const float *wg, *bias;
  float* logits;
  int T, d, N, slices, blocks, stages;   // expert slices, token blocks; ring stages of a tile
  int stride, block_step, slice_step;    // tiles of an XCD from one of a workgroup to its next, in blocks and slices
  unsigned slices_inverse;               // ceil(65536 / slices): i / slices of the first tiles (i < 32) by multiplication
  int warm_lines;                        // 128-byte lines of w_gate that workgroups without a tile read (0: none)
  int32_t* topk_idx;                     // PICK: the picks and their weights
  float* topk_w;
  int k;
};
// PICK (one 16-wide tile holds all experts): the tile's top-k and gate behind its logits, as topk_gate_kernel works them out, in the 16 lanes
// that hold a token's logits.
template <typename XT, int TT, int ET, int QQT, bool PICK = false>
__global__ __launch_bounds__(512) __attribute__((amdgpu_waves_per_eu(2, 2)))
void router_logits_matrix_kernel(RouterJob job) {
  const XT* const x = (const XT*)job.x;
  const float *const wg = job.wg, *const bias = job.bias;
  float* const logits = job.logits;
  const int T = job.T, d = job.d, N = job.N;
  typedef RouterTile<XT, TT, ET, QQT> C;
  constexpr int S = C::S, ES = (int)sizeof(XT), RR = C::RR, M = C::M;
  static_assert(!PICK || (TT == 1 && ET == 1), "all experts of a token in one tile");
  __shared__ __attribute__((aligned(128))) uint4 lds[C::LDS / 16];
  const unsigned lds_at = lds_address(lds);
  const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane((int)threadIdx.x >> 6);
  // Workgroup -> tiles.  Token blocks are dealt to the XCDs in turn and an XCD walks the expert slices of a block one after the
  // other: the block's token rows come from memory once, then from that XCD's L2, and every XCD keeps all of w_gate.
  const int slices = job.slices, blocks = job.blocks, stride = job.stride, block_step = job.block_step, slice_step = job.slice_step;
  const int xcd = (int)(blockIdx.x & 7), tiles = xcd < blocks ? ((blocks - 1 - xcd) / 8 + 1) * slices : 0;
  int tile = (int)(blockIdx.x >> 3);
  const int nq = d / 64, stages = job.stages;             // of a tile
  if (tile >= tiles) {
    // Few tiles: each is one CU's stream of w_gate from memory, at what a CU has in flight.  The XCD's workgroups without a tile
    // read a word of every line, all at once, and the streams find it in the L2.
    if (tiles > 0)
      for (int i = (tile - tiles) * C::THREADS + (int)threadIdx.x; i < job.warm_lines; i += (stride - tiles) * C::THREADS) {
        const float word = wg[(size_t)i * 32];
        asm volatile("" ::"v"(word));
      }
    return;
  }
  int block = (int)((unsigned)tile * job.slices_inverse >> 16), slice = tile - block * slices;
  auto advance = [&](int& bl, int& sl) {
    bl += block_step;
    sl += slice_step;
    if (sl >= slices) { sl -= slices; ++bl; }
  };
  if (bias) {
    float* sb = (float*)(lds + C::BIAS_AT / 16);
    for (int n = threadIdx.x; n < N; n += C::THREADS) sb[n] = bias[n];
    __syncthreads();
  }

  // the wavefront's token tile and c's: (h, p) and instruction row r has q = (r + b) % 4, or (h, p, q % 2) and q / 2 = (r + b) % 2
  const int part = wave % C::WPT, tt = wave / C::WPT;
  const int h = C::WPT == 4 ? part >> 1 : part >> 2, p = C::WPT == 4 ? part & 1 : (part >> 1) & 1;
  auto q_of = [&](int r, int b) { return C::WPT == 4 ? (r + b) & 3 : (part & 1) + 2 * ((r + b) & 1); };

  // requests: lane q of a pass fills chunk q of the stage
  unsigned xoff[C::XL], woff[C::WL], wcol[C::WL];
#pragma unroll
  for (int i = 0; i < C::XL; ++i) {                       // block by block, token rows of 8 (16) chunks, swizzled by the 256-byte window
    const int q = i * C::THREADS + (int)threadIdx.x, row = q / C::XROW, t = row % C::TOKENS, c = (q % C::XROW) ^ (C::XROW == 8 ? (t >> 1) & 7 : t & 15);
    xoff[i] = (unsigned)((t * d + row / C::TOKENS * 64) * ES + c * 16);
  }
#pragma unroll
  for (int i = 0; i < C::WL; ++i) {                       // the four rows of an instruction lie side by side, in the order of their use
    const int q = i * C::THREADS + (int)threadIdx.x, at = q / (4 * ET), b = at & 3, n = (at >> 2) & 15;
    int c;
    if (C::WPT == 4) c = 8 * (n >> 3) + 2 * (((n & 3) + b) & 3) + ((n >> 2) & 1);
    else c = 8 * (n >> 3) + 2 * (((n >> 1) & 1) + 2 * (((n & 1) + b) & 1)) + ((n >> 2) & 1);
    wcol[i] = (unsigned)(q % (4 * ET)) * 4;
    woff[i] = (unsigned)((((at & ~63) + 16 * b + c) * N + (int)wcol[i]) * 4);
  }
  const int wave_chunk = wave * 64;
  int ask_tile = tile, ask_block = block, ask_slice = slice, ask_stage = 0, ask_slot = 0;   // the next stage to request, and its place in the ring
  // (the vector ALU and these matrix instructions do not run side by side, so what changes from stage to stage is kept in scalars)
  // (A tile's stages are filled up in front: `pad` blocks of zeros, which leave the zeros that the sums start from.)
  const int pad = stages * QQT - nq;
  const XT* from_x = x;
  const float* from_w = wg;
  __amdgpu_buffer_rsrc_t rx, rw;
  uint4* to = lds;
  unsigned vx[C::XL], vw[C::WL];
  constexpr unsigned DEAD = 0x80000000u;                  // an offset past the buffers' ends: arrives as zeros
  auto aim = [&]() {                                      // at the next stage to request; past the workgroup's last one: at nothing
    to = lds + ask_slot * (C::STAGE / 16) + wave_chunk;
    if (++ask_slot == S) ask_slot = 0;
    const int bytes = ask_tile < tiles ? (int)DEAD : 0;
    if (ask_stage <= 1 && bytes) {
      const int tb = (ask_block * 8 + xcd) * C::TOKENS, n0 = ask_slice * C::EXPERTS, skip = ask_stage == 0 ? pad : 0;
      if (ask_stage == 0) {
        from_x = x + (long)tb * d - 64 * pad;
        from_w = wg + n0 - (long)64 * pad * N;
      }
#pragma unroll
      for (int i = 0; i < C::XL; ++i) {
        const int row = (i * C::THREADS + (int)threadIdx.x) / C::XROW;
        vx[i] = tb + row % C::TOKENS < T && row / C::TOKENS >= skip ? xoff[i] : DEAD;
      }
#pragma unroll
      for (int i = 0; i < C::WL; ++i)
        vw[i] = n0 + (int)wcol[i] < N && (i * C::THREADS + (int)threadIdx.x) / (256 * ET) >= skip ? woff[i] : DEAD;
    }
    rx = __builtin_amdgcn_make_buffer_rsrc((void*)from_x, 0, bytes, 0x00020000);
    rw = __builtin_amdgcn_make_buffer_rsrc((void*)from_w, 0, bytes, 0x00020000);
    from_x += 64 * QQT;
    from_w += (size_t)64 * QQT * N;
    if (++ask_stage == stages) {
      ask_stage = 0;
      ask_tile += stride;
      advance(ask_block, ask_slice);
    }
  };
  auto request = [&](auto n) {                            // number n of a stage's LPT
#if defined(__HIP_DEVICE_COMPILE__)
    constexpr int I = decltype(n)::value;
    if constexpr (I < C::XL)
      __builtin_amdgcn_raw_ptr_buffer_load_lds(rx, (__attribute__((address_space(3))) void*)(to + I * C::THREADS), 16, vx[I], 0, 0, 0);
    else
      __builtin_amdgcn_raw_ptr_buffer_load_lds(rw, (__attribute__((address_space(3))) void*)(to + C::XCH + (I - C::XL) * C::THREADS), 16, vw[I - C::XL], 0, 0, 0);
#else
    (void)n;
#endif
  };

  // Operands of a 64-row block: lane l holds token or router column l % 16 of residue run b = l / 16.  A bf16 element arrives in the
  // upper half of a register whose lower half is zero for good: no conversion.
  const int tok = lane & 15, b = lane >> 4;
  unsigned xat[RR];
#pragma unroll
  for (int i = 0; i < RR; ++i) {
    const int t = tt * 16 + tok;
    const unsigned e = (unsigned)((16 * b + 8 * h + 2 * q_of(i, b) + p) * ES);   // byte within the block's 64 elements
    xat[i] = lds_at + (unsigned)(t * C::XROW * 16) + (((e >> 4) ^ (unsigned)(C::XROW == 8 ? (t >> 1) & 7 : t & 15)) << 4) + (e & 15);
  }
  unsigned wat = lds_at + (unsigned)(C::XCH * 16 + part * RR * (256 * ET) + lane * 4 * ET);
  // [register set].  Two values of w in one read: neighbouring columns 2 n, 2 n + 1 (ET = 2: column tile j holds the columns
  // 2 n + j), or the two instruction rows
  constexpr int WR = M / 2, READS = RR + WR;
  unsigned xv[2][RR];
  u32x2_t wv[2][WR];
#pragma unroll
  for (int i = 0; i < 2 * RR; ++i) xv[i & 1][i >> 1] = 0u;
  auto read = [&](auto block, auto set, auto n) {         // number n of a block's READS
    constexpr int QQ = decltype(block)::value, R = decltype(set)::value, I = decltype(n)::value;
    auto& xs = xv[R];
    auto& ws = wv[R];
    if constexpr (I < RR) {
      constexpr int OFFSET = QQ * C::TOKENS * C::XROW * 16;
      const unsigned a = xat[I];
      if constexpr (ES == 4) lds_read_b32<OFFSET>(a, xs[I]);
      else lds_read_high_u16<OFFSET>(a, xs[I]);
    } else {
      constexpr int J = I - RR;
      if constexpr (ET == 2) lds_read_b64<QQ * 8192 + J * 512>(wat, ws[J]);
      else lds_read_two_b32<QQ * 4096, QQ * 4096 + 256>(wat, ws[J]);
    }
  };
  auto turn = [&](unsigned step) {                        // to the next stage of the ring
#pragma unroll
    for (int i = 0; i < RR; ++i) xat[i] += step;
    wat += step;
  };
  auto settle = [&](auto set) {
    constexpr int R = decltype(set)::value;
    auto& xs = xv[R];
    auto& ws = wv[R];
    asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
#pragma unroll
    for (int i = 0; i < RR; ++i) asm volatile("" : "+v"(xs[i]));
#pragma unroll
    for (int i = 0; i < WR; ++i) asm volatile("" : "+v"(ws[i]));
  };
  f32x16_t acc[C::M];                                     // [instruction row r, column tile j: r ET + j]
  auto clear = [&]() {
#pragma unroll
    for (int m = 0; m < C::M; ++m)
#pragma unroll
      for (int v = 0; v < 16; ++v) acc[m][v] = 0.0f;
  };
  // instructions FIRST .. LAST - 1 of the block in register set SET, each followed by some of the reads of the next block
  auto multiply = [&](auto set, auto first, auto last, auto&& reads) {
    constexpr int R = decltype(set)::value;
    static_for<decltype(first)::value, decltype(last)::value>([&](auto n) {
      constexpr int m = decltype(n)::value;
      auto& xs = xv[R];
      auto& ws = wv[R];
      acc[m] = __builtin_amdgcn_mfma_f32_16x16x1f32(__uint_as_float(ws[m >> 1][m & 1]), __uint_as_float(xs[m / ET]), acc[m], 0, 0, 0);
      __builtin_amdgcn_sched_barrier(0);
      reads(n);
      __builtin_amdgcn_sched_barrier(0);
    });
  };
  // the sums of a tile: lane l holds router columns 4 (l / 16) + v, v = 0 .. 3, of token l % 16
  auto finish = [&]() {
    const int t0 = (block * 8 + xcd) * C::TOKENS, n0 = slice * C::EXPERTS;
    if constexpr (C::WPT == 4) {
      float sum[4][2][4];                                 // [q][column tile][v]: distances 32 and 16
#pragma unroll
      for (int q = 0; q < 4; ++q)
#pragma unroll
        for (int j = 0; j < 2; ++j)
#pragma unroll
          for (int v = 0; v < 4; ++v) {
            auto of = [&](int bb) { return acc[((q - bb) & 3) * 2 + j][4 * bb + v]; };
            sum[q][j][v] = (of(0) + of(2)) + (of(1) + of(3));
          }
      // distance 8: the two wavefronts of a p keep two of the four v each
      const unsigned to8 = lds_at + (unsigned)(C::SUMS_AT + wave * 4096 + lane * 8), from8 = lds_at + (unsigned)(C::SUMS_AT + (wave ^ 2) * 4096 + lane * 8);
      static_for<0, 8>([&](auto i) {
        constexpr int q = decltype(i)::value >> 1, j = decltype(i)::value & 1;
        u32x2_t v;
        v.x = __float_as_uint(h ? sum[q][j][0] : sum[q][j][2]);
        v.y = __float_as_uint(h ? sum[q][j][1] : sum[q][j][3]);
        lds_write_b64<decltype(i)::value * 512>(to8, v);
      });
      asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
      __builtin_amdgcn_s_barrier();
      u32x2_t theirs[8];
      static_for<0, 8>([&](auto i) {
        auto& v = theirs[decltype(i)::value];
        lds_read_b64<decltype(i)::value * 512>(from8, v);
      });
      lds_wait(theirs);
      float even[2][2];                                   // [column tile][v]: distances 4 and 2
#pragma unroll
      for (int j = 0; j < 2; ++j)
#pragma unroll
        for (int v = 0; v < 2; ++v) {
          float c[4];
#pragma unroll
          for (int q = 0; q < 4; ++q) c[q] = (h ? sum[q][j][2 + v] : sum[q][j][v]) + __uint_as_float(theirs[q * 2 + j][v]);
          even[j][v] = (c[0] + c[2]) + (c[1] + c[3]);
        }
      // distance 1: the two wavefronts of an h keep one v each
      const unsigned to1 = lds_at + (unsigned)(C::SUMS_AT + 32768 + wave * 512 + lane * 8), from1 = lds_at + (unsigned)(C::SUMS_AT + 32768 + (wave ^ 1) * 512 + lane * 8);
      u32x2_t send, got[1];
      send.x = __float_as_uint(p ? even[0][0] : even[0][1]);
      send.y = __float_as_uint(p ? even[1][0] : even[1][1]);
      lds_write_b64<0>(to1, send);
      asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
      __builtin_amdgcn_s_barrier();
      lds_read_b64<0>(from1, got[0]);
      lds_wait(got);
      const int t = t0 + tt * 16 + tok, n = n0 + (b * 4 + h * 2 + p) * 2;
      float out[2] = {(p ? even[0][1] : even[0][0]) + __uint_as_float(got[0].x), (p ? even[1][1] : even[1][0]) + __uint_as_float(got[0].y)};
      if (t < T && n < N) {
        if (bias) {
          u32x2_t add[1];
          lds_read_b64<0>(lds_at + (unsigned)(C::BIAS_AT + n * 4), add[0]);
          lds_wait(add);
          out[0] = out[0] + __uint_as_float(add[0].x);
          out[1] = out[1] + __uint_as_float(add[0].y);
        }
        *(float2*)(logits + (size_t)t * N + n) = make_float2(out[0], out[1]);
      }
    } else {
      // residue by residue through the LDS, 16 bytes per lane; lanes of column group g at token ^ 4 g, which spreads the reads below over the banks
      const unsigned to = lds_at + (unsigned)C::SUMS_AT + (unsigned)((lane ^ (b << 2)) << 4);
#pragma unroll
      for (int i = 0; i < 2; ++i)                         // the wavefront's two q
#pragma unroll
        for (int j = 0; j < ET; ++j) {
          u32x4_t sum;
#pragma unroll
          for (int v = 0; v < 4; ++v) {
            auto of = [&](int bb) { return acc[((i + bb) & 1) * ET + j][4 * bb + v]; };
            sum[v] = __float_as_uint((of(0) + of(2)) + (of(1) + of(3)));
          }
          lds_write_b128(to + (unsigned)(((8 * h + 2 * ((part & 1) + 2 * i) + p) * ET + j) * 1024), sum);
        }
      asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
      __builtin_amdgcn_s_barrier();
      if ((int)threadIdx.x < 256 * ET) {
        const int j = (int)threadIdx.x % ET, row = ((int)threadIdx.x / ET) & 15, token = (int)threadIdx.x / (16 * ET);
        const unsigned from = lds_at + (unsigned)(C::SUMS_AT + j * 1024 + ((((row >> 2) << 4) + (token ^ (row & 12))) << 4) + (row & 3) * 4);
        const int t = t0 + token, n = n0 + row * ET + j;
        unsigned bits[16];
        static_for<0, 16>([&](auto c) {
          auto& v = bits[decltype(c)::value];
          lds_read_b32<decltype(c)::value * ET * 1024>(from, v);
        });
        lds_wait(bits);
        float sum[16];
#pragma unroll
        for (int c = 0; c < 16; ++c) sum[c] = __uint_as_float(bits[c]);
#pragma unroll
        for (int off = 8; off >= 1; off >>= 1)
#pragma unroll
          for (int c = 0; c < off; ++c) sum[c] = sum[c] + sum[c + off];
        if (t < T && n < N) {
          if (bias) {
            unsigned add[1];
            lds_read_b32<0>(lds_at + (unsigned)(C::BIAS_AT + n * 4), add[0]);
            lds_wait(add);
            sum[0] = sum[0] + __uint_as_float(add[0]);
          }
          logits[(size_t)t * N + n] = sum[0];
        }
        if constexpr (PICK) {                             // lane l: expert l % 16 of token 4 wave + l / 16
          const int expert = lane & 15, first = lane & 48;
          unsigned long long key[1] = {expert < N ? logit_key(sum[0], expert) : (unsigned)~expert};
          sort_keys<16>(key, expert);
          const float logit = key_logit(key[0]), m = __shfl(logit, first, 64), e = expert < job.k ? expf(logit - m) : 0.0f;
          float all = 0.0f;
          for (int j = 0; j < job.k; ++j) all += __shfl(e, first + j, 64);
          if (expert < job.k && t < T) {
            job.topk_idx[(size_t)t * job.k + expert] = (int)~(unsigned)key[0];
            job.topk_w[(size_t)t * job.k + expert] = e / all;
          }
        }
      }
    }
  };

  int todo = stages;                                      // of the tile at hand
  int asked = 0;
#pragma clang loop unroll(disable)
  for (; asked < S && ask_tile < tiles; ++asked) {
    aim();
    static_for<0, C::LPT>([&](auto n) { request(n); });
  }
  if (asked == S) BIGMAC_WAIT_VMCNT((S - 1) * C::LPT);     // the first stage
  else BIGMAC_WAIT_VMCNT(0);                               // all of the workgroup's; the waits of the loop then wait for nothing
  __builtin_amdgcn_s_barrier();
  int slot = 0;                                           // the stage at hand
  static_for<0, READS>([&](auto n) { read(StaticIndex<0>{}, StaticIndex<0>{}, n); });
  settle(StaticIndex<0>{});
  clear();
  constexpr StaticIndex<0> I0{};
  constexpr StaticIndex<1> I1{};
  constexpr int EARLY = M / 4, SPREAD = M > 2 ? M - 1 : M;   // instructions of the last block before the barrier; of a block, with reads behind them
  constexpr StaticIndex<EARLY> IE{};
  constexpr StaticIndex<M> END{};
  while (true) {
    // A stage, block by block, each block's operands read between the instructions of the one before it.  Between those of the last
    // block the next stage is awaited, and this one, which everyone has read by then, requested anew.  No branch lies between a read
    // and the wait for it: the compiler may copy a register at a branch, and would copy what is still on its way.
    static_for<0, QQT - 1>([&](auto block) {
      constexpr int QQ = decltype(block)::value, R = QQ & 1;
      multiply(StaticIndex<R>{}, I0, END, [&](auto n) {
        constexpr int K = decltype(n)::value, N0 = K < SPREAD ? K * READS / SPREAD : READS, N1 = K < SPREAD ? (K + 1) * READS / SPREAD : READS;
        static_for<N0, N1>([&](auto i) { read(StaticIndex<QQ + 1>{}, StaticIndex<R ^ 1>{}, i); });
      });
      settle(StaticIndex<R ^ 1>{});
    });
    if constexpr (EARLY == 0) aim();
    multiply(I1, I0, IE, [&](auto n) { if constexpr (decltype(n)::value == 0) aim(); });
    BIGMAC_WAIT_VMCNT((S - 2) * C::LPT);                   // (logits on their way out count too: a longer wait, once a tile)
    __builtin_amdgcn_s_barrier();
    if (++slot == S) slot = 0;
    turn(slot ? (unsigned)C::STAGE : (unsigned)-(S - 1) * C::STAGE);
    multiply(I1, IE, END, [&](auto n) {                    // (past the workgroup's last stage the reads are stale, and never used)
      constexpr int K = decltype(n)::value - EARLY, G = SPREAD - EARLY, N0 = K < G ? K * READS / G : READS, N1 = K < G ? (K + 1) * READS / G : READS;
      static_for<N0, N1>([&](auto i) { read(I0, I0, i); });
      constexpr int ALL = M - EARLY, L0 = K * C::LPT / ALL, L1 = (K + 1) * C::LPT / ALL;
      static_for<L0, L1>([&](auto i) { request(i); });
    });
    settle(I0);
    if (--todo == 0) {
      finish();
      tile += stride;
      if (tile >= tiles) break;
      advance(block, slice);
      todo = stages;
      clear();
    }
  }
  BIGMAC_WAIT_VMCNT(0);                                    // the requests of nothing write the LDS too
}

// (No TopkJob: with its number of workgroups the arguments, the block's size behind them included, pass the first 64-byte line, 0.1 to 0.3 us more.)
template <int PER, int U>
__global__ __launch_bounds__(1024) void topk_gate_kernel(const float* __restrict__ logits, int T, int N, int k, int tokens,
                                                         int32_t* __restrict__ topk_idx, float* __restrict__ topk_w, int32_t* __restrict__ counts) {
  __shared__ int hist[128];
  topk_gate_block<PER, U>(logits, T, N, k, tokens, (int)blockIdx.x, topk_idx, topk_w, counts, hist);
}

__global__ void transpose_f32_kernel(const float* __restrict__ in, float* __restrict__ out, int rows, int cols) {
  __shared__ float tile[32][33];
  int c = blockIdx.x * 32 + threadIdx.x, r0 = blockIdx.y * 32;
  for (int i = threadIdx.y; i < 32; i += 8)
    if (r0 + i < rows && c < cols) tile[i][threadIdx.x] = in[(size_t)(r0 + i) * cols + c];
  __syncthreads();
  int r = r0 + threadIdx.x, c0 = blockIdx.x * 32;
  for (int i = threadIdx.y; i < 32; i += 8)
    if (c0 + i < cols && r < rows) out[(size_t)(c0 + i) * rows + r] = tile[threadIdx.x][i];
}

// Column sums of softmax(logits) over a strided share of the tokens: workgroup b, wavefront w
// takes tokens (b * 4 + w) + i * 4 * gridDim.x.  partial[b][n], the four wavefronts added in order.
template <int PER>
__global__ __launch_bounds__(256) void aux_colsum_kernel(const float* __restrict__ logits, int T, int N, float* __restrict__ partial) {
  __shared__ float sums[4][1024];
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  float col[PER];
#pragma unroll
  for (int i = 0; i < PER; ++i) col[i] = 0.0f;
  for (int t = blockIdx.x * 4 + wave; t < T; t += 4 * gridDim.x) {
    float p[PER];
    softmax_row<PER>(logits + (size_t)t * N, N, lane, p);
#pragma unroll
    for (int i = 0; i < PER; ++i) col[i] += p[i];
  }
#pragma unroll
  for (int i = 0; i < PER; ++i)
    if (i * 64 + lane < N) sums[wave][i * 64 + lane] = col[i];
  __syncthreads();
  for (int n = threadIdx.x; n < N; n += 256)
    partial[(size_t)blockIdx.x * N + n] = ((sums[0][n] + sums[1][n]) + sums[2][n]) + sums[3][n];
}

// One workgroup: pair counts per expert (integer, order-free), P_e from the partial column sums,
// share[e] = f_e, and the loss  alpha N sum_e f_e P_e.  Every sum has a fixed order: the 1024
// threads are G groups x NP experts (NP = N rounded up to a power of two); group g adds its
// contiguous range of partials in order, the G group sums are added in group order, and the N
// terms f_e P_e go through a fixed tree.
// The counts come from the sort's counters of all chunks (chunk_counts [nchunks][N]) or, without them, from the picks.
__global__ __launch_bounds__(1024) void aux_finish_kernel(const int32_t* __restrict__ topk_idx, const int32_t* __restrict__ chunk_counts, int nchunks,
                                                          const float* __restrict__ partial,
                                                          int nparts, int T, int N, int NP, int k, float alpha,
                                                          float* __restrict__ share, float* __restrict__ loss) {
  __shared__ int cnt[1024];
  __shared__ float psum[1024];
  cnt[threadIdx.x] = 0;
  __syncthreads();
  const int Tk = T * k;
  if (chunk_counts) {
    const int n = threadIdx.x % NP;
    int sum = 0;
    if (n < N)
#pragma unroll 8
      for (int c = threadIdx.x / NP; c < nchunks; c += 1024 / NP) sum += chunk_counts[(size_t)c * N + n];
    if (n < N) atomicAdd(&cnt[n], sum);
  } else {
    const int quads = Tk / 4;                      // 16-byte reads; the base pointer is 16-byte aligned
    for (int q = threadIdx.x; q < quads; q += 1024) {
      const int4 v = ((const int4*)topk_idx)[q];
      atomicAdd(&cnt[v.x], 1); atomicAdd(&cnt[v.y], 1); atomicAdd(&cnt[v.z], 1); atomicAdd(&cnt[v.w], 1);
    }
    for (int f = quads * 4 + threadIdx.x; f < Tk; f += 1024) atomicAdd(&cnt[topk_idx[f]], 1);
  }
  const int G = 1024 / NP, e = threadIdx.x % NP, g = threadIdx.x / NP;
  const int per = (nparts + G - 1) / G;
  const int b_beg = min(g * per, nparts), b_end = min(b_beg + per, nparts);
  float mine = 0.0f;
  if (e < N)
#pragma unroll 8
    for (int b = b_beg; b < b_end; ++b) mine += partial[(size_t)b * N + e];
  psum[g * NP + e] = mine;
  __syncthreads();
  float term = 0.0f;
  if ((int)threadIdx.x < N) {
    float P = 0.0f;
    for (int h = 0; h < G; ++h) P += psum[h * NP + threadIdx.x];
    const float f = (float)cnt[threadIdx.x] / (float)Tk;
    share[threadIdx.x] = f;
    term = f * (P / (float)T);
  }
  __syncthreads();
  psum[threadIdx.x] = term;
  __syncthreads();
  for (int half = 512; half >= 1; half >>= 1) {
    if ((int)threadIdx.x < half) psum[threadIdx.x] += psum[threadIdx.x + half];
    __syncthreads();
  }
  if (threadIdx.x == 0) *loss = alpha * (float)N * psum[0];
}

// dlogits[t, :] of the load-balance loss, one wavefront per token
template <int PER>
__global__ __launch_bounds__(256) void aux_grad_kernel(const float* __restrict__ logits, const float* __restrict__ share, int T, int N,
                                                       float scale, float* __restrict__ dlogits) {
  const int lane = threadIdx.x & 63;
  const int t = blockIdx.x * 4 + (threadIdx.x >> 6);
  if (t >= T) return;
  float g[PER];
  aux_grad_row<PER>(logits + (size_t)t * N, share, N, lane, scale, g);
#pragma unroll
  for (int i = 0; i < PER; ++i)
    if (i * 64 + lane < N) dlogits[(size_t)t * N + i * 64 + lane] = g[i];
}

// Backward of the gate (softmax over the k picked logits) and the router's share of dx.
// One wavefront per token.  dL (dense [T, N], storage type DT) feeds d_w_gate = x^T dL.
// With the load-balance loss (logits != NULL) its gradient joins every entry of the row and the
// router's share of dx runs over all N experts instead of the k picked ones (dx == NULL: left to
// the caller).
template <typename DT, int PER>
__global__ __launch_bounds__(256) void gate_backward_kernel(const int32_t* __restrict__ topk_idx, const float* __restrict__ topk_w,
                                                            const float* __restrict__ dgate, const float* __restrict__ wg_t /*[N,d]*/,
                                                            const float* __restrict__ logits, const float* __restrict__ share, float aux_scale,
                                                            DT* __restrict__ dL, float* __restrict__ dx, float* __restrict__ dl_picked,
                                                            int T, int d, int N, int k) {
  const int lane = threadIdx.x & 63;
  const int t = blockIdx.x * 4 + (threadIdx.x >> 6);
  if (t >= T) return;
  float w = 0.0f, g = 0.0f;
  int e = 0;
  if (lane < k) {
    w = topk_w[(size_t)t * k + lane];
    g = dgate[(size_t)t * k + lane];
    e = topk_idx[(size_t)t * k + lane];
  }
  float aux[PER], dl;                     // aux: the whole row of dlogits
  gate_backward_row<DT, PER>(w, g, e, logits ? logits + (size_t)t * N : nullptr, share, aux_scale, N, k, lane, dL + (size_t)t * N,
                             dl_picked ? dl_picked + (size_t)t * k : nullptr, aux, dl);
  if (!dx) return;                        // the caller forms the router's share of dx as a product with dL
  for (int c0 = 0; c0 < d; c0 += 256) {
    const int c = c0 + lane * 4;
    float4 acc = make_float4(0.f, 0.f, 0.f, 0.f);
    if (!logits) {
      for (int j = 0; j < k; ++j) {
        const float dj = __shfl(dl, j, 64);
        const int ej = __shfl(e, j, 64);
        if (c < d) {
          const float4 wv = *(const float4*)(wg_t + (size_t)ej * d + c);
          acc.x = fmaf(dj, wv.x, acc.x); acc.y = fmaf(dj, wv.y, acc.y);
          acc.z = fmaf(dj, wv.z, acc.z); acc.w = fmaf(dj, wv.w, acc.w);
        }
      }
    } else {
#pragma unroll
      for (int i = 0; i < PER; ++i) {
        if (i * 64 >= N) break;
        const int live = min(64, N - i * 64);
        for (int l = 0; l < live; ++l) {
          const float dn = __shfl(aux[i], l, 64);
          if (c < d) {
            const float4 wv = *(const float4*)(wg_t + (size_t)(i * 64 + l) * d + c);
            acc.x = fmaf(dn, wv.x, acc.x); acc.y = fmaf(dn, wv.y, acc.y);
            acc.z = fmaf(dn, wv.z, acc.z); acc.w = fmaf(dn, wv.w, acc.w);
          }
        }
      }
    }
    if (c < d) *(float4*)(dx + (size_t)t * d + c) = acc;
  }
}

// The router's share of dx without the loss:  dx[t, c] = sum_j dl[t, j] w_gate[c, e_j].  A
// workgroup keeps CPL*64 rows of w_gate, transposed (wt[n][c]: one expert's weights for the
// workgroup's columns lie side by side), and its tokens' picks in the LDS, so each pick costs a
// lane one LDS read of its CPL adjacent columns instead of a cached global row.
template <int CPL, int NMAX>
__global__ __launch_bounds__(ROUTER_DX_THREADS) void router_dx_kernel(const int32_t* __restrict__ topk_idx, const float* __restrict__ dl_picked,
                                                        const float* __restrict__ w_gate /*[d,N]*/, float* __restrict__ dx,
                                                        int T, int d, int N, int k, int tokens_per_block) {
  constexpr int TC = CPL * 64, PITCH = TC + 4;
  constexpr int PER_THREAD = TC * NMAX / 4 / ROUTER_DX_THREADS, BATCH = PER_THREAD > 8 ? 8 : (PER_THREAD < 1 ? 1 : PER_THREAD);
  typedef float cols_t __attribute__((ext_vector_type(CPL)));
  __shared__ __attribute__((aligned(16))) float wt[NMAX * PITCH];
  __shared__ float s_dl[ROUTER_DX_PICKS];
  __shared__ int s_e[ROUTER_DX_PICKS];
  const int c0 = blockIdx.x * TC;
  // A workgroup fills its rows of w_gate once and then walks the token groups blockIdx.y,
  // blockIdx.y + gridDim.y, ...: the picks of a group are requested before the work in front of
  // them (the fill; the sums of the group before) and stored into the LDS behind it.
  constexpr int PICK_LOADS = (ROUTER_DX_PICKS + ROUTER_DX_THREADS - 1) / ROUTER_DX_THREADS;
  const int groups = (T + tokens_per_block - 1) / tokens_per_block;
  float pick_dl[PICK_LOADS];
  int pick_e[PICK_LOADS];
  auto request_picks = [&](int group) {
    const int t_beg = group * tokens_per_block, picks_here = (min(T, t_beg + tokens_per_block) - t_beg) * k;
#pragma unroll
    for (int u = 0; u < PICK_LOADS; ++u) {
      const size_t at = (size_t)t_beg * k + min(u * ROUTER_DX_THREADS + (int)threadIdx.x, picks_here - 1);
      pick_dl[u] = dl_picked[at];
      pick_e[u] = topk_idx[at];
    }
  };
  auto stage_picks = [&](int group) {
    const int t_beg = group * tokens_per_block, picks_here = (min(T, t_beg + tokens_per_block) - t_beg) * k;
#pragma unroll
    for (int u = 0; u < PICK_LOADS; ++u) {
      const int i = u * ROUTER_DX_THREADS + (int)threadIdx.x;
      if (i < picks_here) { s_dl[i] = pick_dl[u]; s_e[i] = pick_e[u]; }
    }
  };
  int group = blockIdx.y;
  if (group >= groups) return;
  request_picks(group);
  if ((N & 3) == 0) {
    // 16-byte loads, a batch in flight per lane.  Work item g = (group, quad in row % 4, row % 16):
    // 16 lanes take the same quad of 16 consecutive rows, 4 such sets make a wavefront.  Its four
    // transposing stores then write 16 consecutive words in each of 4 rows of wt that lie
    // 4 * PITCH = 16 (mod 64) words apart: all 64 banks once.  (In row-major order of w_gate the
    // stores of a wavefront would fall on 4 banks.)  Rows past d are clamped to the last one
    // (their outputs are never stored).
    const int qrow = N >> 2, qsets = (qrow + 3) >> 2, items = (TC / 16) * qsets * 64, last_row = d - 1 - c0;
    const float4* src = (const float4*)(w_gate + (size_t)c0 * N);
    for (int g0 = 0; g0 < items; g0 += ROUTER_DX_THREADS * BATCH) {
      float4 v[BATCH];
#pragma unroll
      for (int u = 0; u < BATCH; ++u) {
        const int g = g0 + u * ROUTER_DX_THREADS + (int)threadIdx.x, group = g >> 6;
        const int c = min((group % (TC / 16)) * 16 + (g & 15), last_row);
        const int n4 = min((group / (TC / 16)) * 4 + ((g >> 4) & 3), qrow - 1);
        v[u] = src[c * qrow + n4];
      }
#pragma unroll
      for (int u = 0; u < BATCH; ++u) {
        const int g = g0 + u * ROUTER_DX_THREADS + (int)threadIdx.x, group = g >> 6;
        const int c = (group % (TC / 16)) * 16 + (g & 15), n4 = (group / (TC / 16)) * 4 + ((g >> 4) & 3);
        if (g < items && n4 < qrow) {
          float* dst = wt + n4 * 4 * PITCH + c;
          dst[0] = v[u].x; dst[PITCH] = v[u].y; dst[2 * PITCH] = v[u].z; dst[3 * PITCH] = v[u].w;
        }
      }
    }
  } else {
    for (int i = threadIdx.x; i < TC * N; i += ROUTER_DX_THREADS) {
      const int c = i / N, n = i - c * N;
      wt[n * PITCH + c] = c0 + c < d ? w_gate[(size_t)(c0 + c) * N + n] : 0.0f;
    }
  }
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const float* mine = wt + lane * CPL;
  while (true) {
    stage_picks(group);
    __syncthreads();                    // the picks (and, the first time, the rows of w_gate) are in the LDS
    const int next = group + (int)gridDim.y;
    if (next < groups) request_picks(next);
    const int t_beg = group * tokens_per_block, t_end = min(T, t_beg + tokens_per_block);
    for (int t = t_beg + wave; t < t_end; t += ROUTER_DX_THREADS / 64) {
      const int base = (t - t_beg) * k;
      // lane j holds pick j (k <= 64); every lane then reads them back one by one
      const int at = base + min(lane, k - 1);
      const int dl_bits = __float_as_int(s_dl[at]), e_mine = s_e[at];
      cols_t acc = 0.0f;
      // U picks at a time: their LDS reads are independent, the sums keep the order j = 0, 1, ...
      auto picks = [&](auto width, int j) {
        constexpr int U = decltype(width)::value;
        float dj[U];
        cols_t w[U];
#pragma unroll
        for (int u = 0; u < U; ++u) {
          dj[u] = __int_as_float(__builtin_amdgcn_readlane(dl_bits, j + u));
          w[u] = *(const cols_t*)(mine + __builtin_amdgcn_readlane(e_mine, j + u) * PITCH);
        }
#pragma unroll
        for (int u = 0; u < U; ++u)
#pragma unroll
          for (int q = 0; q < CPL; ++q) acc[q] = fmaf(dj[u], w[u][q], acc[q]);
      };
      int j = 0;
      for (; j + 8 <= k; j += 8) picks(std::integral_constant<int, 8>{}, j);
      if (j + 4 <= k) { picks(std::integral_constant<int, 4>{}, j); j += 4; }
      for (; j < k; ++j) picks(std::integral_constant<int, 1>{}, j);
      const int c = c0 + lane * CPL;
      if (c < d) __builtin_nontemporal_store(acc, (cols_t*)(dx + (size_t)t * d + c));
    }
    if (next >= groups) break;
    __syncthreads();                    // everyone is done with this group's picks
    group = next;
  }
}

}  // namespace

// 16-byte pieces of a router row; 32-bit byte offsets within a tile's up to 32 token rows.  (Router rows are addressed stage by stage, by 64-bit
// bases.  From 2 GiB of them on the kernel with one 64-bit address per load, as ever.)
static bool router_whole_chunks(const bigmac_dims& D) {
  return D.N % 4 == 0 && (size_t)D.d * D.N * 4 < (1ull << 31) && (size_t)D.d * 32 * esize(D.dtype) < (1ull << 31);
}

bool router_picks(const bigmac_dims& D) { return D.N <= 16 && router_whole_chunks(D); }

int launch_router_logits(const bigmac_dims& D, const void* x, const float* w_gate, const float* bias, float* logits, hipStream_t s, int32_t* topk_idx, float* topk_w) {
  if (topk_idx && !router_picks(D)) return BIGMAC_ERR_INVALID_ARG;
  if (!router_whole_chunks(D)) {
    const dim3 block(256);
    const unsigned gy = (unsigned)((D.N + R_NB - 1) / R_NB);
    const dim3 grid((D.T + 31) / 32, gy);
    if (D.dtype == BIGMAC_BF16) hipLaunchKernelGGL(router_logits_kernel<bf16_t>, grid, block, 0, s, (const bf16_t*)x, w_gate, bias, logits, D.T, D.d, D.N);
    else hipLaunchKernelGGL(router_logits_kernel<float>, grid, block, 0, s, (const float*)x, w_gate, bias, logits, D.T, D.d, D.N);
    BIGMAC_CHECK_LAUNCH();
    return BIGMAC_OK;
  }
  // Few tokens of few elements: the kernel on the vector ALU, with the fewest tokens per wavefront that need at most three workgroups per CU.
  // bigmac_route, us, this kernel / the tiles below.  One token, up to 256 workgroups T 32, N 64: d 64 4.9 / 6.2, d 512 6.1 / 6.9, d 1024
  // 7.5 / 7.8, d 1280 8.2 / 8.4 (fp32 8.3 / 8.4; N 20, T 500 8.9 / 8.8); up to 512 T 500, N 64: d 256 5.8 / 6.4, d 768 7.3 / 7.6, d 1024 8.0 / 8.2
  // (fp32 8.4 / 8.3); up to 768 T 700, N 64: d 384 6.7 / 7.2, d 512 7.1 / 7.3, d 768 8.1 / 7.8, T 500, N 96, d 512 8.3 / 8.2; two tokens
  // T 1400, N 64: d 384 7.6 / 8.4, d 512 8.5 / 8.5; up to 1024 of them T 2000, N 64: d 128 7.0 / 7.4, d 384 8.6 / 8.5; T 1400, N 96 (1050): d 128 8.7 / 8.5.
  // Up to 16 experts (that are not picked in the same launch) a tile has one slice only and the tiles gain later.  N 16, bf16 / fp32: T 3000, d 512 7.4 / 7.5
  // and 7.5 / 7.8, d 768 8.2 / 8.1; two tokens T 4500, d 1536 12.7 / 13.2 and 13.3 / 13.9, d 2048 14.7 / 15.0 and 15.5 / 16.3, d 3072 19.4 / 18.7; T 6000,
  // d 2048 15.3 / 15.2; four T 13294, d 256 12.2 / 14.1, d 1024 17.7 / 19.2 and 22.0 / 22.9, d 2048 25.2 / 25.8 and 32.3 / 29.4; T 18000, d 1024 22.9 /
  // 23.4, d 1536 27.8 / 27.5; T 32768, d 512 26.2 / 28.4 and 29.3 / 29.7, d 1024 33.7 / 34.8 and 41.3 / 39.9.
  const long slices = (D.N + R_NB - 1) / R_NB, one = ((long)D.T + 3) / 4 * slices, two = ((long)D.T + 7) / 8 * slices;
  const int most = one <= 256 ? 1024 : one <= 512 ? 768 : slices == 1 ? (one <= 768 ? 512 : two <= 768 ? 1536 : D.T <= 28672 ? 1024 : 512) : two <= 768 ? 384 : two <= 1024 ? 128 : 0;
  if (!topk_idx && D.d <= most) {
    const int tokens = one <= 768 ? 1 : two <= 768 || slices > 1 ? 2 : 4;
    const dim3 grid((unsigned)((((long)D.T + 4 * tokens - 1) / (4 * tokens) + 7) / 8 * 8 * slices));
#define BIGMAC_ROUTER_FEW(XT, TB) hipLaunchKernelGGL((router_logits_few_kernel<XT, TB>), grid, dim3(256), 0, s, (const XT*)x, w_gate, bias, logits, D.T, D.d, D.N)
    if (D.dtype == BIGMAC_BF16) {
      if (tokens == 1) BIGMAC_ROUTER_FEW(bf16_t, 1);
      else if (tokens == 2) BIGMAC_ROUTER_FEW(bf16_t, 2);
      else BIGMAC_ROUTER_FEW(bf16_t, 4);
    } else {
      if (tokens == 1) BIGMAC_ROUTER_FEW(float, 1);
      else if (tokens == 2) BIGMAC_ROUTER_FEW(float, 2);
      else BIGMAC_ROUTER_FEW(float, 4);
    }
#undef BIGMAC_ROUTER_FEW
    BIGMAC_CHECK_LAUNCH();
    return BIGMAC_OK;
  }
  // Tile of a workgroup: 32 x 32 logits keep the multipliers busiest, smaller ones give more workgroups.  A tile takes a time per 64 rows
  // of d and one of its own (start, reduction), and a CU, which holds one workgroup, its share of the tiles one after the other.
  // Measured, us with the top-k, 32 x 32 / 16 x 32 / 16 x 16: d 4096, N 64: T 32 25.2 / 17.8 / 12.9, T 2048 25.5 / 19.5 / 21.8,
  // T 8192 48.3 / 56.9 / 65.0; d 1024, N 64: T 3001 12.7 / 14.9 / 14.3, T 8192 20.7 / 24.8 / 27.7; T 32768, d 4096, N 128 355 / 415 / 542;
  // T 30000, d 1280, N 8 45.1 / 52.9 / 36.6.  Fused multiply-adds on the vector ALU, up to 8 tokens per wavefront: 16.1, 25.5, 67.0; 13.5,
  // 26.3; 504; 37.3.
  auto tile_rounds = [&](int tokens, int experts) {   // tiles of an XCD over its 32 CUs
    const long groups = (((long)D.T + tokens - 1) / tokens + 7) / 8 * ((D.N + experts - 1) / experts);
    return (double)((groups + 31) / 32);
  };
  const double nq = D.d / 64;
  const double us22 = tile_rounds(32, 32) * (0.27 * nq + 2.0), us12 = tile_rounds(16, 32) * (0.155 * nq + 1.7), us11 = tile_rounds(16, 16) * (0.077 * nq + 1.2);
  auto job_of = [&](int tokens, int experts, int blocks_per_stage) {
    RouterJob j = {};
    j.x = x; j.wg = w_gate; j.bias = bias; j.logits = logits;
    j.T = D.T; j.d = D.d; j.N = D.N;
    j.slices = (D.N + experts - 1) / experts;
    j.blocks = (int)(((long)D.T + tokens - 1) / tokens);
    j.stages = (D.d / 64 + blocks_per_stage - 1) / blocks_per_stage;
    const long groups = ((long)j.blocks + 7) / 8 * j.slices, bytes = (long)D.d * D.N * 4;
    // (from 128 KB, a third of a microsecond of a CU's stream, up to half an XCD's L2)
    if (groups <= 24 && bytes >= 131072 && bytes <= 2097152) j.warm_lines = (int)(bytes / 128);
    j.stride = (int)(j.warm_lines ? 32 : std::min(groups, 32l));
    j.block_step = j.stride / j.slices;
    j.slice_step = j.stride % j.slices;
    j.slices_inverse = (65536u + j.slices - 1) / j.slices;
    return j;
  };
#define BIGMAC_ROUTER(XT, TT, ET, ...)                                                                                                       \
  hipLaunchKernelGGL((router_logits_matrix_kernel<XT, TT, ET, __VA_ARGS__>), dim3((unsigned)(8 * job.stride)), dim3(512), 0, s, job)
  RouterJob job;
  if (topk_idx) {
    job = job_of(16, 16, 4);
    job.topk_idx = topk_idx; job.topk_w = topk_w; job.k = D.k;
    if (D.dtype == BIGMAC_BF16) BIGMAC_ROUTER(bf16_t, 1, 1, 4, true);
    else BIGMAC_ROUTER(float, 1, 1, 4, true);
  } else if (us22 <= us12 && us22 <= us11) {
    job = job_of(32, 32, 2);
    if (D.dtype == BIGMAC_BF16) BIGMAC_ROUTER(bf16_t, 2, 2, 2);
    else BIGMAC_ROUTER(float, 2, 2, 2);
  } else if (us12 <= us11) {
    job = job_of(16, 32, D.dtype == BIGMAC_BF16 ? 4 : 2);
    if (D.dtype == BIGMAC_BF16) BIGMAC_ROUTER(bf16_t, 1, 2, 4);
    else BIGMAC_ROUTER(float, 1, 2, 2);
  } else {
    job = job_of(16, 16, 4);
    if (D.dtype == BIGMAC_BF16) BIGMAC_ROUTER(bf16_t, 1, 1, 4);
    else BIGMAC_ROUTER(float, 1, 1, 4);
  }
#undef BIGMAC_ROUTER
  BIGMAC_CHECK_LAUNCH();
  return BIGMAC_OK;
}

// Counting, a workgroup takes a part of the sort's chunks (a part past the end counts nothing), two tokens per wavefront on up to
// 16 wavefronts: several on a SIMD hide each other's latencies.  Else four wavefronts of one token each: level with
// eight tokens in pairs or up to 20 % faster up to 16384 tokens, 1 to 4 % slower from 32768 on.  (Four tokens on wavefronts made for
// pairs had each of them sort the last token beside its own: bigmac_route at d 64, N 128, T 512 / 4096 / 32768
// 8.0 / 17.4 / 90.5 us, 7.2 / 14.7 / 75.9 so.)
TopkGrid topk_grid(int T, int k, int N, bool counting) {
  if (!counting) return {(T + 3) / 4, 256, 4};
  const SortChunks sc = sort_chunks(T, k, N, true);
  return {sc.count * sc.parts, std::min(1024, (sc.tokens + 1) / 2 * 64), sc.tokens};
}

// Beside a product the wavefronts sort two tokens at a time, counting or not: four tokens per workgroup had each of them sort its one token
// twice.  With eight the layer's forward-only call (h 64) at k 1 and T 4096 takes, d 256 / 1024, r = d / 4: 96 experts 53.2 -> 51.2 us, 64.4 ->
// 61.5; 128 experts 54.6 -> 52.6, 63.8 -> 60.7; fewer tokens, or up to 64 experts, level to 1.6 us faster.
TopkJob topk_job_beside(const bigmac_dims& D, const float* logits, int32_t* topk_idx, float* topk_w, int32_t* counts) {
  const TopkGrid G = counts ? topk_grid(D.T, D.k, D.N, true) : TopkGrid{(D.T + 7) / 8, 256, 8};
  return {logits, topk_idx, topk_w, counts, D.T, D.N, D.k, G.tokens, G.workgroups};
}

int launch_topk_gate(const bigmac_dims& D, const float* logits, int32_t* topk_idx, float* topk_w, hipStream_t s, int32_t* counts) {
  if (counts && !topk_counts(D.T, D.k, D.N)) return BIGMAC_ERR_INVALID_ARG;
  const TopkGrid G = topk_grid(D.T, D.k, D.N, counts != nullptr);
  const dim3 g2(G.workgroups), block(G.threads);
  const int per = (D.N + 63) / 64;
#define BIGMAC_TOPK(P, U) hipLaunchKernelGGL((topk_gate_kernel<P, U>), g2, block, 0, s, logits, D.T, D.N, D.k, G.tokens, topk_idx, topk_w, counts)
  if (per <= 1 && counts) BIGMAC_TOPK(1, 2);
  else if (per <= 1) BIGMAC_TOPK(1, 1);
  else if (per <= 2 && counts) BIGMAC_TOPK(2, 2);
  else if (per <= 2) BIGMAC_TOPK(2, 1);
  else if (per <= 4) BIGMAC_TOPK(4, 1);
  else if (per <= 8) BIGMAC_TOPK(8, 1);
  else BIGMAC_TOPK(16, 1);
#undef BIGMAC_TOPK
  BIGMAC_CHECK_LAUNCH();
  return BIGMAC_OK;
}

// How the router's share of dx is formed (see launch_route_backward): on the matrix cores from the dense
// dL (N is the product's K: whole k tiles), or from the picked entries with w_gate's rows in the LDS.
static bool route_dx_by_product(const bigmac_dims& D, bool with_loss) { return with_loss && D.dtype == BIGMAC_BF16 && D.N % 32 == 0; }
static bool route_dx_tiled(const bigmac_dims& D, bool with_loss) { return !with_loss && D.N <= 128 && D.k <= 64 && D.d % 4 == 0; }

bool gate_backward_job(const bigmac_dims& D, const int32_t* topk_idx, const float* logits, const float* share, void* dL_out, void* ws, GateBackward* out) {
  const bool tiled = route_dx_tiled(D, logits != nullptr);
  if (D.dtype != BIGMAC_BF16 || D.N > 128 || !(tiled || route_dx_by_product(D, logits != nullptr))) return false;
  *out = {topk_idx, logits, share, logits ? D.aux_alpha * (float)D.N / (float)D.T : 0.0f, D.N, (bf16_t*)dL_out, tiled ? (float*)ws : nullptr};
  return true;
}

size_t route_backward_ws_bytes(const bigmac_dims& D) {
  // transposed router weights, or the picked entries of dL
  return align_up(std::max((size_t)D.N * D.d, (size_t)D.T * D.k) * sizeof(float));
}

__global__ void router_to_bf16_kernel(const float* __restrict__ in, bf16_t* __restrict__ out, size_t n) {
  const size_t i = (size_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (i < n) out[i] = f2bf(in[i]);
}

int launch_route_backward(const bigmac_dims& D, const float* w_gate, const int32_t* topk_idx,
                          const float* topk_w, const float* dgate, const float* logits, const float* share,
                          float* dx_f32, void* dL_out, void* ws, hipStream_t s, bool gate_done) {
  // With the loss every entry of a dL row is non-zero, and the router's share of dx is the dense
  // product dL w_gate^T: on bf16 runs it goes to the matrix cores (dL is stored in bf16 anyway,
  // w_gate is rounded to bf16 for this product only); otherwise the kernel walks all N rows.
  const bool by_product = route_dx_by_product(D, logits != nullptr), tiled = route_dx_tiled(D, logits != nullptr);
  if (gate_done && !by_product && !tiled) return BIGMAC_ERR_INVALID_ARG;
  float* wg_t = (float*)ws;
  if (tiled) {
    // nothing to prepare: the second kernel reads w_gate as it lies
  } else if (by_product) {
    const size_t n = (size_t)D.d * D.N;
    hipLaunchKernelGGL(router_to_bf16_kernel, dim3((unsigned)((n + 255) / 256)), dim3(256), 0, s, w_gate, (bf16_t*)ws, n);
  } else {
    hipLaunchKernelGGL(transpose_f32_kernel, dim3((D.N + 31) / 32, (D.d + 31) / 32), dim3(32, 8), 0, s, w_gate, wg_t, D.d, D.N);
  }
  BIGMAC_CHECK_LAUNCH();
  const dim3 grid((D.T + 3) / 4), block(256);
  const float aux_scale = logits ? D.aux_alpha * (float)D.N / (float)D.T : 0.0f;
  const int per = (D.N + 63) / 64;
  float* dx_kernel = by_product || tiled ? nullptr : dx_f32;
  float* dl_picked = tiled ? (float*)ws : nullptr;
#define BIGMAC_GATE_BWD(DT, P)                                                                                          \
  hipLaunchKernelGGL((gate_backward_kernel<DT, P>), grid, block, 0, s, topk_idx, topk_w, dgate, wg_t, logits, share, aux_scale, \
                     (DT*)dL_out, dx_kernel, dl_picked, D.T, D.d, D.N, D.k)
#define BIGMAC_GATE_BWD_PER(DT)          \
  if (per <= 1) BIGMAC_GATE_BWD(DT, 1);  \
  else if (per <= 2) BIGMAC_GATE_BWD(DT, 2); \
  else if (per <= 4) BIGMAC_GATE_BWD(DT, 4); \
  else if (per <= 8) BIGMAC_GATE_BWD(DT, 8); \
  else BIGMAC_GATE_BWD(DT, 16)
  if (gate_done) {
    // the combine's backward wrote dL and the picked entries
  } else if (D.dtype == BIGMAC_BF16) {
    BIGMAC_GATE_BWD_PER(bf16_t);
  } else {
    BIGMAC_GATE_BWD_PER(float);
  }
#undef BIGMAC_GATE_BWD_PER
#undef BIGMAC_GATE_BWD
  BIGMAC_CHECK_LAUNCH();
  if (tiled) {
    // tokens per workgroup: as many as the staging holds, fewer while the grid would leave CUs idle
    const int width = ROUTER_DX_CPL * 64;
    const unsigned gx = (unsigned)((D.d + width - 1) / width);
    int tokens = std::min(ROUTER_DX_TOKENS, ROUTER_DX_PICKS / D.k);
    while (tokens > 16 && (long)gx * ((D.T + tokens - 1) / tokens) < 256) tokens /= 2;
    // token groups per workgroup: the rows of w_gate are filled once per workgroup, so each walks
    // several groups once the grid has four workgroups per CU anyway
    unsigned gy_dx = (unsigned)((D.T + tokens - 1) / tokens);
    if ((long)gx * gy_dx > 1024) gy_dx = std::max(1u, 1024u / gx);
    const dim3 grid_dx(gx, gy_dx);
    if (D.N <= 64)
      hipLaunchKernelGGL((router_dx_kernel<ROUTER_DX_CPL, 64>), grid_dx, dim3(ROUTER_DX_THREADS), 0, s,
                         topk_idx, dl_picked, w_gate, dx_f32, D.T, D.d, D.N, D.k, tokens);
    else
      hipLaunchKernelGGL((router_dx_kernel<ROUTER_DX_CPL, 128>), grid_dx, dim3(ROUTER_DX_THREADS), 0, s,
                         topk_idx, dl_picked, w_gate, dx_f32, D.T, D.d, D.N, D.k, tokens);
    BIGMAC_CHECK_LAUNCH();
    return BIGMAC_OK;
  }
  if (by_product) {   // dx_f32[T, d] = dL[T, N] . w_gate[d, N]^T
    GemmDesc g = {};
    g.dtype = BIGMAC_BF16; g.mode = GEMM_DENSE; g.ksplit = 1;
    g.a_kcontig = 1; g.b_kcontig = 1; g.epilogue = EPI_STORE; g.out_f32 = 1;
    g.A = dL_out; g.lda = D.N; g.M = D.T; g.K = D.N;
    g.B = ws; g.ldb = D.N; g.N = D.d;
    g.C = dx_f32; g.ldc = D.d;
    return launch_gemm(g, s);
  }
  return BIGMAC_OK;
}

// Workgroups of the column-sum pass: a fixed function of T, so that the order of the sums is too.
static int aux_parts(int T) {
  const int groups = (T + 3) / 4;
  return groups < 256 ? groups : 256;
}

size_t aux_loss_ws_bytes(const bigmac_dims& D) { return align_up((size_t)aux_parts(D.T) * D.N * sizeof(float)); }

int launch_aux_loss(const bigmac_dims& D, const float* logits, const int32_t* topk_idx, float* share, float* loss,
                    float* dlogits, void* ws, hipStream_t s, const int32_t* counts) {
  float* partial = (float*)ws;
  const int parts = aux_parts(D.T), per = (D.N + 63) / 64;
#define BIGMAC_AUX_PER(KERNEL, GRID, ...)                                                         \
  if (per <= 1) hipLaunchKernelGGL(KERNEL<1>, GRID, dim3(256), 0, s, __VA_ARGS__);                \
  else if (per <= 2) hipLaunchKernelGGL(KERNEL<2>, GRID, dim3(256), 0, s, __VA_ARGS__);           \
  else if (per <= 4) hipLaunchKernelGGL(KERNEL<4>, GRID, dim3(256), 0, s, __VA_ARGS__);           \
  else if (per <= 8) hipLaunchKernelGGL(KERNEL<8>, GRID, dim3(256), 0, s, __VA_ARGS__);           \
  else hipLaunchKernelGGL(KERNEL<16>, GRID, dim3(256), 0, s, __VA_ARGS__)
  BIGMAC_AUX_PER(aux_colsum_kernel, dim3(parts), logits, D.T, D.N, partial);
  BIGMAC_CHECK_LAUNCH();
  int NP = 1;
  while (NP < D.N) NP <<= 1;
  hipLaunchKernelGGL(aux_finish_kernel, dim3(1), dim3(1024), 0, s, topk_idx, counts, counts ? topk_grid(D.T, D.k, D.N, true).workgroups : 0, partial, parts, D.T, D.N, NP, D.k, D.aux_alpha, share, loss);
  BIGMAC_CHECK_LAUNCH();
  if (dlogits) {
    const float scale = D.aux_alpha * (float)D.N / (float)D.T;
    BIGMAC_AUX_PER(aux_grad_kernel, dim3((D.T + 3) / 4), logits, share, D.T, D.N, scale, dlogits);
    BIGMAC_CHECK_LAUNCH();
  }
#undef BIGMAC_AUX_PER
  return BIGMAC_OK;
}

}  // namespace bigmac
