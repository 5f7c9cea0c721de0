// Matrix products on fp32 storage (the debugging and reference precision): fp32 matrix
// instructions, every product and sum in fp32, for the same modes and epilogues as the bf16 kernels.
#include "gemm_core.hpp"

namespace bigmac {

// One wavefront computes a 32 x 32 output tile with v_mfma_f32_32x32x2_f32, operands straight from
// global memory into registers.  The fp32 workloads are small (a few hundred tokens): what bounds
// them is the chain of load latencies of one tile, not arithmetic or bytes, so there is no LDS
// staging and no barrier in the loop, small tiles give many wavefronts, and while there are fewer
// tiles than wavefront slots (KW = 4) the four wavefronts of a workgroup take a quarter of K each
// and add up through the LDS in wavefront order.  With more tiles (KW = 1) a workgroup is four
// tiles side by side.  Measured at T 256, d 256, r 64, h 256 against the 64 x 64 LDS-staged multiply-add
// kernel this replaces: x W_down 42 -> 6.5 us, expert-up 16 -> 6.0,
// expert-down 48 -> 6.8, y' W_up 14 -> 5.2; the layer call 140 -> 40 us.  At T 8192, d 2048, N 16, k 2, h 2048 (KW = 1) the
// training step 7.7 -> 5.5 ms.  Distance of its results from 64 bits: 4 to 8e-7 where that kernel had 6 to 9e-7 at the first
// size, level at 1.4 to 1.7e-6 at T 4096, d 2048.
//
// The matrix instruction takes k = 2 per step: lanes 0..31 hold k even, lanes 32..63 k odd of A's
// rows and B's columns.  Which k that is does not matter as long as A and B agree, so the lower half
// of the wavefront owns k = 0..3 and the upper half k = 4..7 of each group of eight: a k-contiguous
// operand is then read 16 bytes per lane, the other kind 128 contiguous bytes per half.
constexpr int F32_BM = 32;
constexpr int F32_CHUNK = 32;   // k values per loop step: one step's operands are in flight while the previous one's are multiplied

template <bool AK, bool BKC, int EPI, int KW>
__global__ __launch_bounds__(256) void f32_gemm_kernel(GemmDesc p) {
  constexpr int BN = KW == 4 ? 32 : 128;
  constexpr int GROUPS = F32_CHUNK / 8;
  const TileSpace ts = tile_space<F32_BM, BN>(p);
  const int id = tile_at(ts, (int)(blockIdx.x >> 3));
  if (id < 0) return;
  const TileCoord t = resolve_tile<F32_BM, BN>(p, ts, id, 4);
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6, l = lane & 31, half = lane >> 5;
  const int n0 = t.n0 + (KW == 1 ? wave * 32 : 0);
  if (n0 >= p.N) return;                                   // (KW == 1 only: no barrier follows)
  const int per = KW == 4 ? ((t.kend - t.kbeg + 3) / 4 + 7) / 8 * 8 : t.kend - t.kbeg;
  const int kb = min(t.kbeg + (KW == 4 ? wave * per : 0), t.kend), ke = min(t.kend, kb + per);
  const float* A = (const float*)p.A;
  const float* B = (const float*)t.B;
  // rows and columns past the end repeat the last one: their results are not stored
  const size_t row = (size_t)min(t.m0 + l, t.m_end - 1), col = (size_t)min(n0 + l, p.N - 1);
  struct Step { float a[GROUPS][4], b[GROUPS][4]; };
  auto load = [&](int k0, Step& s) {
#pragma unroll
    for (int g = 0; g < GROUPS; ++g) {
      const int k = k0 + g * 8 + half * 4;
      if (AK) {
        const float4 v = k < ke ? *(const float4*)(A + row * p.lda + k) : make_float4(0.f, 0.f, 0.f, 0.f);
        s.a[g][0] = v.x; s.a[g][1] = v.y; s.a[g][2] = v.z; s.a[g][3] = v.w;
      } else {
#pragma unroll
        for (int c = 0; c < 4; ++c) s.a[g][c] = k + c < ke ? A[(size_t)(k + c) * p.lda + row] : 0.0f;
      }
      if (BKC) {
        const float4 v = k < ke ? *(const float4*)(B + col * p.ldb + k) : make_float4(0.f, 0.f, 0.f, 0.f);
        s.b[g][0] = v.x; s.b[g][1] = v.y; s.b[g][2] = v.z; s.b[g][3] = v.w;
      } else {
#pragma unroll
        for (int c = 0; c < 4; ++c) s.b[g][c] = k + c < ke ? B[(size_t)(k + c) * p.ldb + col] : 0.0f;
      }
    }
  };
  f32x16_t acc;
#pragma unroll
  for (int v = 0; v < 16; ++v) acc[v] = 0.0f;
  auto multiply = [&](const Step& s) {
#pragma unroll
    for (int g = 0; g < GROUPS; ++g)
#pragma unroll
      for (int c = 0; c < 4; ++c) acc = __builtin_amdgcn_mfma_f32_32x32x2f32(s.a[g][c], s.b[g][c], acc, 0, 0, 0);
  };
  // three register sets: two steps in flight (a step past the end loads nothing)
  Step s0, s1, s2;
  load(kb, s0);
  load(kb + F32_CHUNK, s1);
  for (int k0 = kb; k0 < ke; k0 += 3 * F32_CHUNK) {
    load(k0 + 2 * F32_CHUNK, s2);
    multiply(s0);
    if (k0 + F32_CHUNK >= ke) break;
    load(k0 + 3 * F32_CHUNK, s0);
    multiply(s1);
    if (k0 + 2 * F32_CHUNK >= ke) break;
    load(k0 + 4 * F32_CHUNK, s1);
    multiply(s2);
  }
  // accumulator value v of a lane: column l, row 8 (v / 4) + 4 half + v % 4
  auto finish = [&](int v, float a) {
    const int r = t.m0 + 8 * (v >> 2) + 4 * half + (v & 3), c = n0 + l;
    if (r >= t.m_end || c >= p.N) return;
    const size_t off = (size_t)r * p.ldc + c;
    if ((EPI == EPI_STORE || EPI == EPI_GELU) && t.bias) a += ((const float*)t.bias)[c];
    float* out = (float*)t.C + off;
    if (EPI == EPI_STORE) *out = a;
    else if (EPI == EPI_GELU) {
      if (p.aux_out) ((float*)p.aux_out)[off] = a;
      *out = gelu_f(a);
    } else if (EPI == EPI_DGELU) *out = a * gelu_grad_f(((const float*)p.aux_in)[off]);
    else *out = p.beta ? *out + a : a;
  };
  if constexpr (KW == 4) {
    __shared__ float part[4][16][64];
#pragma unroll
    for (int v = 0; v < 16; ++v) part[wave][v][lane] = acc[v];
    __syncthreads();
#pragma unroll
    for (int i = 0; i < 4; ++i) {                          // each wavefront finishes a quarter of the tile
      const int v = wave * 4 + i;
      finish(v, ((part[0][v][lane] + part[1][v][lane]) + part[2][v][lane]) + part[3][v][lane]);
    }
  } else {
#pragma unroll
    for (int v = 0; v < 16; ++v) finish(v, acc[v]);
  }
}

namespace {

template <bool AK, bool BKC>
int launch_f32(const GemmDesc& g, hipStream_t s) {
  const long nt = (g.N + 31) / 32;
  const long mt = g.mode == GEMM_RAGGED_M ? g.max_rows / F32_BM + g.groups + 1 : (g.M + F32_BM - 1) / F32_BM;
  const long zt = g.mode == GEMM_RAGGED_K ? g.groups : (g.mode == GEMM_DENSE ? g.ksplit : 1);
  // 2048 tiles: two wavefronts on every SIMD; from there on splitting K adds sums and no parallelism
  const bool split = mt * nt * zt < 2048;
  const long blocks = (mt * zt * (split ? nt : (g.N + 127) / 128) + 7) / 8 * 8;   // a multiple of the 8 XCDs (see tile_space)
  const dim3 grid((unsigned)blocks), block(256);
#define BIGMAC_F32(EPI)                                                                            \
  if (split) hipLaunchKernelGGL((f32_gemm_kernel<AK, BKC, EPI, 4>), grid, block, 0, s, g);         \
  else hipLaunchKernelGGL((f32_gemm_kernel<AK, BKC, EPI, 1>), grid, block, 0, s, g)
  switch (g.epilogue) {
    case EPI_STORE: BIGMAC_F32(EPI_STORE); break;
    case EPI_GELU: BIGMAC_F32(EPI_GELU); break;
    case EPI_DGELU: BIGMAC_F32(EPI_DGELU); break;
    case EPI_ACCUM: BIGMAC_F32(EPI_ACCUM); break;
    default: return BIGMAC_ERR_INVALID_ARG;
  }
#undef BIGMAC_F32
  BIGMAC_CHECK_LAUNCH();
  return BIGMAC_OK;
}

}  // namespace

int launch_gemm_f32(const GemmDesc& g, hipStream_t s) {
  // k-contiguous operands are read 16 bytes at a time
  if ((g.a_kcontig && (g.lda % 4 || g.K % 8)) || (g.b_kcontig && (g.ldb % 4 || g.K % 8)) || g.kwrap_b || g.gather || g.scatter) return BIGMAC_ERR_UNSUPPORTED;
  switch (g.a_kcontig * 2 + g.b_kcontig) {
    case 2: return launch_f32<true, false>(g, s);
    case 3: return launch_f32<true, true>(g, s);
    case 0: return launch_f32<false, false>(g, s);
    default: return BIGMAC_ERR_UNSUPPORTED;
  }
}

int gemm_f32_tile_rows() { return F32_BM; }

}  // namespace bigmac
