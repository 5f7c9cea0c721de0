// Both expert products in one kernel, for narrow experts: o = gelu(x W1[e]) W2[e] with the hidden row in registers.
//
// What bounds it: as two products, the [rows, hidden] activations are written by one kernel and read back by the
// next, which at a narrow width (each of their elements takes part in at most 2 x 256 multiply-adds) costs more
// than the arithmetic.  Here a wavefront owns 32 rows from the first product to the last: its rows' operands
// (32 x width) and its result (32 x width, fp32) stay in registers, the experts' matrices pass through the LDS in chunks of
// 32 hidden columns, and a chunk's activations go from the accumulators of the first product through the GELU
// straight into an operand of the second.  Both products are worked out transposed (matrix fragment first), so a
// lane holds four consecutive hidden columns of its row; exchanging halves between lanes l and l + 32 makes the
// eight consecutive ones that the second product wants, in the order of the separate products: bits unchanged.
// Four wavefronts per workgroup, two workgroups per CU (three at width 128) out of step with each other: one's GELU runs
// beside the other's matrix instructions, which are half of a wavefront's time.  Results leave as whole 128-byte lines through
// the LDS (stored from the registers, 32 bytes of a row at a time, the layer of 8192 tokens at width 256 took 6 % longer).  Measured
// (65536 rows of 64 experts, width 256, 1024 hidden columns): about 100 us where the two products take 68 + 63 and
// the passes over the hidden rows alone 50.  A full round of 512 tiles is some 80 us, a tile that has its CU to itself
// 45; without the GELU the kernel is a fifth faster, without the requests or with half of the LDS reads 5 to
// 10 percent: none of them is what it waits for alone.
#include "gemm_core.hpp"

namespace bigmac {

namespace {

constexpr int EP_ROWS = 128, EP_THREADS = 256, EP_CHUNK = 32;   // rows per workgroup, hidden columns per chunk
static_assert(EP_ROWS == BIGMAC_TILE_BM, "the kernel walks the square tile's map");

template <int R, bool GATHER, bool OUTF32>
__global__ __launch_bounds__(EP_THREADS) __attribute__((amdgpu_waves_per_eu(R <= 128 ? 3 : 2, R <= 128 ? 3 : 2)))
void expert_pair_kernel(ExpertPairDesc p) {
  constexpr int PASSES = R / 64;                  // requests of a lane per matrix and chunk
  constexpr int KS = R / 16, NJ = R / 32;         // k steps of the first product; column sub-tiles of the second
  constexpr unsigned W_BYTES = R * EP_CHUNK * 2, STAGE = 2 * W_BYTES;
  constexpr unsigned OUT_OF_RANGE = 0x80000000u;
  constexpr int FRAGS = KS + 2 * NJ;              // matrix fragments, and instructions, of a chunk
  constexpr int AHEAD = 3;                        // fragments read ahead of their instruction (six: no faster at width 128, spills at 256)
  __shared__ __attribute__((aligned(128))) uint4 ring[2 * STAGE / 16];
  const unsigned ring_at = lds_address(ring);
  const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane((int)threadIdx.x >> 6);
  const int half = lane >> 5;

  // tiles in the map's order, a run of them per XCD (see gemm_core.hpp)
  const int total = table_at(p.tile_map, 0), per_xcd = (total + 7) >> 3;
  const int first = (int)(blockIdx.x & 7) * per_xcd, last = min(first + per_xcd, total);
  const int stride = (int)(gridDim.x >> 3);
  struct Tile {
    int m0, m_end;
    __amdgpu_buffer_rsrc_t w1, w2;
  };
  const size_t matrix = (size_t)R * p.hid * 2;    // bytes
  auto tile_of = [&](int id) {
    Tile t;
    const bool valid = id < last;
    const int g = valid ? table_at(p.tile_map, TILE_MAP_HEADER + p.groups + 2 * id) : 0;
    t.m0 = valid ? table_at(p.tile_map, TILE_MAP_HEADER + p.groups + 1 + 2 * id) : 0;
    t.m_end = valid ? min(table_at(p.offsets, g + 1), t.m0 + EP_ROWS) : 0;
    t.w1 = __builtin_amdgcn_make_buffer_rsrc((void*)((const char*)p.w1 + g * matrix), 0, valid ? (int)matrix : 0, 0x00020000);
    t.w2 = __builtin_amdgcn_make_buffer_rsrc((void*)((const char*)p.w2 + g * matrix), 0, valid ? (int)matrix : 0, 0x00020000);
    return t;
  };
  int id = first + (int)(blockIdx.x >> 3);
  if (id >= last) return;

  // A chunk of W1 is R rows of 64 bytes, as they are (a transposing read takes four of them, 256 bytes in a row); one
  // of W2 is 32 rows of 2 R bytes, whose 64-byte pieces are permuted by the row so that the four that a read takes
  // lie on the four quarters of the banks' 256 bytes.
  auto piece_swap = [](int row) { return R % 128 ? (row >> 1) & 1 : row & 3; };
  const unsigned w1_off = (unsigned)((threadIdx.x >> 2) * (unsigned)p.hid * 2u + (threadIdx.x & 3) * 16u), w1_pass = 64u * (unsigned)p.hid * 2u;
  unsigned w2_off[R % 128 ? PASSES : 1];
#pragma unroll
  for (int i = 0; i < (R % 128 ? PASSES : 1); ++i) {
    const int q = i * EP_THREADS + (int)threadIdx.x, row = q / (R / 8), pc = q % (R / 8);
    w2_off[i] = (unsigned)(row * R * 2 + (((pc >> 2) ^ piece_swap(row)) << 6) + (pc & 3) * 16);
  }
  auto request = [&](const __amdgpu_buffer_rsrc_t& w1, const __amdgpu_buffer_rsrc_t& w2, int chunk, unsigned stage) {
#if defined(__HIP_DEVICE_COMPILE__)
    unsigned first = w1_off + (unsigned)chunk * 64u;
    unsigned first2 = w2_off[0] + (unsigned)chunk * W_BYTES;
    asm volatile("" : "+v"(first), "+v"(first2)); // (or every pass's offset would have a register of its own)
    uint4* at = ring + stage / 16 + wave * 64;
#pragma unroll
    for (int i = 0; i < PASSES; ++i)
      __builtin_amdgcn_raw_ptr_buffer_load_lds(w1, (__attribute__((address_space(3))) void*)(at + i * EP_THREADS), 16,
                                               first + i * w1_pass, 0, 0, 0);
#pragma unroll
    for (int i = 0; i < PASSES; ++i)
      __builtin_amdgcn_raw_ptr_buffer_load_lds(w2, (__attribute__((address_space(3))) void*)(at + W_BYTES / 16 + i * EP_THREADS), 16,
                                               R % 128 ? w2_off[R % 128 ? i : 0] + (unsigned)chunk * W_BYTES : first2 + i * 4096u, 0, 0, 0);
#endif
  };

  // fragment addresses (see Frag): k row (lane / 32) 8 + 4 jj + (lane % 16) / 4 of a k step, four columns
  const int frag_row = half * 8 + ((lane & 15) >> 2), frag_col = ((lane >> 4) & 1) * 16 + (lane & 3) * 4;
  const unsigned w1_at = ring_at + (unsigned)(frag_row * 64 + frag_col * 2);
  constexpr int PIECE_SETS = R % 128 ? 2 : 4;     // piece j sits at j ^ swap: one address per j % 2 or j % 4
  unsigned w2_at[PIECE_SETS];
#pragma unroll
  for (int j = 0; j < PIECE_SETS; ++j) w2_at[j] = ring_at + W_BYTES + (unsigned)(frag_row * R * 2 + ((j ^ piece_swap(frag_row)) << 6) + frag_col * 2);

  // this wavefront's rows as operands: lane l holds row l % 32, k = 16 ks + 8 (l / 32) .. + 7 (rows past the end: zeros)
  bf16x8_t x[KS];
  auto row_offset = [&](const Tile& t) -> unsigned {
    const int row = t.m0 + wave * 32 + (lane & 31);
    unsigned at = (unsigned)row;
    if (GATHER) {
      const __amdgpu_buffer_rsrc_t rg = __builtin_amdgcn_make_buffer_rsrc((void*)p.gather, 0, t.m_end * 4, 0x00020000);
      at = __builtin_amdgcn_raw_buffer_load_b32(rg, (unsigned)row * 4u, 0, 0) / (unsigned)p.gather_div;
    }
    return at | (row < t.m_end ? 0u : OUT_OF_RANGE);
  };
  // (a row index with its top bit set stands for no row; the offset within the table is built from it at the load)
  const __amdgpu_buffer_rsrc_t rx_all = __builtin_amdgcn_make_buffer_rsrc((void*)p.x, 0, (int)((size_t)p.x_rows * R * 2), 0x00020000);
  auto load_rows = [&](const Tile& t, unsigned index) {
    __amdgpu_buffer_rsrc_t rx = rx_all;
    unsigned base = (index & ~OUT_OF_RANGE) * (unsigned)(R * 2);
    if (!GATHER) {                                // (rows in order: the table may be larger than a 32-bit offset, the tile is not)
      rx = __builtin_amdgcn_make_buffer_rsrc((void*)((const char*)p.x + (size_t)t.m0 * R * 2), 0, (t.m_end - t.m0) * R * 2, 0x00020000);
      base = (unsigned)(wave * 32 + (lane & 31)) * (unsigned)(R * 2);
    }
    base = (base + half * 16u) | (index & OUT_OF_RANGE);
#pragma unroll
    for (int ks = 0; ks < KS; ++ks) x[ks] = __builtin_bit_cast(bf16x8_t, __builtin_amdgcn_raw_buffer_load_b128(rx, base + ks * 32u, 0, 0));
  };

  const int chunks = p.hid / EP_CHUNK;
  unsigned stage = 0;
  Tile cur = tile_of(id);
  load_rows(cur, row_offset(cur));
  request(cur.w1, cur.w2, 0, stage);
  f32x16_t acc[NJ];

  // in front of chunk c: it has landed for everyone and everyone has read the stage before, which the next chunk, or
  // the next tile's first, may then fill
  auto turn_stage = [&](int c, const Tile& nxt) {
    BIGMAC_WAIT_VMCNT(0);
    __builtin_amdgcn_s_barrier();
    const bool over = c == chunks - 1;
    request(over ? nxt.w1 : cur.w1, over ? nxt.w2 : cur.w2, over ? 0 : c + 1, stage ^ STAGE);
  };
  auto chunk_step = [&](int c) {
    Frag<false> f[AHEAD + 1];
    const unsigned a1 = w1_at + stage;
    unsigned a2[PIECE_SETS];
#pragma unroll
    for (int j = 0; j < PIECE_SETS; ++j) a2[j] = w2_at[j] + stage;
    // fragment n: the first product's k step n, then sub-tile (n - KS) % NJ of k step (n - KS) / NJ of the second
    auto read = [&](auto n_) {
      constexpr int n = decltype(n_)::value;
      auto& to = f[n % (AHEAD + 1)];
      if constexpr (n < KS) {
        lds_read_tr_b64<n * 16 * 64>(a1, to.h[0]);
        lds_read_tr_b64<n * 16 * 64 + 4 * 64>(a1, to.h[1]);
      } else if constexpr (n < FRAGS) {
        constexpr int ks = (n - KS) / NJ, j = (n - KS) % NJ, at = ks * 16 * R * 2 + j / PIECE_SETS * PIECE_SETS * 64;
        lds_read_tr_b64<at>(a2[j % PIECE_SETS], to.h[0]);
        lds_read_tr_b64<at + 4 * R * 2>(a2[j % PIECE_SETS], to.h[1]);
      }
    };
    auto take = [&](auto n_) -> bf16x8_t {        // fragment n, behind the request for the one AHEAD of it
      constexpr int n = decltype(n_)::value, younger = FRAGS - 1 - n < AHEAD ? FRAGS - 1 - n : AHEAD;
      read(StaticIndex<n + AHEAD>{});
      lds_wait_for<2 * younger>();
      f[n % (AHEAD + 1)].settle();
      return f[n % (AHEAD + 1)].value();
    };
    static_for<0, AHEAD>([&](auto n) { read(n); });
    f32x16_t h;
#pragma unroll
    for (int v = 0; v < 16; ++v) h[v] = 0.0f;
    static_for<0, KS>([&](auto n) {
      constexpr int ks = decltype(n)::value;
      h = __builtin_amdgcn_mfma_f32_32x32x16_bf16(take(n), x[ks], h, 0, 0, 0);
      __builtin_amdgcn_sched_barrier(0);
    });
    // GELU, and the lane's quads of columns exchanged into runs of eight
    auto eights = [&](const u32x2_t (&quad)[4], u32x4_t (&out)[2], int s) {
      const auto lo = __builtin_amdgcn_permlane32_swap(quad[2 * s].x, quad[2 * s + 1].x, false, false);
      const auto hi = __builtin_amdgcn_permlane32_swap(quad[2 * s].y, quad[2 * s + 1].y, false, false);
      out[s].x = lo[0]; out[s].y = hi[0]; out[s].z = lo[1]; out[s].w = hi[1];
    };
    u32x2_t quad[4];
    u32x4_t hidden[2];
    // The second product's first k step needs half of the activations; the others are worked out beside its matrix instructions.
    auto gelu = [&](int q) {
      quad[q].x = f2bf_pair(gelu_bf16_f(h[q * 4 + 0]), gelu_bf16_f(h[q * 4 + 1]));
      quad[q].y = f2bf_pair(gelu_bf16_f(h[q * 4 + 2]), gelu_bf16_f(h[q * 4 + 3]));
    };
    gelu(0);
    __builtin_amdgcn_sched_barrier(0);            // (all sixteen at once would not fit the registers)
    gelu(1);
    __builtin_amdgcn_sched_barrier(0);
    eights(quad, hidden, 0);
    static_for<KS, FRAGS>([&](auto n) {
      constexpr int ks = (decltype(n)::value - KS) / NJ, j = (decltype(n)::value - KS) % NJ;
      acc[j] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(take(n), __builtin_bit_cast(bf16x8_t, hidden[ks]), acc[j], 0, 0, 0);
      if constexpr (ks == 0 && j == 0) gelu(2);
      if constexpr (ks == 0 && j == NJ / 2) gelu(3);
      if constexpr (ks == 0 && j == NJ - 1) eights(quad, hidden, 1);
      __builtin_amdgcn_sched_barrier(0);
    });
  };

  while (true) {
#pragma unroll
    for (int j = 0; j < NJ; ++j)
#pragma unroll
      for (int v = 0; v < 16; ++v) {
        float zero;                               // (a constant would be kept in sixteen registers)
        asm volatile("v_mov_b32 %0, 0" : "=v"(zero));
        acc[j][v] = zero;
      }
    const bool live = cur.m0 + wave * 32 < cur.m_end;
    id += stride;
    const bool more = id < last;
    const Tile nxt = tile_of(id);
    const unsigned index = row_offset(nxt);
    BIGMAC_WAIT_VMCNT(0);                         // the rows and the first chunk
    if (live) {
#pragma clang loop unroll(disable)
      for (int c = 0; c < chunks; ++c) {
        turn_stage(c, nxt);
        chunk_step(c);
        stage ^= STAGE;
      }
    } else {
      for (int c = 0; c < chunks; ++c) {
        turn_stage(c, nxt);
        stage ^= STAGE;
      }
    }
    load_rows(nxt, index);

    // Results: lane l holds columns 32 j + 8 q + 4 (l / 32) .. + 3 of row l % 32.  They leave as whole 128-byte lines (32 columns
    // in fp32, 64 in bf16) through a strip per wavefront in the stage that everyone has read.
    __builtin_amdgcn_s_barrier();
    if (live) {
      constexpr int ESZ = OUTF32 ? 4 : 2, PER_LINE = OUTF32 ? 1 : 2;   // sub-tiles per line
      const __amdgpu_buffer_rsrc_t rc =
          __builtin_amdgcn_make_buffer_rsrc((char*)p.out + (size_t)cur.m0 * R * ESZ, 0, (cur.m_end - cur.m0) * R * ESZ, 0x00020000);
      int l = lane;
      asm volatile("" : "+v"(l));                 // (or the addresses below would have registers of their own throughout)
      // (16-byte chunk c of row r sits at c ^ (r / 2) % 8, see mfma_gemm_kernel)
      const unsigned strip = ring_at + (stage ^ STAGE) + wave * 4096, put = strip + (l & 31) * 128, swz = (l >> 1) & 7;
      const unsigned get = strip + (l >> 3) * 128 + (((l & 7) ^ (l >> 4)) << 4);
      unsigned at = (unsigned)((wave * 32 + (l >> 3)) * R * ESZ + (l & 7) * 16);
#pragma unroll
      for (int j = 0; j < NJ; j += PER_LINE) {
#pragma unroll
        for (int jj = 0; jj < PER_LINE; ++jj)
#pragma unroll
          for (int q = 0; q < 4; ++q) {
            const f32x16_t& v = acc[j + jj];
            if (OUTF32) {
              u32x4_t w;
#pragma unroll
              for (int i = 0; i < 4; ++i) w[i] = __float_as_uint(v[q * 4 + i]);
              lds_write_b128(put + (((unsigned)(q * 2 + (l >> 5)) ^ swz) << 4), w);
            } else {
              u32x2_t w;
              w.x = f2bf_pair(v[q * 4 + 0], v[q * 4 + 1]);
              w.y = f2bf_pair(v[q * 4 + 2], v[q * 4 + 3]);
              lds_write_b64(put + (l >> 5) * 8 + (((unsigned)(jj * 4 + q) ^ swz) << 4), w);
            }
          }
        u32x4_t line[4];
#pragma unroll
        for (int q = 0; q < 4; ++q) lds_read_b128((q & 1 ? get ^ 64u : get) + q * 1024, line[q]);
        lds_wait(line);
#pragma unroll
        for (int q = 0; q < 4; ++q) __builtin_amdgcn_raw_buffer_store_b128(line[q], rc, at + (unsigned)(q * 8 * R * ESZ), 0, 0);
        at += 128;
      }
    }
    if (!more) break;
    cur = nxt;
  }
}

}  // namespace

int launch_expert_pair(const ExpertPairDesc& p, hipStream_t s) {
  if (!p.x || !p.w1 || !p.w2 || !p.out || !p.tile_map || !p.offsets || p.groups <= 0 || p.max_rows <= 0 || p.hid <= 0 || p.hid % EP_CHUNK) return BIGMAC_ERR_INVALID_ARG;
  if ((size_t)p.width * p.hid * 2 >= (1ull << 31) || (p.gather && ((size_t)p.x_rows * p.width * 2 >= (1ull << 31) || p.gather_div <= 0))) return BIGMAC_ERR_INVALID_ARG;
  long blocks = ((long)p.max_rows / EP_ROWS + p.groups + 7) / 8 * 8;
  const long resident = p.width <= 128 ? 768 : 512;
  if (blocks > resident) blocks = resident;
  const dim3 grid((unsigned)blocks), block(EP_THREADS);
#define BIGMAC_PAIR(R)                                                                                                  \
  if (p.gather && p.out_f32) hipLaunchKernelGGL((expert_pair_kernel<R, true, true>), grid, block, 0, s, p);             \
  else if (p.gather) hipLaunchKernelGGL((expert_pair_kernel<R, true, false>), grid, block, 0, s, p);                    \
  else if (p.out_f32) hipLaunchKernelGGL((expert_pair_kernel<R, false, true>), grid, block, 0, s, p);                   \
  else hipLaunchKernelGGL((expert_pair_kernel<R, false, false>), grid, block, 0, s, p);
  switch (p.width) {
    case 128: BIGMAC_PAIR(128) break;
    case 192: BIGMAC_PAIR(192) break;
    case 256: BIGMAC_PAIR(256) break;
    default: return BIGMAC_ERR_UNSUPPORTED;
  }
#undef BIGMAC_PAIR
  BIGMAC_CHECK_LAUNCH();
  return BIGMAC_OK;
}

}  // namespace bigmac
