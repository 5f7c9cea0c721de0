// The 256 x 256 matrix product: eight wavefronts, one workgroup per CU, 64-deep k tiles.
//
// What bounds it: operand delivery.  At 256 x 256 a CU needs 64 KB per k tile, which is 0.85 us of
// matrix instructions; a line that misses the L2 takes 0.5 to 1 us under load.  With the two 64 KB
// stages handed over whole (all of a k tile requested when the one before it starts, all of it
// awaited when that ends) every such line is waited for.  Here a stage is given back in two pieces,
// as soon as its last fragment has been read into registers, and requested again at once: the
// requests run 1.5 to 2 k tiles ahead, no wait in the loop asks for the youngest eight requests of a
// lane, and the stream does not stop at the end of an output tile: the last two k tiles' places go
// to the first two of the workgroup's next tile, so an epilogue starts with all of them on their way.
#include "gemm_core.hpp"

namespace bigmac {

namespace {

constexpr int PH_BM = 256, PH_BN = 256, PH_BK = 64, PH_THREADS = 512;
static_assert(PH_BM == BIGMAC_TALL_BM, "its ragged-M products walk the second tile map");
constexpr unsigned PH_STAGE = 65536, PH_B_AT = 32768, PH_HALF = 16384;   // bytes: a ring stage, B's place in it, half of A's
constexpr int PH_STRIP = 4096;                                          // epilogue staging: 32 rows x 128 bytes per wavefront

// Requests of one lane for a 64-deep k tile: four 16-byte pieces of A (two per 128-row half) and four
// of B.  A pass moves 512 pieces; passes differ by a constant in memory and in the LDS.
template <bool KC, int COLS>   // COLS: chunks (16 bytes) per LDS row
struct PassMover {
  unsigned voff, col;   // byte offsets: of the lane's piece in the first pass, and within its row
  __device__ __forceinline__ void init(long ld) {
    int row, cc;
    if (KC) lds_unchunk_kc<COLS>((int)threadIdx.x, row, cc);
    else lds_unchunk_tr<COLS>((int)threadIdx.x, row, cc);
    col = (unsigned)cc * 16u;
    voff = (unsigned)(row * ld) * 2u + col;
  }
};

__device__ __forceinline__ void load_piece(__amdgpu_buffer_rsrc_t rsrc, uint4* lds, unsigned voff) {
#if defined(__HIP_DEVICE_COMPILE__)
  __builtin_amdgcn_raw_ptr_buffer_load_lds(rsrc, (__attribute__((address_space(3))) void*)lds, 16, voff, 0, 0, 0);
#else
  (void)rsrc; (void)lds; (void)voff;
#endif
}

template <int MODE, bool AK, bool BKC, int EPI, bool OUTF32, bool GATHER = false, bool SCATTER = false>
__global__ __launch_bounds__(PH_THREADS) __attribute__((amdgpu_waves_per_eu(2, 2)))
void phased_gemm_kernel(GemmDesc desc) {
  GemmDesc p = desc;
  p.mode = MODE;                            // a constant from here on, as is what only one mode has
  p.ksplit = 1;
  if (MODE != GEMM_DENSE) p.kwrap_b = 0;
  if (MODE == GEMM_RAGGED_K) p.bias = nullptr;
  constexpr bool SWAP = !(EPI == EPI_ACCUM || OUTF32);   // bf16 results accumulate the transposed tile (see mfma_gemm_kernel)
  constexpr unsigned OUT_OF_RANGE = 0x80000000u;
  constexpr int NON_TEMPORAL = 2;
  constexpr int STREAMING = (EPI == EPI_GELU || EPI == EPI_DGELU) ? NON_TEMPORAL : 0;
  __shared__ uint4 ring[(2 * PH_STAGE + (SWAP ? 8 * PH_STRIP : 256)) / 16];
  const unsigned ring_at = lds_address(ring);
  const unsigned box_at = ring_at + 2 * PH_STAGE;   // the claimed tile, in the first wavefront's strip: written behind its epilogue

  const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane((int)threadIdx.x >> 6);
  const int wr = wave >> 2, wc = wave & 3;
  // A wavefront owns the rows s * 64 + wr * 32 .. + 31 (s = 0 .. 3) and the columns wc * 64 .. + 63 of
  // the tile: its fragments of rows below 128 are read first, which frees that half of A's stage.
  PassMover<AK, AK ? 8 : 16> ma;
  PassMover<BKC, BKC ? 8 : 32> mb;
  ma.init(p.lda);
  mb.init(p.ldb);
  const unsigned a_pass = (unsigned)((AK ? 64 : 32) * p.lda * 2), b_pass = (unsigned)((BKC ? 64 : 16) * p.ldb * 2);
  const int wave_chunk = wave * 64;
  const int wrap_tiles = p.kwrap_b ? p.kwrap_b / PH_BK : 0x7FFFFFFF;

  TileSpace ts = tile_space<PH_BM, PH_BN>(p);
  if (p.mode == GEMM_RAGGED_K && p.tile_map) balance_ragged_k(p, ts);
  // Positions of the XCD's run: its tiles in order; where the last round would keep at most half of the XCD's
  // workgroups, that round's tiles are cut into row halves, one workgroup each.
  const int stride = (int)(gridDim.x >> 3), tiles = ts.last - ts.first;
  const int last_round = tiles > 0 ? tiles % stride : 0;
  int whole = 2 * last_round <= stride ? tiles - last_round : tiles;
  if (MODE == GEMM_RAGGED_K && p.tile_map) {
    // skewed routing: a tile of the heaviest group is one serial chain over all of its rows; where that is more than
    // twice the rows that a workgroup walks on average, every tile is cut
    const long long heaviest = (long long)(table_at(p.tile_map, 10) - 8) * TILE_MAP_K_ROWS, all = table_at(p.offsets, p.groups);
    if (heaviest * (long long)gridDim.x > 2 * all * ts.gx * ts.gy) whole = 0;
  }
  auto operands = [&](int at) {   // of a position; none: empty ranges
    const int half = at - whole, i = half < 0 ? at : whole + (half >> 1);
    TileCoord t = resolve_tile<PH_BM, PH_BN>(p, ts, i < tiles ? ts.first + i : -1, 2);
    if (half >= 0 && t.valid) {
      t.m0 += (half & 1) * (PH_BM / 2);
      t.m_end = max(t.m0, min(t.m_end, t.m0 + PH_BM / 2));
      if (t.m_end == t.m0) t.kend = t.kbeg;   // (a tile of few rows has no second half)
    }
    return tile_operands<PH_BM, PH_BN, PH_BK, AK, BKC, GATHER>(p, t);
  };

  int pos = (int)(blockIdx.x >> 3);
  TileOperands cur = operands(pos), nxt = cur, src = cur;   // src: where the requests stand, k tile `fk` of it is next
  if (!cur.t.valid) return;
  int fk = 0;
  // (a group without rows, or one k tile only: the second k tile is requested out of range, zeros)
  auto tiles_of = [&](const TileOperands& o) { return o.nk < 2 ? 2 : o.nk; };
  // GATHER (see mfma_gemm_kernel): row m of the product is row gather[m] / gather_div of A.  The indices of a
  // tile's 256 rows are requested a tile ahead into the second wavefront's strip, which is idle outside the
  // epilogue, and turned into the lane's four piece offsets where the requests move on to that tile.
  static_assert(!GATHER || (AK && SWAP), "gathered rows are k-contiguous rows of A; the index lies in a strip");
  const unsigned index_at = ring_at + 2 * PH_STAGE + PH_STRIP;
  unsigned row_off[GATHER ? 4 : 1];
  auto index_buffer = [&](const TileCoord& t) { return __builtin_amdgcn_make_buffer_rsrc((void*)p.gather, 0, t.valid ? t.m_end * 4 : 0, 0x00020000); };
  auto request_index = [&](const TileCoord& t) {   // (lanes 256 .. 511 fill the rest of their 2 KB; one request per lane)
    if (GATHER) {
#if defined(__HIP_DEVICE_COMPILE__)
      __builtin_amdgcn_raw_ptr_buffer_load_lds(index_buffer(t), (__attribute__((address_space(3))) void*)(ring + (2 * PH_STAGE + PH_STRIP) / 16 + wave * 16), 4,
                                               (unsigned)(t.m0 + (int)threadIdx.x) * 4u, 0, 0, 0);
#endif
    }
  };
  auto place_rows = [&](const unsigned (&index)[4]) {
#pragma unroll
    for (int i = 0; i < (GATHER ? 4 : 1); ++i) row_off[i] = (index[i] / (unsigned)p.gather_div) * (unsigned)(p.lda * 2) + ma.col;
  };
  auto take_index = [&]() {
    if (GATHER) {
      u32x4_t v;
      const unsigned at = index_at + ((unsigned)threadIdx.x >> 3) * 4u;   // piece i holds row threadIdx / 8 + 64 i
      asm volatile("ds_read_b32 %0, %4\n\tds_read_b32 %1, %4 offset:256\n\tds_read_b32 %2, %4 offset:512\n\tds_read_b32 %3, %4 offset:768\n\ts_waitcnt lgkmcnt(0)"
                   : "=&v"(v.x), "=&v"(v.y), "=&v"(v.z), "=&v"(v.w) : "v"(at) : "memory");
      const unsigned index[4] = {v.x, v.y, v.z, v.w};
      place_rows(index);
    }
  };
  if (GATHER) {   // the first tile's
    unsigned index[4];
#pragma unroll
    for (int i = 0; i < 4; ++i)
      index[i] = __builtin_amdgcn_raw_buffer_load_b32(index_buffer(cur.t), (unsigned)(cur.t.m0 + (int)(threadIdx.x >> 3) + 64 * i) * 4u, 0, 0);
    place_rows(index);
  }
  unsigned off_a = 0, off_a2 = 0, off_b = 0;
  auto rows_over_half = [](const TileCoord& t) { return t.m_end - t.m0 > PH_BM / 2; };
  auto aim = [&]() {   // offsets of the next k tile to request
    if (fk == tiles_of(src)) {
      src = nxt;
      fk = 0;
      take_index();
    }
    const bool live = fk < src.nk;
    off_a = live ? (unsigned)fk * src.step_a : OUT_OF_RANGE;
    off_a2 = rows_over_half(src.t) ? off_a : OUT_OF_RANGE;   // the second row half
    off_b = live ? (unsigned)((fk + src.wrap_first) % wrap_tiles) * src.step_b : OUT_OF_RANGE;
    ++fk;
  };
  auto load_a = [&](unsigned stage, int i) {   // piece i of 4: half i / 2
    const unsigned v = GATHER ? row_off[GATHER ? i : 0] : AK ? ma.voff + i * a_pass : ma.voff + (i & 1) * a_pass + (i >> 1) * 256u;
    load_piece(src.ra, ring + stage / 16 + i * PH_THREADS + wave_chunk, v + (i < 2 ? off_a : off_a2));
  };
  auto load_b = [&](unsigned stage, int i) {
    load_piece(src.rb, ring + (stage + PH_B_AT) / 16 + i * PH_THREADS + wave_chunk, mb.voff + i * b_pass + off_b);
  };

  // fragment addresses (LDS bytes, stage 0).  k-contiguous: one per operand, k step ks is an XOR of
  // ks * 32 away (the swizzle); transposing reads: one per sub-tile, everything else is an offset.
  unsigned pa[2], pb[2];
  if (AK) {
    pa[0] = pa[1] = ring_at + lds_chunk_kc<8>(wr * 32 + (lane & 31), lane >> 5) * 16;
  } else {
#pragma unroll
    for (int i = 0; i < 2; ++i) {
      const int c = i * 64 + wr * 32 + ((lane >> 4) & 1) * 16 + (lane & 3) * 4;
      pa[i] = ring_at + lds_chunk_tr<16>((lane >> 5) * 8 + ((lane & 15) >> 2), c >> 3) * 16 + (c & 7) * 2;
    }
  }
  if (BKC) {
    pb[0] = pb[1] = ring_at + PH_B_AT + lds_chunk_kc<8>(wc * 64 + (lane & 31), lane >> 5) * 16;
  } else {
#pragma unroll
    for (int j = 0; j < 2; ++j) {
      const int c = wc * 64 + j * 32 + ((lane >> 4) & 1) * 16 + (lane & 3) * 4;
      pb[j] = ring_at + PH_B_AT + lds_chunk_tr<32>((lane >> 5) * 8 + ((lane & 15) >> 2), c >> 3) * 16 + (c & 7) * 2;
    }
  }
  Frag<AK> fa[2][2][2];   // [buffer][k step of the k half][sub-tile of the row half]
  Frag<BKC> fb[4][2];     // [k step][column sub-tile]
  auto read_a = [&](auto buf, auto half, auto khalf, auto n, unsigned stage) {   // fragment n of 4
    constexpr int b = decltype(buf)::value, h = decltype(half)::value, q = decltype(khalf)::value, kk = decltype(n)::value >> 1, i = decltype(n)::value & 1;
    constexpr int ks = q * 2 + kk;
    if constexpr (AK) lds_read_b128<h * PH_HALF + i * 8192>((pa[0] ^ (ks * 32)) + stage, fa[b][kk][i].q);
    else {
      lds_read_tr_b64<h * PH_HALF + ks * 4096>(pa[i] + stage, fa[b][kk][i].h[0]);
      lds_read_tr_b64<h * PH_HALF + ks * 4096 + 1024>(pa[i] + stage, fa[b][kk][i].h[1]);
    }
  };
  auto read_b = [&](auto khalf, auto n, unsigned stage) {
    constexpr int ks = decltype(khalf)::value * 2 + (decltype(n)::value >> 1), j = decltype(n)::value & 1;
    if constexpr (BKC) lds_read_b128<j * 4096>((pb[0] ^ (ks * 32)) + stage, fb[ks][j].q);
    else {
      lds_read_tr_b64<ks * 8192>(pb[j] + stage, fb[ks][j].h[0]);
      lds_read_tr_b64<ks * 8192 + 2048>(pb[j] + stage, fb[ks][j].h[1]);
    }
  };
  auto settle = [&](auto buf, auto khalf) {   // behind the wait: the fragments of a phase are usable
    constexpr int b = decltype(buf)::value, q = decltype(khalf)::value;
#pragma unroll
    for (int kk = 0; kk < 2; ++kk)
#pragma unroll
      for (int i = 0; i < 2; ++i) {
        fa[b][kk][i].settle();
        fb[q * 2 + kk][i].settle();
      }
  };
  constexpr StaticIndex<0> I0{};
  constexpr StaticIndex<1> I1{};

  // prologue: the first two k tiles
#pragma unroll
  for (unsigned s = 0; s < 2; ++s) {
    aim();
#pragma unroll
    for (int i = 0; i < 2; ++i) load_a(s * PH_STAGE, i);
#pragma unroll
    for (int i = 0; i < 4; ++i) load_b(s * PH_STAGE, i);
#pragma unroll
    for (int i = 2; i < 4; ++i) load_a(s * PH_STAGE, i);
  }
  unsigned* const ctr = p.claim ? p.claim + (blockIdx.x & 7) * 16 : nullptr;
  // Claims (see TileClaim) run one tile ahead: requested as a tile's k loop starts, taken when it ends (the result of
  // a memory operation is awaited with everything in front of it; behind the epilogue that would be its stores, 3000 to
  // 7000 cycles of the first wavefront and of the others at the next barrier), published behind the epilogue.
  // (The address is hidden from the compiler, which otherwise reduces the addition over the wavefront first and then
  // waits for the result on the spot.)
  unsigned no_offset = 0;
  asm volatile("" : "+v"(no_offset));
  unsigned got = 0;
  auto request_claim = [&]() {
    if (ctr && threadIdx.x == 0) got = __hip_atomic_fetch_add(ctr + no_offset, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
  };
  request_claim();
  int claimed = stride + __builtin_amdgcn_readfirstlane((int)got);   // (the first wavefront's is the one that counts)
  int written = 0;   // sub-tiles that the last epilogue stored
  unsigned stage = 0;

  while (true) {
    // publish the claimed tile; what the previous epilogue left in flight behind the requests may stay
    constexpr int STORES = SWAP ? 4 : 32;   // at least so many instructions per sub-tile are younger than the requests (the counter holds 63)
    if (ctr && threadIdx.x == 0) {
      const unsigned v = (unsigned)claimed;
      asm volatile("ds_write_b32 %0, %1" ::"v"(box_at), "v"(v) : "memory");
    }
    asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
    if (written == 4) BIGMAC_WAIT_VMCNT((4 * STORES < 63 ? 4 * STORES : 63));
    else if (written == 3) BIGMAC_WAIT_VMCNT((3 * STORES < 63 ? 3 * STORES : 63));
    else if (written == 2) BIGMAC_WAIT_VMCNT((2 * STORES < 63 ? 2 * STORES : 63));
    else if (written == 1) BIGMAC_WAIT_VMCNT(STORES);
    else BIGMAC_WAIT_VMCNT(0);
    __builtin_amdgcn_s_barrier();
    // the tile after this one, looked up behind the first matrix instructions: a chain of scalar loads
    auto look_ahead = [&]() {
      if (ctr) {
        unsigned v;
        asm volatile("ds_read_b32 %0, %1\n\ts_waitcnt lgkmcnt(0)" : "=v"(v) : "v"(box_at) : "memory");
        pos = __builtin_amdgcn_readfirstlane((int)v);
      } else {
        pos += stride;
      }
      nxt = operands(pos);
      request_index(nxt.t);
    };
    const TileCoord t = cur.t;
    const int nk = tiles_of(cur);

    f32x16_t acc[4][2];
#pragma unroll
    for (int i = 0; i < 4; ++i)
#pragma unroll
      for (int j = 0; j < 2; ++j)
#pragma unroll
        for (int v = 0; v < 16; ++v) acc[i][j][v] = 0.0f;
    auto mm = [&](auto half, auto khalf, auto buf, auto n) {   // matrix instruction n of 8 of a phase
      constexpr int h = decltype(half)::value, q = decltype(khalf)::value, b = decltype(buf)::value;
      constexpr int kk = decltype(n)::value >> 2, i = (decltype(n)::value >> 1) & 1, j = decltype(n)::value & 1;
      auto& c = acc[h * 2 + i][j];
      c = SWAP ? __builtin_amdgcn_mfma_f32_32x32x16_bf16(fb[q * 2 + kk][j].value(), fa[b][kk][i].value(), c, 0, 0, 0)
               : __builtin_amdgcn_mfma_f32_32x32x16_bf16(fa[b][kk][i].value(), fb[q * 2 + kk][j].value(), c, 0, 0, 0);
      __builtin_amdgcn_sched_barrier(0);
    };
    // a tile of at most 128 rows leaves out the second row half
    const bool tall = rows_over_half(t);

    static_for<0, 4>([&](auto n) { read_a(I0, I0, I0, n, stage); });
    static_for<0, 4>([&](auto n) { read_b(I0, n, stage); });
    request_claim();
    int it = 0;
    asm volatile("" : "+s"(it));   // (the compiler would peel the first turns off the loop for the two conditional waits)
#pragma clang loop unroll(disable)
    for (; it < nk; ++it) {
      // phase 1: rows 0 .. 127, k 0 .. 31; the fragments of k 32 .. 63 arrive meanwhile
      asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
      settle(I0, I0);
      static_for<0, 8>([&](auto n) {
        mm(I0, I0, I0, n);
        if constexpr (decltype(n)::value < 4) {
          read_a(I1, I0, I1, n, stage);
          read_b(I1, n, stage);
        }
      });
      if (it == 0) look_ahead();
      asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
      settle(I1, I1);
      // the second row half of this k tile has landed (all of the first two had before the loop; a tile of two
      // or three k tiles reads the next tile's index below, which was requested after them)
      if (it > 1) BIGMAC_WAIT_VMCNT(8);
      else if (GATHER && it + 2 == nk) { if (it == 0) BIGMAC_WAIT_VMCNT(0); else BIGMAC_WAIT_VMCNT(8); }
      __builtin_amdgcn_s_barrier();          // ... everyone's part of it; everyone has read the first row half and B
      // phase 2: rows 0 .. 127, k 32 .. 63
      aim();
      static_for<0, 8>([&](auto n) {
        constexpr int m = decltype(n)::value;
        mm(I0, I1, I1, n);
        if constexpr (m < 4) read_a(I0, I1, I0, n, stage);
        if constexpr (m >= 1 && m < 3) load_a(stage, m - 1);
        if constexpr (m >= 3 && m < 7) load_b(stage, m - 3);
      });
      // phase 3: rows 128 .. 255, k 0 .. 31
      asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
      settle(I0, I0);
      if (tall) {
        static_for<0, 8>([&](auto n) {
          mm(I1, I0, I0, n);
          if constexpr (decltype(n)::value < 4) read_a(I1, I1, I1, n, stage);
        });
        asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
      }
      settle(I1, I1);
      if (it > 0) BIGMAC_WAIT_VMCNT(8);      // the first row half and B of the next k tile have landed
      __builtin_amdgcn_s_barrier();          // ... everyone's part; everyone has read the second row half
      // phase 4: rows 128 .. 255, k 32 .. 63; the next k tile's first fragments
      const unsigned other = stage ^ PH_STAGE;
      if (tall) {
        static_for<0, 8>([&](auto n) {
          constexpr int m = decltype(n)::value;
          mm(I1, I1, I1, n);
          if constexpr (m < 4) {
            read_a(I0, I0, I0, n, other);
            read_b(I0, n, other);
          }
          if constexpr (m >= 4 && m < 6) load_a(stage, m - 2);
        });
      } else {
        static_for<0, 4>([&](auto n) {
          read_a(I0, I0, I0, n, other);
          read_b(I0, n, other);
        });
        load_a(stage, 2);
        load_a(stage, 3);
      }
      stage = other;
    }
    // (the last turn has read fragments of the next output tile, possibly ahead of their landing; they are read
    // again behind the wait above, and their registers are free once these reads have delivered)
    asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
    settle(I0, I0);
    if (wave == 0) claimed = stride + __builtin_amdgcn_readfirstlane((int)got);

    // ---- epilogue.  Output rows as buffers (see mfma_gemm_kernel).
    // A wavefront leaves at its first sub-tile without rows: the last row tile of a group holds half a tile on
    // average, a decode batch's only one a quarter or less, and the GELU of a whole tile takes longer than what is
    // requested by then (62 rows per expert, K 1024: expert-up 115 -> 107 us, the forward-only call of 500 tokens 276 -> 262; the
    // training step of 8192 tokens at d 1024 603 -> 595 us).
    written = min(max((t.m_end - t.m0 - wr * 32 + 63) >> 6, 0), 4);
    auto rows_of = [&](const void* base, int esz_out) { return output_rows<PH_BM>(p, t, base, esz_out); };
    if ((EPI == EPI_GELU || EPI == EPI_STORE) && t.bias) {
#pragma unroll
      for (int i = 0; i < 4; ++i)
#pragma unroll
        for (int j = 0; j < 2; ++j) {
          if (SWAP) add_bias_transposed(acc[i][j], (const bf16_t*)t.bias, t.n0 + wc * 64 + j * 32, p.N, lane);
          else add_bias_plain(acc[i][j], (const bf16_t*)t.bias, t.n0 + wc * 64 + j * 32, p.N, lane);
        }
    }
    if constexpr (!SWAP) {
      const __amdgpu_buffer_rsrc_t rc = rows_of(t.C, 4);
      const unsigned row_step = (unsigned)(p.ldc * 4);
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        if (i >= written) break;
#pragma unroll
        for (int j = 0; j < 2; ++j) {
          const int col = t.n0 + wc * 64 + j * 32 + (lane & 31);
          unsigned off[4];
#pragma unroll
          for (int vq = 0; vq < 4; ++vq) {
            const int row = i * 64 + wr * 32 + vq * 8 + (lane >> 5) * 4;
            off[vq] = (unsigned)(((size_t)row * p.ldc + col) * 4) | ((unsigned)(p.N - 1 - col) >> 31) * OUT_OF_RANGE;
          }
          if (EPI == EPI_ACCUM && p.beta) {
            float old[16];
#pragma unroll
            for (int v = 0; v < 16; ++v)
              old[v] = __uint_as_float(__builtin_amdgcn_raw_buffer_load_b32(rc, off[v >> 2] + (v & 3) * row_step, 0, 0));
#pragma unroll
            for (int v = 0; v < 16; ++v) acc[i][j][v] += old[v];
          }
#pragma unroll
          for (int v = 0; v < 16; ++v)
            __builtin_amdgcn_raw_buffer_store_b32(__float_as_uint(acc[i][j][v]), rc, off[v >> 2] + (v & 3) * row_step, 0, NON_TEMPORAL);
        }
      }
    } else {
      constexpr int SROW = 128;
      const unsigned strip = ring_at + 2 * PH_STAGE + wave * PH_STRIP;
      const unsigned quad_row = strip + (lane & 31) * SROW + (lane >> 5) * 8;
      const unsigned quad_swz = (lane >> 1) & 7;
      auto quad_at = [&](int j, int vq) { return quad_row + ((((unsigned)(j * 4 + vq)) ^ quad_swz) << 4); };
      const unsigned row_even = strip + (lane >> 3) * SROW + (((lane & 7) ^ (lane >> 4)) << 4);
      const unsigned row_odd = strip + (lane >> 3) * SROW + (((lane & 7) ^ (lane >> 4) ^ 4) << 4);
      auto row_at = [&](int q) { return (q & 1 ? row_odd : row_even) + q * 8 * SROW; };
      const int out_col = t.n0 + wc * 64 + (lane & 7) * 8;
      const __amdgpu_buffer_rsrc_t rc = rows_of(t.C, 2);
      const __amdgpu_buffer_rsrc_t rx = rows_of(EPI == EPI_GELU && p.aux_out ? p.aux_out : t.C, 2);
      const unsigned out_off = (unsigned)(((size_t)(wr * 32 + (lane >> 3)) * p.ldc + out_col) * 2) | ((unsigned)(p.N - 1 - out_col) >> 31) * OUT_OF_RANGE;
      const unsigned pass_step = (unsigned)(8 * p.ldc * 2);
      // EPI_DGELU: the saved pre-activation, a sub-tile (32 rows) at a time, two sub-tiles ahead
      const __amdgpu_buffer_rsrc_t rin = rows_of(EPI == EPI_DGELU ? p.aux_in : t.C, 2);
      uint4 aux[EPI == EPI_DGELU ? 8 : 1];
      auto request_aux = [&](int i) {
        if (EPI == EPI_DGELU) {
          unsigned at = out_off + (unsigned)(i * 8) * pass_step;
          asm volatile("" : "+v"(at));
#pragma unroll
          for (int q = 0; q < 4; ++q)
            aux[(i & 1) * 4 + q] = __builtin_bit_cast(uint4, __builtin_amdgcn_raw_buffer_load_b128(rin, at + (unsigned)q * pass_step, 0, NON_TEMPORAL));
        }
      };
      request_aux(0);
      request_aux(1);
      auto flush_rows = [&](const __amdgpu_buffer_rsrc_t& dst, int i) {
        u32x4_t v[4];
#pragma unroll
        for (int q = 0; q < 4; ++q) lds_read_b128(row_at(q), v[q]);
        lds_wait(v);
#pragma unroll
        for (int q = 0; q < 4; ++q)
          __builtin_amdgcn_raw_buffer_store_b128(v[q], dst, out_off + (unsigned)(i * 8 + q) * pass_step, 0, STREAMING);
      };
      // SCATTER (see mfma_gemm_kernel): the staged rows of a sub-tile leave once per pick, eight picks at a time
      auto flush_scattered = [&](int i) {
        const __amdgpu_buffer_rsrc_t rs = __builtin_amdgcn_make_buffer_rsrc((void*)p.scatter, 0, p.M * p.scatter_k * 4, 0x00020000);
        const __amdgpu_buffer_rsrc_t rd = __builtin_amdgcn_make_buffer_rsrc(p.C, 0, (int)((size_t)p.scatter_rows * p.ldc * 2), 0x00020000);
        const unsigned col_off = (unsigned)out_col * 2u | ((unsigned)(p.N - 1 - out_col) >> 31) * OUT_OF_RANGE;
        const unsigned row_bytes = (unsigned)(p.ldc * 2);
        u32x4_t v[4];
#pragma unroll
        for (int q = 0; q < 4; ++q) lds_read_b128(row_at(q), v[q]);
        lds_wait(v);
        for (int j0 = 0; j0 < p.scatter_k; j0 += 8) {
          int slot[4][8];
          unsigned dead[4][8];
#pragma unroll
          for (int q = 0; q < 4; ++q) {
            const int row = t.m0 + i * 64 + wr * 32 + q * 8 + (lane >> 3);
#pragma unroll
            for (int j = 0; j < 8; ++j) {
              dead[q][j] = ((unsigned)(t.m_end - 1 - row) >> 31) | ((unsigned)(p.scatter_k - 1 - (j0 + j)) >> 31);
              slot[q][j] = (int)__builtin_amdgcn_raw_buffer_load_b32(rs, (unsigned)((row * p.scatter_k + j0 + j) * 4) | dead[q][j] * OUT_OF_RANGE, 0, 0);
            }
          }
#pragma unroll
          for (int q = 0; q < 4; ++q)
#pragma unroll
            for (int j = 0; j < 8; ++j) {
              const unsigned gone = dead[q][j] | ((unsigned)slot[q][j] >> 31);
              __builtin_amdgcn_raw_buffer_store_b128(v[q], rd, ((unsigned)slot[q][j] * row_bytes + col_off) | gone * OUT_OF_RANGE, 0, 0);
            }
        }
      };
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        if (i >= written) break;
        u32x2_t pre[EPI == EPI_DGELU ? 8 : 1];
        if (EPI == EPI_DGELU) {
#pragma unroll
          for (int q = 0; q < 4; ++q) lds_write_b128(row_at(q), __builtin_bit_cast(u32x4_t, aux[(i & 1) * 4 + q]));
#pragma unroll
          for (int j = 0; j < 2; ++j)
#pragma unroll
            for (int vq = 0; vq < 4; ++vq) lds_read_b64(quad_at(j, vq), pre[(j * 4 + vq) % (EPI == EPI_DGELU ? 8 : 1)]);
          lds_wait(pre);
          if (i < 2) request_aux(i + 2);
        }
        // GELU with the pre-activation kept: its rows wait in the strip while the GELU is worked out, so that
        // neither pass through the strip is waited for
        const bool keep = EPI == EPI_GELU && p.aux_out;
        if (keep) {
#pragma unroll
          for (int j = 0; j < 2; ++j)
#pragma unroll
            for (int vq = 0; vq < 4; ++vq) {
              u32x2_t w;
              w.x = f2bf_pair(acc[i][j][vq * 4 + 0], acc[i][j][vq * 4 + 1]);
              w.y = f2bf_pair(acc[i][j][vq * 4 + 2], acc[i][j][vq * 4 + 3]);
              lds_write_b64(quad_at(j, vq), w);
            }
        }
        u32x2_t packed[8];
#pragma unroll
        for (int j = 0; j < 2; ++j)
#pragma unroll
          for (int vq = 0; vq < 4; ++vq) {
            float v[4];
#pragma unroll
            for (int vr = 0; vr < 4; ++vr) v[vr] = acc[i][j][vq * 4 + vr];
            if (EPI == EPI_GELU) {
#pragma unroll
              for (int vr = 0; vr < 4; ++vr) v[vr] = gelu_bf16_f(v[vr]);
            } else if (EPI == EPI_DGELU) {
              const u32x2_t sv = pre[(j * 4 + vq) % (EPI == EPI_DGELU ? 8 : 1)];
              v[0] *= gelu_grad_bf16_f(__uint_as_float(sv.x << 16));
              v[1] *= gelu_grad_bf16_f(__uint_as_float(sv.x & 0xFFFF0000u));
              v[2] *= gelu_grad_bf16_f(__uint_as_float(sv.y << 16));
              v[3] *= gelu_grad_bf16_f(__uint_as_float(sv.y & 0xFFFF0000u));
            }
            packed[j * 4 + vq].x = f2bf_pair(v[0], v[1]);
            packed[j * 4 + vq].y = f2bf_pair(v[2], v[3]);
          }
        if (keep) flush_rows(rx, i);
#pragma unroll
        for (int j = 0; j < 2; ++j)
#pragma unroll
          for (int vq = 0; vq < 4; ++vq) lds_write_b64(quad_at(j, vq), packed[j * 4 + vq]);
        if (SCATTER) flush_scattered(i);
        else flush_rows(rc, i);
      }
    }
    if (!nxt.t.valid) break;
    cur = nxt;
  }
}

}  // namespace

int launch_gemm_phased(const GemmDesc& g, hipStream_t s) {
  long gx = (g.N + PH_BN - 1) / PH_BN, gy, gz = 1;
  if (g.mode == GEMM_RAGGED_M) gy = g.max_rows / PH_BM + g.groups + 1;
  else gy = (g.M + PH_BM - 1) / PH_BM;
  if (g.mode == GEMM_RAGGED_K) gz = g.groups;
  long blocks = (2 * gx * gy * gz + 7) / 8 * 8;   // (few tiles are cut into row halves)
  if (blocks > 256) blocks = 256;
  if ((g.a_kcontig || g.b_kcontig) && g.K % PH_BK) return BIGMAC_ERR_INVALID_ARG;
  const dim3 grid((unsigned)blocks), block(PH_THREADS);
#define BIGMAC_PHASED(MODE, AK, BKC, EPI, ...) hipLaunchKernelGGL((phased_gemm_kernel<MODE, AK, BKC, EPI, __VA_ARGS__>), grid, block, 0, s, g)
  const int combo = g.a_kcontig * 2 + g.b_kcontig;
  if (g.mode == GEMM_RAGGED_M) {
    if (g.gather) {
      if (combo == 2 && g.epilogue == EPI_GELU) BIGMAC_PHASED(GEMM_RAGGED_M, true, false, EPI_GELU, false, true);
      else return BIGMAC_ERR_UNSUPPORTED;
    } else if (combo == 2 && g.epilogue == EPI_STORE && g.out_f32) BIGMAC_PHASED(GEMM_RAGGED_M, true, false, EPI_STORE, true);
    else if (combo == 2 && g.epilogue == EPI_STORE) BIGMAC_PHASED(GEMM_RAGGED_M, true, false, EPI_STORE, false);
    else if (combo == 2 && g.epilogue == EPI_GELU) BIGMAC_PHASED(GEMM_RAGGED_M, true, false, EPI_GELU, false);
    else if (combo == 3 && g.epilogue == EPI_STORE && g.out_f32) BIGMAC_PHASED(GEMM_RAGGED_M, true, true, EPI_STORE, true);
    else if (combo == 3 && g.epilogue == EPI_STORE) BIGMAC_PHASED(GEMM_RAGGED_M, true, true, EPI_STORE, false);
    else if (combo == 3 && g.epilogue == EPI_DGELU) BIGMAC_PHASED(GEMM_RAGGED_M, true, true, EPI_DGELU, false);
    else return BIGMAC_ERR_UNSUPPORTED;
  } else if (g.mode == GEMM_RAGGED_K) {
    if (combo == 0 && g.epilogue == EPI_ACCUM) BIGMAC_PHASED(GEMM_RAGGED_K, false, false, EPI_ACCUM, true);
    else return BIGMAC_ERR_UNSUPPORTED;
  } else {
    if (g.scatter) BIGMAC_PHASED(GEMM_DENSE, true, false, EPI_STORE, false, false, true);
    else if (combo == 2 && g.epilogue == EPI_STORE && g.out_f32) BIGMAC_PHASED(GEMM_DENSE, true, false, EPI_STORE, true);
    else if (combo == 2 && g.epilogue == EPI_STORE) BIGMAC_PHASED(GEMM_DENSE, true, false, EPI_STORE, false);
    else if (combo == 3 && g.epilogue == EPI_STORE && g.out_f32) BIGMAC_PHASED(GEMM_DENSE, true, true, EPI_STORE, true);
    else if (combo == 3 && g.epilogue == EPI_ACCUM) BIGMAC_PHASED(GEMM_DENSE, true, true, EPI_ACCUM, true);
    else return BIGMAC_ERR_UNSUPPORTED;
  }
#undef BIGMAC_PHASED
  BIGMAC_CHECK_LAUNCH();
  return BIGMAC_OK;
}

}  // namespace bigmac
