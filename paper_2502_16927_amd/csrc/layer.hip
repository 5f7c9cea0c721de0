// C ABI of libbigmac: argument checks, workspace planning and the launch sequences of the
// layer (Eq. 2 with the expert of Eq. 4; CDAC order with the expert of Eq. 3) and its backward.
#include <cmath>

#include "common.hpp"
#include "tile_map.hpp"

namespace bigmac {

int check_dims(const bigmac_dims* D) {
  if (!D) return BIGMAC_ERR_INVALID_ARG;
  if (D->T < 1 || D->d < 64 || D->r < 64 || D->N < 1 || D->k < 1) return BIGMAC_ERR_INVALID_ARG;
  if (D->d % 64 || D->r % 64) return BIGMAC_ERR_INVALID_ARG;
  if (D->order != BIGMAC_ORDER_DCCA && D->order != BIGMAC_ORDER_CDAC) return BIGMAC_ERR_INVALID_ARG;
  if (D->order == BIGMAC_ORDER_DCCA && (D->h < 64 || D->h % 64)) return BIGMAC_ERR_INVALID_ARG;
  if (D->k > D->N || D->N > 1024 || D->k > 64) return BIGMAC_ERR_INVALID_ARG;
  if ((long long)D->T * D->k >= (1ll << 31)) return BIGMAC_ERR_INVALID_ARG;
  if (D->dtype != BIGMAC_F32 && D->dtype != BIGMAC_BF16) return BIGMAC_ERR_INVALID_ARG;
  if (D->act != BIGMAC_ACT_GELU_ERF) return BIGMAC_ERR_INVALID_ARG;
  if (D->flags & ~(BIGMAC_FLAG_ACCUMULATE | BIGMAC_FLAG_OUT_BF16 | BIGMAC_FLAG_WIRE_BF16 | BIGMAC_FLAG_TILES_LARGE | BIGMAC_FLAG_TILES_SMALL | BIGMAC_FLAG_ROUTE_LOW |
                   BIGMAC_FLAG_NO_FUSED_DISPATCH)) return BIGMAC_ERR_INVALID_ARG;
  if ((D->flags & BIGMAC_FLAG_TILES_LARGE) && (D->flags & BIGMAC_FLAG_TILES_SMALL)) return BIGMAC_ERR_INVALID_ARG;
  if (D->capacity < 0 || !(D->aux_alpha >= 0.0f) || D->aux_alpha > 1e30f) return BIGMAC_ERR_INVALID_ARG;
  if (D->order == BIGMAC_ORDER_CDAC && D->dtype == BIGMAC_BF16 && (D->flags & BIGMAC_FLAG_OUT_BF16)) return BIGMAC_ERR_UNSUPPORTED;
  if ((D->flags & BIGMAC_FLAG_ROUTE_LOW) && D->order == BIGMAC_ORDER_CDAC) return BIGMAC_ERR_INVALID_ARG;   // the fine-grained layer has no x'
  if ((D->flags & BIGMAC_FLAG_ROUTE_LOW) && D->aux_alpha > 0.0f) return BIGMAC_ERR_UNSUPPORTED;
  return BIGMAC_OK;
}

namespace {

void* const* g_stage_events = nullptr;  // profiling aid, see bigmac_set_stage_events

struct StageTimer {  // records the caller's events around the launches of one stage
  hipStream_t s;
  int stage;
  StageTimer(hipStream_t s_, int stage_) : s(s_), stage(stage_) {
    if (g_stage_events) (void)hipEventRecord((hipEvent_t)g_stage_events[2 * stage], s);
  }
  ~StageTimer() {
    if (g_stage_events) (void)hipEventRecord((hipEvent_t)g_stage_events[2 * stage + 1], s);
  }
};
#ifndef BIGMAC_DEEP_MAX_TILES
#define BIGMAC_DEEP_MAX_TILES 256   // 128 x 128 tiles (one per CU) up to which a dense product takes the 128 x 64 x 64 tile
#endif
// Which products take the square tile with 64-deep k tiles (two ring stages) when they do not
// take the 256 x 256 one: 1 expert-up, 2 expert-down, 4 the GELU' product, 8 the data gradient of the
// first matrix, 16 the data gradient of the descending projection, 32 the ascending projection.
// Measured at gpt_medium: -1 %, +2.5 %, +3 %, -6 %, -11 %, -8 %.
#ifndef BIGMAC_WIDEK_MASK
#define BIGMAC_WIDEK_MASK 56
#endif
#ifndef BIGMAC_DEEP_WGRAD_MAX_TILES
#define BIGMAC_DEEP_WGRAD_MAX_TILES 16   // measured: 16 tiles 15.5 -> 13.2 us; 64 tiles (gpt_xl widths) 43 -> 48 us
#endif
#ifndef BIGMAC_DEEP_K_TILE_US
#define BIGMAC_DEEP_K_TILE_US 0.7
#endif
#define BIGMAC_STAGE(stage) StageTimer stage_timer_##stage(s, stage)

struct Carver {  // hands out 256-byte aligned pieces of one buffer
  size_t off = 0;
  size_t take(size_t bytes) {
    size_t o = off;
    off += align_up(bytes);
    return o;
  }
};

struct SavedPlan {
  size_t topk_idx, topk_w, offsets, slot_of, src_of, tile_map, tile_map_tall, x_perm, act, hact, o_perm, y_low, logits, aux, x_low, total;
};
struct FwdPlan {
  size_t logits, perm, x_low, partials, aux, claims, total;
};
struct BwdPlan {
  size_t dy_low, dgate, do_perm, dx_perm, dact, dx_low, dL, route, dx_f32, part_up, part_gate, part_down, bias_sums, gate_low, claims, total;
};

inline bool bf(const bigmac_dims& D) { return D.dtype == BIGMAC_BF16; }
inline bool route_low(const bigmac_dims& D) { return (D.flags & BIGMAC_FLAG_ROUTE_LOW) != 0; }
// the router's view of the dims: with the router on x' its input is r wide
inline bigmac_dims router_dims(const bigmac_dims& D) {
  bigmac_dims R = D;
  if (route_low(D)) R.d = D.r;
  return R;
}
// y' and dx' feed a bf16 MFMA product; they are carried as two bf16 halves (hi | lo) so that
// the product sees them at fp32 precision.  Row length of that operand:
inline int low_ld(const bigmac_dims& D) { return bf(D) ? 2 * D.r : D.r; }
// Row pitch of the layer's own [rows, hidden] tensors (activations kept for the backward pass and
// their gradients).  In bf16 the pitch is 64 elements more than the width: with a power-of-two
// pitch the k rows that a weight-gradient product walks through map onto few L2 sets, and on
// experts with many rows the operand tiles shared between workgroups were fetched several times
// (measured: up to 1.3x faster weight-gradient products at 16384 rows per expert).
inline int wide_ld(const bigmac_dims& D) { return widths(D).hid + (bf(D) ? 64 : 0); }
// The rows that come back through the second All-to-All (expert outputs O) and, in the backward
// pass, through the first (dx_perm) are only win wide.  With bf16 storage the layer calls keep
// them in fp32 unless BIGMAC_FLAG_WIRE_BF16 asks for the all-bf16 wire format: rounding them
// costs as much precision as rounding the hidden activations, for a fraction of the bytes, and
// the rounding of O is what the gate gradient <dy', O_j> sees.
inline bool wire_f32(const bigmac_dims& D) { return bf(D) && !(D.flags & BIGMAC_FLAG_WIRE_BF16); }
inline int wire_dtype(const bigmac_dims& D) { return wire_f32(D) ? BIGMAC_F32 : D.dtype; }
inline size_t low_bytes(const bigmac_dims& D) { return (size_t)D.T * (bf(D) ? 2 * D.r * 2 : D.r * 4); }

// Per-expert weight gradients on the 256 x 128 tile: up to a fifth of padding in M still pays (measured against the
// square tile: 22-30 % faster at the large shapes, level at gpt_medium).
inline bool tall_wgrad(const bigmac_dims& D, int M) {
  return bf(D) && (long)((M + 255) / 256) * 256 * 5 <= (long)M * 6;
}
// Few 128 x 128 tiles under a long K: the narrower tile with deeper k tiles (see launch_gemm).
inline bool deep_dense(const bigmac_dims& D, int M, int N, int K) {
  return bf(D) && K % 64 == 0 && K >= 512 && (long)((M + 127) / 128) * ((N + 127) / 128) <= BIGMAC_DEEP_MAX_TILES;
}
// Expert weights read line by line as a grouped product starts (GemmDesc::touch); bits: 1 expert-up,
// 2 expert-down, 4 GELU' product, 8 the first matrix's data gradient.  Measured: it pays where
// an expert has so few output tiles that they all run at once and each meets its weights in
// memory (expert-up at gpt_medium, 64 tiles per expert and K = 256: 102 -> 81 us), costs a few us
// where an expert's first tiles fetch the weights for many later ones (8192 rows per expert:
// +6 us) or where every matrix is read by one or two row tiles anyway (up to 256 rows per expert:
// +2 to +3 us), and reading more than a fraction of the 256 MB memory-side cache ahead costs more
// than it saves (128 MB at gpt_xl: +30 us); the other three products lose 1 to 4 us by it.
#ifndef BIGMAC_TOUCH_MASK
#define BIGMAC_TOUCH_MASK 1
#endif
#ifndef BIGMAC_TOUCH_MAX_BYTES
#define BIGMAC_TOUCH_MAX_BYTES ((size_t)64 << 20)
#endif
#ifndef BIGMAC_TOUCH_MAX_TILES
#define BIGMAC_TOUCH_MAX_TILES 256
#endif
#ifndef BIGMAC_TOUCH_MIN_ROWS
#define BIGMAC_TOUCH_MIN_ROWS 512
#endif
inline void touch_weights(const bigmac_dims& D, GemmDesc& g, const void* w, int bit) {
  const size_t bytes = (size_t)D.N * g.K * g.N * 2;
  const long rows_per_expert = ((long)D.T * D.k + D.N - 1) / D.N;
  const long tiles_per_expert = ((rows_per_expert + 127) / 128) * ((g.N + 127) / 128);   // 128 x 128 output tiles
  if (bf(D) && (BIGMAC_TOUCH_MASK & bit) && bytes <= BIGMAC_TOUCH_MAX_BYTES && tiles_per_expert <= BIGMAC_TOUCH_MAX_TILES &&
      rows_per_expert >= BIGMAC_TOUCH_MIN_ROWS) {
    g.touch = w;
    g.touch_bytes = bytes;
  }
}
inline bool wide_k_ok(const bigmac_dims& D, int K, int bit) {
  return bf(D) && (BIGMAC_WIDEK_MASK & bit) && K % 64 == 0;
}
// Which products run on 256 x 256 tiles (gemm_phased.hip).  Times are those of one product, the tiles of gemm.hip -> 256 x 256.
inline bool tiles_forced(const bigmac_dims& D, bool* large) {
  *large = (D.flags & BIGMAC_FLAG_TILES_LARGE) != 0;
  return !bf(D) || (D.flags & (BIGMAC_FLAG_TILES_LARGE | BIGMAC_FLAG_TILES_SMALL));
}
// How full the rounds of 256 tiles are; a last round of at most 128 tiles runs as row halves, three quarters of a round.
inline double round_fill(long tiles) {
  const long last = tiles % 256;
  return (double)tiles / 256.0 / ((double)(tiles / 256) + (last == 0 ? 0.0 : last <= 128 ? 0.75 : 1.0));
}
// Per-expert row products: the tiles that the results would fill (full), and the estimated tiles with each expert's last one
// half empty, against the 256 CUs.  Figures are one product's (or the whole layer's, where said) under even or skewed routing.
// Plain stores pay from about a quarter of the CUs on (K 512 to 2048, 49 to 56 full 1.15 of the time, 56 to 64 0.91, 72 to 99 51 -> 43,
// 24 -> 20, 34 -> 29 us; with a K of 2048 and experts that a single 256-row tile holds, which is two of the smaller ones, from 40: 44
// to 54 full 70 -> 56, 72 -> 58, 87 -> 68 us), the data gradient of the first matrix, whose both operands are k-contiguous and which the
// smaller tile also reads in whole lines, from a third on (56 to 80 full 1.04, 80 to 100 0.99, 100 to 128 0.94).  Results that leave an eighth or
// more of their column tiles empty (widths 192, 320, 384, 576, ...) also want the rounds past the first well filled: K 768 to 2304, 147
// tiles 37 -> 27 us, 236 to 248 tiles 30 -> 28, 46 -> 40, 64 -> 50 us, 270 to 320 tiles 58 -> 66, 63 -> 63, 80 -> 78 us, one call of the
// steps 134 -> 139 us; width 128 51 -> 59 us.
// The activation epilogues are not overlapped by another workgroup's k loop, so they want a longer K and more tiles (GELU and
// GELU', even routing unless said): K 384, 621 full 67 -> 70, 705 full 102 -> 79, 1037 full 140 -> 111 and 121 -> 107 us; K 512 to 768,
// 203 full 36 -> 42, 260 full under skew 71 -> 70 and 60 -> 71, 323 full of 129 rows per expert under skew 78 -> 87, 424 full 81 -> 62 and
// 67 -> 57 us; K 960, 267 full 109 -> 79 and 94 -> 73 us; K 1024, 140 full 60 -> 39 us and under skew 51 -> 58 (GELU'), 200 full 66 -> 45
// and 59 -> 43 us.  K 256 to 320: GELU' 0.85 to 0.98 of the time from 1024 tiles on under every routing (94 -> 88 us, 131 -> 117, 245 ->
// 220; 400 to 500 full 0.86 to 1.13), GELU 1.1 to 1.2 (77 -> 88 us, 100 -> 113) up to 1700 tiles.  (The routing moves these lines: both expert products, K 576, 479 full of 213 rows per expert 163 -> 140 us with
// even, 167 -> 190 us with strongly skewed routing.)
// Few rows per expert, whose products stream the weights, keep more of the smaller workgroups in flight (GELU, 4 rows 102 ->
// 112 us, 16 rows 111 -> 115 us; plain stores of 10 rows, whole layer 195 -> 204 us).  Experts that a 128-row tile holds whole
// leave half of a 256-row one idle, which only a long K makes up for (K 384, 72 rows 47 -> 54 and 44 -> 57 us; K 1024, 75 full 50 ->
// 61, 112 full 44 -> 57 (GELU'), 180 full 82 -> 76, 186 full 94 -> 89, 248 full 136 -> 124 and 135 -> 130 us) and, for plain stores, a
// round that is nearly full (72 rows, 128 tiles 43 -> 48 and 20 -> 25 us, 256 tiles 53 -> 48 and 69 -> 62 us, at K 256 14 -> 15).
inline bool big_rows(const bigmac_dims& D, int cols, int K, GemmEpilogue epilogue, bool data_gradient = false) {
  bool large;
  if (tiles_forced(D, &large)) return bf(D) && large;
  const long rows = (long)D.T * D.k, gx = (cols + 255) / 256, tiles = (rows / 256 + D.N / 2) * gx, full = rows * cols / 65536, each = rows / D.N;
  const bool gelu = epilogue == EPI_GELU;
  if (each < 48 || cols * 4 < gx * 256 * 3) return false;
  if (epilogue == EPI_STORE) {
    if (each < 128) return K >= 512 && D.N * gx * 5 >= (D.N * gx + 255) / 256 * 256 * 4;
    const bool padded = cols * 8 < gx * 256 * 7;
    if (K < 256 || full < (data_gradient ? 96 : K >= 2048 && each <= 256 ? 40 : padded ? 64 : 56)) return false;
    // (rows per expert under even routing stay within two standard deviations)
    const long even = ((long)((double)each + 2.0 * std::sqrt((double)each)) + 255) / 256 * D.N * gx, likely = even < tiles ? even : tiles;
    return !padded || likely <= 256 || round_fill(likely) >= 0.75;
  }
  if (each < 128) return K >= 1024 && full >= (gelu ? 176 : 240);
  if (K >= 512) return tiles >= (K >= 1024 ? 256 : 512) && (full >= 400 || (K >= 896 ? gelu || full >= 192 : gelu && each >= 224));
  return K >= (gelu ? 384 : 256) && full >= 640 && tiles >= (K >= 384 ? 768 : 1024);
}
// Per-expert weight gradients [M, rows] x [rows, N]: enough tiles and rows (under 128 per expert the store is most of it: 1024 x 256
// of 64 experts, 72 rows 20 -> 22 us; 4096 x 1024 112 -> 117), at least one tile high, and not much more padding than on 128-wide tiles:
// a tenth in the columns (2560 x 640: 149 -> 158 us, 640 x 2560: 164 -> 140), a fifth in the rows (576 x 2304: 440 -> 343 us with Zipf
// 1.2; 384 x 1536: 94 -> 84 us under even, 86 -> 127 under skewed routing).
// A tile is one chain over its expert's rows, at most T of them, and the chain of the larger tile is the longer one.  Against the
// rows that a CU walks on average, T k M N / 65536 / 256, by this ratio and for whole tiles: below 1 0.95 of the time, 1 to 2 0.98
// to 1.0, above 2 1.07 to 1.1, with padded rows up to 1.8 (384 x 768, k 8, Zipf 1.2: 192 -> 348 us).  With at least 90 tiles'
// worth of work per token (k M N / 65536) the ratio hardly passes 2 (512 x 2048, k 6, even routing 384 -> 349 us, Zipf 1.2 368 -> 390;
// 448 x 1792, k 8: 132 -> 125, Zipf 0.6 181 -> 201; under it 512 x 1024, k 8: 91 -> 83, Zipf 0.6 135 -> 215).
// Up to four whole tiles per expert are claimed (see launch_gemm) and cut, which levels more (1024 x 256 of 64 experts, k 8, 1024 rows
// each: 52 -> 47 us, Zipf 0.6 161 -> 138, Zipf 1.2 203 -> 172; with 400 rows 33 -> 33, Zipf 1.2 67 -> 88).
inline bool big_wgrad(const bigmac_dims& D, int M, int N) {
  bool large;
  if (tiles_forced(D, &large)) return bf(D) && large;
  const long gy = (M + 255) / 256, gx = (N + 255) / 256, each = (long)D.T * D.k / D.N;
  if (M < 256 || each < 128 || D.N * gx * gy < 256 || gx * 256 * 10 > (long)((N + 127) / 128) * 128 * 11 || gy * 256 * 5 > (long)((M + 127) / 128) * 128 * 6)
    return false;
  const double per_token = (double)M * N * D.k / 65536.0;
  return per_token >= 90 || (gx * gy <= 4 && M % 256 == 0 && N % 256 == 0 && per_token >= 32 && each >= 512);
}
// The shared projections and their data gradients: by how full the rounds of 256 tiles are.  Ascending and its counterpart at 472 and
// 252 tiles: 53 -> 51 us and 73 -> 70, 32 -> 30 and 43 -> 42; at 320 and 128 tiles: 53 -> 59 and 70 -> 74, 20 -> 22 and 26 -> 30.  The one that
// adds to dx (accumulate) keeps it from two rounds on (0.80 to 0.88 of the time); plain stores of a K under 896 are left to the
// smaller tiles (ascending, K 640, 560 tiles 60 -> 70 us, 432 tiles 52 -> 56 us; K 768, 528 tiles 71 -> 78 us).
inline bool big_dense(const bigmac_dims& D, int M, int N, int K, bool accumulate = false) {
  bool large;
  if (K % 64) return false;
  if (tiles_forced(D, &large)) return bf(D) && large;
  const long tiles = (long)((M + 255) / 256) * ((N + 255) / 256);
  if (accumulate) return tiles >= 512 || round_fill(tiles) >= 0.8;
  return K >= 896 && round_fill(tiles) >= 0.8;
}
// dy W_up^T, whose operands are both k-contiguous, gains from 90 tiles on where it does not run on the 128 x 64 tile (53 -> 44 us;
// 128 tiles 62 -> 49 us; 81 tiles 47 -> 59 us, 84 tiles 40 -> 51 us).
inline bool big_ascend_dgrad(const bigmac_dims& D) {
  bool large;
  if (tiles_forced(D, &large) || big_dense(D, D.T, D.r, D.d)) return big_dense(D, D.T, D.r, D.d);
  return !deep_dense(D, D.T, D.r, D.d) && D.d >= 1024 && (long)((D.T + 255) / 256) * ((D.r + 255) / 256) >= 90;
}
// Forward row products on 128 x 256 tiles (launch_mfma_stream), of those that the 256 x 256 tile does not take: experts with so few rows
// that reading the weights is most of it.  Times of one product, the 128 x 128 tile -> here, by experts x 256-wide column tiles.
// Up (GELU): 256 tiles 36 -> 33 us, 37 -> 34, 39 -> 35; 384 tiles 36 -> 31, 43 -> 38; 512 to 1024 tiles 70 -> 53, 77 -> 61, 92 -> 83, 94 -> 88,
// 101 -> 93; 128 and 160 tiles 21 -> 26, 17 -> 19; at K 512 the fewer k tiles want more of them (256 and 384 tiles 18 -> 20, 25 -> 27, 512 and
// 768 tiles 43 -> 38, 57 -> 57); at K 384 29 -> 28, 21 -> 23 us.
// Down (store): a round of at least 144 tiles 74 -> 68 (144), 95 -> 83, 82 -> 70, 34 -> 30 (192), 61 -> 55 us (256); 64 to 128 tiles 47 -> 60, 33 -> 40, 62 -> 76.
// A second round that is nearly empty (288 tiles) 62 -> 66 us, half full (384) 83 -> 75, 63 -> 65.  An eighth of the columns padded 97 -> 118 us.
// Rows: from 24 on (with a K of 512 from 30, stores of a K under 2048 from 40: 24 rows 24 -> 26 us, 31 rows 35 -> 29; 30 rows 20 ->
// 25, 40 rows 28 -> 26) up to 320 (there level, 0.99 to 1.01; larger counts not measured).  257 to 383 tiles: up level (1.01 / 1.02 / 1.02 times as fast
// under even routing / Zipf 0.6 / Zipf 1.2), down level where routing is even (1.00 / 1.06 / 1.07).
// Fewer rows, where next to all of the time is the stream of weights: only widths that are powers of two, whose rows all start on the same
// few memory channels, gain by the larger piece (means over 8300 shapes of 180 to 512 MB of weights per product, 2 rows and more, k 2, 4 and 8, routing as above).  Up,
// K 1024: from 448 tiles on 1.06 / 1.06 / 1.03, 384 tiles 0.98 / 0.99 / 0.99; K 512 1.03 / 1.01 / 0.94; other widths 1.00 / 1.00 / 0.98.  Down, 1024
// columns, from 8 rows on: 224 and 256 tiles 1.07 / 1.11 / 1.08, from 448 on 1.06 / 1.07 / 1.06, 320 and 384 0.99 / 1.02 / 1.07, 192 1.02 / 1.11 / 1.03, up to 160
// 0.88 / 0.91 / 0.85; 512 columns 1.04 / 1.09 / 0.78; other widths 0.99 / 1.03 / 0.98.  Down, 3 to 7 rows: skewed routing leaves CUs without a
// tile, so only where that costs nothing (from 448 tiles on 1.05 / 1.04 / 1.05) or where even routing gains most (224 and 256 tiles: K 4096 1.07 / 1.08 / 0.91, shorter
// 1.03 / 1.06 / 0.93; other widths 0.98 / 0.97 / 0.84); 2 rows 1.04 / 0.99 / 0.84.
inline bool stream_rows(const bigmac_dims& D, int cols, int K, GemmEpilogue epilogue) {
  bool large;
  if (tiles_forced(D, &large) || big_rows(D, cols, K, epilogue)) return false;
  const bool gelu = epilogue == EPI_GELU;
  const long each = (long)D.T * D.k / D.N, gx = (cols + 255) / 256, tiles = D.N * gx;
  if (K < 512 || each > 320 || cols * 10 < gx * 256 * 9 || (tiles > 256 && tiles < 384) || tiles < (!gelu ? 144 : K < 576 ? 512 : 256)) return false;
  if (each >= (gelu ? (K < 576 ? 30 : 24) : K < 2048 ? 40 : 24)) return true;
  if (cols & (cols - 1)) return false;
  if (gelu) return each >= 2 && K >= 1024 && tiles >= 448;
  const bool chip_full = tiles >= 448;
  return K >= 2048 && cols >= 1024 && (chip_full || (tiles >= 224 && tiles <= 256)) && each >= (chip_full || K >= 4096 ? 3 : 8);
}
inline bool any_big_rows(const bigmac_dims& D) {   // a tile map of 256-row tiles is needed
  const Widths W = widths(D);
  return big_rows(D, W.hid, W.win, EPI_GELU) || big_rows(D, W.hid, W.win, EPI_DGELU) || big_rows(D, W.win, W.hid, EPI_STORE) ||
         big_rows(D, W.win, W.hid, EPI_STORE, true);
}

// Both expert products in one kernel (expert_pair.hip): calls that keep no activations, without biases, where no tile
// size is asked for.  A tile walks all hidden columns by itself, where the separate products spread them over the chip.  For
// expert matrices of at most 72 K elements the launch saved outweighs that at any size (whole layer in us, separate products ->
// here, by tiles of 128 rows that the batch fills and experts: width 128, 512 columns: 22 of 16 48 -> 42, 46 of 64 60 -> 56, 12 of 256 86 -> 83;
// width 192, 384 columns: 29 of 48 60 -> 57; width 256, 256 columns: 2 of 128 62 -> 56, 80 of 32 64 -> 60).  Larger ones want tiles
// for a good part of the CUs, counted from the batch: experts with few rows each add nearly empty ones, which cost a whole walk
// under even routing and are not there under skewed routing (width 256: 2 of 256, 2048 columns 135 -> 150, 2 of 256 with Zipf 0.6, 4096
// columns 136 -> 205, 45 of 128 with Zipf 0.6, 4096 columns 215 -> 262, 80 of 8, 1024 columns 87 -> 95 (512 columns: 47 of 4 67 -> 71, 68 of 8 68 -> 69, 112 of 48 69 -> 60), 106 of 16, 4096 columns 161 -> 192, 110 of
// 48 with Zipf 1.2 142 -> 144, 144 of 96, 2048 columns 169 -> 137, 177 of 64 124 -> 110, 512 of 64 224 -> 193; width 192: 31 of 32, 768 columns
// 60 -> 63, 71 of 48 77 -> 73, 86 of 64 79 -> 70, 71 of 48 with Zipf 1.2, 3072 columns 113 -> 134; width 128, 1024 columns: 22 of 8 55 -> 59, 56 of 48 67 -> 64, 84 of 96 94 -> 91).
// Training calls stay with the separate products: stored from this kernel's registers, in pieces of 32 bytes per row, the
// two [rows, hidden] tensors took more than the products saved (width 256, 65536 rows: the step 634 -> 685 us).
inline bool pair_experts(const bigmac_dims& D, const void* b1, const void* b2, const void* act) {
  bool large;
  const Widths W = widths(D);
  if (act || b1 || b2 || tiles_forced(D, &large) || (W.win != 128 && W.win != 192 && W.win != 256) || (size_t)W.win * W.hid * 2 >= (1ull << 31)) return false;
  return (size_t)W.win * W.hid <= 72 * 1024 || (long)D.T * D.k / 128 >= (W.hid > (W.win == 256 ? 512 : 1024) ? 120 : 64);
}

// ... by the expert products of a forward pass (the backward pass has one more with an activation)
inline bool big_forward_rows(const bigmac_dims& D, const void* b1, const void* b2, const void* act) {
  const Widths W = widths(D);
  return !pair_experts(D, b1, b2, act) && (big_rows(D, W.hid, W.win, EPI_GELU) || big_rows(D, W.win, W.hid, EPI_STORE));
}
// big: whether a row product of this call runs on 256 x 256 tiles
TileMapJobs tile_map_jobs(const bigmac_dims& D, bool big, int* tile_map, int* tile_map_tall, unsigned* claims) {
  TileMapJobs maps = {};
  maps.tile_rows[0] = gemm_ragged_tile_rows(D.dtype, 0); maps.map[0] = tile_map;
  if (big) { maps.tile_rows[1] = gemm_ragged_tile_rows(D.dtype, 1); maps.map[1] = tile_map_tall; }
  maps.clear = claims; maps.clear_ints = CLAIM_INTS;
  return maps;
}

SavedPlan plan_saved(const bigmac_dims& D) {
  const Widths W = widths(D);
  const size_t Tk = (size_t)D.T * D.k, es = esize(D.dtype);
  Carver c;
  SavedPlan p;
  p.topk_idx = c.take(Tk * 4);
  p.topk_w = c.take(Tk * 4);
  p.offsets = c.take((size_t)(D.N + 1) * 4);
  p.slot_of = c.take(Tk * 4);
  p.src_of = c.take(Tk * 4);
  p.tile_map = c.take(tile_map_ints((int)Tk, D.N, gemm_ragged_tile_rows(D.dtype, 0)) * 4);
  p.tile_map_tall = c.take(any_big_rows(D) ? tile_map_ints((int)Tk, D.N, gemm_ragged_tile_rows(D.dtype, 1)) * 4 : 0);
  p.x_perm = c.take(Tk * W.win * es);
  p.act = c.take(Tk * wide_ld(D) * es);
  p.hact = c.take(Tk * wide_ld(D) * es);
  p.o_perm = c.take(Tk * W.win * esize(wire_dtype(D)));
  p.y_low = c.take(D.order == BIGMAC_ORDER_DCCA ? low_bytes(D) : 0);
  // load-balance loss: the backward pass needs the logits and the experts' pair shares; aux holds
  // the loss (one float) followed, 256 bytes on, by share[N]
  p.logits = c.take(D.aux_alpha > 0.0f ? (size_t)D.T * D.N * 4 : 0);
  p.aux = c.take(D.aux_alpha > 0.0f ? 256 + (size_t)D.N * 4 : 0);
  // router on x': the backward pass needs x' itself (the router's input) for d_w_gate
  p.x_low = c.take(route_low(D) ? (size_t)D.T * D.r * es : 0);
  p.total = c.off;
  return p;
}

// Split of K for a dense forward product [M,K] x [K,N] with few output tiles and a long K (the
// shared projections at decode sizes: a handful of tiles would otherwise walk K alone on a
// handful of CUs).  fp32 partials, reduced in slice order.  1 = no split.
int forward_ksplit(const bigmac_dims& D, int M, int N, int K) {
  if (!bf(D)) return 1;
  const int tiles = ((M + 127) / 128) * ((N + 127) / 128);
  if (tiles >= 128 && K <= 2048) return 1;
  int ks = K / 256;
  if (ks > 512 / tiles) ks = 512 / tiles;
  if (ks > 32) ks = 32;
  return ks < 1 ? 1 : ks;
}
size_t forward_partials_bytes(const bigmac_dims& D) {
  if (D.order != BIGMAC_ORDER_DCCA) return 0;
  const int ka = forward_ksplit(D, D.T, D.r, D.d), kb = forward_ksplit(D, D.T, D.d, low_ld(D));
  const size_t a = ka > 1 ? (size_t)ka * D.T * D.r * 4 : 0, b = kb > 1 ? (size_t)kb * D.T * D.d * 4 : 0;
  return a > b ? a : b;
}

FwdPlan plan_fwd(const bigmac_dims& D) {
  Carver c;
  FwdPlan p;
  p.logits = c.take((size_t)D.T * D.N * 4);
  p.perm = c.take(permutation_ws_bytes(D.T, D.k, D.N, topk_counts(D.T, D.k, D.N)));
  p.x_low = c.take(D.order == BIGMAC_ORDER_DCCA ? (size_t)D.T * D.r * esize(D.dtype) : 0);
  p.partials = c.take(forward_partials_bytes(D));
  p.aux = c.take(D.aux_alpha > 0.0f ? aux_loss_ws_bytes(D) : 0);
  p.claims = c.take(CLAIM_BYTES);
  p.total = c.off;
  return p;
}

// The weight gradients over the token index take the tall tile when there are enough tall
// tiles and enough tokens to be worth it (measured: zipf_stress, T = 32768, d = 4096: 0.34 ->
// 0.25 ms and 0.38 -> 0.28 ms; at T = 8192 with the same widths level or slower).
inline bool tall_token_wgrad(const bigmac_dims& D, int M, int N) {
  return bf(D) && M % 256 == 0 && (long)(M / 256) * ((N + 127) / 128) >= 128 && D.T >= 16384;
}
// Slices of K for a weight gradient over the token index (few output tiles, K = T).  More slices
// fill more of the chip but write and read back more fp32 partials; the count is the power of
// two (slices of at least 256 rows) with the lowest estimate of product + reduction time:
// rounds of 768 resident workgroups x k tiles per slice x 0.6 us (measured per k tile of 32)
// + partial bytes, written and read once, at 5 TB/s.
// (On the tall tile: 512 resident workgroups, 0.85 us per k tile.)
enum TileShape { TILE_SQUARE, TILE_TALL, TILE_DEEP };
int choose_ksplit(int M, int N, int K, TileShape shape = TILE_SQUARE) {
  const int bm = shape == TILE_TALL ? 256 : 128, bn = shape == TILE_DEEP ? 64 : 128, bk = shape == TILE_DEEP ? 64 : 32;
  const long tiles = (long)((M + bm - 1) / bm) * ((N + bn - 1) / bn);
  const long resident = shape == TILE_SQUARE ? 768 : 512;
  const double k_tile_us = shape == TILE_TALL ? 0.85 : (shape == TILE_DEEP ? BIGMAC_DEEP_K_TILE_US : 0.6);
  const double partial_us = (double)M * N * 4 * 2 / 5e6;
  int best = 1;
  double best_us = 1e30;
  for (int ks = 1; ks <= 64 && K / ks >= 256; ks *= 2) {
    const long rounds = (tiles * ks + resident - 1) / resident;
    const double us = rounds * ((K / ks + bk - 1) / bk) * k_tile_us + (ks > 1 ? ks * partial_us : 0.0);
    if (us <= best_us * 1.05) { best_us = us < best_us ? us : best_us; best = ks; }   // near ties go to more workgroups
  }
  return best;
}
// Tile shape and slice count of a weight gradient over the token index ([M, T] x [T, N]); the
// plan of the partials and the launch both take them from here.
// Few output tiles (K = T is long by nature): the 128 x 64 tile with 64-deep k tiles.
inline TileShape token_wgrad_shape(const bigmac_dims& D, int M, int N) {
  if (tall_token_wgrad(D, M, N)) return TILE_TALL;
  if (bf(D) && (long)((M + 127) / 128) * ((N + 127) / 128) <= BIGMAC_DEEP_WGRAD_MAX_TILES) return TILE_DEEP;
  return TILE_SQUARE;
}
inline int token_wgrad_ksplit(const bigmac_dims& D, int M, int N) { return choose_ksplit(M, N, D.T, token_wgrad_shape(D, M, N)); }

BwdPlan plan_bwd(const bigmac_dims& D) {
  const Widths W = widths(D);
  const size_t Tk = (size_t)D.T * D.k, es = esize(D.dtype);
  const bool dcca = D.order == BIGMAC_ORDER_DCCA;
  Carver c;
  BwdPlan p;
  p.dy_low = c.take(dcca ? (size_t)D.T * W.win * 4 : 0);
  p.dgate = c.take(Tk * 4);
  p.do_perm = c.take(Tk * W.win * es);
  p.dx_perm = wire_f32(D) ? c.take(Tk * W.win * 4) : p.do_perm;   // same width: do_perm is dead once the second matrix's gradients are done
  p.dact = c.take(Tk * wide_ld(D) * es);
  p.dx_low = c.take(dcca ? low_bytes(D) : 0);
  p.dL = c.take((size_t)D.T * D.N * es);
  p.route = c.take(route_backward_ws_bytes(router_dims(D)));
  p.dx_f32 = c.take((bf(D) && (D.flags & BIGMAC_FLAG_OUT_BF16)) ? (size_t)D.T * D.d * 4 : 0);
  // split-K partials of the three weight gradients over the token index: one region each, so
  // that one launch at the end can reduce all three
  const int dg = router_dims(D).d;   // rows of w_gate
  p.part_gate = c.take((size_t)token_wgrad_ksplit(D, dg, D.N) * dg * D.N * 4);
  p.part_up = c.take(dcca ? (size_t)token_wgrad_ksplit(D, D.r, D.d) * D.r * D.d * 4 : 0);
  p.part_down = c.take(dcca ? (size_t)token_wgrad_ksplit(D, D.d, D.r) * D.d * D.r * 4 : 0);
  // expert biases: partial column sums (sized for the wider of the two bias vectors; taken always,
  // the plan does not see the parameters); router on x': its share of dx' in fp32
  p.bias_sums = c.take(ragged_colsum_ws_bytes(D.N, W.hid > W.win ? W.hid : W.win));
  p.gate_low = c.take(route_low(D) ? (size_t)D.T * D.r * 4 : 0);
  p.claims = c.take(CLAIM_BYTES);
  p.total = c.off;
  return p;
}

size_t ffn_ws_bytes(const bigmac_dims& D) {
  const Widths W = widths(D);
  const size_t Tk = (size_t)D.T * D.k;
  return align_up(Tk * W.hid * esize(D.dtype)) + 2 * align_up(tile_map_ints((int)Tk, D.N, gemm_ragged_tile_rows(D.dtype, 0)) * 4) +
         align_up(CLAIM_BYTES);
}

__global__ void f32_to_bf16_kernel(const float* __restrict__ in, bf16_t* __restrict__ out, size_t n) {
  size_t i = (size_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (i < n) out[i] = f2bf(in[i]);
}
inline dim3 grid1d(size_t n) { return dim3((unsigned)((n + 255) / 256)); }

GemmDesc base_desc(const bigmac_dims& D) {
  GemmDesc g = {};
  g.dtype = D.dtype;
  g.ksplit = 1;
  g.mode = GEMM_DENSE;
  return g;
}

// The two expert products on permuted rows (ragged per-expert row ranges).
int run_experts_forward(const bigmac_dims& D, const void* x_perm, const int* offsets, const int* tile_map, const int* tile_map_tall,
                        const void* w1, const void* w2, const void* b1, const void* b2, void* act, void* hact, int ld_wide, void* o_perm, int o_f32,
                        hipStream_t s, const int* gather = nullptr) {
  const Widths W = widths(D);
  const int Tk = D.T * D.k;
  if (pair_experts(D, b1, b2, act)) {
    ExpertPairDesc e = {};
    e.x = x_perm; e.gather = gather; e.x_rows = D.T; e.gather_div = D.k;
    e.w1 = w1; e.w2 = w2; e.out = o_perm; e.out_f32 = o_f32;
    e.offsets = offsets; e.tile_map = tile_map; e.groups = D.N; e.max_rows = Tk; e.width = W.win; e.hid = W.hid;
    BIGMAC_STAGE(BIGMAC_STAGE_EXPERT_UP);         // both products; the stage of the second records nothing
    return launch_expert_pair(e, s);
  }
  GemmDesc g = base_desc(D);
  g.mode = GEMM_RAGGED_M;
  g.a_kcontig = 1; g.b_kcontig = 0;
  g.groups = D.N; g.max_rows = Tk; g.offsets = offsets;
  // hact = gelu(x_perm W1[e])
  g.epilogue = EPI_GELU;
  g.big_tile = big_rows(D, W.hid, W.win, EPI_GELU);
  g.stream_tile = stream_rows(D, W.hid, W.win, EPI_GELU);
  g.tile_map = g.big_tile ? tile_map_tall : tile_map;
  g.wide_k = !g.big_tile && !g.stream_tile && !gather && wide_k_ok(D, W.win, 1);
  g.A = x_perm; g.lda = W.win; g.K = W.win;
  g.gather = gather; g.gather_rows = D.T; g.gather_div = D.k;   // with an index, x_perm is the [T, win] rows before the dispatch
  g.B = w1; g.ldb = W.hid; g.gstride_b = (long)W.win * W.hid; g.N = W.hid;
  g.C = hact; g.ldc = ld_wide; g.aux_out = act;
  g.bias = b1; g.gstride_bias = W.hid;
  if (!g.big_tile) touch_weights(D, g, w1, 1);
  // measured: -3 % at K = 512 (gpt_xl); at K = 256 (gpt_medium) +2 % while the weights came from
  // memory, -4.6 % with the warm-up
  g.kloop_priority = W.win >= 512 || g.touch_bytes != 0;
  int rc;
  {
    BIGMAC_STAGE(BIGMAC_STAGE_EXPERT_UP);
    rc = launch_gemm(g, s);
  }
  if (rc) return rc;
  // o_perm = hact W2[e]
  g.gather = nullptr; g.gather_rows = 0;
  g.epilogue = EPI_STORE; g.out_f32 = o_f32; g.aux_out = nullptr;
  g.A = hact; g.lda = ld_wide; g.K = W.hid;
  g.B = w2; g.ldb = W.win; g.gstride_b = (long)W.hid * W.win; g.N = W.win;
  g.C = o_perm; g.ldc = W.win;
  g.bias = b2; g.gstride_bias = W.win;
  g.big_tile = big_rows(D, W.win, W.hid, EPI_STORE);
  g.stream_tile = stream_rows(D, W.win, W.hid, EPI_STORE);
  g.tile_map = g.big_tile ? tile_map_tall : tile_map;
  g.wide_k = !g.big_tile && !g.stream_tile && wide_k_ok(D, W.hid, 2);
  g.kloop_priority = 1;
  g.touch = nullptr; g.touch_bytes = 0;
  if (!g.big_tile) touch_weights(D, g, w2, 2);
  BIGMAC_STAGE(BIGMAC_STAGE_EXPERT_DOWN);
  return launch_gemm(g, s);
}

// dense fp32 C (+)= A^T-style product over the token index, split over K into fp32 partials; the
// reduction (fixed slice order) is left to the caller as a job for launch_reduce_partials_multi
int run_token_wgrad(const bigmac_dims& D, const void* A, long lda, int M, const void* B, long ldb, int N,
                    float* out, float* partials, ReduceJob* job, hipStream_t s) {
  GemmDesc g = base_desc(D);
  g.a_kcontig = 0; g.b_kcontig = 0;
  g.epilogue = EPI_ACCUM; g.beta = 0;
  g.A = A; g.lda = lda; g.M = M; g.B = B; g.ldb = ldb; g.N = N; g.K = D.T;
  const TileShape shape = token_wgrad_shape(D, M, N);
  g.tall_tile = shape == TILE_TALL;
  g.deep_tile = shape == TILE_DEEP;
  g.ksplit = token_wgrad_ksplit(D, M, N);
  g.C = partials; g.ldc = N; g.gstride_c = (long)M * N;
  job->part = partials; job->out = out; job->n = (size_t)M * N; job->nslices = g.ksplit;
  return launch_gemm(g, s);
}

}  // namespace
}  // namespace bigmac

using namespace bigmac;

extern "C" {

size_t bigmac_workspace_bytes(const bigmac_dims* D, int kind) {
  if (check_dims(D) != BIGMAC_OK) return 0;
  switch (kind) {
    case BIGMAC_WS_ROUTE: return align_up((size_t)D->T * D->N * 4);
    case BIGMAC_WS_DISPATCH: return permutation_ws_bytes(D->T, D->k, D->N, false);
    case BIGMAC_WS_GROUPED_FFN: return ffn_ws_bytes(*D);
    case BIGMAC_WS_LAYER_FORWARD: return plan_fwd(*D).total + plan_saved(*D).total;
    case BIGMAC_WS_LAYER_TRAIN: {
      const size_t f = plan_fwd(*D).total, b = plan_bwd(*D).total;
      return f > b ? f : b;
    }
    case BIGMAC_WS_SAVED: return plan_saved(*D).total;
    case BIGMAC_WS_AUX_LOSS: return aux_loss_ws_bytes(*D);
    default: return 0;
  }
}

const char* bigmac_status_string(int status) {
  switch (status) {
    case BIGMAC_OK: return "ok";
    case BIGMAC_ERR_INVALID_ARG: return "invalid argument (null pointer, bad dimension or enum)";
    case BIGMAC_ERR_WORKSPACE: return "workspace too small";
    case BIGMAC_ERR_UNSUPPORTED: return "unsupported combination";
    case BIGMAC_ERR_HIP: return "HIP launch failed";
    case BIGMAC_ERR_TOO_LARGE: return "problem exceeds the static scratch of the allocation-free entry point";
    default: return "unknown status";
  }
}

double bigmac_forward_matrix_flops(const bigmac_dims* D) {
  if (check_dims(D) != BIGMAC_OK) return 0.0;
  const Widths W = widths(*D);
  double f = 4.0 * (double)D->T * D->k * W.win * W.hid;
  if (D->order == BIGMAC_ORDER_DCCA) f += 4.0 * (double)D->T * D->d * D->r;
  return f;
}

double bigmac_permute_bytes(const bigmac_dims* D) {
  if (check_dims(D) != BIGMAC_OK) return 0.0;
  return 4.0 * (double)D->T * D->k * widths(*D).win * esize(D->dtype);
}

int bigmac_gather_probe(const void* table, const int32_t* order, int64_t rows, int64_t row_bytes, int streaming, uint32_t* sink, void* stream) {
  if (!table || !order || !sink || rows <= 0 || rows % 8 || row_bytes <= 0 || row_bytes % 32 || rows > (1ll << 31) - 8 || row_bytes > (1ll << 24) ||
      rows * row_bytes >= (1ll << 40))
    return BIGMAC_ERR_INVALID_ARG;
  return launch_gather_probe(table, order, (long)rows, (long)row_bytes, streaming, sink, (hipStream_t)stream);
}

int bigmac_mfma_probe(int blocks, int iters, float* sink, double* flops, void* stream) {
  if (blocks <= 0 || blocks > 65536 || iters <= 0 || iters > (1 << 20) || !sink || !flops) return BIGMAC_ERR_INVALID_ARG;
  const double f = launch_mfma_probe(blocks, iters, sink, (hipStream_t)stream);
  if (f < 0) return BIGMAC_ERR_HIP;
  *flops = f;
  return BIGMAC_OK;
}

int bigmac_set_stage_events(void* const* events) {
  g_stage_events = events;
  return BIGMAC_OK;
}

namespace {
// training forward: the descending projection writes x' straight into the permuted copy (see
// bigmac_layer_forward)
bool descend_scatters(const bigmac_dims& D) {
  if (D.order != BIGMAC_ORDER_DCCA || !bf(D) || route_low(D) || (D.flags & BIGMAC_FLAG_NO_FUSED_DISPATCH)) return false;
  if (forward_ksplit(D, D.T, D.r, D.d) != 1) return false;
  return (size_t)D.T * D.k * (size_t)D.r * 2 < (1ull << 31) && (size_t)D.T * D.k * 4 < (1ull << 31);
}
GemmDesc descend_product(const bigmac_dims& D) {   // x' = x W_down, without its pointers
  GemmDesc g = base_desc(D);
  g.ksplit = forward_ksplit(D, D.T, D.r, D.d);
  g.a_kcontig = 1; g.b_kcontig = 0; g.epilogue = EPI_STORE; g.out_f32 = bf(D) && g.ksplit == 1 ? 0 : 1;
  g.lda = D.d; g.M = D.T; g.K = D.d;
  g.ldb = D.r; g.N = D.r; g.ldc = D.r;
  g.big_tile = g.ksplit == 1 && big_dense(D, D.T, D.r, D.d);
  g.deep_tile = g.ksplit == 1 && !g.big_tile && deep_dense(D, D.T, D.r, D.d);
  return g;
}
// Where a layer forward picks the experts (the values of bigmac_topk_folding).  With the logits: all experts in one tile of them, and no pairs
// to count for the sort.  Beside the descending projection: neither needs the other (the loss reads the picks in front of it).  A workgroup there is four
// wavefronts, which take eight tokens in 1.3 us; where the sort wants large parts counted that chain outlasts the projection, and a launch
// of its own has up to 16 wavefronts for a part.  Forward-only calls (h 64, k 1 to 8), own launch -> beside: parts of up to 32 tokens 0 to 6.8 us less; 64
// tokens (T 9000 / 13000) d 512 4 to 7 us more, d 1024 2.7 less to 1.8 more / 5 to 12 more, d 2048 6 to 11 / 4 to 8 less, d 4096 7 to 13 / 7 to
// 11 less; 128 tokens (T 20000 / 32000) d 512 9 to 17 / 16 to 29 more, d 1024 4 to 9 / 4 to 13 more, d 2048 and 4096 21 more to 2 less.
enum TopkPlace { TOPK_OWN_LAUNCH = 0, TOPK_WITH_LOGITS = 1, TOPK_BESIDE_DESCEND = 2 };
TopkPlace topk_place(const bigmac_dims& D, bool training) {
  const bool counted = topk_counts(D.T, D.k, D.N);
  if (!counted && router_picks(router_dims(D))) return TOPK_WITH_LOGITS;
  if (D.order != BIGMAC_ORDER_DCCA || route_low(D) || D.aux_alpha > 0.0f || (training && descend_scatters(D))) return TOPK_OWN_LAUNCH;
  const GemmDesc g = descend_product(D);
  const int part = counted ? topk_grid(D.T, D.k, D.N, true).tokens : 0;
  return gemm_takes_topk(g, D.N) && (part <= 32 || (part <= 64 && g.K / g.ksplit >= 2048)) ? TOPK_BESIDE_DESCEND : TOPK_OWN_LAUNCH;
}
// forward-only call: the expert-up product reads its rows through src_of (see bigmac_layer_forward);
// the rows behind the index must lie within one 32-bit byte offset
bool expert_up_gathers(const bigmac_dims& D) {
  return bf(D) && !(D.flags & BIGMAC_FLAG_NO_FUSED_DISPATCH) && (size_t)D.T * (size_t)widths(D).win * 2 < (1ull << 31);
}
}  // namespace

int bigmac_dispatch_folding(const bigmac_dims* D, int training) {
  const int rc = check_dims(D);
  if (rc) return rc;
  if (training) return descend_scatters(*D) ? 2 : 0;
  return expert_up_gathers(*D) ? 1 : 0;
}

int bigmac_expert_pairing(const bigmac_dims* D, int training) {
  const int rc = check_dims(D);
  if (rc) return rc;
  return !training && pair_experts(*D, nullptr, nullptr, nullptr) ? 1 : 0;
}

int bigmac_topk_folding(const bigmac_dims* D, int training) {
  const int rc = check_dims(D);
  return rc ? rc : topk_place(*D, training != 0);
}

const char* bigmac_stage_name(int stage) {
  static const char* names[BIGMAC_STAGE_COUNT] = {
      "router_logits", "topk_gate", "descend", "permutation", "dispatch", "expert_up", "expert_down", "combine", "ascend",
      "bwd_ascend_dgrad", "bwd_ascend_wgrad", "bwd_combine", "bwd_down_dgrad", "bwd_down_wgrad", "bwd_up_wgrad",
      "bwd_up_dgrad", "bwd_dispatch", "bwd_gate", "bwd_router_wgrad", "bwd_descend_wgrad", "bwd_descend_dgrad",
      "bwd_output_cast"};
  return stage >= 0 && stage < BIGMAC_STAGE_COUNT ? names[stage] : "?";
}

int bigmac_saved_layout(const bigmac_dims* D, size_t* off_topk_idx, size_t* off_topk_w, size_t* off_expert_offsets,
                        size_t* off_slot_of) {
  int rc = check_dims(D);
  if (rc) return rc;
  const SavedPlan p = plan_saved(*D);
  if (off_topk_idx) *off_topk_idx = p.topk_idx;
  if (off_topk_w) *off_topk_w = p.topk_w;
  if (off_expert_offsets) *off_expert_offsets = p.offsets;
  if (off_slot_of) *off_slot_of = p.slot_of;
  return BIGMAC_OK;
}

int bigmac_saved_aux_layout(const bigmac_dims* D, size_t* off_aux_loss, size_t* off_aux_share) {
  int rc = check_dims(D);
  if (rc) return rc;
  if (!(D->aux_alpha > 0.0f)) return BIGMAC_ERR_INVALID_ARG;
  const SavedPlan p = plan_saved(*D);
  if (off_aux_loss) *off_aux_loss = p.aux;
  if (off_aux_share) *off_aux_share = p.aux + 256;
  return BIGMAC_OK;
}

int bigmac_aux_loss(const bigmac_dims* D, const float* logits, const int32_t* topk_idx, float* loss, float* share,
                    float* dlogits, void* ws, size_t ws_bytes, void* stream) {
  int rc = check_dims(D);
  if (rc) return rc;
  if (!logits || !topk_idx || !loss || !share || !ws) return BIGMAC_ERR_INVALID_ARG;
  if (ws_bytes < aux_loss_ws_bytes(*D)) return BIGMAC_ERR_WORKSPACE;
  return launch_aux_loss(*D, logits, topk_idx, share, loss, dlogits, ws, (hipStream_t)stream);
}

int bigmac_route(const bigmac_dims* D, const void* x, const float* w_gate, const float* gate_bias, int32_t* topk_idx,
                 float* topk_w, float* logits_out, void* ws, size_t ws_bytes, void* stream) {
  int rc = check_dims(D);
  if (rc) return rc;
  if (!x || !w_gate || !topk_idx || !topk_w) return BIGMAC_ERR_INVALID_ARG;
  float* logits = logits_out;
  if (!logits) {
    if (!ws) return BIGMAC_ERR_INVALID_ARG;
    if (ws_bytes < bigmac_workspace_bytes(D, BIGMAC_WS_ROUTE)) return BIGMAC_ERR_WORKSPACE;
    logits = (float*)ws;
  }
  const bool picks = router_picks(*D);
  rc = launch_router_logits(*D, x, w_gate, gate_bias, logits, (hipStream_t)stream, picks ? topk_idx : nullptr, picks ? topk_w : nullptr);
  if (rc || picks) return rc;
  return launch_topk_gate(*D, logits, topk_idx, topk_w, (hipStream_t)stream);
}

int bigmac_dispatch(const bigmac_dims* D, const void* x_low, const int32_t* topk_idx, void* x_perm, int32_t* expert_offsets,
                    int32_t* slot_of, int32_t* src_of, void* ws, size_t ws_bytes, void* stream) {
  int rc = check_dims(D);
  if (rc) return rc;
  if (!topk_idx || !expert_offsets || !slot_of || !src_of || !ws) return BIGMAC_ERR_INVALID_ARG;
  if ((x_low == nullptr) != (x_perm == nullptr)) return BIGMAC_ERR_INVALID_ARG;
  if (ws_bytes < bigmac_workspace_bytes(D, BIGMAC_WS_DISPATCH)) return BIGMAC_ERR_WORKSPACE;
  hipStream_t s = (hipStream_t)stream;
  rc = launch_build_permutation(D->T, D->k, D->N, D->capacity, topk_idx, expert_offsets, slot_of, src_of, ws, s);
  if (rc || !x_low) return rc;
  return launch_dispatch_rows(D->dtype, D->T, D->k, widths(*D).win, x_low, slot_of, x_perm, s);
}

int bigmac_grouped_ffn(const bigmac_dims* D, const void* x_perm, const int32_t* expert_offsets, const void* w1, const void* w2,
                       const void* b1, const void* b2, void* act_saved, void* o_perm, void* ws, size_t ws_bytes, void* stream) {
  int rc = check_dims(D);
  if (rc) return rc;
  if (!x_perm || !expert_offsets || !w1 || !w2 || !o_perm || !ws) return BIGMAC_ERR_INVALID_ARG;
  if (ws_bytes < ffn_ws_bytes(*D)) return BIGMAC_ERR_WORKSPACE;
  hipStream_t s = (hipStream_t)stream;
  const Widths W = widths(*D);
  const size_t Tk = (size_t)D->T * D->k;
  void* hact = ws;
  int* tile_map = (int*)((char*)ws + align_up(Tk * W.hid * esize(D->dtype)));
  int* tile_map_tall = (int*)((char*)tile_map + align_up(tile_map_ints((int)Tk, D->N, gemm_ragged_tile_rows(D->dtype, 0)) * 4));
  unsigned* claim_counters = (unsigned*)((char*)tile_map_tall + align_up(tile_map_ints((int)Tk, D->N, gemm_ragged_tile_rows(D->dtype, 0)) * 4));
  ClaimScope claims(claim_counters);
  rc = launch_build_tile_map(expert_offsets, D->N, tile_map_jobs(*D, big_forward_rows(*D, b1, b2, act_saved), tile_map, tile_map_tall, claim_counters), s);
  if (rc) return rc;
  return run_experts_forward(*D, x_perm, expert_offsets, tile_map, tile_map_tall, w1, w2, b1, b2, act_saved, hact, W.hid, o_perm, 0, s);
}

int bigmac_combine(const bigmac_dims* D, const void* o_perm, const int32_t* slot_of, const float* topk_w, float* y_low, void* stream) {
  int rc = check_dims(D);
  if (rc) return rc;
  if (!o_perm || !slot_of || !y_low) return BIGMAC_ERR_INVALID_ARG;
  return launch_combine_rows(D->dtype, D->T, D->k, widths(*D).win, o_perm, slot_of, topk_w, y_low, COMBINE_F32, (hipStream_t)stream);
}

int bigmac_layer_forward(const bigmac_dims* D, const bigmac_params* P, const void* x, void* y, void* saved, void* ws,
                         size_t ws_bytes, void* stream) {
  int rc = check_dims(D);
  if (rc) return rc;
  const bool dcca = D->order == BIGMAC_ORDER_DCCA;
  if (!P || !x || !y || !ws || !P->w_gate || !P->w1 || !P->w2) return BIGMAC_ERR_INVALID_ARG;
  if (dcca && (!P->w_down || !P->w_up)) return BIGMAC_ERR_INVALID_ARG;
  if (ws_bytes < bigmac_workspace_bytes(D, saved ? BIGMAC_WS_LAYER_TRAIN : BIGMAC_WS_LAYER_FORWARD)) return BIGMAC_ERR_WORKSPACE;
  hipStream_t s = (hipStream_t)stream;
  const Widths W = widths(*D);
  const FwdPlan F = plan_fwd(*D);
  const SavedPlan S = plan_saved(*D);
  char* wsb = (char*)ws;
  char* sv = saved ? (char*)saved : wsb + F.total;  // inference keeps the same pieces in the workspace
  ClaimScope claims(wsb + F.claims);
  int32_t* topk_idx = (int32_t*)(sv + S.topk_idx);
  float* topk_w = (float*)(sv + S.topk_w);
  int32_t* offsets = (int32_t*)(sv + S.offsets);
  int32_t* slot_of = (int32_t*)(sv + S.slot_of);
  int32_t* src_of = (int32_t*)(sv + S.src_of);
  int* tile_map = (int*)(sv + S.tile_map);
  int* tile_map_tall = (int*)(sv + S.tile_map_tall);
  void* x_perm = sv + S.x_perm;
  void* act = saved ? sv + S.act : nullptr;
  void* hact = sv + S.hact;
  void* o_perm = sv + S.o_perm;
  void* y_low = sv + S.y_low;
  const bool out_bf16 = bf(*D) && (D->flags & BIGMAC_FLAG_OUT_BF16);
  const bool aux = D->aux_alpha > 0.0f;                       // the loss lives in the saved block
  float* logits = aux ? (float*)(sv + S.logits) : (float*)(wsb + F.logits);

  // the top-k kernel may count the pairs of the sort's chunks on its way
  int32_t* chunk_counts = topk_counts(D->T, D->k, D->N) ? (int32_t*)(wsb + F.perm) : nullptr;
  const bool low_router = route_low(*D);
  // x' is the workspace's piece, or (router on x': the backward pass reads it again) the saved block's
  void* x_low_buf = (low_router && saved) ? (void*)(sv + S.x_low) : (void*)(wsb + F.x_low);
  const TopkPlace place = topk_place(*D, saved != nullptr);
  auto route = [&](const void* router_in) -> int {
    const bool picks = place == TOPK_WITH_LOGITS;
    int rr;
    {
      BIGMAC_STAGE(BIGMAC_STAGE_ROUTER_LOGITS);
      rr = launch_router_logits(router_dims(*D), router_in, P->w_gate, P->gate_bias, logits, s, picks ? topk_idx : nullptr, picks ? topk_w : nullptr);
    }
    if (rr || (place != TOPK_OWN_LAUNCH && !aux)) return rr;
    BIGMAC_STAGE(BIGMAC_STAGE_TOPK_GATE);
    if (place == TOPK_OWN_LAUNCH) rr = launch_topk_gate(*D, logits, topk_idx, topk_w, s, chunk_counts);
    if (!rr && aux)
      rr = launch_aux_loss(*D, logits, topk_idx, (float*)(sv + S.aux + 256), (float*)(sv + S.aux), nullptr, wsb + F.aux, s, chunk_counts);
    return rr;
  };
  auto permute = [&](const SliceSum* beside = nullptr) -> int {
    BIGMAC_STAGE(BIGMAC_STAGE_PERMUTATION);
    const bool big = saved ? any_big_rows(*D) : big_forward_rows(*D, P->b1, P->b2, nullptr);
    const TileMapJobs maps = tile_map_jobs(*D, big, tile_map, tile_map_tall, (unsigned*)(wsb + F.claims));
    return launch_build_permutation(D->T, D->k, D->N, D->capacity, topk_idx, offsets, slot_of, src_of, wsb + F.perm, s, &maps, chunk_counts != nullptr, beside);
  };
  // A training forward on bf16 storage whose router reads x folds the dispatch into the descending
  // projection: the permutation is built first, and the product's epilogue writes every token's
  // narrow row straight into the places of its pairs in the permuted copy (x' itself is not
  // stored: nothing else reads it).  Not where the product is summed from K slices, nor where the
  // copy is too large for one 32-bit byte offset.
  const bool scatter_descend = saved && descend_scatters(*D);
  GemmDesc down = {};
  if (dcca) {
    down = descend_product(*D);
    down.A = x; down.B = P->w_down; down.C = x_low_buf;
    if (scatter_descend) {
      down.scatter = slot_of; down.scatter_k = D->k; down.scatter_rows = D->T * D->k;
      down.C = x_perm;
    }
    if (place == TOPK_BESIDE_DESCEND) down.topk = topk_job_beside(*D, logits, topk_idx, topk_w, chunk_counts);
  }
  if (!low_router) {   // Section 3.1's default: the router reads the full-width token
    rc = route(x);
    if (rc) return rc;
  }
  if (scatter_descend) {
    rc = permute();
    if (rc) return rc;
  }
  // The sum of the projection's slices and the sort do not need each other either: in one launch, unless the router reads the sum.
  // Every thread of a workgroup sums, whatever the sort's workgroups are (256 threads to 1024 past 64 experts; only their first
  // wavefronts summing was up to 5 us slower than two launches from 2000 tokens on).  A forward-only call with small experts (h 64, k 4), two
  // launches -> one: d 4096, r 1024: 64 experts T 16 66.0 -> 62.6 us, T 500 85.8 -> 82.1, T 2048 128.4 -> 124.3, T 4096 196.5 -> 190.4; 128 experts
  // 72.7 -> 68.9, 93.6 -> 87.2, 144.3 -> 136.5, 220.8 -> 213.1; 256 experts 97.1 -> 93.7, 126.4 -> 117.8, 194.5 -> 187.0, 298.5 -> 290.7.
  const bool sum_beside_sort = !low_router;
  SliceSum descend_sum = {};
  const void* x_low = x;
  if (dcca) {
    {
      BIGMAC_STAGE(BIGMAC_STAGE_DESCEND);
      if (down.ksplit > 1) {   // fp32 partials, then one rounding to bf16
        down.C = wsb + F.partials; down.gstride_c = (long)D->T * D->r;
        rc = launch_gemm(down, s);
        if (rc) return rc;
        if (sum_beside_sort) descend_sum = {(const float*)(wsb + F.partials), x_low_buf, (size_t)D->T * D->r, down.ksplit};
        else rc = launch_reduce_partials_bf16({(const float*)(wsb + F.partials), x_low_buf, (size_t)D->T * D->r, down.ksplit}, s);
      } else {
        rc = launch_gemm(down, s);
      }
    }
    if (rc) return rc;
    x_low = x_low_buf;
  }
  if (low_router) {    // the alternative Section 3.1 names: the router reads x' (as stored)
    rc = route(x_low);
    if (rc) return rc;
  }
  if (!scatter_descend) {
    rc = permute(descend_sum.part ? &descend_sum : nullptr);
    if (rc) return rc;
  }
  // Forward-only calls on bf16 storage fold the dispatch into the expert-up product: its A rows are
  // read from x' (or x) through src_of and no permuted copy is written.  A training forward
  // keeps the copy: the backward pass contracts over its rows.
  const bool fuse_dispatch = !saved && expert_up_gathers(*D);
  if (!fuse_dispatch && !scatter_descend) {
    BIGMAC_STAGE(BIGMAC_STAGE_DISPATCH);
    rc = launch_dispatch_rows(D->dtype, D->T, D->k, W.win, x_low, slot_of, x_perm, s);
  }
  if (rc) return rc;
  rc = run_experts_forward(*D, fuse_dispatch ? x_low : x_perm, offsets, tile_map, tile_map_tall, P->w1, P->w2, P->b1, P->b2, act, hact, wide_ld(*D), o_perm,
                           wire_f32(*D) ? 1 : 0, s, fuse_dispatch ? src_of : nullptr);
  if (rc) return rc;
  if (!dcca) {  // fine-grained layer: the weighted sum is the output
    BIGMAC_STAGE(BIGMAC_STAGE_COMBINE);
    return launch_combine_rows(wire_dtype(*D), D->T, D->k, W.win, o_perm, slot_of, topk_w, y, COMBINE_F32, s);
  }
  {
    BIGMAC_STAGE(BIGMAC_STAGE_COMBINE);
    rc = launch_combine_rows(wire_dtype(*D), D->T, D->k, W.win, o_perm, slot_of, topk_w, y_low, bf(*D) ? COMBINE_SPLIT_BF16 : COMBINE_F32, s);
  }
  if (rc) return rc;
  {  // y = y' W_up
    GemmDesc g = base_desc(*D);
    g.a_kcontig = 1; g.b_kcontig = 0; g.epilogue = EPI_STORE; g.out_f32 = out_bf16 ? 0 : 1;
    g.A = y_low; g.lda = low_ld(*D); g.M = D->T; g.K = low_ld(*D);
    g.B = P->w_up; g.ldb = D->d; g.N = D->d; g.kwrap_b = bf(*D) ? D->r : 0;
    g.C = y; g.ldc = D->d;
    BIGMAC_STAGE(BIGMAC_STAGE_ASCEND);
    g.ksplit = forward_ksplit(*D, D->T, D->d, low_ld(*D));
    g.big_tile = g.ksplit == 1 && big_dense(*D, D->T, D->d, low_ld(*D));
    // up to one square tile per CU the 128 x 64 tile, twice as many of half the size (whole layer of 8 experts at d 4096, T 500
    // / 700 / 1000: 113 -> 105, 117 -> 115, 130 -> 131 us; d 2048, T 1000 / 2000: 75 -> 72, 83 -> 81; d 1024, T 2000: 59 -> 57)
    g.deep_tile = g.ksplit == 1 && !g.big_tile && deep_dense(*D, D->T, D->d, low_ld(*D));
    g.wide_k = g.ksplit == 1 && !g.big_tile && !g.deep_tile && wide_k_ok(*D, low_ld(*D), 32);
    if (g.ksplit > 1) {
      g.out_f32 = 1; g.C = wsb + F.partials; g.gstride_c = (long)D->T * D->d;
      rc = launch_gemm(g, s);
      if (rc) return rc;
      if (out_bf16) rc = launch_reduce_partials_bf16({(const float*)(wsb + F.partials), y, (size_t)D->T * D->d, g.ksplit}, s);
      else rc = launch_reduce_partials((const float*)(wsb + F.partials), g.ksplit, (size_t)D->T * D->d, (float*)y, 0, s);
    } else {
      rc = launch_gemm(g, s);
    }
  }
  return rc;
}

int bigmac_layer_backward(const bigmac_dims* D, const bigmac_params* P, const void* x, const void* dy, const void* saved,
                          void* dx, float* d_w_down, float* d_w_up, float* d_w_gate, float* d_w1, float* d_w2, float* d_b1,
                          float* d_b2, void* ws, size_t ws_bytes, void* stream) {
  int rc = check_dims(D);
  if (rc) return rc;
  const bool dcca = D->order == BIGMAC_ORDER_DCCA;
  if (!P || !x || !dy || !saved || !dx || !ws || !d_w_gate || !d_w1 || !d_w2 || !P->w_gate || !P->w1 || !P->w2)
    return BIGMAC_ERR_INVALID_ARG;
  if (dcca && (!P->w_down || !P->w_up || !d_w_down || !d_w_up)) return BIGMAC_ERR_INVALID_ARG;
  if ((P->b1 != nullptr) != (d_b1 != nullptr) || (P->b2 != nullptr) != (d_b2 != nullptr)) return BIGMAC_ERR_INVALID_ARG;
  if (bf(*D) && D->N % 8) return BIGMAC_ERR_UNSUPPORTED;  // the dense logit gradient has 16-byte rows
  if (ws_bytes < bigmac_workspace_bytes(D, BIGMAC_WS_LAYER_TRAIN)) return BIGMAC_ERR_WORKSPACE;
  hipStream_t s = (hipStream_t)stream;
  const Widths W = widths(*D);
  const SavedPlan S = plan_saved(*D);
  const BwdPlan B = plan_bwd(*D);
  const char* sv = (const char*)saved;
  char* wsb = (char*)ws;
  ClaimScope claims(wsb + B.claims);
  const int32_t* topk_idx = (const int32_t*)(sv + S.topk_idx);
  const float* topk_w = (const float*)(sv + S.topk_w);
  const int32_t* offsets = (const int32_t*)(sv + S.offsets);
  const int32_t* slot_of = (const int32_t*)(sv + S.slot_of);
  const int* tile_map = (const int*)(sv + S.tile_map);
  const int* tile_map_tall = (const int*)(sv + S.tile_map_tall);
  const void* x_perm = sv + S.x_perm;
  const void* act = sv + S.act;
  const void* hact = sv + S.hact;
  const void* o_perm = sv + S.o_perm;
  const void* y_low = sv + S.y_low;
  float* dy_low = (float*)(wsb + B.dy_low);
  float* dgate = (float*)(wsb + B.dgate);
  void* do_perm = wsb + B.do_perm;
  void* dact = wsb + B.dact;
  void* dx_perm = wsb + B.dx_perm;
  void* dx_low = wsb + B.dx_low;
  void* dL = wsb + B.dL;
  ReduceJob jobs[3];
  int njobs = 0;
  const bool out_bf16 = bf(*D) && (D->flags & BIGMAC_FLAG_OUT_BF16);
  float* dx_f32 = out_bf16 ? (float*)(wsb + B.dx_f32) : (float*)dx;
  const int accumulate = (D->flags & BIGMAC_FLAG_ACCUMULATE) ? 1 : 0;
  const int Tk = D->T * D->k;
  const size_t Td = (size_t)D->T * D->d;

  if (dcca) {
    // dy' = dy W_up^T (kept in fp32)
    GemmDesc g = base_desc(*D);
    g.a_kcontig = 1; g.b_kcontig = 1; g.epilogue = EPI_STORE; g.out_f32 = 1;
    g.A = dy; g.lda = D->d; g.M = D->T; g.K = D->d;
    g.B = P->w_up; g.ldb = D->d; g.N = D->r;
    g.C = dy_low; g.ldc = D->r;
    g.big_tile = big_ascend_dgrad(*D);
    g.deep_tile = !g.big_tile && deep_dense(*D, D->T, D->r, D->d);
    {
      BIGMAC_STAGE(BIGMAC_STAGE_BWD_ASCEND_DGRAD);
      rc = launch_gemm(g, s);
    }
    if (rc) return rc;
    // dW_up (+)= y'^T dy
    BIGMAC_STAGE(BIGMAC_STAGE_BWD_ASCEND_WGRAD);
    rc = run_token_wgrad(*D, y_low, low_ld(*D), D->r, dy, D->d, D->d, d_w_up, (float*)(wsb + B.part_up), &jobs[njobs++], s);
    if (rc) return rc;
  }
  // weighted-sum backward: gate gradients and the scaled scatter of dy' to the expert rows
  // (the fine-grained layer's rows of dy' are dy itself)
  const bool low_router = route_low(*D), aux = D->aux_alpha > 0.0f;
  const bigmac_dims R = router_dims(*D);
  const float* logits = aux ? (const float*)(sv + S.logits) : nullptr;
  const float* share = aux ? (const float*)(sv + S.aux + 256) : nullptr;
  GateBackward gate_job;
  const bool gate_fused = gate_backward_job(R, topk_idx, logits, share, dL, wsb + B.route, &gate_job);
  {
    BIGMAC_STAGE(BIGMAC_STAGE_BWD_COMBINE);
    rc = launch_combine_backward(D->dtype, dcca ? BIGMAC_F32 : D->dtype, wire_dtype(*D), D->T, D->k, W.win, dcca ? (const void*)dy_low : dy, o_perm, slot_of,
                                 topk_w, dgate, do_perm, gate_fused ? &gate_job : nullptr, (unsigned*)(wsb + B.claims), s);
  }
  if (rc) return rc;
  if (d_b2) {  // the second bias adds to every expert output: its gradient is the column sum of do_perm over the expert's rows
    rc = launch_ragged_colsum(D->dtype, do_perm, W.win, W.win, offsets, D->N, d_b2, accumulate, wsb + B.bias_sums, s);
    if (rc) return rc;
  }
  {  // dact = (do_perm W2[e]^T) * act'(act)
    GemmDesc g = base_desc(*D);
    g.mode = GEMM_RAGGED_M; g.groups = D->N; g.max_rows = Tk; g.offsets = offsets; g.tile_map = tile_map;
    g.a_kcontig = 1; g.b_kcontig = 1; g.epilogue = EPI_DGELU;
    g.A = do_perm; g.lda = W.win; g.K = W.win;
    g.B = P->w2; g.ldb = W.win; g.gstride_b = (long)W.hid * W.win; g.N = W.hid;
    g.C = dact; g.ldc = wide_ld(*D); g.aux_in = act;
    g.big_tile = big_rows(*D, W.hid, W.win, EPI_DGELU);
    if (g.big_tile) g.tile_map = tile_map_tall;
    g.wide_k = !g.big_tile && wide_k_ok(*D, W.win, 4);
    g.kloop_priority = 1;              // measured: -3.5 % (gpt_medium), -1.7 % (gpt_xl)
    if (!g.big_tile) touch_weights(*D, g, P->w2, 4);
    {
      BIGMAC_STAGE(BIGMAC_STAGE_BWD_DOWN_DGRAD);
      rc = launch_gemm(g, s);
    }
    if (rc) return rc;
    if (d_b1) {  // the first bias adds to the pre-activation: column sums of dact
      rc = launch_ragged_colsum(D->dtype, dact, wide_ld(*D), W.hid, offsets, D->N, d_b1, accumulate, wsb + B.bias_sums, s);
      if (rc) return rc;
    }
  }
  {  // dW2[e] (+)= hact_e^T do_perm_e
    GemmDesc g = base_desc(*D);
    g.mode = GEMM_RAGGED_K; g.groups = D->N; g.max_rows = Tk; g.offsets = offsets; g.tile_map = tile_map;
    g.a_kcontig = 0; g.b_kcontig = 0; g.epilogue = EPI_ACCUM; g.beta = accumulate;
    g.A = hact; g.lda = wide_ld(*D); g.M = W.hid;
    g.B = do_perm; g.ldb = W.win; g.N = W.win;
    g.C = d_w2; g.ldc = W.win; g.gstride_c = (long)W.hid * W.win;
    g.big_tile = big_wgrad(*D, W.hid, W.win);
    g.tall_tile = !g.big_tile && tall_wgrad(*D, W.hid);
    {
      BIGMAC_STAGE(BIGMAC_STAGE_BWD_DOWN_WGRAD);
      rc = launch_gemm(g, s);
    }
    if (rc) return rc;
    // dW1[e] (+)= x_perm_e^T dact_e
    g.A = x_perm; g.lda = W.win; g.M = W.win;
    g.B = dact; g.ldb = wide_ld(*D); g.N = W.hid;
    g.C = d_w1; g.ldc = W.hid; g.gstride_c = (long)W.win * W.hid;
    g.big_tile = big_wgrad(*D, W.win, W.hid);
    g.tall_tile = !g.big_tile && tall_wgrad(*D, W.win);
    BIGMAC_STAGE(BIGMAC_STAGE_BWD_UP_WGRAD);
    rc = launch_gemm(g, s);
    if (rc) return rc;
  }
  {  // dx_perm = dact W1[e]^T
    GemmDesc g = base_desc(*D);
    g.mode = GEMM_RAGGED_M; g.groups = D->N; g.max_rows = Tk; g.offsets = offsets; g.tile_map = tile_map;
    g.a_kcontig = 1; g.b_kcontig = 1; g.epilogue = EPI_STORE; g.out_f32 = (bf(*D) && !wire_f32(*D)) ? 0 : 1;
    g.A = dact; g.lda = wide_ld(*D); g.K = W.hid;
    g.B = P->w1; g.ldb = W.hid; g.gstride_b = (long)W.win * W.hid; g.N = W.win;
    g.C = dx_perm; g.ldc = W.win;
    g.big_tile = big_rows(*D, W.win, W.hid, EPI_STORE, true);
    if (g.big_tile) g.tile_map = tile_map_tall;
    g.wide_k = !g.big_tile && wide_k_ok(*D, W.hid, 8);
    g.kloop_priority = 1;
    if (!g.big_tile) touch_weights(*D, g, P->w1, 8);
    BIGMAC_STAGE(BIGMAC_STAGE_BWD_UP_DGRAD);
    rc = launch_gemm(g, s);
    if (rc) return rc;
  }
  // Gate backward.  The router's share of the input gradient goes to dx (router on x) or, with the
  // router on x', into an fp32 [T, r] row that the sum of dx' below starts from.
  float* gate_low = low_router ? (float*)(wsb + B.gate_low) : nullptr;
  {
    BIGMAC_STAGE(BIGMAC_STAGE_BWD_GATE);
    rc = launch_route_backward(R, P->w_gate, topk_idx, topk_w, dgate, logits, share, low_router ? gate_low : dx_f32, dL, wsb + B.route, s, gate_fused);
  }
  if (rc) return rc;
  // dispatch backward: dx' = sum_j dx_perm[slot_of[t, j]] (+ the router's share); the fine-grained
  // layer's dx' is dx itself and starts from the router's share that lies there
  {
    BIGMAC_STAGE(BIGMAC_STAGE_BWD_DISPATCH);
    rc = launch_combine_rows(wire_dtype(*D), D->T, D->k, W.win, dx_perm, slot_of, nullptr, dcca ? dx_low : (void*)dx_f32,
                             (dcca && bf(*D)) ? COMBINE_SPLIT_BF16 : COMBINE_F32, s, dcca ? gate_low : dx_f32,
                             /*stream_out=*/low_bytes(*D) >= (32u << 20));   // (smaller results are read back from the caches)
  }
  if (rc) return rc;
  {  // dW_g (+)= x^T dL  (router on x': x'^T dL)
    BIGMAC_STAGE(BIGMAC_STAGE_BWD_ROUTER_WGRAD);
    const void* router_in = low_router ? (const void*)(sv + S.x_low) : x;
    rc = run_token_wgrad(*D, router_in, R.d, R.d, dL, D->N, D->N, d_w_gate, (float*)(wsb + B.part_gate), &jobs[njobs++], s);
  }
  if (rc) return rc;
  if (dcca) {
    {  // dx += dx' W_down^T
      GemmDesc g = base_desc(*D);
      g.a_kcontig = 1; g.b_kcontig = 1; g.epilogue = EPI_ACCUM; g.beta = low_router ? 0 : 1;   // dx holds the router's share, or nothing yet
      g.A = dx_low; g.lda = low_ld(*D); g.M = D->T; g.K = low_ld(*D);
      g.B = P->w_down; g.ldb = D->r; g.N = D->d; g.kwrap_b = bf(*D) ? D->r : 0;
      g.C = dx_f32; g.ldc = D->d;
      g.big_tile = big_dense(*D, D->T, D->d, low_ld(*D), true);
      g.wide_k = !g.big_tile && wide_k_ok(*D, low_ld(*D), 16);
      BIGMAC_STAGE(BIGMAC_STAGE_BWD_DESCEND_DGRAD);
      rc = launch_gemm(g, s);
      if (rc) return rc;
    }
    // dW_down (+)= x^T dx', and the reduction of all three token-index weight gradients
    BIGMAC_STAGE(BIGMAC_STAGE_BWD_DESCEND_WGRAD);
    rc = run_token_wgrad(*D, x, D->d, D->d, dx_low, low_ld(*D), D->r, d_w_down, (float*)(wsb + B.part_down), &jobs[njobs++], s);
    if (rc) return rc;
    rc = launch_reduce_partials_multi(jobs, njobs, (D->flags & BIGMAC_FLAG_ACCUMULATE) ? 1 : 0, s);
    if (rc) return rc;
  } else {
    BIGMAC_STAGE(BIGMAC_STAGE_BWD_OUTPUT_CAST);
    rc = launch_reduce_partials_multi(jobs, njobs, (D->flags & BIGMAC_FLAG_ACCUMULATE) ? 1 : 0, s);
    if (rc) return rc;
  }
  if (out_bf16) {
    BIGMAC_STAGE(BIGMAC_STAGE_BWD_OUTPUT_CAST);
    hipLaunchKernelGGL(f32_to_bf16_kernel, grid1d(Td), dim3(256), 0, s, dx_f32, (bf16_t*)dx, Td);
    BIGMAC_CHECK_LAUNCH();
  }
  return BIGMAC_OK;
}

}  // extern "C"
