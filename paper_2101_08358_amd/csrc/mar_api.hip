// C ABI of the training-step library: argument checks, workspace carve-up, launch order.
#include <stdarg.h>
#include <stdio.h>
#include <stdlib.h>
#include <string.h>
#include <new>

#include "mar_common.h"

static thread_local char g_err[512] = "";

void mar_set_error(const char* fmt, ...) {
  va_list ap;
  va_start(ap, fmt);
  vsnprintf(g_err, sizeof(g_err), fmt, ap);
  va_end(ap);
}

extern "C" const char* mar_last_error(const mar_ctx*) { return g_err; }

static int fail(int code, const char* fmt, ...) {
  va_list ap;
  va_start(ap, fmt);
  vsnprintf(g_err, sizeof(g_err), fmt, ap);
  va_end(ap);
  return code;
}

static int hip_fail(hipError_t e, const char* what) {
  return fail(MAR_EHIP, "%s: %s", what, hipGetErrorString(e));
}

// ------------------------------------------------------------------ configuration -----
#define MAR_FLASH_TARGET_WGS 640

static int wgs_per_cu(const MarDims& d, int pass) { return mar_on_images(d) ? mar_split_wgs_per_cu(d.dk, pass) : mar_flash_wgs_per_cu(d.dk, pass); }

// Small batches give too few (chunk-side, stripe) units to fill 256 CUs: several workgroups share a unit, each
// streaming a slice of the other matrix.  fp32 instructions: until a pass has at least MAR_FLASH_TARGET_WGS workgroups;
// passes 1 and 3 then take the number of parts with the least work on the busiest CU, a part costing its tiles and one
// more (10,000 edges, 100 floats: 4 parts 106 us, 2 parts 121, 8 parts 116), in pass 3 two more (52 x 101 edges, 200
// candidates of 400 floats: 1 part 48 us, 4 parts 60).  16-bit instructions: as many parts as the least estimated time
// of the busiest CU asks for -- a workgroup costs its tiles plus about three tiles' time for its operand fragments, its
// first tile and its rows (pass 3, whose tiles are half the work and whose close comparisons are settled at the end:
// eight, from the time when every lane settled its own); a CU that holds one of two possible workgroups runs it at about 0.6 of its full rate.
void mar_plan_parts(const MarDims& d, int pass, long units, int n_y, int32_t* sy, int32_t* tps) {
  const int ty = mar_tile_rows(d, pass);
  const int ntiles = (n_y + ty - 1) / ty;
  long want = 1;
  if (!mar_on_images(d)) {
    want = (MAR_FLASH_TARGET_WGS + units - 1) / units;
    if (want > MAR_MAX_PARTS) want = MAR_MAX_PARTS;
    if (want > ntiles) want = ntiles;
    if (pass != 2 && want > 1) {
      long best = 1L << 60;
      for (long k = 1; k <= MAR_MAX_PARTS && k <= ntiles; ++k) {
        const long cost = (units * k + 255) / 256 * ((ntiles + k - 1) / k + (pass == 3 ? 2 : 1));
        if (cost < best) { best = cost; want = k; }
      }
    }
  } else if (units < 256L * wgs_per_cu(d, pass) || pass == 3) {
    double best = 1e30;
    const bool two = wgs_per_cu(d, pass) >= 2;
    const int most = pass == 3 ? 64 : MAR_MAX_PARTS;
    for (long k = 1; k <= most && k <= ntiles; ++k) {
      const long t = (ntiles + k - 1) / k, per_cu = (units * k + 255) / 256;
      const double cost = (two && per_cu == 1 ? 1.6 : (double)per_cu) * (double)(t + (pass == 3 ? 8 : 3));
      if (cost < best * 0.97) { best = cost; want = k; }
    }
  }
  if (want < 1) want = 1;
  *tps = (int32_t)((ntiles + want - 1) / want);
  *sy = (int32_t)((ntiles + *tps - 1) / *tps);
}

// Evaluation of rows above 256 floats (a workgroup a CU): equal shares, one a CU, in place of parts.  A share has no last,
// partly filled round, but its workgroup begins anew at every unit it enters; where that does not save a tenth by the estimate
// above, parts of units stay.  400 floats, gather included, us (parts / shares): 20 x 1,000 edges, 1,000 candidates 201 / 186,
// 37 x 611, 777: 207 / 205, 100 x 1,000, 1,000: 912 / 934, 60 x 1,000, 1,000: 531 / 546, 10 x 700, 1,000: 75 / 82, 1 x 900, 3,000:
// 39 / 45.  With two or three workgroups a CU the other ones fill the round: shares of 100 floats took 2 to 8 % longer at all sizes.
bool mar_plan_shares(const MarDims& d, long units, int ntiles, int sy, int tps) {
  if (!mar_split_shares(d.dk) || ntiles < 3 || units * ntiles < 8 * MAR_SHARES) return false;   // fewer than 3: sp_share_border
  const long share = (units * ntiles + MAR_SHARES - 1) / MAR_SHARES, pieces = 1 + (share - 2 + ntiles) / ntiles;
  return (double)(share + 8 * pieces) < 0.9 * (double)((units * sy + 255) / 256 * (tps + 8));
}

// Large batches: the units of a pass rarely fill a whole number of rounds of the chip's workgroup slots (256 CUs x
// workgroups per CU), and the last, partly filled round costs as much time as a full one.  The units beyond the last
// whole round are split into k parts.  TransE (pass 1 only): as many as fill one round.  Bilinear models: the
// remainder often exceeds half a round (units of 128 rows), so the parts may take several rounds of their own; every
// part beyond the first costs a write and a read of the units' output rows.  Estimated in microseconds from the rates
// these passes reach (about 1,000 TFLOP/s of 16-bit work over all slots -- 100 floats 970 and 880, 400 floats 1,150 and 1,020 --
// and 4.5 TB/s of memory traffic).
static void plan_rem(const MarDims& d, int pass, long units, int n_y, int sy, int sr, MarRem* r) {
  r->whole_units = (int32_t)units; r->k = 1; r->tps = 0; r->rows = 0;
  const long slots = 256L * wgs_per_cu(d, pass);
  if (sy != 1 || units < slots || units % slots == 0 || (!mar_on_images(d) && pass == 2)) return;
  const int ty = mar_tile_rows(d, pass);
  const long ntiles = (n_y + ty - 1) / ty, rem = units % slots;
  long k = slots / rem;
  if (k > MAR_MAX_PARTS) k = MAR_MAX_PARTS;
  if (k > ntiles) k = ntiles;
  if (mar_on_images(d)) {
    const double unit_us = 12.0 * sr * (double)n_y * d.dk * (double)slots / 1.0e9;
    double best = 1e30;
    k = 1;
    for (long kk = 1; kk <= MAR_MAX_PARTS && kk <= ntiles; ++kk) {
      const double cost = (double)((rem * kk + slots - 1) / slots) / (double)kk * unit_us + (double)(kk - 1) * rem * sr * d.dk * 8.0 / 4.5e6;
      if (cost < best) { best = cost; k = kk; }
    }
  }
  if (k < 2) return;
  r->whole_units = (int32_t)(units - rem);
  r->tps = (int32_t)((ntiles + k - 1) / k);
  r->k = (int32_t)((ntiles + r->tps - 1) / r->tps);
  r->rows = (int64_t)rem * sr;
}

// Evaluation of the bilinear models: on images and 16-bit products (mar_split.hip), or on dense fp32 operands and fp32
// matrix instructions (k_flash, PASS 4), whose gather writes no images and whose two kernels are a third of the code to be
// fetched.  What the images cost goes with a chunk's rows, S edges and N candidates, what the faster products save with
// its S N pairs, so the line is one of S N / (S + N); and where all pairs together are few, latency decides.  fp32 / images,
// us, 50 and 100 floats: 20 x 400 edges, 100 candidates 12 / 19, 16 / 23; 20 x 400, 400 (on the line) 20 / 23, 32 / 29; 100 x 300, 600
// (on the line) 54 / 53, 89 / 78; 4 x 1,000, 600: 13 / 19, 18 / 21; 100 x 1,000, 1,000: 216 / 144, 373 / 231; 28 x 370, 213 of 78
// floats 34 / 38.  Above 128 floats products cost more and the line lies nearer: 512 edges, 4 chunks, all 12,326 nodes of 374 floats
// 247 / 132; 15,500, 77, 515 of 262 223 / 180; 768, 4, all 7,371 of 244 119 / 87; 290, 1, all 4,137 of 185 (1.2e6 pairs) 59 / 34; 11,800, 18,
// 132 of 240 (S N / (S + N) = 110) 48 / 44; 33,000, 43, 112 of 279 (98) 115 / 119.  Ranks are the same bits either way.
bool mar_eval_dense(const MarDims& d, const MarBatch& b) {
  const double S = b.n < d.S ? b.n : d.S, N = d.N;
  const bool wide = d.dk > 128;
  return d.bilinear && (S * N <= (wide ? 100.0 : 200.0) * (S + N) || (double)b.n * N <= (wide ? 1.1e6 : 2.0e6));
}

// Training passes of TransE: on images and 16-bit products (k_split_dist), or on dense fp32 operands with stored weights (k_flash,
// k_flash_bwd), whose code is a quarter as long and whose gather writes no images.  What the faster products save goes with
// pairs x columns.  A step, us, dense / images: 1e9 (10,000 edges, 1,000 negatives, 100 floats, outputs) 222 / 177, 4e9 (the same,
// 400 floats) 776 / 578; 5e8 178 / 139 (84 floats), 296 / 265 (320); 2 to 2.5e8: 143 / 133 (61), 145 / 136 (191), 150 / 152 (304);
// 1e8: 126 / 113 (144), 95 / 113 (58), 114 / 126 (148); 200 to 2,000 edges mostly 5 to 20 % slower on images.
// And images pad: a workgroup owns 128 rows and streams 32 where the dense ones own 64 and stream 64, so chunks of few edges or few
// negatives are left to those.  Passes of full chunks take 48 and 58 us on images, 111 and 61 dense (10,000 edges, 1,000 negatives, 100
// floats), which weighs the padded work of either; from 0.77 on images are slower (steps of 1e8 to 8e8, dense / images, us: 722
// edges a chunk, 29 negatives 190 / 237; 55 and 644 243 / 294; 50 and 100 373 / 405; 20 and 50 425 / 523; 1,000 and 64 194 / 208, and 50
// 159 / 157; below: 272 and 564 174 / 131; 70 and 703 169 / 151; 94 and 566 189 / 165; 209 and 144 176 / 148; 696 and 185 162 / 127).
// Above 256 floats, one workgroup a CU, eight parts of fewer than 25 stripes leave a fifth of them idle (3 chunks of 875 edges, 345 negatives
// of 372 floats: 18 stripes 150 / 167; 24 of 397 127 / 150; 20 of 336 154 / 162; 26 of 280 179 / 149).  80 measured batches from 2e8 on lie
// at 0.69 to 1.07 of the dense form, most of them below 0.95.
bool mar_dist_images(const MarDims& d) {
  auto up = [](int32_t rows, int32_t to) { return (double)((rows + to - 1) / to * to); };
  const double images = 48 * up(d.S, 128) * up(d.N, 32) + 58 * up(d.N, 128) * up(d.S, 32);
  const double dense = 111 * up(d.S, 64) * up(d.N, 64) + 61 * up(d.N, 64) * up(d.S, 64);
  const int32_t rows = d.S < d.N ? d.S : d.N;
  const bool idle = d.dk > 256 && 2L * d.C * ((rows + MAR_SPLIT_STRIPE_ROWS - 1) / MAR_SPLIT_STRIPE_ROWS) < 200 / MAR_MAX_PARTS;
  return !d.bilinear && (double)d.B * d.N * d.dk >= 2.0e8 && images < 0.77 * dense && !idle;
}

// Whether the step's own launches carry the row order along (MarSortJob), or the second stream takes it.  Carried along it costs
// neither launches nor events, which bound small steps, but its workgroups (a tile of 1,024 gradient rows each, about 10 us) take
// slots of the passes.  us a step, second stream / carried along: 1,000 edges of 50 floats, 100 negatives 73 / 54; 20,000 gradient
// rows (2,000 edges, 5 chunks, 31 floats) 81 / 50; 32,000 (13,600 edges, 28 chunks of 88 negatives, 39 floats) 107 / 91; 60,000 where
// they fit beside both passes (18,700 edges, 111 negatives of 36) 92 / 76; 90,000 beside passes of 33 us (10,000 edges, 1,000 negatives of
// 100) 139 / 128, of 64 floats, TransE 135 / 124, 81,000 (9,000, 950 of 120) 127 / 117, 88,000 (8,000, 2,000 of 100) 150 / 149, 75,000
// (5,000, 1,500 of 100, three sort passes) 126 / 127, 86,000 (22,000, 300 of 200) 208 / 211; where neither holds 120,000 (33,000
// edges, 191 negatives of 76) 135 / 141, 230,000 (57,000 edges of 20 floats) 135 / 168, 72,000 (4,200 edges, 755 negatives of 272: one
// workgroup a CU) 194 / 201.  Images above 128 floats have one workgroup a CU and no slots beside their own: there the order costs more
// than the second stream from 36,000 rows with three sort passes (a scatter beside each of pass 1, the chain rule and pass 2: 45,700
// rows of 154 floats 162 / 170, 40,600 of 133 108 / 112, 61,000 of 192 148 / 154; 33,500 of 208 107 / 104), from 50,000 with two
// (54,000 of 140 141 / 149, 58,800 of 176 110 / 113; 44,000 of 196 97 / 90, 49,900 of 152, TransE 171 / 158).
static bool order_rides(const MarDims& d, long units1, long units2) {
  if (d.index_after_gather || d.sort_items != MAR_SORT_RIDE_ITEMS || d.sort_passes > 3 || d.n_pos_max > 96 * 1024) return false;
  const bool crowded = wgs_per_cu(d, 1) == 1 && d.n_pos_max > (d.sort_passes > 2 ? 36 : 50) * 1024;
  if (d.n_pos_max <= 72 * 1024 && d.dk <= 256 && !crowded) return true;
  const long tiles = (d.n_pos_max + 1023) / 1024 + 7;
  if (units1 * d.sy1 + tiles <= 256L * wgs_per_cu(d, 1) && units2 * d.sy2 + tiles <= 256L * wgs_per_cu(d, 2)) return true;
  return d.long_passes && d.dk <= 256;
}

int mar_check_config(const mar_config* cfg, MarDims* d) {
  if (!cfg) return fail(MAR_EINVAL, "config is NULL");
  if (cfg->num_nodes < 1 || cfg->num_rels < 1) return fail(MAR_EINVAL, "num_nodes and num_rels must be >= 1");
  if (cfg->num_nodes + (int64_t)cfg->num_rels >= ((int64_t)1 << 31))
    return fail(MAR_ERANGE, "num_nodes + num_rels must be below 2^31");
  if (cfg->model < MAR_MODEL_DISTMULT || cfg->model > MAR_MODEL_DOT) return fail(MAR_EINVAL, "unknown model %d", cfg->model);
  if (cfg->dim < 1 || cfg->dim > MAR_MAX_DIM) return fail(MAR_ERANGE, "dim %d outside 1..%d", cfg->dim, MAR_MAX_DIM);
  if (cfg->model == MAR_MODEL_COMPLEX && (cfg->dim & 1)) return fail(MAR_EINVAL, "ComplEx needs an even dim");
  if (cfg->precision != MAR_PRECISION_FP32 && cfg->precision != MAR_PRECISION_SPLIT_BF16) return fail(MAR_EINVAL, "unknown precision %d", cfg->precision);
  if (cfg->precision == MAR_PRECISION_SPLIT_BF16 && cfg->model == MAR_MODEL_TRANSE)
    return fail(MAR_EINVAL, "the split-precision contraction serves the bilinear models (DistMult, ComplEx, Dot) only");
  if (cfg->reserved != 0) return fail(MAR_EINVAL, "reserved must be 0");
  if (cfg->batch_size < 1 || cfg->num_chunks < 1 || cfg->negs_per_chunk < 1)
    return fail(MAR_EINVAL, "batch_size, num_chunks and negs_per_chunk must be >= 1");
  if (cfg->batch_size % cfg->num_chunks) return fail(MAR_ERANGE, "batch_size must be a multiple of num_chunks");
  if (cfg->deg_negs_per_chunk < 0 || cfg->deg_negs_per_chunk > cfg->negs_per_chunk)
    return fail(MAR_EINVAL, "deg_negs_per_chunk outside 0..negs_per_chunk");
  if (!(cfg->lr > 0.f) || !(cfg->eps >= 0.f)) return fail(MAR_EINVAL, "lr must be > 0 and eps >= 0");
  const int64_t cn = (int64_t)cfg->num_chunks * cfg->negs_per_chunk;
  const int roles = cfg->model == MAR_MODEL_DOT ? 2 : 3;
  const int64_t n_occ = roles * (int64_t)cfg->batch_size + 2 * cn;
  if (3 * (int64_t)cfg->batch_size + 2 * cn >= ((int64_t)1 << 30)) return fail(MAR_ERANGE, "batch too large: 3*batch_size + 2*chunks*negatives must be below 2^30");
  d->dim = cfg->dim;
  d->dk = (cfg->dim + 3) & ~3;
  d->B = cfg->batch_size; d->C = cfg->num_chunks; d->S = cfg->batch_size / cfg->num_chunks;
  d->N = cfg->negs_per_chunk; d->Ndeg = cfg->deg_negs_per_chunk; d->roles = roles;
  d->num_nodes = cfg->num_nodes; d->num_rels = cfg->num_rels;
  d->n_occ_max = n_occ;
  const int64_t ids = cfg->num_nodes + cfg->num_rels;
  d->u_max = ids < n_occ ? ids : n_occ;
  if (!mar_flash_supported(d->dk)) return fail(MAR_ERANGE, "row width %d not supported by the contraction kernels", d->dk);
  d->bilinear = cfg->model != MAR_MODEL_TRANSE;
  d->split_bf16 = cfg->precision == MAR_PRECISION_SPLIT_BF16;
  if (d->bilinear && !mar_split_supported(d->dk)) return fail(MAR_ERANGE, "row width %d not supported by the contraction kernels", d->dk);
  // The contraction kernels of TransE address one chunk-side's rows of either operand, and its block of weights, with
  // 32-bit byte offsets; the limit holds for every model.
  {
    const int64_t rows = d->S > d->N ? d->S : d->N;
    const int64_t tp = (d->N + 127) & ~(int64_t)127, tr_ = (d->S + 63) & ~(int64_t)63;
    if (rows * d->dk * 4 >= ((int64_t)1 << 31) || tp * tr_ * 4 >= ((int64_t)1 << 31))
      return fail(MAR_ERANGE, "chunk too large: rows x row bytes of a chunk's edges or negatives, and chunk edges x negatives x 4, must be below 2^31");
    if (d->split_bf16 && ((rows + 31) / 32) * (int64_t)mar_split_image_bytes(d->dk) >= ((int64_t)1 << 31))
      return fail(MAR_ERANGE, "chunk too large for the split-precision operand images (2^31 bytes per chunk and side)");
  }
  d->dist_img = mar_dist_images(*d);
  const int sr1 = mar_stripe_rows(*d, 1), sr2 = mar_stripe_rows(*d, 2);
  const long units1 = 2L * d->C * ((d->S + sr1 - 1) / sr1), units2 = 2L * d->C * ((d->N + sr2 - 1) / sr2);
  mar_plan_parts(*d, 1, units1, d->N, &d->sy1, &d->tps1);
  mar_plan_parts(*d, 2, units2, d->S, &d->sy2, &d->tps2);
  plan_rem(*d, 1, units1, d->N, d->sy1, sr1, &d->rem1);
  plan_rem(*d, 2, units2, d->S, d->sy2, sr2, &d->rem2);
  d->n_pos_max = roles * (int64_t)cfg->batch_size + 2 * cn * d->sy2;
  // Few positions per lane group while whole ones would leave CUs without a workgroup of the reduce.  Above that the
  // segments that cross the smaller workgroups' borders cost more than the shorter chains gain (52,000 gradient rows of 75
  // floats: a step 125 -> 116 us; 90,000 of 100: 147 -> 156).
  // And half as many again while those would: what a task costs beside its rows is then the same (1,000 edges of 50 floats, 11,000
  // gradient rows in 86 workgroups: the reduce 15 -> 12 us, a step 49 -> 45; 300 edges 70 -> 66); with a workgroup a CU or more it is slower
  // (55,000 rows of 75 floats 91 -> 98, 21,000 of 148 84 -> 90).
  d->reduce_small = d->n_pos_max < 256 * 256 ? 8 : 0;
  if (d->n_pos_max < 256 * (256 / mar_lane_group(d->dk) * 8)) d->reduce_small = 4;
  // Sort keys are unified ids: as few passes as digits of at most MAR_SORT_MAX_BITS bits allow.
  int nbits = 1;
  while (((int64_t)1 << nbits) < ids) ++nbits;
  d->sort_passes = (nbits + MAR_SORT_MAX_BITS - 1) / MAR_SORT_MAX_BITS;
  d->sort_bits = (nbits + d->sort_passes - 1) / d->sort_passes;
  // Every tile of a pass reads the counts of all tiles: small tiles while that is at most 128 KB.
  d->sort_items = ((d->n_pos_max + 1023) / 1024) << d->sort_bits <= 32768 ? 4 : 16;
  // score pairs x row width per step: above ~2e9 the contraction passes are long enough to hide the index build
  d->index_after_gather = (double)cfg->batch_size * cfg->negs_per_chunk * d->dk >= 2.0e9;
  d->sort_one = mar_sort_one_limit(d->dk, false);
  d->long_passes = (double)cfg->batch_size * cfg->negs_per_chunk * d->dk >= 6.0e8;
  d->order_rides = order_rides(*d, units1, units2);
  // The smallest steps that cannot carry it, for ids above 27 bits take a fourth pass, have it on the caller's stream all the same: the
  // fork and the join are half of the host's time (1,400 gradient rows 65 -> 51 us a step, 1,100 64 -> 52, 3,800 65 -> 64).  Wide rows
  // beside passes that fill the chip stay on two (1,280 edges of 300 floats, 3,840 rows 78 and 77, with outputs 80 and 86).
  d->one_stream = d->order_rides || (d->sort_passes > 3 && d->n_pos_max <= MAR_SORT_ONE / 4 && !d->index_after_gather);
  return MAR_OK;
}

// Carves the workspace; with base == NULL only measures.
static size_t carve(const MarDims& d, char* base, MarLayout* L) {
  size_t off = 0;
  auto take = [&](size_t bytes) -> void* {
    void* p = base ? base + off : nullptr;
    off += (bytes + 255) & ~(size_t)255;
    return p;
  };
  const size_t n_pos = (size_t)d.n_pos_max, u1 = (size_t)d.u_max + 1;
  const size_t B = d.B, CN = (size_t)d.C * d.N, dk = d.dk;
  const size_t rb = (size_t)mar_reduce_block(d), blocks = (n_pos + rb - 1) / rb;
  const size_t tiles = ((n_pos + 256 * d.sort_items - 1) / (256 * d.sort_items) + 3) & ~(size_t)3, rank_tiles = n_pos / MAR_RANK_TILE + 1;
  MarLayout l;
  l.scalars = (int32_t*)take(16 * 4);
  l.uniq = (int32_t*)take(u1 * 4);
  l.keys0 = (uint32_t*)take(n_pos * 4);
  for (int i = 0; i < 2; ++i) {
    l.kbuf[i] = (uint32_t*)take(d.sort_passes > i + 1 ? n_pos * 4 : 0);
    l.vbuf[i] = (int32_t*)take(d.sort_passes > i + 1 ? n_pos * 4 : 0);
  }
  const size_t counts = (tiles << d.sort_bits) * (d.order_rides ? d.sort_passes : 1);
  l.hist = (uint32_t*)take((counts > rank_tiles ? counts : rank_tiles) * 4);
  l.perm = (int32_t*)take(n_pos * 4);
  l.ids_sorted = (uint32_t*)take(n_pos * 4);
  l.rank_sorted = (int32_t*)take(n_pos * 4);
  l.owners = (int32_t*)take(blocks * 4);
  // On images no weights are stored (pass 2 computes the scores again).  TransE keeps its fp32 edge-side operands and the norms
  // there too; its evaluation, on dense operands, then has the negatives' rows in the gradient rows' place.
  const bool bl = d.bilinear != 0, img = mar_on_images(d);
  l.Q = (float*)take(bl ? 0 : 2 * B * dk * 4);
  l.Km = (float*)take(img ? 0 : 2 * CN * dk * 4);
  l.qq = (float*)take(bl ? 0 : 2 * B * 4);
  l.kk = (float*)take(bl ? 0 : 2 * CN * 4);
  l.pos = (float*)take(B * 4);
  l.gQ = (float*)take((size_t)d.sy1 * 2 * B * dk * 4);
  l.ml = (float*)take((size_t)d.sy1 * 2 * B * 2 * 4);
  l.gQx = (float*)take((size_t)(d.rem1.k - 1) * (size_t)d.rem1.rows * dk * 4);
  l.mlx = (float*)take((size_t)(d.rem1.k - 1) * (size_t)d.rem1.rows * 2 * 4);
  l.T = (float*)take(img ? 0 : 2 * (size_t)d.C * (size_t)((d.S + 63) & ~63) * (size_t)((d.N + 127) & ~127) * 4);
  l.R = (float*)take(img ? 0 : 2 * (size_t)d.C * (size_t)((d.S + 63) & ~63) * (size_t)(((d.N + 127) & ~127) / 16) * 4);
  const size_t ktiles = 2 * (size_t)d.C * (size_t)((d.N + 31) / 32), qtiles = 2 * (size_t)d.C * (size_t)((d.S + 31) / 32);
  l.Kimg = (char*)take(img ? ktiles * mar_split_image_bytes(d.dk) : 0);
  l.Qimg = (char*)take(img ? qtiles * mar_split_image_bytes(d.dk) : 0);
  l.Gx = (float*)take((size_t)(d.rem2.k - 1) * (size_t)d.rem2.rows * dk * 4);
  const size_t eval_floats = bl ? ktiles * (2 + 2 + MAR_SPLIT_TILE_ROWS) + qtiles * 2 : 0;
  l.G = (float*)take((n_pos * dk > eval_floats ? n_pos * dk : eval_floats) * 4);
  if (d.dist_img) l.Km = l.G;
  // evaluation's norms, and with bf16 images (which have no exponents) its exponents, lie in the gradient rows, for which it
  // has no other use
  const bool own_exp = img && !d.split_bf16;
  l.Kexp = own_exp ? (float*)take(ktiles * 8) : l.G;
  l.Qexp = own_exp ? (float*)take(qtiles * 8) : l.G + ktiles * 2;
  l.Knorm = l.G + ktiles * 2 + qtiles * 2;
  l.carry = (float*)take(blocks * 2 * dk * 4);
  l.loss_part = (float*)take((B / 4 + 2) * 4);
  l.shift = (float*)take(d.dist_img ? 512 * 4 : 0);
  l.metric_part = take((size_t)MAR_METRIC_MAX_PARTS * MAR_METRIC_PART_BYTES);
  if (L) *L = l;
  return off;
}

extern "C" int mar_workspace_bytes(const mar_config* cfg, size_t* out_bytes) {
  MarDims d;
  const int rc = mar_check_config(cfg, &d);
  if (rc) return rc;
  if (!out_bytes) return fail(MAR_EINVAL, "out_bytes is NULL");
  *out_bytes = carve(d, nullptr, nullptr);
  return MAR_OK;
}

extern "C" int mar_init_tables(const mar_config* cfg, float* node_emb, float* node_state, float* rel_emb,
                               float* rel_state, void* workspace, size_t workspace_bytes, int fill,
                               void* hip_stream, mar_ctx** out) {
  MarDims d;
  const int rc = mar_check_config(cfg, &d);
  if (rc) return rc;
  if (!out) return fail(MAR_EINVAL, "out is NULL");
  if (!node_emb || !node_state || !rel_emb || !rel_state) return fail(MAR_EINVAL, "a table pointer is NULL");
  if (((uintptr_t)node_emb | (uintptr_t)node_state | (uintptr_t)rel_emb | (uintptr_t)rel_state) & 15)
    return fail(MAR_EINVAL, "table pointers must be 16-byte aligned");
  if (!workspace || ((uintptr_t)workspace & 255)) return fail(MAR_EINVAL, "workspace must be non-NULL and 256-byte aligned");
  const size_t need = carve(d, nullptr, nullptr);
  if (workspace_bytes < need) return fail(MAR_ENOMEM, "workspace has %zu bytes, %zu needed", workspace_bytes, need);
  {
    hipError_t e_ = mar_flash_prepare(d.dk);
    if (e_ == hipSuccess && mar_on_images(d)) e_ = mar_split_prepare(d.dk);
    if (e_ != hipSuccess) return hip_fail(e_, "kernel attributes");
  }
  mar_ctx* c = new (std::nothrow) mar_ctx();
  if (!c) return fail(MAR_ENOMEM, "out of host memory");
  c->cfg = *cfg; c->dm = d;
  c->node_emb = node_emb; c->node_state = node_state; c->rel_emb = rel_emb; c->rel_state = rel_state;
  c->workspace = workspace; c->workspace_bytes = workspace_bytes;
  carve(d, (char*)workspace, &c->L);
  c->prof_max = 0; c->prof_steps = 0; c->prof_mask = 0; c->prof_events = nullptr;
  c->aux = nullptr; c->ev_fork = c->ev_index = c->ev_pass1 = c->ev_chain = nullptr;
  hipError_t e = hipStreamCreateWithFlags(&c->aux, hipStreamNonBlocking);
  hipEvent_t* evs[4] = {&c->ev_fork, &c->ev_index, &c->ev_pass1, &c->ev_chain};
  for (int i = 0; i < 4 && e == hipSuccess; ++i) e = hipEventCreateWithFlags(evs[i], hipEventDisableTiming);
  if (e == hipSuccess) e = mar_launch_init(c, fill, (hipStream_t)hip_stream);
  if (e != hipSuccess) { mar_destroy(c); return hip_fail(e, "context set-up"); }
  *out = c;
  return MAR_OK;
}

extern "C" int mar_destroy(mar_ctx* c) {
  if (!c) return MAR_OK;
  if (c->prof_events) {
    for (int i = 0; i < c->prof_max * 2 * MAR_NUM_PHASES; ++i) (void)hipEventDestroy(c->prof_events[i]);
    free(c->prof_events);
  }
  hipEvent_t evs[4] = {c->ev_fork, c->ev_index, c->ev_pass1, c->ev_chain};
  for (int i = 0; i < 4; ++i) if (evs[i]) (void)hipEventDestroy(evs[i]);
  if (c->aux) { (void)hipStreamSynchronize(c->aux); (void)hipStreamDestroy(c->aux); }
  delete c;
  return MAR_OK;
}

extern "C" int mar_sample_negatives(mar_ctx* c, uint64_t step, const int32_t* edge_src, const int32_t* edge_dst,
                                    int64_t num_edges, int32_t* neg_src, int32_t* neg_dst, void* hip_stream) {
  if (!c) return fail(MAR_EINVAL, "context is NULL");
  if (!neg_src || !neg_dst) return fail(MAR_EINVAL, "an output pointer is NULL");
  if (step >> 63) return fail(MAR_ERANGE, "step must be below 2^63");
  if (c->dm.Ndeg > 0) {
    if (!edge_src || !edge_dst) return fail(MAR_EINVAL, "degree-based negatives need the edge list");
    if (num_edges < 1) return fail(MAR_EINVAL, "degree-based negatives need num_edges >= 1");
  }
  if (num_edges < 0) return fail(MAR_EINVAL, "num_edges is negative");
  const hipError_t e = mar_launch_sample(c, step, edge_src, edge_dst, num_edges, neg_src, neg_dst, (hipStream_t)hip_stream);
  return e == hipSuccess ? MAR_OK : hip_fail(e, "sampling kernel");
}

static int make_batch(const mar_ctx* c, const int32_t* src, const int32_t* rel, const int32_t* dst, int32_t n,
                      const int32_t* neg_src, const int32_t* neg_dst, MarBatch* b) {
  if (!c) return fail(MAR_EINVAL, "context is NULL");
  if (n < 0 || n > c->dm.B) return fail(MAR_ERANGE, "n_edges %d outside 0..batch_size %d", n, c->dm.B);
  if (n > 0 && (!src || (!rel && c->dm.roles == 3) || !dst || !neg_src || !neg_dst)) return fail(MAR_EINVAL, "an id array is NULL");
  b->src = src; b->rel = rel; b->dst = dst; b->neg_src = neg_src; b->neg_dst = neg_dst;
  b->n = n;
  b->nchunks = (n + c->dm.S - 1) / c->dm.S;
  b->cn = b->nchunks * c->dm.N;
  b->n_occ = c->dm.roles * (int64_t)n + 2 * (int64_t)b->cn;
  b->n_pos = c->dm.roles * (int64_t)n + 2 * (int64_t)b->cn * c->dm.sy2;
  return MAR_OK;
}

#define HIP_TRY(expr, what) do { const hipError_t e_ = (expr); if (e_ != hipSuccess) return hip_fail(e_, what); } while (0)

extern "C" int mar_train_batch(mar_ctx* c, const int32_t* src, const int32_t* rel, const int32_t* dst, int32_t n_edges,
                               const int32_t* neg_src, const int32_t* neg_dst, float* loss_sum_out,
                               const mar_debug_out* dbg, void* hip_stream) {
  MarBatch b;
  const int rc = make_batch(c, src, rel, dst, n_edges, neg_src, neg_dst, &b);
  if (rc) return rc;
  hipStream_t st = (hipStream_t)hip_stream;
  if (n_edges == 0) {
    if (loss_sum_out) HIP_TRY(mar_launch_fill_u32((uint32_t*)loss_sum_out, 1, 0u, st), "loss reset");
    if (dbg && dbg->num_uniq) HIP_TRY(mar_launch_fill_u32((uint32_t*)dbg->num_uniq, 2, 0u, st), "debug reset");
    return MAR_OK;
  }
  // Two streams: the caller's carries the gather and the two contraction passes; the index build
  // (needed only by the per-row reduce) and the chain rule (needs pass 1 only) run beside them on `aux`.
  // Small batches stay on the caller's, whose launches carry the row order along (MarSortJob).
  const bool rides = c->dm.order_rides;
  hipStream_t ax = c->dm.one_stream ? st : c->aux;
  hipEvent_t* ev = nullptr;
  if (c->prof_events && c->prof_steps < c->prof_max) ev = c->prof_events + (size_t)c->prof_steps * 2 * MAR_NUM_PHASES;
#define MARK(phase, end, stream) do { if (ev && (c->prof_mask >> (phase) & 1u)) HIP_TRY(hipEventRecord(ev[2 * (phase) + (end)], stream), "event record"); } while (0)
  // Two orders of the first launches.  Large batches: the gather runs alone at memory speed and the index build
  // starts behind it, beside the first contraction pass that hides it.  Others whose order is not carried along (order_rides):
  // the index build is the longer path to the reduce, so it starts first and the gather runs beside it.
  if (c->dm.index_after_gather) {
    MARK(1, 0, st);
    HIP_TRY(mar_launch_prep(c, b, dbg ? dbg->pos : nullptr, c->dm.split_bf16, nullptr, nullptr, st), "gather kernel");
    MARK(1, 1, st);
  }
  if (ax != st) {
    HIP_TRY(hipEventRecord(c->ev_fork, st), "fork");
    HIP_TRY(hipStreamWaitEvent(ax, c->ev_fork, 0), "fork");
  }
  MARK(0, 0, ax);
  const int ranks = dbg && (dbg->num_uniq || dbg->uniq_nodes || dbg->uniq_rels || dbg->grad_rows);
  MarSortJob job[4];
  if (rides) {
    for (int k = 0; k < 4; ++k) job[k] = mar_sort_slot(c, b, k, ranks, dbg);
  } else {
    HIP_TRY(mar_launch_index(c, b, ranks, ax), "index kernels");
    if (dbg) HIP_TRY(mar_launch_debug_copy(c, b, dbg, ax), "debug copy");
  }
  MARK(0, 1, ax);
  if (ax != st) HIP_TRY(hipEventRecord(c->ev_index, ax), "join");
  if (!c->dm.index_after_gather) {
    MARK(1, 0, st);
    HIP_TRY(mar_launch_prep(c, b, dbg ? dbg->pos : nullptr, c->dm.split_bf16, nullptr, nullptr, st, rides ? &job[0] : nullptr), "gather kernel");
    MARK(1, 1, st);
  }
  MARK(2, 0, st);
  HIP_TRY(mar_launch_flash(c, b, 1, nullptr, nullptr, st, rides ? &job[1] : nullptr), "score/softmax kernel");
  MARK(2, 1, st);
  HIP_TRY(mar_launch_flash_merge(c, b, st), "stripe merge kernel");
  // The chain rule needs pass 1 only.  Large batches run it on `aux` beside pass 2, which leaves memory bandwidth
  // unused; for small batches `aux` is the longer path to the reduce (the index build), so it stays on the
  // caller's stream.
  if (c->dm.index_after_gather) {
    HIP_TRY(hipEventRecord(c->ev_pass1, st), "fork");
    HIP_TRY(hipStreamWaitEvent(ax, c->ev_pass1, 0), "fork");
    MARK(4, 0, ax);
    HIP_TRY(mar_launch_chain(c, b, dbg, ax), "chain-rule kernel");
    MARK(4, 1, ax);
    HIP_TRY(hipEventRecord(c->ev_chain, ax), "join");
  } else {
    MARK(4, 0, st);
    HIP_TRY(mar_launch_chain(c, b, dbg, st, rides ? &job[2] : nullptr), "chain-rule kernel");
    MARK(4, 1, st);
  }
  MARK(3, 0, st);
  HIP_TRY(mar_launch_flash(c, b, 2, nullptr, nullptr, st, rides ? &job[3] : nullptr), "negative-gradient kernel");
  MARK(3, 1, st);
  if (rides && ranks && job[3].kind != MAR_SORT_RANKS) {   // three passes over the ids: pass 2 carries the last of them
    HIP_TRY(mar_launch_ranks(c, b, st), "rank kernels");
    HIP_TRY(mar_launch_debug_copy(c, b, dbg, st), "debug copy");
  }
  if (ax != st) HIP_TRY(hipStreamWaitEvent(st, c->ev_index, 0), "join");
  if (c->dm.index_after_gather) HIP_TRY(hipStreamWaitEvent(st, c->ev_chain, 0), "join");
  MARK(5, 0, st);
  HIP_TRY(mar_launch_reduce(c, b, loss_sum_out, dbg ? dbg->grad_rows : nullptr, nullptr, st), "reduce/Adagrad kernels");
  MARK(5, 1, st);
#undef MARK
  if (ev) c->prof_steps++;
  return MAR_OK;
}

extern "C" int mar_eval_scores(mar_ctx* c, const int32_t* src, const int32_t* rel, const int32_t* dst, int32_t n_edges,
                               const int32_t* neg_src, const int32_t* neg_dst, float* pos_scores, int32_t* rank_dst,
                               int32_t* rank_src, void* hip_stream) {
  MarBatch b;
  const int rc = make_batch(c, src, rel, dst, n_edges, neg_src, neg_dst, &b);
  if (rc) return rc;
  if (!rank_dst || !rank_src) return fail(MAR_EINVAL, "a rank output pointer is NULL");
  if (n_edges == 0) return MAR_OK;
  hipStream_t st = (hipStream_t)hip_stream;
  HIP_TRY(mar_launch_prep(c, b, pos_scores, 0, rank_dst, rank_src, st), "gather kernel");
  HIP_TRY(mar_launch_flash(c, b, 3, rank_dst, rank_src, st), "rank kernel");
  return MAR_OK;
}

extern "C" int mar_eval_filter(mar_ctx* c, const int32_t* src, const int32_t* rel, const int32_t* dst, int32_t n_edges,
                               const int64_t* dst_off, const int32_t* dst_ids, const int64_t* src_off,
                               const int32_t* src_ids, const float* pos_scores, int32_t* rank_dst, int32_t* rank_src,
                               void* hip_stream) {
  if (!c) return fail(MAR_EINVAL, "context is NULL");
  if (n_edges < 0 || n_edges > c->dm.B) return fail(MAR_ERANGE, "n_edges %d outside 0..batch_size %d", n_edges, c->dm.B);
  if (n_edges == 0) return MAR_OK;
  if (!src || (!rel && c->dm.roles == 3) || !dst) return fail(MAR_EINVAL, "an id array is NULL");
  if (!dst_off || !src_off || !pos_scores || !rank_dst || !rank_src) return fail(MAR_EINVAL, "an argument is NULL");
  MarBatch b;
  b.src = src; b.rel = rel; b.dst = dst; b.neg_src = nullptr; b.neg_dst = nullptr;
  b.n = n_edges; b.nchunks = 0; b.cn = 0; b.n_occ = 0; b.n_pos = 0;
  HIP_TRY(mar_launch_filter(c, b, dst_off, dst_ids, src_off, src_ids, pos_scores, rank_dst, rank_src, (hipStream_t)hip_stream),
          "filter kernel");
  return MAR_OK;
}

extern "C" int mar_rank_metrics(mar_ctx* c, const int32_t* ranks, int64_t n_ranks, const int32_t* ks, int32_t num_k,
                                double* out, void* hip_stream) {
  if (!c) return fail(MAR_EINVAL, "context is NULL");
  if (!out) return fail(MAR_EINVAL, "out is NULL");
  if (n_ranks < 0 || (n_ranks > 0 && !ranks)) return fail(MAR_EINVAL, "ranks is NULL or n_ranks negative");
  if (num_k < 0 || num_k > 8 || (num_k > 0 && !ks)) return fail(MAR_ERANGE, "num_k outside 0..8 or ks NULL");
  for (int j = 0; j < num_k; ++j) if (ks[j] < 1) return fail(MAR_EINVAL, "thresholds must be >= 1");
  HIP_TRY(mar_launch_rank_metrics(ranks, n_ranks, ks, num_k, out, c->L.metric_part, (hipStream_t)hip_stream), "metrics kernel");
  return MAR_OK;
}

// ------------------------------------------------------- out-of-memory pipelined training -----
// Sec. 3: node embeddings and their optimiser state live outside device memory; a batch goes through
//   in   : unique set + staging of its node rows into a compact device table          (stream s_in)
//   step : gather / score / loss / backward on the staged rows, relation rows updated  (caller's stream)
//   out  : Adagrad on the host table with the batch's summed node gradients            (stream s_out)
// and up to `depth` batches are in flight.  Events order the stages so that batch j stages its rows after the
// updates of batches <= j - depth and before the update of batch j - depth + 1: the staleness is exactly
// depth - 1 batches in every run.
struct PipeSlot {
  mar_ctx* ctx;                // context over the compact table (node_emb = compact) and the resident relation tables
  MarStage sg;
  int32_t *src, *rel, *dst, *neg_src, *neg_dst;    // the slot's copy of the batch's ids
  MarBatch b_ids, b_rank;      // the batch over real ids (index build) and over ranks (gather, chain rule)
  hipEvent_t ev_in, ev_step, ev_out;
};

struct mar_pipe {
  mar_config cfg; MarDims dm;
  int32_t depth;
  float *host_emb, *host_state, *rel_emb, *rel_state;
  hipStream_t s_in, s_out;
  hipEvent_t ev_call;
  PipeSlot* slots;
  int64_t submitted, applied;  // batches submitted / the batch behind the one whose update was enqueued last
  int64_t drained;             // batches submitted when the last drain was called: it enqueued all their updates
};

static size_t pipe_slot_extra(const MarDims& d, char* base, PipeSlot* ps) {
  size_t off = 0;
  auto take = [&](size_t bytes) -> void* {
    void* p = base ? base + off : nullptr;
    off += (bytes + 255) & ~(size_t)255;
    return p;
  };
  const size_t B = d.B, CN = (size_t)d.C * d.N;
  const size_t rows = (size_t)(2 * B + 2 * CN < (size_t)d.num_nodes ? 2 * B + 2 * CN : (size_t)d.num_nodes);
  PipeSlot t;
  t.sg.compact = (float*)take(rows * d.dim * 4 + 16);
  t.sg.gsum = (float*)take((size_t)d.u_max * d.dk * 4);
  t.sg.shared = (uint8_t*)take(rows);
  t.sg.c_src = (int32_t*)take(B * 4); t.sg.c_dst = (int32_t*)take(B * 4);
  t.sg.c_neg_dst = (int32_t*)take(CN * 4); t.sg.c_neg_src = (int32_t*)take(CN * 4);
  t.src = (int32_t*)take(B * 4); t.rel = (int32_t*)take(B * 4); t.dst = (int32_t*)take(B * 4);
  t.neg_src = (int32_t*)take(CN * 4); t.neg_dst = (int32_t*)take(CN * 4);
  if (ps) { ps->sg.compact = t.sg.compact; ps->sg.gsum = t.sg.gsum; ps->sg.shared = t.sg.shared; ps->sg.c_src = t.sg.c_src; ps->sg.c_dst = t.sg.c_dst;
            ps->sg.c_neg_dst = t.sg.c_neg_dst; ps->sg.c_neg_src = t.sg.c_neg_src; ps->src = t.src; ps->rel = t.rel; ps->dst = t.dst;
            ps->neg_src = t.neg_src; ps->neg_dst = t.neg_dst; }
  return off;
}

static int pipe_check(const mar_config* cfg, int32_t depth, MarDims* d) {
  const int rc = mar_check_config(cfg, d);
  if (rc) return rc;
  if (depth < 1 || depth > MAR_PIPE_MAX_DEPTH) return fail(MAR_ERANGE, "depth %d outside 1..%d", depth, MAR_PIPE_MAX_DEPTH);
  return MAR_OK;
}

extern "C" int mar_pipe_workspace_bytes(const mar_config* cfg, int32_t depth, size_t* out_bytes) {
  MarDims d;
  const int rc = pipe_check(cfg, depth, &d);
  if (rc) return rc;
  if (!out_bytes) return fail(MAR_EINVAL, "out_bytes is NULL");
  *out_bytes = (size_t)depth * (carve(d, nullptr, nullptr) + pipe_slot_extra(d, nullptr, nullptr));
  return MAR_OK;
}

extern "C" int mar_pipe_destroy(mar_pipe* p) {
  if (!p) return MAR_OK;
  if (p->s_in) { (void)hipStreamSynchronize(p->s_in); (void)hipStreamDestroy(p->s_in); }
  if (p->s_out) { (void)hipStreamSynchronize(p->s_out); (void)hipStreamDestroy(p->s_out); }
  if (p->ev_call) (void)hipEventDestroy(p->ev_call);
  if (p->slots) {
    for (int i = 0; i < p->depth; ++i) {
      hipEvent_t evs[3] = {p->slots[i].ev_in, p->slots[i].ev_step, p->slots[i].ev_out};
      for (int k = 0; k < 3; ++k) if (evs[k]) (void)hipEventDestroy(evs[k]);
      mar_destroy(p->slots[i].ctx);
    }
    delete[] p->slots;
  }
  delete p;
  return MAR_OK;
}

extern "C" int mar_pipe_create(const mar_config* cfg, float* host_node_emb, float* host_node_state, float* rel_emb,
                               float* rel_state, void* workspace, size_t workspace_bytes, int32_t depth, void* hip_stream,
                               mar_pipe** out) {
  MarDims d;
  const int rc = pipe_check(cfg, depth, &d);
  if (rc) return rc;
  if (!out) return fail(MAR_EINVAL, "out is NULL");
  if (!host_node_emb || !host_node_state || !rel_emb || !rel_state) return fail(MAR_EINVAL, "a table pointer is NULL");
  if (((uintptr_t)host_node_emb | (uintptr_t)host_node_state | (uintptr_t)rel_emb | (uintptr_t)rel_state) & 15)
    return fail(MAR_EINVAL, "table pointers must be 16-byte aligned");
  if (!workspace || ((uintptr_t)workspace & 255)) return fail(MAR_EINVAL, "workspace must be non-NULL and 256-byte aligned");
  // the host tables must be memory the GPU can address; kernels use the device-side alias the runtime reports
  float* host_tabs[2] = {host_node_emb, host_node_state};
  for (int i = 0; i < 2; ++i) {
    hipPointerAttribute_t at;
    const hipError_t pe = hipPointerGetAttributes(&at, host_tabs[i]);
    if (pe != hipSuccess) { (void)hipGetLastError(); return fail(MAR_EINVAL, "host table %d is not memory known to the HIP runtime (allocate it pinned)", i); }
    if (at.type != hipMemoryTypeHost || !at.devicePointer) return fail(MAR_EINVAL, "host table %d is not pinned, device-accessible host memory", i);
    host_tabs[i] = (float*)at.devicePointer;
  }
  host_node_emb = host_tabs[0]; host_node_state = host_tabs[1];
  const size_t ctx_bytes = carve(d, nullptr, nullptr), extra = pipe_slot_extra(d, nullptr, nullptr);
  if (workspace_bytes < (size_t)depth * (ctx_bytes + extra))
    return fail(MAR_ENOMEM, "workspace has %zu bytes, %zu needed", workspace_bytes, (size_t)depth * (ctx_bytes + extra));
  mar_pipe* p = new (std::nothrow) mar_pipe();
  if (!p) return fail(MAR_ENOMEM, "out of host memory");
  p->cfg = *cfg; p->dm = d; p->depth = depth;
  p->host_emb = host_node_emb; p->host_state = host_node_state; p->rel_emb = rel_emb; p->rel_state = rel_state;
  p->s_in = p->s_out = nullptr; p->ev_call = nullptr; p->submitted = p->applied = p->drained = 0;
  p->slots = new (std::nothrow) PipeSlot[depth]();
  if (!p->slots) { delete p; return fail(MAR_ENOMEM, "out of host memory"); }
  hipError_t e = hipStreamCreateWithFlags(&p->s_in, hipStreamNonBlocking);
  if (e == hipSuccess) e = hipStreamCreateWithFlags(&p->s_out, hipStreamNonBlocking);
  if (e == hipSuccess) e = hipEventCreateWithFlags(&p->ev_call, hipEventDisableTiming);
  char* base = (char*)workspace;
  for (int i = 0; i < depth && e == hipSuccess; ++i) {
    PipeSlot& ps = p->slots[i];
    char* sb = base + (size_t)i * (ctx_bytes + extra);
    pipe_slot_extra(d, sb + ctx_bytes, &ps);
    ps.sg.host_emb = host_node_emb; ps.sg.host_state = host_node_state;
    // the slot's context: the compact table stands in for the node table (no fill; its accumulators are never used)
    const int rc2 = mar_init_tables(cfg, ps.sg.compact, ps.sg.compact, rel_emb, rel_state, sb, ctx_bytes, 0, hip_stream, &ps.ctx);
    if (rc2) { mar_pipe_destroy(p); return rc2; }
    ps.ctx->dm.sort_one = mar_sort_one_limit(d.dk, true);
    hipEvent_t* evs[3] = {&ps.ev_in, &ps.ev_step, &ps.ev_out};
    for (int k = 0; k < 3 && e == hipSuccess; ++k) e = hipEventCreateWithFlags(evs[k], hipEventDisableTiming);
  }
  if (e != hipSuccess) { mar_pipe_destroy(p); return hip_fail(e, "pipeline set-up"); }
  *out = p;
  return MAR_OK;
}

__global__ void __launch_bounds__(256)
k_copy_ids(const int32_t* __restrict__ s0, const int32_t* __restrict__ r0, const int32_t* __restrict__ d0,
           const int32_t* __restrict__ ns0, const int32_t* __restrict__ nd0, int n, int cn, int32_t* __restrict__ s1,
           int32_t* __restrict__ r1, int32_t* __restrict__ d1, int32_t* __restrict__ ns1, int32_t* __restrict__ nd1) {
  const int i = blockIdx.x * 256 + threadIdx.x;
  if (i < n) { s1[i] = s0[i]; d1[i] = d0[i]; if (r0) r1[i] = r0[i]; }
  if (i < cn) { ns1[i] = ns0[i]; nd1[i] = nd0[i]; }
}

#define PIPE_TRY(expr, what) do { const hipError_t e_ = (expr); if (e_ != hipSuccess) return hip_fail(e_, what); } while (0)

// Enqueues the update stage of batch i on s_out; `gather_of` >= 0: it must also wait for the staging of that batch.
static int pipe_enqueue_update(mar_pipe* p, int64_t i, int64_t gather_of) {
  PipeSlot& ps = p->slots[i % p->depth];
  PIPE_TRY(hipStreamWaitEvent(p->s_out, ps.ev_step, 0), "update stage");
  if (gather_of >= 0) PIPE_TRY(hipStreamWaitEvent(p->s_out, p->slots[gather_of % p->depth].ev_in, 0), "update stage");
  // The staged values of a batch whose update a drain has enqueued already are not the newest: a submit that follows the
  // drain reads everything from the host table.
  MarStage sg = ps.sg;
  if (i < p->drained) sg.shared = nullptr;
  PIPE_TRY(mar_launch_stage_out(ps.ctx, ps.b_ids, sg, p->s_out), "update kernel");
  PIPE_TRY(hipEventRecord(ps.ev_out, p->s_out), "update stage");
  p->applied = i + 1;
  return MAR_OK;
}

extern "C" int mar_pipe_submit(mar_pipe* p, const int32_t* src, const int32_t* rel, const int32_t* dst, int32_t n_edges,
                               const int32_t* neg_src, const int32_t* neg_dst, float* loss_sum_out, void* ids_stream,
                               void* hip_stream) {
  if (!p) return fail(MAR_EINVAL, "pipeline is NULL");
  if (n_edges < 1) return fail(MAR_EINVAL, "n_edges must be >= 1");
  const int64_t j = p->submitted;
  PipeSlot& ps = p->slots[j % p->depth];
  mar_ctx* c = ps.ctx;
  int rc = make_batch(c, src, rel, dst, n_edges, neg_src, neg_dst, &ps.b_ids);
  if (rc) return rc;
  hipStream_t st = (hipStream_t)hip_stream;
  const int roles = c->dm.roles;
  // ---- in: after the work enqueued so far on the stream the ids come from, and after the update of the batch that
  // used this slot before (batch j - depth: its buffers are free, and its update is the newest one batch j may see)
  PIPE_TRY(hipEventRecord(p->ev_call, (hipStream_t)ids_stream), "submit");
  PIPE_TRY(hipStreamWaitEvent(p->s_in, p->ev_call, 0), "submit");
  if (j >= p->depth) PIPE_TRY(hipStreamWaitEvent(p->s_in, ps.ev_out, 0), "stage in");
  // the first batch behind a drain: the drain enqueued the updates up to batch j - 1, and the staging must not run beside
  // them (the caller need not have waited for the drain on the stream the ids come from)
  if (j > 0 && j == p->drained) PIPE_TRY(hipStreamWaitEvent(p->s_in, p->slots[(j - 1) % p->depth].ev_out, 0), "stage in");
  const int work = n_edges > ps.b_ids.cn ? n_edges : ps.b_ids.cn;
  hipLaunchKernelGGL(k_copy_ids, dim3((work + 255) / 256), dim3(256), 0, p->s_in, src, roles == 3 ? rel : nullptr, dst, neg_src, neg_dst,
                     n_edges, ps.b_ids.cn, ps.src, ps.rel, ps.dst, ps.neg_src, ps.neg_dst);
  PIPE_TRY(hipGetLastError(), "id copy");
  ps.b_ids.src = ps.src; ps.b_ids.rel = ps.rel; ps.b_ids.dst = ps.dst; ps.b_ids.neg_src = ps.neg_src; ps.b_ids.neg_dst = ps.neg_dst;
  ps.b_rank = ps.b_ids;
  ps.b_rank.src = ps.sg.c_src; ps.b_rank.dst = ps.sg.c_dst; ps.b_rank.neg_src = ps.sg.c_neg_src; ps.b_rank.neg_dst = ps.sg.c_neg_dst;
  PIPE_TRY(mar_launch_index(c, ps.b_ids, 1, p->s_in), "index kernels");
  // the updates of the batches between j - depth and j come after this batch's staging and before its own update; their
  // unique lists were written earlier on s_in and stay until their slots are used again, also on s_in
  const int64_t first = j - p->depth + 1 > 0 ? j - p->depth + 1 : 0;
  ps.sg.num_prev = j - first <= MAR_STAGE_PREV ? (int32_t)(j - first) : -1;
  for (int q = 0; q < MAR_STAGE_PREV; ++q) {
    const mar_ctx* pc = q < ps.sg.num_prev ? p->slots[(first + q) % p->depth].ctx : nullptr;
    ps.sg.prev_uniq[q] = pc ? pc->L.uniq : nullptr; ps.sg.prev_scalars[q] = pc ? pc->L.scalars : nullptr;
  }
  PIPE_TRY(mar_launch_stage_in(c, ps.b_ids, ps.sg, p->s_in), "staging kernels");
  PIPE_TRY(hipEventRecord(ps.ev_in, p->s_in), "stage in");
  // ---- step on the caller's stream: staged rows, ranks as ids; node gradients are left in gsum, relation rows updated
  PIPE_TRY(hipStreamWaitEvent(st, ps.ev_in, 0), "step");
  PIPE_TRY(mar_launch_prep(c, ps.b_rank, nullptr, c->dm.split_bf16, nullptr, nullptr, st), "gather kernel");
  PIPE_TRY(mar_launch_flash(c, ps.b_rank, 1, nullptr, nullptr, st), "score/softmax kernel");
  PIPE_TRY(mar_launch_flash_merge(c, ps.b_rank, st), "stripe merge kernel");
  PIPE_TRY(mar_launch_chain(c, ps.b_rank, nullptr, st), "chain-rule kernel");
  PIPE_TRY(mar_launch_flash(c, ps.b_rank, 2, nullptr, nullptr, st), "negative-gradient kernel");
  PIPE_TRY(mar_launch_reduce(c, ps.b_ids, loss_sum_out, nullptr, ps.sg.gsum, st), "reduce kernels");
  PIPE_TRY(hipEventRecord(ps.ev_step, st), "step");
  p->submitted = j + 1;
  // ---- out: the update of batch j - depth + 1 goes behind this batch's staging
  const int64_t i = j - p->depth + 1;
  if (i >= 0) { rc = pipe_enqueue_update(p, i, j); if (rc) return rc; }
  return MAR_OK;
}

extern "C" int mar_pipe_drain(mar_pipe* p, void* hip_stream) {
  if (!p) return fail(MAR_EINVAL, "pipeline is NULL");
  for (int64_t i = p->applied; i < p->submitted; ++i) { const int rc = pipe_enqueue_update(p, i, -1); if (rc) return rc; }
  p->drained = p->submitted;
  if (p->submitted > 0)
    PIPE_TRY(hipStreamWaitEvent((hipStream_t)hip_stream, p->slots[(p->submitted - 1) % p->depth].ev_out, 0), "drain");
  return MAR_OK;
}

// ----------------------------------------------------------------------- profiling -----
extern "C" int mar_profile_enable(mar_ctx* c, int32_t max_steps, uint32_t phase_mask) {
  if (!c) return fail(MAR_EINVAL, "context is NULL");
  if (max_steps < 0 || max_steps > MAR_MAX_PROFILE_STEPS) return fail(MAR_ERANGE, "max_steps outside 0..%d", MAR_MAX_PROFILE_STEPS);
  if (c->prof_events) {
    for (int i = 0; i < c->prof_max * 2 * MAR_NUM_PHASES; ++i) (void)hipEventDestroy(c->prof_events[i]);
    free(c->prof_events);
    c->prof_events = nullptr;
  }
  c->prof_max = 0; c->prof_steps = 0; c->prof_mask = phase_mask & ((1u << MAR_NUM_PHASES) - 1u);
  if (max_steps == 0) return MAR_OK;
  const size_t ne = (size_t)max_steps * 2 * MAR_NUM_PHASES;
  c->prof_events = (hipEvent_t*)calloc(ne, sizeof(hipEvent_t));
  if (!c->prof_events) return fail(MAR_ENOMEM, "out of host memory");
  for (size_t i = 0; i < ne; ++i) {
    const hipError_t e = hipEventCreate(&c->prof_events[i]);
    if (e != hipSuccess) {
      for (size_t j = 0; j < i; ++j) (void)hipEventDestroy(c->prof_events[j]);
      free(c->prof_events); c->prof_events = nullptr;
      return hip_fail(e, "event create");
    }
  }
  c->prof_max = max_steps;
  return MAR_OK;
}

extern "C" int mar_profile_read(mar_ctx* c, double* ms, int32_t* steps) {
  if (!c || !ms || !steps) return fail(MAR_EINVAL, "an argument is NULL");
  for (int p = 0; p < MAR_NUM_PHASES; ++p) ms[p] = 0.0;
  *steps = c->prof_steps;
  for (int s = 0; s < c->prof_steps; ++s) {
    hipEvent_t* ev = c->prof_events + (size_t)s * 2 * MAR_NUM_PHASES;
    for (int p = 0; p < MAR_NUM_PHASES; ++p) {
      if (!(c->prof_mask >> p & 1u)) continue;
      hipError_t e = hipEventSynchronize(ev[2 * p + 1]);
      if (e != hipSuccess) return hip_fail(e, "event synchronize");
      float t = 0.f;
      e = hipEventElapsedTime(&t, ev[2 * p], ev[2 * p + 1]);
      if (e != hipSuccess) return hip_fail(e, "event elapsed time");
      ms[p] += t;
    }
  }
  c->prof_steps = 0;
  return MAR_OK;
}
