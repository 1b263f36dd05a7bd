// Contraction passes of the bilinear models (DistMult, ComplEx, Dot) on the 16-bit matrix pipe (gfx950): scores with
// online softmax and the edge-side gradient, the negatives' gradient, and rank counts; and TransE's training passes (k_split_dist).
//
// fp32 precision (F16 = true).  Every operand value is written as v 2^e = hi + lo, both f16 (mar_split.h; one exponent
// per 16 rows puts the largest value just below 2^15), and every product a b is taken as
//     a_hi b_hi + a_lo b_hi + a_hi b_lo
// with 16-bit matrix instructions (fp32 accumulation), which run at 16 times the rate of the fp32 ones.
// hi + lo holds 23-24 significant bits of every value down to 2^-17 of its block's largest (below that an absolute
// 2^-40 of the largest), the dropped product is below 2^-22 of its pair, and the sums are rounded less often than the fp32
// instruction's, so a pass is as accurate as its fp32 form: against 64 bits a dot product of 128 (1,024) normal values is
// off by 1.5e-7 (3.6e-7) of its norm on 16x16x32 and on 32x32x16, with v_mfma_f32_16x16x4_f32 by 2.0e-7 (5.7e-7).
// SPLIT_BF16 (F16 = false): v = hi + lo in bf16 without exponents, the same three products; errors of 2^-16 .. 2^-17
// per product.
//
// fp32 precision: softmax weights are formed as 2^(t - ref) with t = score log2(e) - e_y and an integer reference per stationary row
// that moves only when some t exceeds it by more than 15 (it is then put 8 below the maximum): the weights stay below
// the largest f16, values down to 2^-33 of the largest weight keep their place in hi + lo, moving the reference
// multiplies by powers of two only, and the streamed block's exponent e_y needs no operation of its own.  The
// reference is folded into the statistics at the end (mantissa of the sum, integer in log2 units), so parts merge
// exactly.
// SPLIT_BF16: hi + lo of a weight is off by up to 2^-17 of it, the same in every copy of a repeated negative, while the
// sum keeps the weight itself.  Pass 1's reference is therefore the running maximum (moved when some t exceeds it by more
// than 16 in natural units): a negative that dominates its row has weight 1, which bf16 holds exactly.
//
// Operand images come from the gather.  The images of the matrix a pass streams (pass 1 and 3: the negatives, pass 2:
// the edge-side operands) are copied into LDS by buffer loads that write LDS directly, one tile ahead, in two
// alternating buffers; the stationary rows' fragments are read from their own images once and stay in registers.
//
// All passes but the evaluation of narrow rows (sp_eval_32) run on v_mfma_f32_16x16x32_f16 / bf16: with operands as random as
// these the chip holds its power limit by its clock, and a 16 x 16 block over 32 slots takes 12 % less energy a product than a 32
// x 32 block over 16 (fed from LDS, two waves a SIMD, 1,735 to 1,770 against 1,550 TFLOP/s whatever the order of the products;
// zeros 2,200), and pads less: rows of 100 take 80 instructions of 16 cycles a tile, where 32 x 32 blocks took 45 of 32.  (50,000
// edges, 100 floats: passes 127 and 152 us -> 122 and 138; 100,000, 400 floats: 872 and 1,033 -> 852 and 1,027, where one wave a
// SIMD issues such an instruction every 19.6 cycles; evaluation of 100,000 edges against 1,000 candidates of 400 floats, gather
// included, 995 -> 955.)
// Tried: a tile's weights formed between the next tile's score products, three tiles in LDS: the same cycles; counters in LDS
// in place of the barrier: 8 % slower.
//
// Lane layouts (lane = 16 g + i):
//   v_mfma_f32_16x16x32: A lane holds row i, contraction slots 8 g .. 8 g + 7; B lane holds column i, the same slots; D lane
//   holds column i, register r = row 4 g + r.  Which contraction index a slot stands for is free as long as A and B agree.
//   Score product S^T[y][x] = sum_c Y[y][c] X[x][c], two halves of 16 of the tile's rows y, two of the wave's rows x: A = Y
//   from LDS (16-byte read of row i, columns 32 s + 8 g ..), B = X fragments in registers.
//   Second product O^T[c][x] += sum_y Y[y][c] W[y][x] over the tile's 32 rows: B = W of the lane's own score registers, so slot
//   8 g + j stands for row 4 g + j (j < 4), 16 + 4 g + j - 4 (j >= 4).  A = Y^T by the LDS transpose read
//   (ds_read_b64_tr_b16): within 16 lanes, lane i passes the address of 4 consecutive 16-bit values and receives, as its
//   j-th value, value (i % 4) of lane 4 j + i / 4; with lane i pointing at row 4 g + i / 4, columns 16 cb + 4 (i % 4), it
//   receives Y[4 g + j][16 cb + i].
//   Evaluation then swaps halves between the lane groups g and g ^ 1 (v_permlane16_swap, 8 a tile), so that lane 32 h + m holds
//   half of the tile's rows against the one edge m, whose comparisons it keeps.
//   v_mfma_f32_32x32x16 (sp_eval_32; lane = 32 h + m): A lane holds row m, contraction slots 8 h .. 8 h + 7; B lane
//   holds column m, the same slots; D lane holds column m, register r = row 8 (r / 4) + 4 h + r % 4.
#include <type_traits>

#include "mar_common.h"
#include "mar_split_dev.h"
#include "mar_sort_dev.h"

// Evaluation compares scores with the positive's, and where the two are within rounding of one another the outcome
// belongs to the arithmetic (an edge's own endpoint among the candidates scores what the edge does).  Comparisons
// closer than the passes' error are settled by the fp32 score as v_mfma_f32_16x16x4_f32 forms it -- a chain of fused
// multiply-adds -- in the column order of the fp32 contraction kernels: blocks of 16 columns up to column `chain`, each
// as columns 4 g + i for i = 0..3, g = 0..3; the rest in sequence.  So do blocks that hold an infinity or a NaN.
constexpr int sp_chain(int dk) { return dk <= 52 ? 48 : (dk <= 100 ? 96 : 400); }
template <bool VEC, int UB>
__device__ __forceinline__ float sp_exact_score(const float* __restrict__ q, const float* __restrict__ y, int dim, int chain) {
  float s = 0.f;
  const int nb = (min(chain, dim) + 15) / 16;
  for (int b0 = 0; b0 < nb; b0 += UB) {
    float a[UB][16], c[UB][16];
#pragma unroll
    for (int b = 0; b < UB; ++b) {
#pragma unroll
      for (int i = 0; i < 16; i += 4) {
        const int k = 16 * (b0 + b) + i;
        if (VEC) {
          float4 u = make_float4(0.f, 0.f, 0.f, 0.f), v = u;
          if (b0 + b < nb && k < dim) { u = *reinterpret_cast<const float4*>(y + k); v = *reinterpret_cast<const float4*>(q + k); }
          a[b][i] = u.x; a[b][i + 1] = u.y; a[b][i + 2] = u.z; a[b][i + 3] = u.w;
          c[b][i] = v.x; c[b][i + 1] = v.y; c[b][i + 2] = v.z; c[b][i + 3] = v.w;
        } else {
#pragma unroll
          for (int j = 0; j < 4; ++j) {
            const bool in = b0 + b < nb && k + j < dim;
            a[b][i + j] = in ? y[k + j] : 0.f; c[b][i + j] = in ? q[k + j] : 0.f;
          }
        }
      }
    }
#pragma unroll
    for (int b = 0; b < UB; ++b) {
#pragma unroll
      for (int i = 0; i < 4; ++i) {
#pragma unroll
        for (int g = 0; g < 4; ++g) s = __builtin_fmaf(a[b][4 * g + i], c[b][4 * g + i], s);
      }
    }
  }
  for (int k = chain; k < dim; ++k) s = __builtin_fmaf(y[k], q[k], s);
  return s;
}
// Columns k .. k+3 of a row, zeros from column n on (VEC: n is a multiple of 4).
template <bool VEC> __device__ __forceinline__ float4 sp_row_cols(const float* __restrict__ row, int k, int n) {
  if (VEC) {
    const float4 v = *reinterpret_cast<const float4*>(row + (k < n ? k : 0));
    return k < n ? v : make_float4(0.f, 0.f, 0.f, 0.f);
  }
  float4 v;
  v.x = k < n ? row[k] : 0.f; v.y = k + 1 < n ? row[k + 1] : 0.f; v.z = k + 2 < n ? row[k + 2] : 0.f; v.w = k + 3 < n ? row[k + 3] : 0.f;
  return v;
}
// A whole tile settled: the wave's 32 edges (fp32 operands q0, q1 of edges i and 16 + i; i = lane % 16, G = lane / 16)
// against 32 candidates (rows y0, y1 of candidates i and 16 + i) on v_mfma_f32_16x16x4_f32 itself, in the order above:
// in step j of a 16-column block lane group G holds column 4 G + j of it.  acc[y half][x half]: register r is candidate
// 4 G + r against edge i.  16 matrix instructions and four 16-byte loads a lane per 16 columns.  All 14,951 nodes as
// candidates, 100 floats, half of the rows equal: 1,050 us; one comparison after the other 16,700, as fp32 contraction
// throughout 1,110, no two rows equal 230.  (20,000 edges, 1,000 candidates of 400 floats, half equal: 1,000 us, 25,000
// and 355; 186 without.  One wave per SIMD hides little of the loads.)
template <bool VEC>
__device__ __forceinline__ void sp_exact_tile(const float* __restrict__ q0, const float* __restrict__ q1, const float* __restrict__ y0,
                                              const float* __restrict__ y1, int G, int dim, int dk, int chain, v4f (&acc)[2][2]) {
  const int nb = (min(chain, dim) + 15) / 16;
#pragma unroll 1
  for (int b = 0; b < nb; ++b) {
    const int k = 16 * b + 4 * G;
    const float4 ya = sp_row_cols<VEC>(y0, k, dim), yb = sp_row_cols<VEC>(y1, k, dim);
    const float4 qa = sp_row_cols<true>(q0, k, dk), qb = sp_row_cols<true>(q1, k, dk);
    const float a0[4] = {ya.x, ya.y, ya.z, ya.w}, a1[4] = {yb.x, yb.y, yb.z, yb.w};
    const float b0[4] = {qa.x, qa.y, qa.z, qa.w}, b1[4] = {qb.x, qb.y, qb.z, qb.w};
#pragma unroll
    for (int j = 0; j < 4; ++j) {
      acc[0][0] = mfma16(a0[j], b0[j], acc[0][0]); acc[0][1] = mfma16(a0[j], b1[j], acc[0][1]);
      acc[1][0] = mfma16(a1[j], b0[j], acc[1][0]); acc[1][1] = mfma16(a1[j], b1[j], acc[1][1]);
    }
  }
  if (chain < dim) {                                       // at most four columns are left: one step, a column per lane group
    const int k = chain + G;
    const float a0 = k < dim ? y0[k] : 0.f, a1 = k < dim ? y1[k] : 0.f, b0 = k < dim ? q0[k] : 0.f, b1 = k < dim ? q1[k] : 0.f;
    acc[0][0] = mfma16(a0, b0, acc[0][0]); acc[0][1] = mfma16(a0, b1, acc[0][1]);
    acc[1][0] = mfma16(a1, b0, acc[1][0]); acc[1][1] = mfma16(a1, b1, acc[1][1]);
  }
}

// Up to 16 pairs settled: lanes (G, i) pass the rows of pair i; the lanes with G = i / 4 receive its score.  The loads of UB
// blocks of 16 columns are in flight at once (blocks the rows do not have read the last one again), then comes their chain.
// Rows above 128 floats, all of whose columns lie in the chain's blocks.
template <bool VEC, int UB>
__device__ __forceinline__ float sp_exact_pairs(const float* __restrict__ q, const float* __restrict__ y, int G, int i, int dim, int dk) {
  static_assert(sp_chain(129) >= 400, "no column behind the chain");
  const int whole = dim / 16, part = 16 * whole + 4 * G;   // uniform: whole
  const float4 ap = sp_row_cols<VEC>(y, part, dim), bp = sp_row_cols<true>(q, part, dk);
  v4f acc = (v4f)(0.f);
#pragma unroll 1
  for (int n0 = 0; n0 < whole; n0 += UB) {
    float4 a[UB], b[UB];
#pragma unroll
    for (int n = 0; n < UB; ++n) {
      const int at = 4 * G + 16 * min(n0 + n, whole - 1);
      a[n] = VEC ? *reinterpret_cast<const float4*>(y + at) : make_float4(y[at], y[at + 1], y[at + 2], y[at + 3]);
      b[n] = *reinterpret_cast<const float4*>(q + at);
    }
#pragma unroll
    for (int n = 0; n < UB; ++n) {
      if (n0 + n < whole) {
        acc = mfma16(a[n].x, b[n].x, acc); acc = mfma16(a[n].y, b[n].y, acc);
        acc = mfma16(a[n].z, b[n].z, acc); acc = mfma16(a[n].w, b[n].w, acc);
      }
    }
  }
  acc = mfma16(ap.x, bp.x, acc); acc = mfma16(ap.y, bp.y, acc);
  acc = mfma16(ap.z, bp.z, acc); acc = mfma16(ap.w, bp.w, acc);
  return i & 2 ? (i & 1 ? acc[3] : acc[2]) : (i & 1 ? acc[1] : acc[0]);
}

#ifndef SP_PD
#define SP_PD 2
#endif
#ifndef SP_PG
#define SP_PG 2
#endif
// One step of a score product: the three products of 32 rows' parts (0: rows i, 1: rows 16 + i) with 32 columns'.
// Consecutive instructions share an operand.
template <bool F16> __device__ __forceinline__ void sp_score_step(v8s h0, v8s h1, v8s l0, v8s l1, v8s xh0, v8s xh1, v8s xl0, v8s xl1, v4f (&sc)[2][2]) {
  sc[0][0] = mfma16h<F16>(h0, xl0, sc[0][0]); sc[0][0] = mfma16h<F16>(h0, xh0, sc[0][0]); sc[0][0] = mfma16h<F16>(l0, xh0, sc[0][0]);
  sc[0][1] = mfma16h<F16>(l0, xh1, sc[0][1]); sc[0][1] = mfma16h<F16>(h0, xh1, sc[0][1]); sc[0][1] = mfma16h<F16>(h0, xl1, sc[0][1]);
  sc[1][1] = mfma16h<F16>(h1, xl1, sc[1][1]); sc[1][1] = mfma16h<F16>(h1, xh1, sc[1][1]); sc[1][1] = mfma16h<F16>(l1, xh1, sc[1][1]);
  sc[1][0] = mfma16h<F16>(l1, xh0, sc[1][0]); sc[1][0] = mfma16h<F16>(h1, xh0, sc[1][0]); sc[1][0] = mfma16h<F16>(h1, xl0, sc[1][0]);
}
template <bool F16> __device__ __forceinline__ void sp_tail_step(v8s t0, v8s t1, v8s x0, v8s x1, v4f (&sc)[2][2]) {
  sc[0][0] = mfma16h<F16>(t0, x0, sc[0][0]); sc[0][1] = mfma16h<F16>(t0, x1, sc[0][1]);
  sc[1][1] = mfma16h<F16>(t1, x1, sc[1][1]); sc[1][0] = mfma16h<F16>(t1, x0, sc[1][0]);
}
__device__ __forceinline__ float sum_of_squares(v8s v) {
  const v8h f = __builtin_bit_cast(v8h, v);
  float n2 = 0.f;
#pragma unroll
  for (int i = 0; i < 8; ++i) n2 += (float)f[i] * (float)f[i];
  return n2;
}

// Waves per SIMD = workgroups per CU: pass 3 keeps no output accumulators.
constexpr int sp_waves(int nk, int pass) { return pass == 3 ? (nk <= 8 ? 3 : (nk <= 16 ? 2 : 1)) : (nk <= 8 ? 2 : 1); }

// ---------------------------------------------------------------------------- evaluation -----
// What a workgroup takes of all units' tiles, counted one unit after the other: a unit's part, or (rows above 256 floats) an
// equal share wherever it ends, for counts need no merging.  As in flash_unit an XCD's workgroups take neighbouring shares.
constexpr bool sp_shares(int nk) { return nk > 16; }
template <typename A> __device__ __forceinline__ bool eval_tiles(const A& a, int64_t& at, int64_t& at_end) {
  const int ntiles = (a.N + SP_TY - 1) / SP_TY;
  if (!a.share) {
    FlashUnit u;
    if (!flash_unit(a, u)) return false;
    at = (int64_t)u.unit * ntiles + u.part * a.tps;
    at_end = min(at + a.tps, (int64_t)(u.unit + 1) * ntiles);
    return true;
  }
  const int p = (int)(blockIdx.x & 7) * (int)(gridDim.x >> 3) + (int)(blockIdx.x >> 3);
  at = sp_share_border(a.share, a.share_rest, ntiles, p);
  at_end = sp_share_border(a.share, a.share_rest, ntiles, p + 1);
  return at < at_end;
}
typedef const __attribute__((address_space(4))) FlashArgs KernelArgs;

// Rows up to 96 floats, and from 105 to 112, take their scores in one 32 x 32 block over 16 columns a step, whose accumulators hold
// a lane's one edge as they are: the comparisons, which take as long as the products there, do without the 8 exchanges that 16 x 16
// blocks need.  Wider rows are bound by the products, which 16 x 16 x 32 forms at less energy (7 blocks: unless the last one, more
// than half full, takes a second step).  10,000 edges, all 14,951 nodes, 16 x 16 / 32 x 32 blocks, us a call, ten in a row: 32
// floats 153 / 140, 64: 181 / 173, 96: 216 / 209, 100: 231 / 227 (thirty in a row 216 / 222: the chip then holds its power limit),
// 112: 246 / 230, 128: 253 / 256; a tenth of the rows small: 166 / 151, 204 / 193, 259 / 253, 264 / 260, 295 / 265, 308 / 300; 60,000
// edges, 1,000 candidates: 78 / 76, 102 / 99, 134 / 137, 145 / 147, 159 / 153, 160 / 161.
constexpr bool sp_eval_32(int nk, int dk) { return nk <= 6 || (nk == 7 && dk > 16 * (nk - 1) + 8); }

// PASS 3: counts the negatives that score above the positive; ranks start at 1 and the parts of a stripe add their counts.
template <int NK, bool B32>                                // B32: 32 x 32 blocks, NK steps of 16 columns, no tail
__device__ __forceinline__ void split_eval() {
  typedef SplitGeom<NK> SG;
  constexpr int UNITS = SG::UNITS, PA = SG::PA, PLANE = SG::PLANE, IMG = SG::IMG;
  constexpr int TY = SP_TY;
  constexpr int NCW = (SG::NCH + 3) / 4;                   // 1 KB pieces of an image per wave
  constexpr int NS = NK / 2;                               // whole steps of 32 columns
  constexpr bool SHARES = sp_shares(NK);
  constexpr bool TAIL = !B32 && NK % 2 != 0;              // and 16 columns more
  extern __shared__ __attribute__((aligned(256))) char smem[];

  KernelArgs* args = (KernelArgs*)__builtin_amdgcn_kernarg_segment_ptr();
  int64_t at, at_end;
  if (!eval_tiles(*args, at, at_end)) return;
  do {                                                     // one piece: tiles t_begin .. ntiles - 1 of one unit
  // the arguments are read again, and the lane's coordinates formed again, for every piece: kept across them they spill
  int tid = threadIdx.x;
  if (SHARES) asm volatile("" : "+s"(args), "+v"(tid));
  KernelArgs& a = *args;
  const int lane = tid & 63, wave = tid >> 6;
  const int g = lane >> 4, i = lane & 15;                  // of the matrix instructions
  const int h = lane >> 5, m = lane & 31;                  // of the comparisons: edge m, half of the tile's rows
  const int n_y = a.N, ntiles_all = (n_y + TY - 1) / TY;  // streamed rows and their tiles
  const int unit = (int)(at / ntiles_all), t_begin = (int)(at - (int64_t)unit * ntiles_all);
  const int ntiles = (int)min((int64_t)ntiles_all, t_begin + (at_end - at));
  at += ntiles - t_begin;
  const int cs = unit / a.nstripes, stripe = unit % a.nstripes, side = cs & 1, c = cs >> 1;
  const int n_x = min(a.S, a.n - c * a.S);                // stationary rows: edges in this chunk
  if (stripe * SP_SR >= n_x) continue;
  const size_t q_base = (size_t)side * a.B + (size_t)c * a.S;        // first Q row of the chunk
  const int dk = a.dk;

  const int wave_s = __builtin_amdgcn_readfirstlane(wave);
  // ---- images of the streamed rows, copied into LDS one tile ahead; a register load issued behind the copies is the
  // fence (memory operations of a wave complete in order): once its value is there the image is in LDS.  The fence is
  // the load of the tile's two exponents and of its blocks' norms.
  const char* ybase = a.yimg + (size_t)cs * a.yimg_tiles * IMG;
  const BufRsrc expsrc = buf_rsrc(a.yexp + (size_t)cs * a.yimg_tiles * 2, (uint32_t)a.yimg_tiles * 8);
  float2 ye_next = make_float2(0.f, 0.f), yn_next = make_float2(0.f, 0.f);
  const BufRsrc normsrc = buf_rsrc(a.ynorm + (size_t)cs * a.yimg_tiles * SP_NORMS, (uint32_t)a.yimg_tiles * (SP_NORMS * 4));
  int token = 0;
  auto dma_piece = [&](int t, int buf, int q) {            // piece q of this wave of tile t into buffer `buf`
    const v4i ywords = buf_words(ybase + (size_t)t * IMG, IMG);
    const int pc = 4 * q + wave_s;
    if (pc < SG::NCH) buf_load4_to_lds(ywords, lds_address_b(smem) + buf * IMG + pc * 1024, lane * 16, pc * 1024, token);
  };
  auto dma_fence = [&](int t) {
    ye_next = buf_load2(expsrc, token, t * 8);
    yn_next = buf_load2(normsrc, token, t * (SP_NORMS * 4));
  };
  auto dma_land = [&]() { asm volatile("" : "+v"(ye_next.x), "+v"(ye_next.y)); };
  // The first tile is on its way while the stationary fragments are fetched.
  if (SHARES) __syncthreads();                             // every wave is done with the piece before
#pragma unroll
  for (int q = 0; q < NCW; ++q) dma_piece(t_begin, 0, q);
  dma_fence(t_begin);

  // ---- stationary fragments and their tail, as in split_pass; 32 x 32 blocks: xh[s & 1][s / 2] are columns 16 s + 8 h .. +7 of row m
  const int x0 = stripe * SP_SR + wave_s * 32, x = x0 + m;   // the wave's first row, the lane's
  const bool xv = x < n_x;
  const size_t xtile = (size_t)cs * a.ximg_tiles + stripe * (SP_SR / TY) + wave_s;
  const int swz = 16 * sp_swizzle(UNITS, B32 ? m : i);    // of row m, or of rows i and 16 + i, of a tile, in bytes
  const v8s zero8 = {0, 0, 0, 0, 0, 0, 0, 0};
  constexpr int NF = B32 ? (NK + 1) / 2 : NS;
  v8s xh[2][NF], xl[2][NF], xt[2][2];
  const bool tail2 = TAIL && NK > 7 && dk > 16 * (NK - 1) + 8;   // uniform; 7 blocks: such rows take 32 x 32 blocks
#pragma unroll
  for (int b = 0; b < 2; ++b) {
    const bool in = B32 ? xv : x0 + 16 * b + i < n_x;
    const char* xrow = a.ximg + xtile * IMG + (B32 ? m : 16 * b + i) * PA;
#pragma unroll
    for (int s = 0; s < NF; ++s) {
      const int col = (B32 ? 64 * s + 32 * b + 16 * h : 64 * s + 16 * g) ^ swz;
      xh[b][s] = xl[b][s] = zero8;
      if (in && (!B32 || 2 * s + b < NK)) {
        xh[b][s] = *reinterpret_cast<const v8s*>(xrow + col);
        xl[b][s] = *reinterpret_cast<const v8s*>(xrow + PLANE + col);
      }
    }
    xt[b][0] = xt[b][1] = zero8;
    if (TAIL && in) {
      const int unit = 64 * NS + (tail2 ? 16 * (g & 1) : 0);
      if (tail2 || g < 3) xt[b][0] = *reinterpret_cast<const v8s*>(xrow + (!tail2 && g == 2 ? PLANE : 0) + (unit ^ swz));
      if (tail2 && g < 2) xt[b][1] = *reinterpret_cast<const v8s*>(xrow + PLANE + (unit ^ swz));
    }
  }
  float ex = 0.f;                                         // exponent of the row's block
  bool xbad = false;
  if (xv) {
    ex = a.xexp[xtile * 2 + (m >> 4)];
    xbad = ex > 0.5f * SP_NONFINITE;
    if (xbad) ex -= SP_NONFINITE;
  }
  // A comparison is close if the score is within sqrt(dk) (2^-23 |q| + 2^-25) |n| of the positive's, q and n
  // scaled by their blocks' exponents, |n| the largest of the block.  The rounding errors of a chain of dk steps are
  // independent and each below 2^-24 |q| |n| (the partial sums are), 0.3 of that on average: the first term is seven
  // standard deviations where all products have one sign, and ten times that where they do not.  hi + lo holds a value to
  // 2^-24 of itself and no better than 2^-25: over a row that is the second term, which matters where q is far below its
  // block's largest row (or its block's exponent at the limit); for n it lies inside the first, the block's |n| being
  // 2^14 at least.  A zero row's scores are exactly zero.
  float posx = 0.f, tolx = 0.f;
  const float* qrow = nullptr;
  int* const pend = reinterpret_cast<int*>(smem + 2 * IMG) + tid;
  int npend = 0;                                           // pending candidates; + SP_FULL: no more are taken
  float n2;
  {
    float q[2] = {0.f, 0.f};
#pragma unroll
    for (int b = 0; b < 2; ++b) {
#pragma unroll
      for (int s = 0; s < NF; ++s) q[b] += sum_of_squares(xh[b][s]);
      if (TAIL && g < (tail2 ? 2 : 1)) q[b] += sum_of_squares(xt[b][0]);
      if (!B32) q[b] += __shfl_xor(q[b], 16);
      q[b] += __shfl_xor(q[b], 32);
    }
    n2 = B32 ? q[0] + q[1] : (g & 1 ? q[1] : q[0]);
  }
  if (xv) { posx = a.pos[(size_t)c * a.S + x]; qrow = a.qrows + (q_base + x) * dk; }
  bool zero = n2 == 0.f;
  if (xv && zero) {                                      // or merely below the f16 range
    for (int k = 4 * h; k < dk; k += 8) {
      const float4 q = *reinterpret_cast<const float4*>(qrow + k);
      zero = zero && q.x == 0.f && q.y == 0.f && q.z == 0.f && q.w == 0.f;
    }
  }
  zero = (__shfl_xor(zero ? 1 : 0, 32) & (zero ? 1 : 0)) != 0;
  tolx = zero ? 0.f : sqrtf((float)dk) * (0x1p-23f * sqrtf(n2) + 0x1p-25f);
  xbad |= !(fabsf(posx) <= 3.4028234663852886e38f);     // no difference to a positive score outside the range
  const int32_t* const cand = (side == MAR_SIDE_DST ? a.neg_dst : a.neg_src) + (size_t)c * a.N;   // ids of the streamed rows
  int own = -1, nown = 0;                                  // the replaced endpoint's id, how often it came up close
  if (xv) own = (side == MAR_SIDE_DST ? a.dst : a.src)[(size_t)c * a.S + x];
  // All lanes of the wave: candidates of the tile at y0 that score above this lane's edge, settled as a whole (in
  // the lanes of the wave's first half).
  auto exact_tile = [&](int y0) -> int {
    int ln = lane;
    asm volatile("" : "+v"(ln));                          // what follows is rare: nothing of it is kept across tiles
    const int i = ln & 15, G = ln >> 4;
    const float* qr = a.qrows + q_base * dk;
    v4f acc[2][2];
#pragma unroll
    for (int k = 0; k < 4; ++k) acc[k >> 1][k & 1] = (v4f)(0.f);
    const float *q0 = qr + (size_t)min(x0 + i, n_x - 1) * dk, *q1 = qr + (size_t)min(x0 + 16 + i, n_x - 1) * dk;
    const float *r0 = a.table + (size_t)cand[min(y0 + i, n_y - 1)] * a.dim, *r1 = a.table + (size_t)cand[min(y0 + 16 + i, n_y - 1)] * a.dim;
    if (a.dim % 4 == 0) sp_exact_tile<true>(q0, q1, r0, r1, G, a.dim, dk, sp_chain(dk), acc);
    else sp_exact_tile<false>(q0, q1, r0, r1, G, a.dim, dk, sp_chain(dk), acc);
    int above[2] = {0, 0};
#pragma unroll
    for (int xb = 0; xb < 2; ++xb) {
      const float p = __shfl(posx, 16 * xb + i);
#pragma unroll
      for (int k = 0; k < 8; ++k) above[xb] += y0 + 16 * (k >> 2) + 4 * G + (k & 3) < n_y && acc[k >> 2][xb][k & 3] > p ? 1 : 0;
      above[xb] += __shfl_xor(above[xb], 16);
      above[xb] += __shfl_xor(above[xb], 32);
    }
    return h == 0 ? ((G & 1) ? above[1] : above[0]) : 0;
  };

  int cnt = 0;
  auto row_of = [&](int v) { return B32 ? 8 * (v >> 2) + 4 * h + (v & 3) : 16 * (v >> 3) + 8 * h + (v & 7); };   // of a lane's pair v within the tile

  // Where a lane reads in a tile's buffer (as in split_pass)
  constexpr int GU = sp_group(UNITS);
  const int fofs = (B32 ? m : i) * PA + ((16 * (B32 ? h : g)) ^ swz);
  const int tfofs = i * PA + (tail2 ? (g & 2 ? PLANE : 0) + ((64 * NS + 16 * (g & 1)) ^ swz) : (g == 1 ? PLANE : 0) + ((64 * NS) ^ swz));
  auto at = [](unsigned base, int byte) { return (base ^ (byte % (16 * GU))) + byte / (16 * GU) * (16 * GU); };
  dma_land();
  __syncthreads();
  for (int t = t_begin; t < ntiles; ++t) {
    const int buf = (t - t_begin) & 1;
    const int bofs = buf * IMG;
    const bool has_next = t + 1 < ntiles;                  // uniform
    const float2 ye = ye_next, yn = yn_next;
    const int y0 = t * TY;
    const bool masked = y0 + TY > n_y;

    // -- scores as in split_pass; then lane groups g and g ^ 1 exchange halves, so that lane (h, m) holds its one edge's:
    // sacc[v] = row row_of(v).  32 x 32 blocks need no exchange.
    float sacc[16];
    if constexpr (B32) {
      v16f sc = (v16f)(0.f);
      constexpr int PD = NK < 2 * SP_PD ? NK : 2 * SP_PD;
      v8s fh[PD], fl[PD];
      const unsigned fb = lds_address_b(smem) + bofs + fofs;   // smem lies at a whole group: exclusive or on addresses
      auto read_step = [&](int s) {
        const unsigned p = at(fb, 32 * s);
        fh[s % PD] = lds_read16(p); fl[s % PD] = lds_read16(p + PLANE);
      };
#pragma unroll
      for (int s = 0; s < PD; ++s) read_step(s);
#pragma unroll
      for (int s = 0; s < NK; ++s) {
        const v8s yh = fh[s % PD], yl = fl[s % PD];
        if (s + PD < NK) read_step(s + PD);
        sc = mfma32h(yl, xh[s & 1][s / 2], sc); sc = mfma32h(yh, xl[s & 1][s / 2], sc); sc = mfma32h(yh, xh[s & 1][s / 2], sc);
        if (has_next) {                                    // the next tile's pieces, as below
#pragma unroll
          for (int q = s * NCW / NK; q < (s + 1) * NCW / NK; ++q) dma_piece(t + 1, buf ^ 1, q);
          if (s == NK - 1) dma_fence(t + 1);
        }
        __builtin_amdgcn_sched_barrier(0);                 // keeps the reads PD steps ahead of their use
      }
      if (masked) {                                        // the chunk's last, partial tile (uniform): rows beyond it weigh nothing
#pragma unroll
        for (int v = 0; v < 16; ++v) sc[v] = y0 + row_of(v) < n_y ? sc[v] : -__builtin_inff();
      }
#pragma unroll
      for (int v = 0; v < 16; ++v) sacc[v] = sc[v];
    } else {
      v4f sc[2][2];
      sc[0][0] = sc[0][1] = sc[1][0] = sc[1][1] = (v4f)(0.f);
      constexpr int PD = NS < SP_PD ? NS : SP_PD;
      v8s fh[PD][2], fl[PD][2];
      const unsigned fb = lds_address_b(smem) + bofs + fofs;
      auto read_step = [&](int s, v8s (&vh)[2], v8s (&vl)[2]) {
        const unsigned p = at(fb, 64 * s);
#pragma unroll
        for (int r = 0; r < 2; ++r) { vh[r] = lds_read16(p + 16 * r * PA); vl[r] = lds_read16(p + 16 * r * PA + PLANE); }
      };
#pragma unroll
      for (int s = 0; s < PD; ++s) read_step(s, fh[s], fl[s]);
#pragma unroll
      for (int s = 0; s < NS; ++s) {
        const v8s h0 = fh[s % PD][0], h1 = fh[s % PD][1], l0 = fl[s % PD][0], l1 = fl[s % PD][1];
        if (s + PD < NS) read_step(s + PD, fh[s % PD], fl[s % PD]);
        sp_score_step<true>(h0, h1, l0, l1, xh[0][s], xh[1][s], xl[0][s], xl[1][s], sc);
        // the next tile's pieces are issued between the steps: a burst of them holds the wave at the memory pipeline's
        // queue (rows of 400: a pass 1075 us with the copies at the tile's start, 915 spread, 810 without any)
        if (has_next) {
#pragma unroll
          for (int q = s * NCW / NS; q < (s + 1) * NCW / NS; ++q) dma_piece(t + 1, buf ^ 1, q);
          if (s == NS - 1) dma_fence(t + 1);
        }
        __builtin_amdgcn_sched_barrier(0);                 // keeps the reads PD steps ahead of their use
      }
      if (TAIL) {
        const unsigned p = lds_address_b(smem) + bofs + tfofs;
        sp_tail_step<true>(lds_read16(p), lds_read16(p + 16 * PA), xt[0][0], xt[1][0], sc);
        if (tail2) {                                       // its hi fragments again (groups 2, 3 meet zeros)
          const unsigned p2 = lds_address_b(smem) + bofs + i * PA + ((64 * NS + 16 * (g & 1)) ^ swz);
          sp_tail_step<true>(lds_read16(p2), lds_read16(p2 + 16 * PA), xt[0][1], xt[1][1], sc);
        }
      }
      if (masked) {
#pragma unroll
        for (int k = 0; k < 8; ++k) {
          if (y0 + 16 * (k >> 2) + 4 * g + (k & 3) >= n_y) sc[k >> 2][0][k & 3] = sc[k >> 2][1][k & 3] = -__builtin_inff();
        }
      }
      asm volatile("" : "+v"(sc[0][0]), "+v"(sc[0][1]), "+v"(sc[1][0]), "+v"(sc[1][1]));   // exchanged where they lie, without moves
#pragma unroll
      for (int k = 0; k < 8; ++k) {
        const auto w = __builtin_amdgcn_permlane16_swap(__float_as_uint(sc[k >> 2][0][k & 3]), __float_as_uint(sc[k >> 2][1][k & 3]), false, false);
        sacc[8 * (k >> 2) + (k & 3)] = __uint_as_float(w[0]);
        sacc[8 * (k >> 2) + 4 + (k & 3)] = __uint_as_float(w[1]);
      }
    }
    // -- scale of the two 16-row blocks: score = sacc 2^-(ex + ey); never 0, or a masked row's -inf would become NaN
    // (two blocks at the largest exponent: scores below 2^-100 either way)
    const bool ybad = ye.x > 0.5f * SP_NONFINITE || ye.y > 0.5f * SP_NONFINITE;
    const float e0 = ye.x > 0.5f * SP_NONFINITE ? ye.x - SP_NONFINITE : ye.x;
    const float e1 = ye.y > 0.5f * SP_NONFINITE ? ye.y - SP_NONFINITE : ye.y;
    const float k0 = __builtin_ldexpf(1.f, max(-140, min(126, -(int)(ex + e0))));
    const float k1 = __builtin_ldexpf(1.f, max(-140, min(126, -(int)(ex + e1))));
    bool settle = __any(ybad || xbad);                     // uniform over the wave: the tile is settled as a whole
    int ct = 0;
    if (!settle) {
      float near0 = __builtin_inff(), near1 = near0;
#pragma unroll
      for (int v = 0; v < 16; ++v) {
        const float dif = __builtin_fmaf(sacc[v], v < 8 ? k0 : k1, -posx);
        ct += dif > 0.f ? 1 : 0;
        if (v < 8) near0 = fminf(near0, fabsf(dif)); else near1 = fminf(near1, fabsf(dif));
      }
      // scores at the ends of the exponents' range: every comparison is close
      const float t0 = tolx * (fabsf(ex + e0) > 126.f ? __builtin_inff() : k0), t1 = tolx * (fabsf(ex + e1) > 126.f ? __builtin_inff() : k1);
      const float tol0 = t0 * yn.x, tol1 = t1 * yn.y;
      if (__any(xv && (near0 < tol0 || near1 < tol1))) {
        // An edge's close candidates are mostly its own endpoint, as often as the candidates hold it: it is counted, and
        // compared once at the end, like up to SP_PEND others.  Where there are more the tile is settled as a whole.
        // (20,000 edges, 1,000 candidates of 100 floats drawn by degree from a power law: 78 to 85 us, 1,200 to 3,100 with
        // every copy compared, 91 as fp32 contraction, 58 for uniform candidates.)
        // lane i: id and norm of the tile's row i % TY, on their way while the comparisons are made again (unless most tiles of
        // this wave are settled as a whole)
        int id_t = 0;
        float nrm = 0.f;
        auto look = [&] { id_t = cand[min(y0 + lane % TY, n_y - 1)]; nrm = buf_load1(normsrc, (2 + lane % TY) * 4, t * (SP_NORMS * 4)); };
        const bool early = !__any(npend >= SP_FULL);
        if (early) look();
        unsigned close = 0u, same = 0u;                  // bit v: pair v is close / is with the own endpoint
        float p = posx;
        asm volatile("" : "+v"(p));                      // the comparisons are made again, one after the other: kept, their lane
                                                         // masks would take 32 scalar registers
#pragma unroll
        for (int v = 15; v >= 0; --v) {
          const float dif = __builtin_fmaf(sacc[v], v < 8 ? k0 : k1, -p);
          const bool cl = fabsf(dif) < (v < 8 ? tol0 : tol1);
          close = close + close + (cl ? 1u : 0u);
          ct -= cl && dif > 0.f ? 1 : 0;
          asm volatile("" : "+v"(close), "+v"(ct));
        }
        if (!xv) close = 0u;
        // Several in a lane, or again and again: most are copies of the own endpoint; the others are looked at with their
        // own norms in place of the block's largest (2^-25 of q is at most a quarter of tolx).
        settle = __any(close != 0u && npend >= SP_FULL);
        const bool many = __any((close & (close - 1u)) != 0u || (close != 0u && npend >= 2));
        if (!settle && !many && close) {                 // one at most: by its place, without a look at its id
          const int v = __ffs((int)close) - 1;
          pend[256 * npend] = ~(y0 + row_of(v));
          pend[256 * (SP_PEND + npend++)] = 1;
        }
        if (!settle && many) {
          if (!early) look();
#pragma unroll
          for (int v = 0; v < 16; ++v) {
            same |= __shfl(id_t, row_of(v)) == own ? 1u << v : 0u;
            asm volatile("" : "+v"(same));
          }
          same &= close;
          if (__any((close & ~same) != 0u)) {
#pragma unroll
            for (int v = 0; v < 16; ++v) {
              const float dif = __builtin_fmaf(sacc[v], v < 8 ? k0 : k1, -p), nv = __shfl(nrm, row_of(v));
              const bool far = ((close & ~same) >> v & 1u) && !(fabsf(dif) < (v < 8 ? t0 : t1) * (nv + 0.25f) && nv >= 0.f);
              close &= far ? ~(1u << v) : ~0u;
              ct += far && dif > 0.f ? 1 : 0;
              asm volatile("" : "+v"(close), "+v"(ct));
            }
          }
          unsigned rest = close & ~same, times = 0u;     // times: 5 bits per pending candidate, how often the tile has it
          int npend_t = npend, nown_t = nown + __popc(same);
          bool over = rest != 0u && npend >= SP_PEND;
          settle = __any(over);
          if (!settle) {
            for (; rest; rest &= rest - 1u) {
              const int v = __ffs((int)rest) - 1, id = cand[y0 + row_of(v)];
              int j = npend_t;
#pragma unroll
              for (int q = SP_PEND - 1; q >= 0; --q) j = q < npend_t && pend[256 * q] == id ? q : j;
              const bool put = id != own && j < SP_PEND;
              if (put && j == npend_t) { pend[256 * j] = id; pend[256 * (SP_PEND + j)] = 0; ++npend_t; }
              times += put ? 1u << (5 * j) : 0u;
              nown_t += id == own ? 1 : 0;
              over |= id != own && !put;
            }
            settle = __any(over);
            if (over) npend += SP_FULL;                  // so many more at once: later tiles are settled without another look
          }
          if (!settle) {
            nown = nown_t;
            npend = npend_t;
            for (int j = 0; times; ++j, times >>= 5) pend[256 * (SP_PEND + j)] += (int)(times & 31u);
          }
        }
      }
    }
    cnt += settle ? exact_tile(y0) : ct;
    if (has_next) {
      dma_land();
      __syncthreads();                                     // tile t + 1 is in LDS; every wave is done with tile t
    }
  }

  // ---- epilogue
  // What is pending.  Up to 128 floats every lane settles its own, a chain of multiply-adds.  Wider rows 16 pairs of the wave at a
  // time: every lane with something left offers its next one, the first 16 are taken; each lane by itself, a row's loads eight
  // blocks at a time, was several times a load's latency at the end of every workgroup: 20,000 edges, 1,000 candidates of 400
  // floats 222 -> 206 us, gather included; 900 edges, 3,000 candidates 54 -> 43.  (Up to 128 floats a row is two loads' latencies
  // either way and most lanes have their own endpoint to settle, four times 16: candidates of 100 floats by degree 88 -> 95.)
  int ln = lane;
  asm volatile("" : "+v"(ln));                            // lane coordinates formed afresh: kept across the tiles they would spill
  const int gl = ln >> 4, il = ln & 15, xe = x0 + (ln & 31);
  const int items = npend % SP_FULL;
  if constexpr (NK <= 8) {
    const float* qrow = a.qrows + (q_base + min(xe, n_x - 1)) * dk;
    for (int item = nown ? -1 : 0; item < items; ++item) {
      const int e = item < 0 ? own : pend[256 * item], id = e < 0 ? cand[~e] : e;
      const float* yrow = a.table + (size_t)id * a.dim;
      const float s = a.dim % 4 == 0 ? sp_exact_score<true, 4>(qrow, yrow, a.dim, sp_chain(dk)) : sp_exact_score<false, 2>(qrow, yrow, a.dim, sp_chain(dk));
      if (s > posx) cnt += item < 0 ? nown : pend[256 * (SP_PEND + item)];
    }
  } else {
    constexpr int UB = NK > 16 ? NK : (NK + 1) / 2;        // as many blocks as the registers hold
    for (int item = nown ? -1 : 0; const unsigned long long left = __builtin_amdgcn_ballot_w64(item < items);) {
      const int slot = __builtin_amdgcn_mbcnt_hi((unsigned)(left >> 32), __builtin_amdgcn_mbcnt_lo((unsigned)left, 0));
      const bool take = item < items && slot < 16;
      int id = own;
      if (item >= 0 && item < items) {
        const int e = pend[256 * item];
        id = e < 0 ? cand[~e] : e;
      }
      // lane `slot` learns who holds pair `slot`; pairs beyond the last are the first again
      const int who = __builtin_amdgcn_ds_permute(4 * (take ? slot : 63), ln);
      const int from = __shfl(who, il < __popcll(left) ? il : 0);
      const float* yrow = a.table + (size_t)__shfl(id, from) * a.dim;
      const float* qrow = a.qrows + (q_base + x0 + (from & 31)) * dk;
      const float s = __shfl(a.dim % 4 == 0 ? sp_exact_pairs<true, UB>(qrow, yrow, gl, il, a.dim, dk)
                                            : sp_exact_pairs<false, UB>(qrow, yrow, gl, il, a.dim, dk), 16 * ((slot & 15) >> 2) + (slot & 15));
      if (take) {
        if (s > posx) cnt += item < 0 ? nown : pend[256 * (SP_PEND + item)];
        ++item;
      }
    }
  }
  cnt += __shfl_xor(cnt, 32);
  if (ln < 32 && xe < n_x && cnt) atomicAdd((side == MAR_SIDE_DST ? a.rank_dst : a.rank_src) + (size_t)c * a.S + xe, cnt);
  } while (SHARES && at < at_end);
}

// ------------------------------------------------------------------------ the training passes -----
// Squared norm of a row of TransE as the passes use it; none above 1e37, so that a squared distance stays finite (a NaN makes every
// pair of the row a near one, whose distance is formed from the rows).
__device__ __forceinline__ float dist_norm(float n2) { return n2 < 1e37f ? n2 : __builtin_nanf(""); }

// PASS 1: scores, online softmax and gQ = P K for 128 edges of one chunk-side (32 per wave) against the chunk's
// negatives.
// PASS 2: gK = P^T Q for 128 negatives of one chunk-side against the chunk's edges, with the scores computed again and
// P = exp(score - lse) from the finished log-sum-exp.  Writing the weights out and reading them back costs 8 bytes of
// memory traffic per pair, computing a score again 6 d 16-bit flops: at this matrix rate the second is cheaper.
// TransE: a row in fp32 (EDGE: of the edge-side operands; else a negative's, of the node table).  Formed from
// arguments that the compiler cannot see through: what the addresses take would otherwise be kept across the tiles.
template <bool EDGE> struct DistRow {
  const float* row;
  const float* shift;
  int left;
  __device__ __forceinline__ DistRow(int cs, int x) {
    KernelArgs* args = (KernelArgs*)__builtin_amdgcn_kernarg_segment_ptr();
    asm volatile("" : "+s"(args));
    KernelArgs& a = *args;
    const int side = cs & 1, c = cs >> 1;
    if (EDGE) row = a.qrows + ((size_t)side * a.B + (size_t)c * a.S + x) * a.dk;
    else row = a.table + (size_t)((side == MAR_SIDE_DST ? a.neg_dst : a.neg_src) + (size_t)c * a.N)[x] * a.dim;
    left = EDGE ? a.dk : a.dim;
    shift = a.shift;
  }
  __device__ __forceinline__ float4 cols(int k) const { return sp_row_cols<EDGE>(row, k, left); }
  __device__ __forceinline__ float4 shifted(int k) const { // as the images have it (k below 16 NK)
    const float4 v = cols(k), m = *reinterpret_cast<const float4*>(shift + k);
    return make_float4(v.x - m.x, v.y - m.y, v.z - m.z, v.w - m.w);
  }
};

// Close pairs: 2^-15 of the root of their norms' sum, squared.
#define SP_CLOSE 0x1p-30f
// DIST (TransE): the score is -|x - y|, its square expanded as |x|^2 + |y|^2 - 2 x.y with the norms in fp32.  Pairs for which the
// expansion cancels (below 2^-8 of the norms' sum) are formed from the differences of their columns (rare in training; a wave
// without one skips the loop).  The second product then runs with W = softmax weight / distance, less x times the sum of the W.
// A close pair (SP_CLOSE) stays out of the product: its weight over its distance would leave the others' no bits of the f16 range, and
// W y - W x cancels.  Its lane keeps it, two at most (further ones go through the product), and the end adds W (y - x) from the rows.
// CARRY: the first a.carried workgroups do a piece of the row order (small batches).
template <int NK, int PASS, bool F16, bool DIST, bool CARRY>
__device__ __forceinline__ void split_pass(const FlashArgs& a) {
  static_assert(F16 || !DIST, "TransE's operands are f16 pairs");
  typedef SplitGeom<NK> SG;
  constexpr int UNITS = SG::UNITS, PA = SG::PA, PLANE = SG::PLANE, IMG = SG::IMG;
  constexpr int TY = SP_TY;
  constexpr int NCW = (SG::NCH + 3) / 4;                   // 1 KB pieces of an image per wave
  constexpr int NS = NK / 2;                               // whole steps of 32 columns of the score product
  constexpr bool TAIL = NK % 2 != 0;                       // and 16 columns more
  constexpr int NO = NK;                                   // 16-column output blocks
  constexpr float LOG2E = 1.44269504088896341f;
  extern __shared__ __attribute__((aligned(16))) char smem[];
  if (CARRY && __builtin_expect((int)blockIdx.x < a.carried, 0)) { sort_job<PASS == 1 ? MAR_SORT_SCATTER : MAR_SORT_SCATTER | MAR_SORT_RANKS>(a.sort, reinterpret_cast<uint32_t*>(smem)); return; }
  float* const aux_all = reinterpret_cast<float*>(smem + 2 * IMG);   // PASS 2: [2][2][TY] log-sum-exp of the tile's edges, log2 units
  float* const nrm_all = aux_all + 4 * TY;                // DIST: [2][TY] squared norms of the tile's rows

  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const int g = lane >> 4, i = lane & 15;
  FlashUnit u;
  if (!flash_unit(a, u)) return;
  const int cs = u.cs, side = cs & 1, c = cs >> 1;
  const int ne = min(a.S, a.n - c * a.S);                 // edges in this chunk
  const int n_x = PASS == 2 ? a.N : ne;                   // stationary rows
  const int n_y = PASS == 2 ? ne : a.N;                   // streamed rows
  if (u.stripe * SP_SR >= n_x) return;
  const size_t q_base = (size_t)side * a.B + (size_t)c * a.S;        // first Q row of the chunk
  const int dk = a.dk;
  const int wave_s = __builtin_amdgcn_readfirstlane(wave);
  float neg1 = -1.f;
  asm volatile("" : "+v"(neg1));

  // ---- stationary fragments from the rows' own images: column b of lane (g, i) is row x0 + 16 b + i, its slots of step s
  // are columns 32 s + 8 g .. +7
  const int x0 = u.stripe * SP_SR + wave * 32;
  const size_t xtile = (size_t)cs * a.ximg_tiles + u.stripe * (SP_SR / TY) + wave_s;
  const int swz = 16 * sp_swizzle(UNITS, i);              // of rows i and 16 + i of a tile, in bytes
  const v8s zero8 = {0, 0, 0, 0, 0, 0, 0, 0};
  // DIST, widest rows: the fragments of the last XL steps lie in LDS, each lane's own (its registers would spill; 400 floats: 351 of them)
  constexpr int XL = DIST ? sp_dist_lds_steps(NK) : 0;
  char* const xlds = smem + SG::LDS_BYTES + 2 * TY * 4 + threadIdx.x * 16;   // [4 XL][256] 16-byte units
  // DIST: a lane's close pairs, added at the end: streamed row and column block (-1: none), weight, its reference: [3][2][256]
  int* const close_id = reinterpret_cast<int*>(smem + SG::LDS_BYTES + 2 * TY * 4 + XL * 4 * 4096);
  // formed anew where it is rarely used: kept across the tiles it would cost a register
  const auto fresh_lane = []() { int l = __builtin_amdgcn_mbcnt_hi(~0u, __builtin_amdgcn_mbcnt_lo(~0u, 0u)); asm volatile("" : "+v"(l)); return l; };
  v8s xh[2][NS], xl[2][NS], xt[2][2];
  // Tail: 16 columns more as one or two steps of 32 slots.  At most 8 of them: lane groups 0, 1, 2 hold the first 8
  // columns of hi * hi, lo * hi and hi * lo.  Else groups 0, 1 / 2, 3 hold both halves of hi * hi and lo * hi, and a second step hi * lo.
  const bool tail2 = TAIL && dk > 16 * (NK - 1) + 8;      // uniform
  bool xv[2];
  int ex[2] = {0, 0};                                     // exponents of the rows' blocks
#pragma unroll
  for (int b = 0; b < 2; ++b) {
    xv[b] = x0 + 16 * b + i < n_x;
    const char* xrow = a.ximg + xtile * IMG + (16 * b + i) * PA;
#pragma unroll
    for (int s = 0; s < NS; ++s) {
      xh[b][s] = xl[b][s] = zero8;
      if (xv[b]) {
        xh[b][s] = *reinterpret_cast<const v8s*>(xrow + ((64 * s + 16 * g) ^ swz));
        xl[b][s] = *reinterpret_cast<const v8s*>(xrow + PLANE + ((64 * s + 16 * g) ^ swz));
      }
      if (s >= NS - XL) {
        char* const p = xlds + (4 * (s - (NS - XL)) + 2 * b) * 4096;
        *reinterpret_cast<v8s*>(p) = xh[b][s];
        *reinterpret_cast<v8s*>(p + 4096) = xl[b][s];
      }
    }
    xt[b][0] = xt[b][1] = zero8;
    if (TAIL && xv[b]) {
      const int unit = 64 * NS + (tail2 ? 16 * (g & 1) : 0);
      if (tail2 || g < 3) xt[b][0] = *reinterpret_cast<const v8s*>(xrow + (!tail2 && g == 2 ? PLANE : 0) + (unit ^ swz));
      if (tail2 && g < 2) xt[b][1] = *reinterpret_cast<const v8s*>(xrow + PLANE + (unit ^ swz));
    }
    if (F16 && x0 + 16 * b < n_x) {                        // uniform
      const float e = a.xexp[xtile * 2 + b];
      ex[b] = __builtin_amdgcn_readfirstlane((int)(e > 0.5f * SP_NONFINITE ? e - SP_NONFINITE : e));
    }
  }

  if (DIST) close_id[threadIdx.x] = close_id[256 + threadIdx.x] = -1;
  v4f oacc[NO][2];
#pragma unroll
  for (int cb = 0; cb < NO; ++cb) oacc[cb][0] = oacc[cb][1] = (v4f)(0.f);
  float mref[2] = {-3.0e38f, -3.0e38f}, lrun[2] = {0.f, 0.f};   // softmax reference (log2 units; F16: an integer) and sum
  // DIST: squared norms (of rows there are not: 1, so that no pair with them is near), sums of the weights, where rows lie
  const size_t k_base = (size_t)side * a.C * a.N + (size_t)c * a.N;   // first row of the chunk's negatives
  float xn[2] = {1.f, 1.f}, wsum[2] = {0.f, 0.f};
  if (DIST) {
#pragma unroll
    for (int b = 0; b < 2; ++b) if (xv[b]) xn[b] = dist_norm(PASS == 1 ? a.xx[q_base + x0 + 16 * b + i] : a.yy[k_base + x0 + 16 * b + i]);
  }
  const int ntiles_all = (n_y + TY - 1) / TY;
  const int t_begin = u.part * u.tps;
  const int ntiles = min(ntiles_all, t_begin + u.tps);

  // ---- images of the streamed rows, copied into LDS one tile ahead; a register load issued behind the copies is the
  // fence (memory operations of a wave complete in order): once its value is there the image is in LDS.  The fence is
  // the load of the tile's two exponents; pass 2 also loads the softmax statistics of edge threadIdx % TY behind it.
  const char* ybase = a.yimg + (size_t)cs * a.yimg_tiles * IMG;
  const BufRsrc expsrc = buf_rsrc(F16 ? (const void*)(a.yexp + (size_t)cs * a.yimg_tiles * 2) : (const void*)ybase, (uint32_t)a.yimg_tiles * 8);
  const BufRsrc mlsrc = buf_rsrc(a.ml + q_base * 2, PASS == 2 ? (uint32_t)ne * 8 : 0u);
  const int f_row = threadIdx.x % TY;
  const size_t ml_stride = (size_t)2 * a.B;               // rows per part of pass 1's statistics
  const BufRsrc nrmsrc = buf_rsrc(!DIST ? (const void*)ybase : (const void*)(PASS == 1 ? a.yy + k_base : a.xx + q_base), DIST ? (uint32_t)n_y * 4 : 0u);
  float2 ye_next = make_float2(0.f, 0.f), st_ml = make_float2(0.f, 0.f);
  float st_nrm = 0.f;
  int token = 0;
  auto dma_piece = [&](int t, int buf, int q) {            // piece q of this wave of tile t into buffer `buf`
    const v4i ywords = buf_words(ybase + (size_t)t * IMG, IMG);
    const int pc = 4 * q + wave_s;
    if (pc < SG::NCH) buf_load4_to_lds(ywords, lds_address_b(smem) + buf * IMG + pc * 1024, lane * 16, pc * 1024, token);
  };
  auto dma_fence = [&](int t) {
    ye_next = buf_load2(expsrc, token, t * 8);
    if (PASS == 2) st_ml = buf_load2(mlsrc, f_row * 8 + token, t * TY * 8);
    if (DIST) st_nrm = buf_load1(nrmsrc, f_row * 4 + token, t * TY * 4);
  };
  auto dma_land = [&](int t, int buf) {
    asm volatile("" : "+v"(ye_next.x), "+v"(ye_next.y));
    if (DIST) nrm_all[buf * TY + f_row] = t * TY + f_row < n_y ? dist_norm(st_nrm) : 1.f;   // threads that share a row write the same value
    if (PASS == 2) {
      const int yr = t * TY + f_row;
      float mm = st_ml.x, ll = st_ml.y;
      if (a.sy_ml > 1 && yr < n_y) {                       // pass 1 was split (small batches): merge the parts
        const float2* __restrict__ mlp = reinterpret_cast<const float2*>(a.ml) + q_base + yr;
        for (int p = 1; p < a.sy_ml; ++p) mm = fmaxf(mm, mlp[p * ml_stride].x);
        ll *= __builtin_amdgcn_exp2f(st_ml.x - mm);
        for (int p = 1; p < a.sy_ml; ++p) { const float2 v = mlp[p * ml_stride]; ll += v.y * __builtin_amdgcn_exp2f(v.x - mm); }
      }
      // Rows beyond the chunk: +inf, so that their weights are 2^-inf = 0 (threads that share a row write the same value).
      // fp32: the integer and the logarithm of the mantissa stay apart (their sum would be rounded to 2^-21, an error that
      // all of an edge's weights share).
      const float lg = log2f(ll);
      aux_all[2 * buf * TY + f_row] = yr < n_y ? (F16 ? lg : mm + lg) : __builtin_inff();
      if (F16) aux_all[(2 * buf + 1) * TY + f_row] = mm;
    }
  };
  if (t_begin < ntiles) {
#pragma unroll
    for (int q = 0; q < NCW; ++q) dma_piece(t_begin, 0, q);
    dma_fence(t_begin);
    dma_land(t_begin, 0);
    __syncthreads();
  }

  // Where a lane reads in a tile's buffer: rows start at whole groups of units, so a unit of the same group is a bit pattern
  // away and the other groups are immediate offsets.  Rows y and y + 16 have the same swizzle.
  constexpr int GU = sp_group(UNITS);                      // units to a group
  const int fofs = i * PA + ((16 * g) ^ swz);              // score product, row half a, step s: at(fofs, 64 s) + 16 a PA
  const int tfofs = i * PA + (tail2 ? (g & 2 ? PLANE : 0) + ((64 * NS + 16 * (g & 1)) ^ swz) : (g == 1 ? PLANE : 0) + ((64 * NS) ^ swz));
  const int ty = 4 * g + (i >> 2), tswz = 16 * sp_swizzle(UNITS, ty);   // second product: rows ty, ty + 16, columns 16 cb + 4 (i % 4) .. +3
  const int trofs = ty * PA + ((8 * (i & 3)) ^ tswz);      // at(trofs, 32 cb)
  auto at = [](int base, int byte) { return (base ^ (byte % (16 * GU))) + byte / (16 * GU) * (16 * GU); };
  // Last output block: where at most 8 columns are left, its rows 0 .. 7 are their hi parts and 8 .. 15 their lo parts
  const bool pack = dk <= 16 * (NO - 1) + 8;               // uniform
  const int ptrofs = ty * PA + (pack && (i & 2) ? PLANE : 0) + ((32 * (NO - 1) + 8 * (i & (pack ? 1 : 3))) ^ tswz);

  for (int t = t_begin; t < ntiles; ++t) {
    const int buf = (t - t_begin) & 1, bofs = buf * IMG;
    const bool has_next = t + 1 < ntiles;                  // uniform
    const int e0 = F16 ? __builtin_amdgcn_readfirstlane((int)(ye_next.x > 0.5f * SP_NONFINITE ? ye_next.x - SP_NONFINITE : ye_next.x)) : 0;
    const int e1 = F16 ? __builtin_amdgcn_readfirstlane((int)(ye_next.y > 0.5f * SP_NONFINITE ? ye_next.y - SP_NONFINITE : ye_next.y)) : 0;
    const int y0 = t * TY;
    const bool masked = PASS != 2 && y0 + TY > n_y;

    // -- scores S^T: block (ah, b) = rows 16 ah + 4 g + r, column 16 b + i; the streamed rows' fragments are read PD steps ahead
    v4f sc[2][2];
    sc[0][0] = sc[0][1] = sc[1][0] = sc[1][1] = (v4f)(0.f);
    {
      constexpr int PD = NS < SP_PD ? NS : SP_PD;
      v8s fh[PD][2], fl[PD][2];
      const int fb = bofs + fofs;
      auto read_step = [&](int s, v8s (&vh)[2], v8s (&vl)[2]) {
        const char* p = smem + at(fb, 64 * s);
#pragma unroll
        for (int r = 0; r < 2; ++r) { vh[r] = *reinterpret_cast<const v8s*>(p + 16 * r * PA); vl[r] = *reinterpret_cast<const v8s*>(p + 16 * r * PA + PLANE); }
      };
#pragma unroll
      for (int s = 0; s < PD; ++s) read_step(s, fh[s], fl[s]);
#pragma unroll
      for (int s = 0; s < NS; ++s) {
        const v8s h0 = fh[s % PD][0], h1 = fh[s % PD][1], l0 = fl[s % PD][0], l1 = fl[s % PD][1];
        if (s + PD < NS) read_step(s + PD, fh[s % PD], fl[s % PD]);
        if (s >= NS - XL) {
          const char* const p = xlds + 4 * (s - (NS - XL)) * 4096;
          sp_score_step<F16>(h0, h1, l0, l1, *reinterpret_cast<const v8s*>(p), *reinterpret_cast<const v8s*>(p + 2 * 4096),
                             *reinterpret_cast<const v8s*>(p + 4096), *reinterpret_cast<const v8s*>(p + 3 * 4096), sc);
        } else {
          sp_score_step<F16>(h0, h1, l0, l1, xh[0][s], xh[1][s], xl[0][s], xl[1][s], sc);
        }
        // the next tile's pieces are issued between the steps: a burst of them holds the wave at the memory pipeline's
        // queue (rows of 400: a pass 1075 us with the copies at the tile's start, 915 spread, 810 without any)
        if (has_next) {
#pragma unroll
          for (int q = s * NCW / NS; q < (s + 1) * NCW / NS; ++q) dma_piece(t + 1, buf ^ 1, q);
          if (s == NS - 1) dma_fence(t + 1);
        }
        __builtin_amdgcn_sched_barrier(0);                 // keeps the reads PD steps ahead of their use
      }
      if (TAIL) {
        const char* p = smem + bofs + tfofs;
        sp_tail_step<F16>(*reinterpret_cast<const v8s*>(p), *reinterpret_cast<const v8s*>(p + 16 * PA), xt[0][0], xt[1][0], sc);
        if (tail2) {                                       // its hi fragments again (groups 2, 3 meet zeros)
          const char* p2 = smem + bofs + i * PA + ((64 * NS + 16 * (g & 1)) ^ swz);
          sp_tail_step<F16>(*reinterpret_cast<const v8s*>(p2), *reinterpret_cast<const v8s*>(p2 + 16 * PA), xt[0][1], xt[1][1], sc);
        }
      }
    }
    const float ef[2] = {(float)e0, (float)e1};
    // image row of row `row` of the wave (there is one only where xv says so); formed anew from the arguments, as DistRow is
    auto dist_image_row = [&](int row) {
      KernelArgs* args = (KernelArgs*)__builtin_amdgcn_kernarg_segment_ptr();
      asm volatile("" : "+s"(args), "+v"(row));
      return args->ximg + ((size_t)u.cs * args->ximg_tiles + u.stripe * (SP_SR / TY) + wave_s) * IMG + row * PA;
    };
    // -- weights of the lane's 2 x 8 pairs: w[b][4 ah + r] is row 16 ah + 4 g + r against column 16 b + i
    float w[2][8];
    if constexpr (DIST) {
#pragma unroll
      for (int b = 0; b < 2; ++b) {
        // squared distances; near: the expansion is left with fewer than 14 good bits (or is no number)
        float d2[8];
        bool near = false;
        const auto is_near = [&](int v, float yn) { return xv[b] && !(d2[v] > 0.00390625f * (xn[b] + yn)); };
        const float4 yn4[2] = {*reinterpret_cast<const float4*>(nrm_all + buf * TY + 4 * g), *reinterpret_cast<const float4*>(nrm_all + buf * TY + 16 + 4 * g)};
        const float yn[8] = {yn4[0].x, yn4[0].y, yn4[0].z, yn4[0].w, yn4[1].x, yn4[1].y, yn4[1].z, yn4[1].w};
        const float k2[2] = {-__builtin_ldexpf(1.f, 1 - ex[b] - e0), -__builtin_ldexpf(1.f, 1 - ex[b] - e1)};
#pragma unroll
        for (int v = 0; v < 8; ++v) {
          d2[v] = __builtin_fmaf(sc[v >> 2][b][v & 3], k2[v >> 2], xn[b] + yn[v]);
          near |= is_near(v, yn[v]);
        }
        unsigned none = 0u;                                // pairs at distance 0: no gradient; << 8, << 16: close pairs in slots 0 and 1
        if (__builtin_expect(__any(near), 0)) {
          unsigned left = 0u;
#pragma unroll
          for (int v = 0; v < 8; ++v) left |= is_near(v, yn[v]) ? 1u << (16 * (v >> 2) + 4 * g + (v & 3)) : 0u;
          left |= __shfl_xor(left, 16);                    // near pairs of the column: a bit for each of the tile's rows
          left |= __shfl_xor(left, 32);
          for (; __any(left != 0u); left &= left - 1u) {
            // one pair of every column at a time: its four lanes each take the columns they hold fragments of
            const int at_row = left ? __ffs((int)left) - 1 : 0;
            const int ey = at_row < 16 ? e0 : e1;
            const float r = __builtin_ldexpf(1.f, max(-126, min(126, ey - ex[b])));   // differences in units of the streamed row's block
            const char* const yp = smem + bofs + at_row * PA;
            const int ysw = 16 * sp_swizzle(UNITS, at_row);
            float part = 0.f;
            auto add_unit = [&](const v8h& x0h, const v8h& x0l, int byte) {
              const v8h y0h = *reinterpret_cast<const v8h*>(yp + (byte ^ ysw)), y0l = *reinterpret_cast<const v8h*>(yp + PLANE + (byte ^ ysw));
#pragma unroll
              for (int j = 0; j < 8; ++j) {
                float d = __builtin_fmaf((float)x0h[j], r, -(float)y0h[j]);
                d = __builtin_fmaf((float)x0l[j], r, d);
                d = __builtin_fmaf((float)y0l[j], neg1, d);
                part = __builtin_fmaf(d, d, part);
              }
            };
            const char* const xp = dist_image_row(16 * b + i);
            auto add_image = [&](int byte) { add_unit(*reinterpret_cast<const v8h*>(xp + (byte ^ swz)), *reinterpret_cast<const v8h*>(xp + PLANE + (byte ^ swz)), byte); };
            if (XL > 0) {                                  // registers are full: all columns from the row's image
              if (left) {
#pragma unroll 1
                for (int s = 0; s < NS; ++s) add_image(64 * s + 16 * g);
              }
            } else {
#pragma unroll
              for (int s = 0; s < NS; ++s) {
                v8s ah = xh[b][s], al = xl[b][s];
                asm volatile("" : "+v"(ah), "+v"(al));     // or their conversions are moved out of the loop, into registers that there are not
                add_unit(__builtin_bit_cast(v8h, ah), __builtin_bit_cast(v8h, al), 64 * s + 16 * g);
                if (s % 2) __builtin_amdgcn_sched_barrier(0);
              }
            }
            if (TAIL && left && g < 2) add_image(64 * NS + 16 * g);   // the 16 columns behind: units 0 and 1 (zeros from dk on)
            part += __shfl_xor(part, 16);
            part = __builtin_ldexpf(part + __shfl_xor(part, 32), -2 * ey);
            // close (2^-15 of the norm): by the rows themselves, for hi + lo of two rows tell them apart to 2^-20 of the norm, and
            // rows that are the same have to be found to be
            const float both = xn[b] + nrm_all[buf * TY + at_row];
            const bool close = left && !(part > SP_CLOSE * both);
            if (__builtin_expect(__any(close), 0)) {
              const int xr = min(u.stripe * SP_SR + wave_s * 32 + 16 * b + (fresh_lane() & 15), n_x - 1), yr = min(y0 + at_row, n_y - 1);
              const DistRow<true> q(u.cs, PASS == 1 ? xr : yr);
              const DistRow<false> n(u.cs, PASS == 1 ? yr : xr);
              float exact = 0.f;
#pragma unroll 1
              for (int k = 4 * g; k < dk; k += 16) {
                const float4 qc = q.cols(k), nc = n.cols(k);
                const float d[4] = {qc.x - nc.x, qc.y - nc.y, qc.z - nc.z, qc.w - nc.w};
                exact += (d[0] * d[0] + d[1] * d[1]) + (d[2] * d[2] + d[3] * d[3]);
              }
              exact += __shfl_xor(exact, 16);
              exact += __shfl_xor(exact, 32);
              part = close ? exact : part;
              // a close pair's weight over its distance would leave the others' no bits of the f16 range, and its part in the sums
              // of W y cancels: it stays out of the product where its lane has a slot left
              if (close && part >= 2e-38f && g == (at_row & 15) >> 2) {
                int* const own = close_id + wave_s * 64 + fresh_lane();
                const int slot = own[0] < 0 ? 0 : (own[256] < 0 ? 1 : 2);
                if (slot < 2) {
                  own[256 * slot] = (y0 + at_row) | b << 30;
                  none |= 256u << (8 * slot + 4 * (at_row >> 4) + (at_row & 3));
                }
              }
            }
#pragma unroll
            for (int v = 0; v < 8; ++v) {
              if (left && at_row == 16 * (v >> 2) + 4 * g + (v & 3)) {
                d2[v] = part < 2e-38f ? 2e-38f : (part > 3e38f ? 3e38f : part);   // normal numbers; a NaN stays one
                none |= part < 2e-38f ? 1u << v : 0u;
              }
            }
          }
        }
        // log2 of the softmax weight (pass 2: of the probability) of a pair at 1 / rs, less the pieces of the reference
        float lg[8], mm[8];
        auto read_lse = [&]() {
          if (PASS == 2) {
#pragma unroll
            for (int h = 0; h < 2; ++h) {
              const float4 l4 = *reinterpret_cast<const float4*>(aux_all + 2 * buf * TY + 16 * h + 4 * g);
              const float4 m4 = *reinterpret_cast<const float4*>(aux_all + (2 * buf + 1) * TY + 16 * h + 4 * g);
              lg[4 * h] = l4.x; lg[4 * h + 1] = l4.y; lg[4 * h + 2] = l4.z; lg[4 * h + 3] = l4.w;
              mm[4 * h] = m4.x; mm[4 * h + 1] = m4.y; mm[4 * h + 2] = m4.z; mm[4 * h + 3] = m4.w;
            }
          }
        };
        auto log2w = [&](int v, float rs) {
          const float dist = d2[v] * rs;
          if (PASS == 2) return __builtin_fmaf(dist, -LOG2E, -lg[v]) - mm[v];
          return masked && y0 + 16 * (v >> 2) + 4 * g + (v & 3) >= n_y ? -__builtin_inff() : -LOG2E * dist;
        };
        float l[2];
        auto weigh = [&]() {                               // the weights; returns the largest
          read_lse();
          l[0] = l[1] = 0.f;
#pragma unroll
          for (int v = 0; v < 8; ++v) {
            float rs = __builtin_amdgcn_rsqf(d2[v]);       // and a Newton step: the instruction's errors lean to one side, which sums over
            rs = __builtin_fmaf(0.5f * rs, __builtin_fmaf(-(d2[v] * rs), rs, 1.f), rs);   // many pairs keep (relation rows 3.3e-7 off, 2.4e-7 with it)
            const float p = __builtin_amdgcn_exp2f(log2w(v, rs) - (ef[v >> 2] + mref[b]));
            if (PASS == 1) l[v >> 2] += p;
            w[b][v] = p * rs;
          }
          if (__builtin_expect(__any(none != 0u), 0)) {
            float* const close_w = reinterpret_cast<float*>(close_id) + 2 * 256 + wave_s * 64 + fresh_lane();
#pragma unroll
            for (int v = 0; v < 8; ++v) {
              if (none >> v & 0x10100u) {
                float* const at = close_w + (none >> v & 0x100u ? 0 : 256);
                at[0] = fminf(w[b][v], 3e38f);
                at[2 * 256] = ef[v >> 2] + mref[b];
              }
              w[b][v] = none >> v & 0x10101u ? 0.f : w[b][v];
            }
          }
          float most = w[b][0];
#pragma unroll
          for (int v = 1; v < 8; ++v) most = fmaxf(most, w[b][v]);
          return fmaxf(most, fmaxf(l[0], l[1]) * 0x1p-64f);   // (a pair at distance 0, and a close one, has only a softmax weight here)
        };
        if (__builtin_expect(__any(weigh() > 32768.f), 0)) {
          float tall = -3.0e38f;
#pragma unroll
          for (int v = 0; v < 8; ++v) {
            const float rs = __builtin_amdgcn_rsqf(d2[v]);
            tall = fmaxf(tall, log2w(v, rs) - ef[v >> 2] + (none >> v & 0x10101u ? 0.f : __builtin_amdgcn_logf(rs)));
          }
          tall = fmaxf(tall, __shfl_xor(tall, 16));
          tall = fmaxf(tall, __shfl_xor(tall, 32));
          const float mnew = fmaxf(mref[b], __builtin_ceilf(tall) - 8.f);
          float alpha = __builtin_amdgcn_exp2f(mref[b] - mnew);
          asm volatile("" : "+v"(alpha));
          lrun[b] *= alpha;
          wsum[b] *= alpha;
#pragma unroll
          for (int cb = 0; cb < NO; ++cb) {
            if (NK > 8) asm volatile("" : "+a"(oacc[cb][b]));
            oacc[cb][b] *= alpha;
            if (NK > 8) asm volatile("" : "+a"(oacc[cb][b]));
          }
          mref[b] = mnew;
          (void)weigh();
        }
        if (PASS == 1) lrun[b] += __builtin_ldexpf(l[0], e0) + __builtin_ldexpf(l[1], e1);
        float ws[2] = {0.f, 0.f};
#pragma unroll
        for (int v = 0; v < 8; ++v) ws[v >> 2] += w[b][v];
        wsum[b] += __builtin_ldexpf(ws[0], e0) + __builtin_ldexpf(ws[1], e1);
      }
    } else {
      // -- score log2(e) = sc k, k = log2(e) 2^-(ex + ey): never 0, or a masked row's -inf would become NaN (two blocks at the
      // largest exponent: scores below 2^-85 either way)
      float k[2][2];
#pragma unroll
      for (int b = 0; b < 2; ++b) {
        k[0][b] = F16 ? __int_as_float(0x3fb8aa3b - (max(-126, min(125, ex[b] + e0)) << 23)) : LOG2E;
        k[1][b] = F16 ? __int_as_float(0x3fb8aa3b - (max(-126, min(125, ex[b] + e1)) << 23)) : LOG2E;
      }
      if (masked) {                                          // the chunk's last, partial tile (uniform): rows beyond it weigh nothing
#pragma unroll
        for (int r = 0; r < 8; ++r) {
          if (y0 + 16 * (r >> 2) + 4 * g + (r & 3) >= n_y) sc[r >> 2][0][r & 3] = sc[r >> 2][1][r & 3] = -__builtin_inff();
        }
      }
      if (PASS == 1 || F16) {
        float tmax[2];
        if (PASS == 1) {
#pragma unroll
          for (int b = 0; b < 2; ++b) {
            float m[2];
#pragma unroll
            for (int h = 0; h < 2; ++h) m[h] = __builtin_fmaf(fmaxf(fmaxf(sc[h][b][0], sc[h][b][1]), fmaxf(sc[h][b][2], sc[h][b][3])), k[h][b], -ef[h]);
            tmax[b] = fmaxf(m[0], m[1]);
          }
        } else {
          float m[2][2];
#pragma unroll
          for (int h = 0; h < 2; ++h) {
            const float4 l4 = *reinterpret_cast<const float4*>(aux_all + 2 * buf * TY + 16 * h + 4 * g);
            const float4 m4 = *reinterpret_cast<const float4*>(aux_all + (2 * buf + 1) * TY + 16 * h + 4 * g);
#pragma unroll
            for (int b = 0; b < 2; ++b) {
              w[b][4 * h] = __builtin_fmaf(sc[h][b][0], k[h][b], -l4.x) - m4.x;
              w[b][4 * h + 1] = __builtin_fmaf(sc[h][b][1], k[h][b], -l4.y) - m4.y;
              w[b][4 * h + 2] = __builtin_fmaf(sc[h][b][2], k[h][b], -l4.z) - m4.z;
              w[b][4 * h + 3] = __builtin_fmaf(sc[h][b][3], k[h][b], -l4.w) - m4.w;
              m[h][b] = fmaxf(fmaxf(w[b][4 * h], w[b][4 * h + 1]), fmaxf(w[b][4 * h + 2], w[b][4 * h + 3])) - ef[h];
            }
          }
#pragma unroll
          for (int b = 0; b < 2; ++b) tmax[b] = fmaxf(m[0][b], m[1][b]);
        }
        constexpr float SLACK = F16 ? 15.f : 16.f * LOG2E;
        if (__any(tmax[0] > mref[0] + SLACK || tmax[1] > mref[1] + SLACK)) {
#pragma unroll
          for (int b = 0; b < 2; ++b) {
            float tall = fmaxf(tmax[b], __shfl_xor(tmax[b], 16));
            tall = fmaxf(tall, __shfl_xor(tall, 32));
            const float mnew = fmaxf(mref[b], F16 ? __builtin_ceilf(tall) - 8.f : tall);
            float alpha = __builtin_amdgcn_exp2f(mref[b] - mnew);
            asm volatile("" : "+v"(alpha));                  // a real branch: keeps the rescale from being executed speculatively
            lrun[b] *= alpha;
#pragma unroll
            for (int cb = 0; cb < NO; ++cb) {
              if (NK > 8) asm volatile("" : "+a"(oacc[cb][b]));
              oacc[cb][b] *= alpha;
              if (NK > 8) asm volatile("" : "+a"(oacc[cb][b]));   // wide rows: back to the accumulation registers, one block at a time
            }
            mref[b] = mnew;
          }
        }
#pragma unroll
        for (int b = 0; b < 2; ++b) {
          float l[2] = {0.f, 0.f};
#pragma unroll
          for (int v = 0; v < 8; ++v) {
            const float ref = ef[v >> 2] + mref[b];          // exact: integers (bf16: no exponents)
            w[b][v] = __builtin_amdgcn_exp2f(PASS == 1 ? __builtin_fmaf(sc[v >> 2][b][v & 3], k[v >> 2][b], -ref) : w[b][v] - ref);
            if (PASS == 1) l[v >> 2] += w[b][v];
          }
          if (PASS == 1) lrun[b] += F16 ? __builtin_ldexpf(l[0], e0) + __builtin_ldexpf(l[1], e1) : l[0] + l[1];
        }
      } else {                                               // pass 2, bf16: no reference needed
#pragma unroll
        for (int h = 0; h < 2; ++h) {
          const float4 l4 = *reinterpret_cast<const float4*>(aux_all + 2 * buf * TY + 16 * h + 4 * g);
#pragma unroll
          for (int b = 0; b < 2; ++b) {
            w[b][4 * h] = __builtin_amdgcn_exp2f(__builtin_fmaf(sc[h][b][0], LOG2E, -l4.x));
            w[b][4 * h + 1] = __builtin_amdgcn_exp2f(__builtin_fmaf(sc[h][b][1], LOG2E, -l4.y));
            w[b][4 * h + 2] = __builtin_amdgcn_exp2f(__builtin_fmaf(sc[h][b][2], LOG2E, -l4.z));
            w[b][4 * h + 3] = __builtin_amdgcn_exp2f(__builtin_fmaf(sc[h][b][3], LOG2E, -l4.w));
          }
        }
      }
    }
    v8s wh[2], wl[2];
    split8<F16>(w[0], neg1, wh[0], wl[0]);
    split8<F16>(w[1], neg1, wh[1], wl[1]);
    // -- O^T[c][x] += sum_y Y[y][c] W[y][x], one 16-column block after the other, read PG blocks ahead
    constexpr int PG = SP_PG < NO ? SP_PG : NO;
    const int tb = bofs + trofs;
    v8s gh[PG], gl[PG];
    auto read_block = [&](int cb, v8s& vh, v8s& vl) {
      const char* p = smem + (cb == NO - 1 ? bofs + ptrofs : at(tb, 32 * cb));
      vh = join8(lds_read_tr(p), lds_read_tr(p + 16 * PA));
      if (cb == NO - 1) p = smem + at(tb, 32 * cb);
      if (cb < NO - 1 || !pack) vl = join8(lds_read_tr(p + PLANE), lds_read_tr(p + 16 * PA + PLANE));
    };
#pragma unroll
    for (int cb = 0; cb < PG; ++cb) read_block(cb, gh[cb], gl[cb]);
#pragma unroll
    for (int cb = 0; cb < NO; ++cb) {
      const v8s ah = gh[cb % PG], al = gl[cb % PG];
      if (cb + PG < NO) read_block(cb + PG, gh[cb % PG], gl[cb % PG]);
      const int p = cb & 1, q = p ^ 1;                     // consecutive instructions share an operand
      oacc[cb][p] = mfma16h<F16>(ah, wl[p], oacc[cb][p]); oacc[cb][p] = mfma16h<F16>(ah, wh[p], oacc[cb][p]);
      if (cb < NO - 1 || !pack) { oacc[cb][p] = mfma16h<F16>(al, wh[p], oacc[cb][p]); oacc[cb][q] = mfma16h<F16>(al, wh[q], oacc[cb][q]); }
      oacc[cb][q] = mfma16h<F16>(ah, wh[q], oacc[cb][q]); oacc[cb][q] = mfma16h<F16>(ah, wl[q], oacc[cb][q]);
      __builtin_amdgcn_sched_barrier(0);
    }
    if (has_next) {
      dma_land(t + 1, buf ^ 1);
      __syncthreads();                                     // tile t + 1 is in LDS; every wave is done with tile t
    }
  }

  // ---- epilogue
#pragma unroll
  for (int b = 0; b < 2; ++b) {
    if (pack) {                                            // lo parts back to the hi parts' columns
#pragma unroll
      for (int r = 0; r < 4; ++r) oacc[NO - 1][b][r] += __shfl_xor(oacc[NO - 1][b][r], 32);
    }
    const int x = x0 + 16 * b + i;
    int oshift = 0;                                        // gradient rows are written as accumulator x 2^oshift
    float* orow;
    if (PASS == 1) {                                       // the part's statistics and unnormalised gradient rows
      float ltot = lrun[b] + __shfl_xor(lrun[b], 16);
      ltot += __shfl_xor(ltot, 32);
      // sum = mantissa 2^p, reference + p: the statistics' reference is close to the log-sum-exp itself
      int p = 0;
      if (F16 && ltot > 0.f && ltot < 3.0e38f) p = (int)((__float_as_uint(ltot) >> 23) & 255u) - 127;
      oshift = -p;
      const size_t part_row = (size_t)u.part * 2 * a.B + q_base + x;
      const bool extra = u.rem && u.part > 0;              // parts 1.. of a split stripe
      const size_t xr = (size_t)(u.part - 1) * a.rem_rows + (size_t)(u.unit - a.whole_units) * SP_SR + wave * 32 + 16 * b + i;
      float* ml_out = extra ? a.mlx + xr * 2 : a.ml + (u.rem ? q_base + x : part_row) * 2;
      orow = extra ? a.outx + xr * dk : a.out + (u.rem ? q_base + x : part_row) * dk;
      if (g == 0 && xv[b]) *reinterpret_cast<float2*>(ml_out) = make_float2(mref[b] + (float)p, __builtin_ldexpf(ltot, -p));
    } else {                                               // gradient row of part `part` of each negative's occurrence
      if (F16) oshift = mref[b] > -1.0e38f ? (int)mref[b] : 0;   // weights were formed relative to the reference
      orow = a.out + (a.roles * (size_t)a.n + ((side == MAR_SIDE_DST ? 0 : (size_t)a.cn) + (size_t)c * a.N + x) * a.sy + (u.rem ? 0 : u.part)) * dk;
      if (u.rem && u.part > 0) orow = a.outx + ((size_t)(u.part - 1) * a.rem_rows + (size_t)(u.unit - a.whole_units) * SP_SR + wave * 32 + 16 * b + i) * dk;
    }
    float ws = 0.f;
    if (DIST) {                                            // sum of W (y - x): less the stationary row times the sum of its weights
      ws = wsum[b] + __shfl_xor(wsum[b], 16);
      ws += __shfl_xor(ws, 32);
    }
    bool has_close = false;
    if (DIST) has_close = __any(close_id[wave_s * 64 + fresh_lane()] >= 0);   // (slot 0 is taken first)
    int go = g;
    if (DIST) go = fresh_lane() >> 4;                      // nor are the rows' columns to be kept
    if (xv[b]) {
      if constexpr (DIST) {
        const DistRow<PASS == 1> row(u.cs, x);
#pragma unroll
        for (int cb = 0; cb < NO; ++cb) {
          const float4 xs = row.shifted(16 * cb + 4 * go);
          oacc[cb][b] -= (v4f){xs.x * ws, xs.y * ws, xs.z * ws, xs.w * ws};
          if (cb % 4 == 3) __builtin_amdgcn_sched_barrier(0);   // a few blocks' loads at a time: registers are full
        }
        if (__builtin_expect(has_close, 0)) {
          // the column's close pairs, which its four lanes keep: W (y - x) from the rows, at the end's reference
#pragma unroll 1
          for (int k = 0; k < 8; ++k) {
            const int lane_c = fresh_lane(), at = 256 * (k >> 2) + wave_s * 64 + 16 * (k & 3) + (lane_c & 15), id = close_id[at];
            if (id < 0 || id >> 30 != b) continue;
            const float* const close_w = reinterpret_cast<const float*>(close_id) + 2 * 256 + at;
            const float wc = __builtin_ldexpf(close_w[0], (int)fmaxf(-300.f, fminf(300.f, close_w[2 * 256] - mref[b])));
            const int y = id & 0x3fffffff;
            const DistRow<true> q(u.cs, PASS == 1 ? x : y);
            const DistRow<false> n(u.cs, PASS == 1 ? y : x);
#pragma unroll
            for (int cb = 0; cb < NO; ++cb) {
              const int col = 16 * cb + 4 * (lane_c >> 4);
              const float4 qc = q.cols(col), nc = n.cols(col);
              const v4f d = {nc.x - qc.x, nc.y - qc.y, nc.z - qc.z, nc.w - qc.w};
              oacc[cb][b] += d * (PASS == 1 ? wc : -wc);
              if (cb % 4 == 3) __builtin_amdgcn_sched_barrier(0);
            }
          }
        }
      }
#pragma unroll
      for (int cb = 0; cb < NO; ++cb) {
        const int col = 16 * cb + 4 * go;
        if (col < dk && (cb < NO - 1 || !pack || go < 2))
          *reinterpret_cast<float4*>(orow + col) =
              make_float4(__builtin_ldexpf(oacc[cb][b][0], oshift), __builtin_ldexpf(oacc[cb][b][1], oshift),
                          __builtin_ldexpf(oacc[cb][b][2], oshift), __builtin_ldexpf(oacc[cb][b][3], oshift));
      }
    }
  }
}

template <int NK, int PASS, bool F16>
__global__ void __launch_bounds__(256) MAR_WAVES_PER_SIMD(sp_waves(NK, PASS))
k_split(FlashArgs a) {
  if constexpr (PASS == 3) split_eval<NK, sp_eval_32(NK, 16 * NK - 8)>();
  else split_pass<NK, PASS, F16, false, false>(a);
}

template <int NK, int PASS, bool F16>
__global__ void __launch_bounds__(256) MAR_WAVES_PER_SIMD(sp_waves(NK, PASS))
k_split_carry(FlashArgs a) { split_pass<NK, PASS, F16, false, true>(a); }

// The training passes of TransE.  Counted, a pair takes 40 vector instructions, matrix ones included, in a bilinear model's pass 18; the
// vector pipe is busy 0.46 and 0.37 of the time, the matrix pipe 0.22 and 0.18, the rest is one tile's chain of products, distances,
// weights and products with two waves a SIMD.  10,000 edges, 1,000 negatives of 100 floats: 47 and 58 us where fp32 matrix
// instructions with stored weights (k_flash, k_flash_bwd) take 111 and 61.  Errors against 64 bits over 42 drawn steps, fp32 instructions / these, mean: node gradients 1.1e-7 / 9e-8, relation gradients 4.1e-7 / 3.1e-7, log-sum-exps 2.1e-7 /
// 8e-8, worst row 8.8e-7 / 4.9e-7.  Near pairs: 3e-2 to 3e-5 apart as on fp32 instructions (100 floats, 1e-3: 6.3e-7 / 6.7e-7), closer
// ones (SP_CLOSE) exact to 1.6e-7 where those have 3e-5 (1e-5 apart) to 7e-2 (one unit in the last place, 400 floats).  Tables whose
// rows share an offset are taken without it (common_offset); the loop over near pairs is for few (after 200 and 1,000 steps of training
// from 0 +- 0.3: 153 and 156 us a step, 210 on fp32 instructions).
// Registers decide: nothing may spill (a step of 10,000 edges, 1,000 negatives of 400 floats 585 us with 351 registers spilled, 511 with
// three steps' fragments in LDS and the near loop on the row's image; 50,000 edges 2,390 and 1,880).
template <int NK, int PASS, bool CARRY>
__global__ void __launch_bounds__(256) MAR_WAVES_PER_SIMD(sp_waves(NK, PASS))
k_split_dist(FlashArgs a) { split_pass<NK, PASS, true, true, CARRY>(a); }

// The form of pass 3 that the fullest rows of an instantiation take, where it is not that of the others.
template <int NK>
__global__ void __launch_bounds__(256) MAR_WAVES_PER_SIMD(sp_waves(NK, 3))
k_split_eval_full(FlashArgs a) { split_eval<NK, true>(); }

// Adds parts 1.. of pass 2's split stripes to the gradient rows that part 0 wrote, in the parts' order.  One group of
// 32 lanes per row.
__global__ void __launch_bounds__(256) k_split_merge2(FlashArgs a) {
  const int grp = threadIdx.x >> 5, l = threadIdx.x & 31;
  const long rrow = (long)blockIdx.x * 8 + grp;
  if (rrow >= a.rem_rows) return;
  const int unit = a.whole_units + (int)(rrow / SP_SR);
  const int cs = unit / a.nstripes, x = (unit % a.nstripes) * SP_SR + (int)(rrow % SP_SR);
  if (x >= a.N) return;
  const int side = cs & 1, c = cs >> 1;
  float* o0 = a.out + (a.roles * (size_t)a.n + ((side == MAR_SIDE_DST ? 0 : (size_t)a.cn) + (size_t)c * a.N + x)) * a.dk;
  for (int k = 4 * l; k < a.dk; k += 128) {
    float4 o = *reinterpret_cast<const float4*>(o0 + k);
    for (int p = 1; p < a.rem_k; ++p) {
      const float4 q = *reinterpret_cast<const float4*>(a.outx + ((size_t)(p - 1) * a.rem_rows + rrow) * a.dk + k);
      o.x += q.x; o.y += q.y; o.z += q.z; o.w += q.w;
    }
    *reinterpret_cast<float4*>(o0 + k) = o;
  }
}

// ------------------------------------------------------------------- launchers -----
int mar_split_supported(int dk) { return dk >= 4 && dk <= 400; }
int mar_split_wgs_per_cu(int dk, int pass) { return sp_waves(sp_nk(dk), pass); }
bool mar_split_shares(int dk) { return sp_shares(sp_nk(dk)); }
size_t mar_split_image_bytes(int dk) { return (size_t)sp_image(sp_nk(dk)); }

template <int NK> static hipError_t sp_prepare() {
  constexpr size_t lds = SplitGeom<NK>::LDS_BYTES;
  hipError_t e = hipSuccess;
#define PREP(P, F) if (e == hipSuccess) e = hipFuncSetAttribute(reinterpret_cast<const void*>(&k_split<NK, P, F>), hipFuncAttributeMaxDynamicSharedMemorySize, (int)(P == 3 ? SplitGeom<NK>::LDS_BYTES3 : lds))
  PREP(1, true); PREP(2, true); PREP(3, true); PREP(1, false); PREP(2, false);
#undef PREP
#define PREP(P, C) if (e == hipSuccess) e = hipFuncSetAttribute(reinterpret_cast<const void*>(&k_split_dist<NK, P, C>), hipFuncAttributeMaxDynamicSharedMemorySize, (int)SplitGeom<NK>::LDS_BYTES_DIST)
  PREP(1, false); PREP(2, false); PREP(1, true); PREP(2, true);
#undef PREP
#define PREP(P, F) if (e == hipSuccess) e = hipFuncSetAttribute(reinterpret_cast<const void*>(&k_split_carry<NK, P, F>), hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds)
  PREP(1, true); PREP(2, true); PREP(1, false); PREP(2, false);
#undef PREP
  return e;
}
hipError_t mar_split_prepare(int dk) {
  switch (sp_nk(dk)) {
    case 12: return sp_prepare<12>();
    case 16: return sp_prepare<16>();
    case 25: return sp_prepare<25>();
    default: static_assert(SplitGeom<8>::LDS_BYTES <= 64 * 1024 && SplitGeom<8>::LDS_BYTES3 <= 64 * 1024 && SplitGeom<8>::LDS_BYTES_DIST <= 64 * 1024, "narrower instantiations stay below the default limit"); return hipSuccess;
  }
}

template <int NK> static hipError_t sp_launch(const FlashArgs& a, int pass, bool f16, dim3 grid, hipStream_t st) {
  constexpr size_t lds = SplitGeom<NK>::LDS_BYTES, ldsd = SplitGeom<NK>::LDS_BYTES_DIST;
  static_assert(SplitGeom<NK>::LDS_BYTES3 <= 160 * 1024 && SplitGeom<NK>::LDS_BYTES_DIST <= 160 * 1024, "two images in LDS");
  if constexpr (sp_eval_32(NK, 16 * NK) && !sp_eval_32(NK, 16 * NK - 8)) {
    if (pass == 3 && sp_eval_32(NK, a.dk)) {
      hipLaunchKernelGGL((k_split_eval_full<NK>), grid, dim3(256), SplitGeom<NK>::LDS_BYTES3, st, a);
      return hipGetLastError();
    }
  }
  if (a.dist) {
    if (pass == 1) {
      if (a.carried) hipLaunchKernelGGL((k_split_dist<NK, 1, true>), grid, dim3(256), ldsd, st, a);
      else hipLaunchKernelGGL((k_split_dist<NK, 1, false>), grid, dim3(256), ldsd, st, a);
    }
    else if (a.carried) hipLaunchKernelGGL((k_split_dist<NK, 2, true>), grid, dim3(256), ldsd, st, a);
    else hipLaunchKernelGGL((k_split_dist<NK, 2, false>), grid, dim3(256), ldsd, st, a);
  }
  else if (pass == 3) hipLaunchKernelGGL((k_split<NK, 3, true>), grid, dim3(256), SplitGeom<NK>::LDS_BYTES3, st, a);
  else if (pass == 1) {
    if (a.carried) {
      if (f16) hipLaunchKernelGGL((k_split_carry<NK, 1, true>), grid, dim3(256), lds, st, a);
      else hipLaunchKernelGGL((k_split_carry<NK, 1, false>), grid, dim3(256), lds, st, a);
    }
    else if (f16) hipLaunchKernelGGL((k_split<NK, 1, true>), grid, dim3(256), lds, st, a);
    else hipLaunchKernelGGL((k_split<NK, 1, false>), grid, dim3(256), lds, st, a);
  } else {
    if (a.carried) {
      if (f16) hipLaunchKernelGGL((k_split_carry<NK, 2, true>), grid, dim3(256), lds, st, a);
      else hipLaunchKernelGGL((k_split_carry<NK, 2, false>), grid, dim3(256), lds, st, a);
    }
    else if (f16) hipLaunchKernelGGL((k_split<NK, 2, true>), grid, dim3(256), lds, st, a);
    else hipLaunchKernelGGL((k_split<NK, 2, false>), grid, dim3(256), lds, st, a);
  }
  return hipGetLastError();
}

// `a` is filled by mar_launch_flash (units, parts, buffers); this picks the instantiation for a.dk.
hipError_t mar_split_launch(const FlashArgs& a, int pass, bool f16, dim3 grid, hipStream_t st) {
  hipError_t e = hipErrorInvalidValue;
  switch (sp_nk(a.dk)) {
    case 2: e = sp_launch<2>(a, pass, f16, grid, st); break;
    case 4: e = sp_launch<4>(a, pass, f16, grid, st); break;
    case 6: e = sp_launch<6>(a, pass, f16, grid, st); break;
    case 7: e = sp_launch<7>(a, pass, f16, grid, st); break;
    case 8: e = sp_launch<8>(a, pass, f16, grid, st); break;
    case 12: e = sp_launch<12>(a, pass, f16, grid, st); break;
    case 16: e = sp_launch<16>(a, pass, f16, grid, st); break;
    case 25: e = sp_launch<25>(a, pass, f16, grid, st); break;
  }
  if (e == hipSuccess && pass == 2 && a.rem_k > 1) {
    hipLaunchKernelGGL(k_split_merge2, dim3((unsigned)((a.rem_rows + 7) / 8)), dim3(256), 0, st, a);
    e = hipGetLastError();
  }
  return e;
}
