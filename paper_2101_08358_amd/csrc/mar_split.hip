// Contraction passes of the bilinear models (DistMult, ComplEx, Dot) on the 16-bit matrix pipe (gfx950): scores with
// online softmax and the edge-side gradient, the negatives' gradient, and rank counts.
//
// fp32 precision (F16 = true).  Every operand value is written as v 2^e = hi + lo, both f16 (mar_split.h; one exponent
// per 16 rows puts the largest value just below 2^15), and every product a b is taken as
//     a_hi b_hi + a_lo b_hi + a_hi b_lo
// with v_mfma_f32_32x32x16_f16 (fp32 accumulation), which runs at 16 times the rate of the fp32 matrix instructions.
// hi + lo holds 23-24 significant bits of every value down to 2^-17 of its block's largest (below that an absolute
// 2^-40 of the largest), the dropped product is below 2^-22 of its pair, and the sums see 3 roundings per 16 terms
// where the fp32 instruction sees 4, so a pass is as accurate as its fp32 form: against 64 bits a dot product of 128
// (1024) normal values is off by 1.5e-7 (3.5e-7) of its norm, with v_mfma_f32_16x16x4_f32 by 1.9e-7 (5.6e-7).
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
// Lane layouts (lane = 32 h + m; i = lane % 16, G = lane / 16):
//   v_mfma_f32_32x32x16_f16 / bf16: A lane holds row m, contraction slots 8h .. 8h+7; B lane holds column m, the same
//   slots; D lane holds column m, register v = row 8 (v / 4) + 4h + v % 4.  Which contraction index a slot stands for
//   is free as long as A and B agree.
//   Score product S^T[y][x] = sum_c Y[y][c] X[x][c]: A = Y from LDS (16-byte read of row m, columns 16 s + 8h ..),
//   B = X fragments in registers.
//   Second product O^T[c][x] += sum_y Y[y][c] W[y][x] over the tile's 32 rows in two steps of 16: B of step k = W of
//   the lane's own score registers 8k .. 8k+7, so slot 8h + j stands for row 16k + 4h + j (j < 4), 16k + 8 + 4h + j - 4
//   (j >= 4).  A = Y^T by the LDS transpose read (ds_read_b64_tr_b16): within 16 lanes, lane i passes the address of 4
//   consecutive 16-bit values and receives, as its j-th value, value (i % 4) of lane 4j + i / 4; with lane i pointing
//   at row 4h + i / 4, columns 32 cb + 16 (G % 2) + 4 (i % 4), lane m receives Y[4h + j][32 cb + m].  (With NK odd the
//   last block reads units that no one has written: columns beyond dk, whose outputs are not stored.)
#include <type_traits>

#include "mar_common.h"
#include "mar_flash.h"
#include "mar_split.h"

typedef float v16f __attribute__((ext_vector_type(16)));
typedef _Float16 v8h __attribute__((ext_vector_type(8)));
typedef __bf16 v8b __attribute__((ext_vector_type(8)));
typedef short v4s __attribute__((ext_vector_type(4)));
typedef short v8s __attribute__((ext_vector_type(8)));
typedef float v2f __attribute__((ext_vector_type(2)));
typedef _Float16 v2h __attribute__((ext_vector_type(2)));
typedef __bf16 v2b __attribute__((ext_vector_type(2)));

template <bool F16> __device__ __forceinline__ v16f mfma32(v8s a, v8s b, v16f c) {
  if (F16) return __builtin_amdgcn_mfma_f32_32x32x16_f16(__builtin_bit_cast(v8h, a), __builtin_bit_cast(v8h, b), c, 0, 0, 0);
  return __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(v8b, a), __builtin_bit_cast(v8b, b), c, 0, 0, 0);
}

// v = hi + lo, two values per step: one packed conversion and two mixed-precision multiply-adds (f16; neg1 = -1 in a
// register the compiler cannot see through, or it would turn the multiply-add into a conversion and a subtraction),
// two packed conversions with the unpacking between them (bf16).
template <bool F16, int O> __device__ __forceinline__ void split8(const float (&v)[16], float neg1, v8s& hi, v8s& lo) {
  v4i hw, lw;                                              // two 16-bit values per word
#pragma unroll
  for (int i = 0; i < 4; ++i) {
    const float p0 = v[O + 2 * i], p1 = v[O + 2 * i + 1];
    if (F16) {
      const v2h h = __builtin_convertvector((v2f){p0, p1}, v2h);
      const v2h l = {(_Float16)__builtin_fmaf((float)h[0], neg1, p0), (_Float16)__builtin_fmaf((float)h[1], neg1, p1)};
      hw[i] = __builtin_bit_cast(int, h); lw[i] = __builtin_bit_cast(int, l);
    } else {
      const v2b h = __builtin_convertvector((v2f){p0, p1}, v2b);
      const v2b l = __builtin_convertvector((v2f){p0 - (float)h[0], p1 - (float)h[1]}, v2b);
      hw[i] = __builtin_bit_cast(int, h); lw[i] = __builtin_bit_cast(int, l);
    }
  }
  hi = __builtin_bit_cast(v8s, hw); lo = __builtin_bit_cast(v8s, lw);
}

__device__ __forceinline__ unsigned lds_address_b(const char* p) {
  return (unsigned)(unsigned long long)(__attribute__((address_space(3))) const char*)p;
}
__device__ __forceinline__ v4s lds_read_tr(const char* p) {
  return __builtin_amdgcn_ds_read_tr16_b64_v4i16((__attribute__((address_space(3))) v4s*)p);
}
__device__ __forceinline__ v8s join8(v4s a, v4s b) { return __builtin_shufflevector(a, b, 0, 1, 2, 3, 4, 5, 6, 7); }

#define SP_PEND 6                                          // candidates whose comparisons a lane of pass 3 keeps for the end (5 bits of a word each)
#define SP_FULL 8                                          // added to their number: this lane takes no more (above SP_PEND)
template <int NK>
struct SplitGeom {
  static constexpr int NB = sp_nb(NK);
  static constexpr int UNITS = sp_units(NK);
  static constexpr int PA = sp_pitch(NK);
  static constexpr int PLANE = sp_plane(NK);
  static constexpr int IMG = sp_image(NK);
  static constexpr int NCH = IMG / 1024;                   // 1 KB pieces of an image
  static constexpr size_t LDS_BYTES = 2 * (size_t)IMG + 4 * SP_TY * 4;   // two images, and (pass 2) the log-sum-exp of a tile's edges
  static constexpr size_t LDS_BYTES3 = 2 * (size_t)IMG + 2 * SP_PEND * 256 * 4;   // two images, and the lanes' pending candidates: id, how often
};

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
// throughout 1,110, no two rows equal 229.  (20,000 edges, 1,000 candidates of 400 floats, half equal: 1,075 us, 25,000
// and 355; 233 without.  One wave per SIMD hides little of the loads.)
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

#ifndef SP_PD
#define SP_PD 4
#endif
#ifndef SP_PG
#define SP_PG 2
#endif
// Waves per SIMD = workgroups per CU: pass 3 keeps no output accumulators.
constexpr int sp_waves(int nk, int pass) { return pass == 3 ? (nk <= 8 ? 3 : (nk <= 16 ? 2 : 1)) : (nk <= 8 ? 2 : 1); }

// ------------------------------------------------------------------------ the passes -----
// PASS 1: scores, online softmax and gQ = P K for 128 edges of one chunk-side (32 per wave) against the chunk's
// negatives.  No weights are kept for pass 2:
// PASS 2: gK = P^T Q for 128 negatives of one chunk-side against the chunk's edges, with the scores computed again and
// P = exp(score - lse) from the finished log-sum-exp.  Writing the weights out and reading them back costs 8 bytes of
// memory traffic per pair, computing a score again 6 d 16-bit flops: at this matrix rate the second is cheaper.
// PASS 3 (evaluation): counts the negatives that score above the positive; ranks start at 1 and the parts of a stripe add
// their counts.
template <int NK, int PASS, bool F16>
__global__ void __launch_bounds__(256) MAR_WAVES_PER_SIMD(sp_waves(NK, PASS))
k_split(FlashArgs a) {
  typedef SplitGeom<NK> SG;
  constexpr int NB = SG::NB, UNITS = SG::UNITS, PA = SG::PA, PLANE = SG::PLANE, IMG = SG::IMG;
  constexpr int TY = SP_TY;
  constexpr int NCW = (SG::NCH + 3) / 4;                   // 1 KB pieces of an image per wave
  constexpr float LOG2E = 1.44269504088896341f;
  extern __shared__ __attribute__((aligned(16))) char smem[];
  float* const aux_all = reinterpret_cast<float*>(smem + 2 * IMG);   // PASS 2: [2][2][TY] log-sum-exp of the tile's edges, log2 units

  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const int h = lane >> 5, m = lane & 31;
  FlashUnit u;
  if (!flash_unit(a, u)) return;
  const int cs = u.cs, side = cs & 1, c = cs >> 1;
  const int ne = min(a.S, a.n - c * a.S);                 // edges in this chunk
  const int n_x = PASS == 2 ? a.N : ne;                   // stationary rows
  const int n_y = PASS == 2 ? ne : a.N;                   // streamed rows
  if (u.stripe * SP_SR >= n_x) return;
  const size_t q_base = (size_t)side * a.B + (size_t)c * a.S;        // first Q row of the chunk
  const int dk = a.dk;
  float neg1 = -1.f;
  asm volatile("" : "+v"(neg1));

  // ---- stationary fragments from the rows' own images: slots of step s = columns 16 s + 8h .. +7 of row x
  const int x = u.stripe * SP_SR + wave * 32 + m;
  const bool xv = x < n_x;
  const size_t xtile = (size_t)cs * a.ximg_tiles + u.stripe * (SP_SR / TY) + wave;
  const int swz = 16 * sp_swizzle(UNITS, m);              // of row m of a tile, in bytes
  const char* xrow = a.ximg + xtile * IMG + m * PA;
  v8s xh[NK], xl[NK];
#pragma unroll
  for (int s = 0; s < NK; ++s) {
    xh[s] = (v8s){0, 0, 0, 0, 0, 0, 0, 0};
    xl[s] = (v8s){0, 0, 0, 0, 0, 0, 0, 0};
    if (xv) {
      xh[s] = *reinterpret_cast<const v8s*>(xrow + ((16 * h + 32 * s) ^ swz));
      xl[s] = *reinterpret_cast<const v8s*>(xrow + PLANE + ((16 * h + 32 * s) ^ swz));
    }
  }
  float ex = 0.f;                                         // exponent of the row's block
  bool xbad = false;
  if (F16 && xv) {
    ex = a.xexp[xtile * 2 + (m >> 4)];
    xbad = ex > 0.5f * SP_NONFINITE;
    if (xbad) ex -= SP_NONFINITE;
  }
  // Pass 3.  A comparison is close if the score is within sqrt(dk) (2^-23 |q| + 2^-25) |n| of the positive's, q and n
  // scaled by their blocks' exponents, |n| the largest of the block.  The rounding errors of a chain of dk steps are
  // independent and each below 2^-24 |q| |n| (the partial sums are), 0.3 of that on average: the first term is seven
  // standard deviations where all products have one sign, and ten times that where they do not.  hi + lo holds a value to
  // 2^-24 of itself and no better than 2^-25: over a row that is the second term, which matters where q is far below its
  // block's largest row (or its block's exponent at the limit); for n it lies inside the first, the block's |n| being
  // 2^14 at least.  A zero row's scores are exactly zero.
  float posx = 0.f, tolx = 0.f;
  const float* qrow = nullptr;
  int* const pend = reinterpret_cast<int*>(smem + 2 * IMG) + threadIdx.x;
  int npend = 0;                                           // pending candidates; + SP_FULL: no more are taken
  if (PASS == 3) {
    float n2 = 0.f;
#pragma unroll
    for (int s = 0; s < NK; ++s) {
      const v8h f = __builtin_bit_cast(v8h, xh[s]);
#pragma unroll
      for (int i = 0; i < 8; ++i) n2 += (float)f[i] * (float)f[i];
    }
    n2 += __shfl_xor(n2, 32);
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
  }
  const int32_t* const cand = (side == MAR_SIDE_DST ? a.neg_dst : a.neg_src) + (size_t)c * a.N;   // ids of the streamed rows
  int own = -1, nown = 0;                                  // pass 3: the replaced endpoint's id, how often it came up close
  if (PASS == 3 && xv) own = (side == MAR_SIDE_DST ? a.dst : a.src)[(size_t)c * a.S + x];
  // Pass 3, all lanes of the wave: candidates of the tile at y0 that score above this lane's edge, settled as a whole (in
  // the lanes of the wave's first half).
  auto exact_tile = [&](int y0) -> int {
    int ln = lane;
    asm volatile("" : "+v"(ln));                          // what follows is rare: nothing of it is kept across tiles
    const int i = ln & 15, G = ln >> 4, x0 = u.stripe * SP_SR + wave * 32;
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

  constexpr int NO = PASS == 3 ? 1 : NB;
  v16f oacc[NO];
#pragma unroll
  for (int cb = 0; cb < NO; ++cb) oacc[cb] = (v16f)(0.f);
  float mref = -3.0e38f, lrun = 0.f;                      // softmax reference (log2 units; F16: an integer) and sum
  int cnt = 0;

  const int ntiles_all = (n_y + TY - 1) / TY;
  const int t_begin = u.part * u.tps;
  const int ntiles = min(ntiles_all, t_begin + u.tps);

  // ---- images of the streamed rows, copied into LDS one tile ahead; a register load issued behind the copies is the
  // fence (memory operations of a wave complete in order): once its value is there the image is in LDS.  The fence is
  // the load of the tile's two exponents; pass 2 also loads the softmax statistics of edge threadIdx % TY behind it.
  const char* ybase = a.yimg + (size_t)cs * a.yimg_tiles * IMG;
  const BufRsrc expsrc = buf_rsrc(F16 ? (const void*)(a.yexp + (size_t)cs * a.yimg_tiles * 2) : (const void*)ybase, (uint32_t)a.yimg_tiles * 8);
  const BufRsrc mlsrc = buf_rsrc(a.ml + q_base * 2, PASS == 2 ? (uint32_t)ne * 8 : 0u);
  const int wave_s = __builtin_amdgcn_readfirstlane(wave);
  const int f_row = threadIdx.x % TY;
  const size_t ml_stride = (size_t)2 * a.B;               // rows per part of pass 1's statistics
  float2 ye_next = make_float2(0.f, 0.f), yn_next = make_float2(0.f, 0.f), st_ml = make_float2(0.f, 0.f);
  const BufRsrc normsrc = buf_rsrc(PASS == 3 ? (const void*)(a.ynorm + (size_t)cs * a.yimg_tiles * SP_NORMS) : (const void*)ybase, PASS == 3 ? (uint32_t)a.yimg_tiles * (SP_NORMS * 4) : 0u);
  int token = 0;
  auto dma_piece = [&](int t, int buf, int q) {            // piece q of this wave of tile t into buffer `buf`
    const v4i ywords = buf_words(ybase + (size_t)t * IMG, IMG);
    const int pc = 4 * q + wave_s;
    if (pc < SG::NCH) buf_load4_to_lds(ywords, lds_address_b(smem) + buf * IMG + pc * 1024, lane * 16, pc * 1024, token);
  };
  auto dma_fence = [&](int t) {
    ye_next = buf_load2(expsrc, token, t * 8);
    if (PASS == 3) yn_next = buf_load2(normsrc, token, t * (SP_NORMS * 4));
    if (PASS == 2) st_ml = buf_load2(mlsrc, f_row * 8 + token, t * TY * 8);
  };
  auto dma_land = [&](int t, int buf) {
    asm volatile("" : "+v"(ye_next.x), "+v"(ye_next.y));
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
  // away and the other groups are immediate offsets.
  constexpr int FB = sp_group(UNITS) / 2, TB = sp_group(UNITS) / 4;   // steps of the score product / column blocks to a group
  const int fofs = m * PA + ((16 * h) ^ swz);              // score product, step s = FB q + j: (fofs ^ 32 j) + 32 FB q
  const int ty = 4 * h + ((lane & 15) >> 2), tc = 32 * ((lane >> 4) & 1) + 8 * (lane & 3);   // second product, rows ty and ty + 8
  const int trofs0 = ty * PA + (tc ^ (16 * sp_swizzle(UNITS, ty))), trofs1 = (ty + 8) * PA + (tc ^ (16 * sp_swizzle(UNITS, ty + 8)));
                                                           // column block cb = TB q + j: (trofs ^ 64 j) + 64 TB q
  auto frag_at = [](int fb, int s) { return (fb ^ (s % FB * 32)) + s / FB * FB * 32; };
  for (int t = t_begin; t < ntiles; ++t) {
    const int buf = (t - t_begin) & 1;
    const int fb = buf * IMG + fofs;
    const bool has_next = t + 1 < ntiles;                  // uniform
    const float2 ye = ye_next, yn = yn_next;
    const int y0 = t * TY;
    const bool masked = PASS != 2 && y0 + TY > n_y;

    // -- scores; the fragments of the streamed rows are read PD steps ahead of the instructions that consume them
    v16f sacc = (v16f)(0.f);
    {
      constexpr int PD = NK < SP_PD ? NK : SP_PD;
      v8s fh[PD], fl[PD];
#pragma unroll
      for (int s = 0; s < PD; ++s) {
        fh[s] = *reinterpret_cast<const v8s*>(smem + frag_at(fb, s));
        fl[s] = *reinterpret_cast<const v8s*>(smem + PLANE + frag_at(fb, s));
      }
#pragma unroll
      for (int s = 0; s < NK; ++s) {
        const v8s ah = fh[s % PD], al = fl[s % PD];
        if (s + PD < NK) {
          fh[s % PD] = *reinterpret_cast<const v8s*>(smem + frag_at(fb, s + PD));
          fl[s % PD] = *reinterpret_cast<const v8s*>(smem + PLANE + frag_at(fb, s + PD));
        }
        sacc = mfma32<F16>(al, xh[s], sacc);
        sacc = mfma32<F16>(ah, xl[s], sacc);
        sacc = mfma32<F16>(ah, xh[s], sacc);
        // the next tile's pieces are issued between the steps: a burst of them holds the wave at the memory pipeline's
        // queue (rows of 400: a pass 1075 us with the copies at the tile's start, 915 spread, 810 without any)
        if (has_next) {
#pragma unroll
          for (int q = s * NCW / NK; q < (s + 1) * NCW / NK; ++q) dma_piece(t + 1, buf ^ 1, q);
          if (s == NK - 1) dma_fence(t + 1);
        }
        __builtin_amdgcn_sched_barrier(0);                 // keeps the reads PD steps ahead of their use
      }
    }
    // -- scale of the two 16-row blocks: score = sacc 2^-(ex + ey); never 0, or a masked row's -inf would become NaN
    // (two blocks at the largest exponent: scores below 2^-100 either way)
    float k0 = PASS == 3 ? 1.f : LOG2E, k1 = k0, e0 = 0.f, e1 = 0.f;
    bool settle = false;                                   // pass 3, uniform over the wave: the tile is settled as a whole
    if (F16) {
      const bool ybad = ye.x > 0.5f * SP_NONFINITE || ye.y > 0.5f * SP_NONFINITE;
      e0 = ye.x > 0.5f * SP_NONFINITE ? ye.x - SP_NONFINITE : ye.x;
      e1 = ye.y > 0.5f * SP_NONFINITE ? ye.y - SP_NONFINITE : ye.y;
      k0 = __builtin_ldexpf(k0, max(-140, min(126, -(int)(ex + e0))));
      k1 = __builtin_ldexpf(k1, max(-140, min(126, -(int)(ex + e1))));
      settle = PASS == 3 && __any(ybad || xbad);
    }
    if (masked) {                                          // the chunk's last, partial tile (uniform): rows beyond it weigh nothing
#pragma unroll
      for (int v = 0; v < 16; ++v) {
        if (y0 + 8 * (v / 4) + 4 * h + v % 4 >= n_y) sacc[v] = -__builtin_inff();
      }
    }
    if (PASS == 3) {
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
          // (20,000 edges, 1,000 candidates of 100 floats drawn by degree from a power law: 78 to 90 us, 1,200 to 3,100 with
          // every copy compared, 91 as fp32 contraction, 59 for uniform candidates.)
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
            pend[256 * npend] = ~(y0 + 8 * (v >> 2) + 4 * h + (v & 3));
            pend[256 * (SP_PEND + npend++)] = 1;
          }
          if (!settle && many) {
            const int id_t = cand[min(y0 + lane % TY, n_y - 1)];   // lane i: the tile's row i % TY
#pragma unroll
            for (int v = 0; v < 16; ++v) {
              same |= __shfl(id_t, 8 * (v / 4) + 4 * h + v % 4) == own ? 1u << v : 0u;
              asm volatile("" : "+v"(same));
            }
            same &= close;
            if (__any((close & ~same) != 0u)) {
              const float nrm = buf_load1(normsrc, (2 + lane % TY) * 4, t * (SP_NORMS * 4));
#pragma unroll
              for (int v = 0; v < 16; ++v) {
                const float dif = __builtin_fmaf(sacc[v], v < 8 ? k0 : k1, -p), nv = __shfl(nrm, 8 * (v / 4) + 4 * h + v % 4);
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
                const int v = __ffs((int)rest) - 1, id = cand[y0 + 8 * (v >> 2) + 4 * h + (v & 3)];
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
    } else {
      // -- weights of the lane's 16 pairs, split; register v <-> row y0 + 8 (v / 4) + 4h + v % 4
      float w[16];
      if (PASS == 1 || F16) {
        float tmax;
        if (PASS == 1) {
          float a0 = sacc[0], a1 = sacc[8];
#pragma unroll
          for (int v = 1; v < 8; ++v) { a0 = fmaxf(a0, sacc[v]); a1 = fmaxf(a1, sacc[8 + v]); }
          tmax = fmaxf(__builtin_fmaf(a0, k0, -e0), __builtin_fmaf(a1, k1, -e1));
        } else {
#pragma unroll
          for (int q = 0; q < 4; ++q) {
            const float4 l4 = *reinterpret_cast<const float4*>(aux_all + 2 * buf * TY + 8 * q + 4 * h);
            const float4 m4 = *reinterpret_cast<const float4*>(aux_all + (2 * buf + 1) * TY + 8 * q + 4 * h);
            const float kq = q < 2 ? k0 : k1;
            w[4 * q] = __builtin_fmaf(sacc[4 * q], kq, -l4.x) - m4.x;
            w[4 * q + 1] = __builtin_fmaf(sacc[4 * q + 1], kq, -l4.y) - m4.y;
            w[4 * q + 2] = __builtin_fmaf(sacc[4 * q + 2], kq, -l4.z) - m4.z;
            w[4 * q + 3] = __builtin_fmaf(sacc[4 * q + 3], kq, -l4.w) - m4.w;
          }
          float a0 = w[0], a1 = w[8];
#pragma unroll
          for (int v = 1; v < 8; ++v) { a0 = fmaxf(a0, w[v]); a1 = fmaxf(a1, w[8 + v]); }
          tmax = fmaxf(a0 - e0, a1 - e1);
        }
        if (__any(tmax > mref + (F16 ? 15.f : 16.f * LOG2E))) {
          const float tall = fmaxf(tmax, __shfl_xor(tmax, 32));
          const float mnew = fmaxf(mref, F16 ? __builtin_ceilf(tall) - 8.f : tall);
          float alpha = __builtin_amdgcn_exp2f(mref - mnew);
          asm volatile("" : "+v"(alpha));                  // a real branch: keeps the rescale from being executed speculatively
          lrun *= alpha;
#pragma unroll
          for (int cb = 0; cb < NO; ++cb) {
            if (NK > 8) asm volatile("" : "+a"(oacc[cb]));
            oacc[cb] *= alpha;
            if (NK > 8) asm volatile("" : "+a"(oacc[cb]));   // wide rows: back to the accumulation registers, one block at a time
          }
          mref = mnew;
        }
        const float r0 = e0 + mref, r1 = e1 + mref;        // exact: integers (bf16: no exponents)
        if (PASS == 1) {
          float l0 = 0.f, l1 = 0.f;
#pragma unroll
          for (int v = 0; v < 16; ++v) w[v] = __builtin_amdgcn_exp2f(__builtin_fmaf(sacc[v], v < 8 ? k0 : k1, v < 8 ? -r0 : -r1));
#pragma unroll
          for (int v = 0; v < 8; ++v) { l0 += w[v]; l1 += w[8 + v]; }
          lrun += F16 ? __builtin_ldexpf(l0, (int)e0) + __builtin_ldexpf(l1, (int)e1) : l0 + l1;
        } else {
#pragma unroll
          for (int v = 0; v < 16; ++v) w[v] = __builtin_amdgcn_exp2f(w[v] - (v < 8 ? r0 : r1));
        }
      } else {                                             // pass 2, bf16: no reference needed
#pragma unroll
        for (int q = 0; q < 4; ++q) {
          const float4 l4 = *reinterpret_cast<const float4*>(aux_all + 2 * buf * TY + 8 * q + 4 * h);
          w[4 * q] = __builtin_amdgcn_exp2f(__builtin_fmaf(sacc[4 * q], LOG2E, -l4.x));
          w[4 * q + 1] = __builtin_amdgcn_exp2f(__builtin_fmaf(sacc[4 * q + 1], LOG2E, -l4.y));
          w[4 * q + 2] = __builtin_amdgcn_exp2f(__builtin_fmaf(sacc[4 * q + 2], LOG2E, -l4.z));
          w[4 * q + 3] = __builtin_amdgcn_exp2f(__builtin_fmaf(sacc[4 * q + 3], LOG2E, -l4.w));
        }
      }
      v8s wh[2], wl[2];
      split8<F16, 0>(w, neg1, wh[0], wl[0]);
      split8<F16, 8>(w, neg1, wh[1], wl[1]);
      // -- O^T[c][x] += sum_y Y[y][c] W[y][x]: group q = (column block q / 2, step q % 2), read PG groups ahead
      constexpr int NG = 2 * NO, PG = SP_PG < NG ? SP_PG : NG;
      const int tb0 = buf * IMG + trofs0, tb1 = buf * IMG + trofs1;
      v8s gh[PG], gl[PG];
      auto read_group = [&](int q, v8s& vh, v8s& vl) {
        const int cb = q / 2, o = (q % 2) * 16 * PA + cb / TB * TB * 64;
        const char *r0 = smem + ((tb0 ^ (cb % TB * 64)) + o), *r1 = smem + ((tb1 ^ (cb % TB * 64)) + o);
        vh = join8(lds_read_tr(r0), lds_read_tr(r1));
        vl = join8(lds_read_tr(r0 + PLANE), lds_read_tr(r1 + PLANE));
      };
#pragma unroll
      for (int q = 0; q < PG; ++q) read_group(q, gh[q], gl[q]);
#pragma unroll
      for (int q = 0; q < NG; ++q) {
        const v8s ah = gh[q % PG], al = gl[q % PG];
        if (q + PG < NG) read_group(q + PG, gh[q % PG], gl[q % PG]);
        oacc[q / 2] = mfma32<F16>(al, wh[q % 2], oacc[q / 2]);
        oacc[q / 2] = mfma32<F16>(ah, wl[q % 2], oacc[q / 2]);
        oacc[q / 2] = mfma32<F16>(ah, wh[q % 2], oacc[q / 2]);
        __builtin_amdgcn_sched_barrier(0);
      }
    }
    if (has_next) {
      dma_land(t + 1, buf ^ 1);
      __syncthreads();                                     // tile t + 1 is in LDS; every wave is done with tile t
    }
  }

  // ---- epilogue
  if (PASS == 3) {
    constexpr int UB = NK <= 16 ? 4 : 8;                   // 16-column blocks whose loads are in flight at once
    for (int i = nown ? -1 : 0; i < npend % SP_FULL; ++i) {
      const int e = i < 0 ? own : pend[256 * i], id = e < 0 ? cand[~e] : e;
      const float* yrow = a.table + (size_t)id * a.dim;
      const float s = a.dim % 4 == 0 ? sp_exact_score<true, UB>(qrow, yrow, a.dim, sp_chain(dk)) : sp_exact_score<false, UB / 2>(qrow, yrow, a.dim, sp_chain(dk));
      if (s > posx) cnt += i < 0 ? nown : pend[256 * (SP_PEND + i)];
    }
    cnt += __shfl_xor(cnt, 32);
    if (h == 0 && xv && cnt) atomicAdd((side == MAR_SIDE_DST ? a.rank_dst : a.rank_src) + (size_t)c * a.S + x, cnt);
    return;
  }
  int oshift = 0;                                          // gradient rows are written as accumulator x 2^oshift
  float* orow;
  if (PASS == 1) {                                         // the part's statistics and unnormalised gradient rows
    float ltot = lrun + __shfl_xor(lrun, 32);
    // sum = mantissa 2^p, reference + p: the statistics' reference is close to the log-sum-exp itself
    int p = 0;
    if (F16 && ltot > 0.f && ltot < 3.0e38f) p = (int)((__float_as_uint(ltot) >> 23) & 255u) - 127;
    oshift = -p;
    const size_t part_row = (size_t)u.part * 2 * a.B + q_base + x;
    const bool extra = u.rem && u.part > 0;                // parts 1.. of a split stripe
    const size_t xr = (size_t)(u.part - 1) * a.rem_rows + (size_t)(u.unit - a.whole_units) * SP_SR + wave * 32 + m;
    float* ml_out = extra ? a.mlx + xr * 2 : a.ml + (u.rem ? q_base + x : part_row) * 2;
    orow = extra ? a.outx + xr * dk : a.out + (u.rem ? q_base + x : part_row) * dk;
    if (h == 0 && xv) *reinterpret_cast<float2*>(ml_out) = make_float2(mref + (float)p, __builtin_ldexpf(ltot, -p));
  } else {                                                 // gradient row of part `part` of each negative's occurrence
    if (F16) oshift = mref > -1.0e38f ? (int)mref : 0;     // weights were formed relative to the reference
    orow = a.out + (a.roles * (size_t)a.n + ((side == MAR_SIDE_DST ? 0 : (size_t)a.cn) + (size_t)c * a.N + x) * a.sy + (u.rem ? 0 : u.part)) * dk;
    if (u.rem && u.part > 0) orow = a.outx + ((size_t)(u.part - 1) * a.rem_rows + (size_t)(u.unit - a.whole_units) * SP_SR + wave * 32 + m) * dk;
  }
  if (xv) {
#pragma unroll
    for (int cb = 0; cb < NO; ++cb) {
#pragma unroll
      for (int q = 0; q < 4; ++q) {
        const int col = 32 * cb + 8 * q + 4 * h;
        if (col < dk)
          *reinterpret_cast<float4*>(orow + col) =
              make_float4(__builtin_ldexpf(oacc[cb][4 * q], oshift), __builtin_ldexpf(oacc[cb][4 * q + 1], oshift),
                          __builtin_ldexpf(oacc[cb][4 * q + 2], oshift), __builtin_ldexpf(oacc[cb][4 * q + 3], oshift));
      }
    }
  }
}

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
size_t mar_split_image_bytes(int dk) { return (size_t)sp_image(sp_nk(dk)); }

template <int NK> static hipError_t sp_prepare() {
  constexpr size_t lds = SplitGeom<NK>::LDS_BYTES;
  hipError_t e = hipSuccess;
#define PREP(P, F) if (e == hipSuccess) e = hipFuncSetAttribute(reinterpret_cast<const void*>(&k_split<NK, P, F>), hipFuncAttributeMaxDynamicSharedMemorySize, (int)(P == 3 ? SplitGeom<NK>::LDS_BYTES3 : lds))
  PREP(1, true); PREP(2, true); PREP(3, true); PREP(1, false); PREP(2, false);
#undef PREP
  return e;
}
hipError_t mar_split_prepare(int dk) {
  switch (sp_nk(dk)) {
    case 16: return sp_prepare<16>();
    case 25: return sp_prepare<25>();
    default: static_assert(SplitGeom<12>::LDS_BYTES3 <= 64 * 1024, "narrower instantiations stay below the default limit"); return hipSuccess;
  }
}

template <int NK> static hipError_t sp_launch(const FlashArgs& a, int pass, bool f16, dim3 grid, hipStream_t st) {
  constexpr size_t lds = SplitGeom<NK>::LDS_BYTES;
  static_assert(SplitGeom<NK>::LDS_BYTES3 <= 160 * 1024, "two images in LDS");
  if (pass == 3) hipLaunchKernelGGL((k_split<NK, 3, true>), grid, dim3(256), SplitGeom<NK>::LDS_BYTES3, st, a);
  else if (pass == 1) {
    if (f16) hipLaunchKernelGGL((k_split<NK, 1, true>), grid, dim3(256), lds, st, a);
    else hipLaunchKernelGGL((k_split<NK, 1, false>), grid, dim3(256), lds, st, a);
  } else {
    if (f16) hipLaunchKernelGGL((k_split<NK, 2, true>), grid, dim3(256), lds, st, a);
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
