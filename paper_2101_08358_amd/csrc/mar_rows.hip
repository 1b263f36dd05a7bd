// Row-wise (bandwidth-bound) kernels of the training step (gfx950): gather of the batch's
// rows into dense contraction operands, the chain rule from operand gradients back to the
// source / relation / destination rows, the per-row gradient reduction over the row-sorted
// order, and the sparse Adagrad scatter.
#include <type_traits>

#include "mar_common.h"
#include "mar_split.h"
#include "mar_sort_dev.h"

struct RowArgs {
  const float *node_emb, *rel_emb;
  const int32_t *src, *rel, *dst, *neg_src, *neg_dst;
  int32_t n, cn, B, C, N, S, dim, dk, model;
  float* shift;          // TransE on images: what all rows of the batch have in common (common_offset), for the passes
  int32_t num_nodes;
  int32_t sy1, sy2;      // parts per stripe in the two contraction passes
  int32_t roles;         // 3, or 2 for the relation-free Dot score
  float ml_log2;         // natural-log units of one unit of the softmax references (see FlashArgs)
};

template <int GL> __device__ __forceinline__ float group_sum(float v) {
#pragma unroll
  for (int o = GL / 2; o >= 1; o >>= 1) v += __shfl_xor(v, o);
  return v;
}

// ---------------------------------------------------------------------- gather -----
// Edge blocks build the two edge-side operands of each edge
//     side DST (negatives replace d): a_ej = <q, n_j>,  q = s*r (DistMult), s.r complex (ComplEx)
//     side SRC (negatives replace s): b_ej = <q, m_j>,  q = r*d,            conj(r).d
//   for TransE the scores are -|q - n_j| with q = s + r and q = d - r; also the positive score.
// Negative blocks bring the negatives' rows into the layout the contraction reads.
// Dense fp32 matrices, one row after the other, or hi/lo images (mar_split.h); for images a workgroup takes
// 16, 32 or 64 consecutive rows of one chunk (whole 16-row blocks, so a block's exponent is found through LDS), the
// rows of the chunk's last tile beyond its own being written as zeros.
// A lane group issues the loads of all its rows (E edges, P negatives) before the first use: the gathers are bound by
// the latency of scattered row reads (address translation included), so bytes in flight per lane are what counts.
// A lane holds NV float4s of a row.  VEC (dim is a multiple of 4): float4 v holds columns 4 (l + GL v) .. +3; for ComplEx
// columns 2 (l + GL v), +1 of the real half and of the imaginary half (re, re, im, im).  Otherwise element c of float4 v
// is column l + GL (4 v + c); for ComplEx columns l + GL 2v and l + GL (2v + 1) of either half (re, re, im, im).
// MODEL: the score function, resolved at compile time.  FORM: images of scaled f16 parts, images of bf16 parts without
// exponents, or dense matrices (TransE; small evaluations of the bilinear models).
constexpr int PREP_F16 = 0, PREP_BF16 = 1, PREP_DENSE = 2;
template <int GL, bool VEC, bool CPLX>
__device__ __forceinline__ float4 load_cols(const float* __restrict__ row, int l, int v, int dim) {
  float4 x = make_float4(0.f, 0.f, 0.f, 0.f);
  const int h = dim >> 1;
  if (VEC && CPLX) {
    const int k = 2 * (l + GL * v);
    if (k < h) {
      const float2 re = *reinterpret_cast<const float2*>(row + k), im = *reinterpret_cast<const float2*>(row + h + k);
      x = make_float4(re.x, re.y, im.x, im.y);
    }
  } else if (VEC) {
    const int k = 4 * (l + GL * v);
    if (k < dim) x = *reinterpret_cast<const float4*>(row + k);
  } else if (CPLX) {
    const int k0 = l + GL * (2 * v), k1 = k0 + GL;
    if (k0 < h) { x.x = row[k0]; x.z = row[h + k0]; }
    if (k1 < h) { x.y = row[k1]; x.w = row[h + k1]; }
  } else {
    const int k = l + GL * (4 * v);
    if (k < dim) x.x = row[k];
    if (k + GL < dim) x.y = row[k + GL];
    if (k + 2 * GL < dim) x.z = row[k + 2 * GL];
    if (k + 3 * GL < dim) x.w = row[k + 3 * GL];
  }
  return x;
}
// sum += x . y over a lane's float4, in the order of its columns.  The fused multiply-adds are written out, here and in
// dst_operand, so that the gather and the filter give a triple the same bits whatever surrounds the expression.
template <bool VEC, bool CPLX> __device__ __forceinline__ void add_dot(float& sum, const float4& x, const float4& y) {
  if (VEC && CPLX) sum += __builtin_fmaf(x.x, y.x, x.z * y.z) + __builtin_fmaf(x.y, y.y, x.w * y.w);
  else if (VEC) sum += __builtin_fmaf(x.x, y.x, x.y * y.y) + __builtin_fmaf(x.z, y.z, x.w * y.w);
  else if (CPLX) { sum += __builtin_fmaf(x.x, y.x, x.z * y.z); sum += __builtin_fmaf(x.y, y.y, x.w * y.w); }
  else {
    sum = __builtin_fmaf(x.x, y.x, sum); sum = __builtin_fmaf(x.y, y.y, sum);
    sum = __builtin_fmaf(x.z, y.z, sum); sum = __builtin_fmaf(x.w, y.w, sum);
  }
}
// largest finite magnitude so far
__device__ __forceinline__ float finite_max(float m, float v) { const float f = fabsf(v); return f <= 3.4028234663852886e38f ? fmaxf(m, f) : m; }
__device__ __forceinline__ float finite_max4(float m, const float4& v) { return finite_max(finite_max(finite_max(finite_max(m, v.x), v.y), v.z), v.w); }
__device__ __forceinline__ bool finite1(float v) { return fabsf(v) <= 3.4028234663852886e38f; }
__device__ __forceinline__ bool finite4(const float4& v) { return finite1(v.x) && finite1(v.y) && finite1(v.z) && finite1(v.w); }

template <int GL> __device__ __forceinline__ float group_max(float v) {
#pragma unroll
  for (int o = GL / 2; o >= 1; o >>= 1) v = fmaxf(v, __shfl_xor(v, o));
  return v;
}

// The edge-side operand whose product with (TransE: distance to) a destination's row is the score.
__device__ __forceinline__ float4 sub4(const float4& x, const float4& y) { return make_float4(x.x - y.x, x.y - y.y, x.z - y.z, x.w - y.w); }
template <int MODEL> __device__ __forceinline__ float4 dst_operand(const float4& s, const float4& r) {
  if (MODEL == MAR_MODEL_COMPLEX)
    return make_float4(__builtin_fmaf(s.x, r.x, -(s.z * r.z)), __builtin_fmaf(s.y, r.y, -(s.w * r.w)),
                       __builtin_fmaf(s.z, r.x, s.x * r.z), __builtin_fmaf(s.w, r.y, s.y * r.w));
  if (MODEL == MAR_MODEL_DISTMULT) return make_float4(s.x * r.x, s.y * r.y, s.z * r.z, s.w * r.w);
  if (MODEL == MAR_MODEL_TRANSE) return make_float4(s.x + r.x, s.y + r.y, s.z + r.z, s.w + r.w);
  return s;
}

// Calls f(column, value) for the elements, or f2 / f4 for aligned pairs / quadruples of columns, that a lane holds of a row.
template <int GL, int NV, bool VEC, bool CPLX, class F1, class F2, class F4>
__device__ __forceinline__ void each_col(const float4 (&v)[NV], int l, int dim, F1 f1, F2 f2, F4 f4) {
  const int h = dim >> 1;
#pragma unroll
  for (int i = 0; i < NV; ++i) {
    if (VEC && CPLX) {
      const int k = 2 * (l + GL * i);
      if (k < h) { f2(k, make_float2(v[i].x, v[i].y)); f2(h + k, make_float2(v[i].z, v[i].w)); }
    } else if (VEC) {
      const int k = 4 * (l + GL * i);
      if (k < dim) f4(k, v[i]);
    } else if (CPLX) {
      const int k0 = l + GL * (2 * i), k1 = k0 + GL;
      if (k0 < h) { f1(k0, v[i].x); f1(h + k0, v[i].z); }
      if (k1 < h) { f1(k1, v[i].y); f1(h + k1, v[i].w); }
    } else {
      const int k = l + GL * (4 * i);
      if (k < dim) f1(k, v[i].x);
      if (k + GL < dim) f1(k + GL, v[i].y);
      if (k + 2 * GL < dim) f1(k + 2 * GL, v[i].z);
      if (k + 3 * GL < dim) f1(k + 3 * GL, v[i].w);
    }
  }
}

// One image row from a lane group's registers: columns scaled and split, zeros from dim up to the images' width.
template <int GL, int NV, bool VEC, bool CPLX, bool F16>
__device__ __forceinline__ void store_image_row(const SplitImages& g, const SplitRow& row, const float4 (&v)[NV], float scale, int l, int dim) {
  if (VEC) {
    for (int k = dim + 4 * l; k < g.dkp; k += 4 * GL) sp_store4<F16>(row, k, make_float4(0.f, 0.f, 0.f, 0.f), 1.f);
  } else {
    for (int k = dim + l; k < g.dkp; k += GL) sp_store1<F16>(row, k, 0.f, 1.f);
  }
  each_col<GL, NV, VEC, CPLX>(v, l, dim, [&](int k, float x) { sp_store1<F16>(row, k, x, scale); },
                              [&](int k, const float2& x) { sp_store2<F16>(row, k, x, scale); },
                              [&](int k, const float4& x) { sp_store4<F16>(row, k, x, scale); });
}

// Dense fp32 row, zero-padded from dim to dk.
template <int GL, int NV, bool VEC, bool CPLX>
__device__ __forceinline__ void store_dense_row(float* row, const float4 (&v)[NV], int l, int dim, int dk) {
  if (!VEC) { for (int k = dim + l; k < dk; k += GL) row[k] = 0.f; }
  each_col<GL, NV, VEC, CPLX>(v, l, dim, [&](int k, float x) { row[k] = x; },
                              [&](int k, const float2& x) { *reinterpret_cast<float2*>(row + k) = x; },
                              [&](int k, const float4& x) { *reinterpret_cast<float4*>(row + k) = x; });
}

// TransE on images: a vector that k_prep takes off every operand, which leaves all distances as they are.  Per column the mean of eight of
// the batch's negatives where they are of one sign and within a factor of 4 of one another, else 0 (columns drawn around 0: one in
// some 500 is taken for more by chance; it then grows by less than it varies).  Rows that share an offset are closer to one another
// than to 0: |x|^2 + |y|^2 - 2 x.y cancels, and nearly all pairs are near ones.  10,000 edges, 1,000 negatives of 100 floats, values of
// 5 +- 0.3: a step 568 us without, 154 with (fp32 instructions: 325; 0 +- 0.3: 157 and 159); 400 floats, 1 +- 0.2: relation gradients
// 3.4e-6 off without, 1.0e-6 with (fp32 instructions on the rows as they are: 1.5e-6), which is what rounding s + r to fp32 takes.
constexpr int SHIFT_ROWS = 8;
__device__ __forceinline__ float common_offset(const float (&v)[SHIFT_ROWS]) {
  float sum = v[0], lo = v[0], hi = v[0];
#pragma unroll
  for (int j = 1; j < SHIFT_ROWS; ++j) { sum += v[j]; lo = fminf(lo, v[j]); hi = fmaxf(hi, v[j]); }
  const bool close = (lo > 0.f && hi <= 4.f * lo) || (hi < 0.f && lo >= 4.f * hi);
  return close && fabsf(sum) <= 1e37f ? sum * (1.f / SHIFT_ROWS) : 0.f;   // (a NaN among them: 0)
}
// Node of row j of the eight: of either side, spread over the chunks and, from the last on, over a chunk's negatives (the first ones may
// be drawn by degree).
__device__ __forceinline__ int32_t shift_node(const RowArgs& a, int j) {
  const size_t at = (size_t)(j * (int64_t)(a.cn / a.N) / SHIFT_ROWS) * a.N + (a.N - 1 - (int)(j * (int64_t)a.N / SHIFT_ROWS));
  return (j & 1 ? a.neg_src : a.neg_dst)[at];
}

// Rows per lane group: edges, negatives.
constexpr int prep_edges(int gl, bool img) { return img && gl == 64 ? 4 : 2; }
constexpr int PREP_NEGS = 4;

// CARRY: the first `carried` workgroups do a piece of the row order (small batches; instantiations of their own, because the piece
// costs the others registers: 50,000 edges 1.2 % of a step, 20,000 edges' evaluation of 400 floats 2.7 %).
template <int GL, int NV, bool VEC, int MODEL, int FORM, bool CARRY>
__global__ void __launch_bounds__(256)
k_prep(RowArgs a, int carried, int nbB, int wpc_e, int wpc_n, float* __restrict__ Q, float* __restrict__ Km, float* __restrict__ qq,
       float* __restrict__ kk, float* __restrict__ pos, float* __restrict__ pos_user, int32_t* __restrict__ rank_dst,
       int32_t* __restrict__ rank_src, SplitImages qi, SplitImages ki, MarSortJob job) {
  extern __shared__ uint32_t sort_lds[];         // launched with the digits' counts where a job rides along
  if (CARRY && (int)blockIdx.x < carried) { sort_job<MAR_SORT_HIST>(job, sort_lds); return; }
  const int block = CARRY ? (int)blockIdx.x - carried : (int)blockIdx.x;
  constexpr bool IMG = FORM != PREP_DENSE, CPLX = MODEL == MAR_MODEL_COMPLEX, F16 = FORM == PREP_F16;
  constexpr int GPB = 256 / GL;                  // lane groups per block
  constexpr int E = prep_edges(GL, IMG), P = PREP_NEGS;
  constexpr int RE = GPB * E, RN = GPB * P;      // rows per workgroup
  static_assert(!IMG || (RE % SP_EB == 0 && RN % SP_EB == 0 && SP_EB % E == 0 && SP_EB % P == 0), "whole 16-row blocks per workgroup");
  constexpr int MB = (RN > RE ? RN : RE) / 16 + 1;
  __shared__ int s_max[2][MB];                   // per 16-row block: bits of the largest finite magnitude (two operands of an edge block)
  __shared__ int s_bad[2][MB];                   // the block holds an infinity or a NaN
  __shared__ int s_n2[MB];                       // evaluation: bits of the largest squared row norm of a block of negatives
  const bool eval = rank_dst != nullptr;         // uniform
  if (IMG && F16) {
    if (threadIdx.x < 2 * MB) { (&s_max[0][0])[threadIdx.x] = 0; (&s_bad[0][0])[threadIdx.x] = 0; }
    if (threadIdx.x < MB) s_n2[threadIdx.x] = 0;
    __syncthreads();
  }
  const int grp = threadIdx.x / GL, l = threadIdx.x % GL;
  const int dim = a.dim, dk = a.dk;
  // The rows of the shift: fetched by a lane group or two each, their ids and then they in flight with the workgroup's own, and
  // exchanged through LDS
  constexpr bool SHIFT = MODEL == MAR_MODEL_TRANSE && IMG;
  constexpr int SPG = (SHIFT_ROWS + GPB - 1) / GPB;
  __shared__ float4 s_rows[SHIFT ? SHIFT_ROWS : 1][NV][GL];
  int32_t sample_id[SPG];
  float4 sample[SPG][NV], shift[NV];
  if constexpr (SHIFT) {
#pragma unroll
    for (int k = 0; k < SPG; ++k) sample_id[k] = shift_node(a, min(grp * SPG + k, SHIFT_ROWS - 1));
  }
  auto fetch_shift = [&]() {
    if constexpr (SHIFT) {
#pragma unroll
      for (int k = 0; k < SPG; ++k) {
#pragma unroll
        for (int v = 0; v < NV; ++v) sample[k][v] = load_cols<GL, VEC, false>(a.node_emb + (size_t)sample_id[k] * dim, l, v, dim);
      }
    }
  };
  auto take_shift = [&]() {
    if constexpr (SHIFT) {
#pragma unroll
      for (int k = 0; k < SPG; ++k) {
        if (grp * SPG + k < SHIFT_ROWS) {
#pragma unroll
          for (int v = 0; v < NV; ++v) s_rows[grp * SPG + k][v][l] = sample[k][v];
        }
      }
      __syncthreads();
#pragma unroll
      for (int v = 0; v < NV; ++v) {
        float c[4][SHIFT_ROWS];
#pragma unroll
        for (int j = 0; j < SHIFT_ROWS; ++j) { const float4 x = s_rows[j][v][l]; c[0][j] = x.x; c[1][j] = x.y; c[2][j] = x.z; c[3][j] = x.w; }
        shift[v] = make_float4(common_offset(c[0]), common_offset(c[1]), common_offset(c[2]), common_offset(c[3]));
      }
      if (block == 0 && grp == 0) {
        store_dense_row<GL, NV, VEC, false>(a.shift, shift, l, dim, dk);
        for (int k = dk + l; k < qi.dkp; k += GL) a.shift[k] = 0.f;
      }
    }
  };
  // exponent of the 16-row block of workgroup row `rw` (two operands: which), after all groups have put in their maxima
  auto put_max = [&](int which, int rw, float mx, bool bad) {
    mx = group_max<GL>(mx);
    if (l == 0) atomicMax(&s_max[which][rw / SP_EB], __float_as_int(mx));
    if (bad) s_bad[which][rw / SP_EB] = 1;
  };
  if (block < nbB) {
    const int chunk = IMG ? block / wpc_e : 0;
    const int r0 = (IMG ? block % wpc_e : block) * RE + grp * E;         // first row of the group in its chunk
    const int nr = IMG ? min(a.S, a.n - chunk * a.S) : a.n;                         // edges of the chunk
    if (IMG) { if (r0 - grp * E >= ((nr + SP_TY - 1) & ~(SP_TY - 1))) return; }     // uniform over the workgroup
    else if (r0 >= nr) return;
    const size_t eb = IMG ? (size_t)chunk * a.S : 0;
    const float *s_row[E], *r_row[E], *d_row[E];
#pragma unroll
    for (int j = 0; j < E; ++j) {
      const size_t e = eb + min(r0 + j, nr - 1);                                    // surplus rows repeat the last edge (not stored)
      s_row[j] = a.node_emb + (size_t)a.src[e] * dim;
      r_row[j] = a.rel_emb + (size_t)(MODEL == MAR_MODEL_DOT ? 0 : a.rel[e]) * dim;     // unused by Dot
      d_row[j] = a.node_emb + (size_t)a.dst[e] * dim;
    }
    fetch_shift();
    float acc[E], nd[E], ns[E];
    float4 u[E][NV], w[E][NV], s[E][NV], r[E][NV], d[E][NV];
#pragma unroll
    for (int j = 0; j < E; ++j) {
      acc[j] = nd[j] = ns[j] = 0.f;
#pragma unroll
      for (int v = 0; v < NV; ++v) {
        s[j][v] = load_cols<GL, VEC, CPLX>(s_row[j], l, v, dim);
        d[j][v] = load_cols<GL, VEC, CPLX>(d_row[j], l, v, dim);
        r[j][v] = MODEL == MAR_MODEL_DOT ? make_float4(0.f, 0.f, 0.f, 0.f) : load_cols<GL, VEC, CPLX>(r_row[j], l, v, dim);
      }
    }
    take_shift();
    float mxu = 0.f, mxw = 0.f;
    bool badu = false, badw = false;
#pragma unroll
    for (int j = 0; j < E; ++j) {
      float4 qu[NV], qw[NV];
#pragma unroll
      for (int v = 0; v < NV; ++v) {
        const float4 S = s[j][v], R = r[j][v], D = d[j][v];
        float4 U, W;
        U = dst_operand<MODEL>(S, R);
        if (CPLX) W = make_float4(R.x * D.x + R.z * D.z, R.y * D.y + R.w * D.w, R.x * D.z - R.z * D.x, R.y * D.w - R.w * D.y);
        else if (MODEL == MAR_MODEL_DISTMULT) W = make_float4(R.x * D.x, R.y * D.y, R.z * D.z, R.w * D.w);
        else if (MODEL == MAR_MODEL_DOT) W = D;
        else W = sub4(D, R);
        if (MODEL == MAR_MODEL_TRANSE) {
          const float4 df = sub4(U, D);
          add_dot<VEC, false>(acc[j], df, df);
          if constexpr (SHIFT) {                           // the rows as they are: for near pairs and the passes' ends
            qu[v] = U; qw[v] = W;
            U = sub4(U, shift[v]); W = sub4(W, shift[v]);
          }
          add_dot<VEC, false>(nd[j], U, U);
          add_dot<VEC, false>(ns[j], W, W);
        } else {
          add_dot<VEC, CPLX>(acc[j], U, D);
        }
        u[j][v] = U; w[j][v] = W;
        if (IMG && F16 && r0 + j < nr) {
          mxu = finite_max4(mxu, U); mxw = finite_max4(mxw, W);
          badu |= !finite4(U); badw |= !finite4(W);
        }
      }
      if constexpr (SHIFT) {
        if (r0 + j < nr) {
          store_dense_row<GL, NV, VEC, false>(Q + ((size_t)MAR_SIDE_DST * a.B + eb + r0 + j) * dk, qu, l, dim, dk);
          store_dense_row<GL, NV, VEC, false>(Q + ((size_t)MAR_SIDE_SRC * a.B + eb + r0 + j) * dk, qw, l, dim, dk);
        }
      }
    }
    if (IMG && F16) {
      put_max(MAR_SIDE_DST, grp * E, mxu, badu);
      put_max(MAR_SIDE_SRC, grp * E, mxw, badw);
      __syncthreads();
    }
    float scu = 1.f, scw = 1.f;
    if (IMG && F16) {
      const int eu = sp_exponent(s_max[MAR_SIDE_DST][grp * E / SP_EB]), ew = sp_exponent(s_max[MAR_SIDE_SRC][grp * E / SP_EB]);
      scu = ldexpf(1.f, eu); scw = ldexpf(1.f, ew);
      if (l == 0 && r0 % SP_EB == 0 && r0 / SP_TY < qi.tiles) {
        qi.exps[((size_t)(2 * chunk + MAR_SIDE_DST) * qi.tiles) * 2 + r0 / SP_EB] = (float)eu + (s_bad[MAR_SIDE_DST][grp * E / SP_EB] ? SP_NONFINITE : 0.f);
        qi.exps[((size_t)(2 * chunk + MAR_SIDE_SRC) * qi.tiles) * 2 + r0 / SP_EB] = (float)ew + (s_bad[MAR_SIDE_SRC][grp * E / SP_EB] ? SP_NONFINITE : 0.f);
      }
    }
#pragma unroll
    for (int j = 0; j < E; ++j) {
      const int row = r0 + j;
      const size_t e = eb + row;
      const bool valid = row < nr;
      if (IMG) {
        if (row / SP_TY < qi.tiles) {
          if (!valid) {
#pragma unroll
            for (int v = 0; v < NV; ++v) u[j][v] = w[j][v] = make_float4(0.f, 0.f, 0.f, 0.f);
          }
          store_image_row<GL, NV, VEC, CPLX, F16>(qi, sp_row(qi, 2 * chunk + MAR_SIDE_DST, row), u[j], scu, l, dim);
          store_image_row<GL, NV, VEC, CPLX, F16>(qi, sp_row(qi, 2 * chunk + MAR_SIDE_SRC, row), w[j], scw, l, dim);
        }
      }
      if (!SHIFT && valid && (!IMG || Q)) {                  // dense; evaluation
        store_dense_row<GL, NV, VEC, CPLX>(Q + ((size_t)MAR_SIDE_DST * a.B + e) * dk, u[j], l, dim, dk);
        store_dense_row<GL, NV, VEC, CPLX>(Q + ((size_t)MAR_SIDE_SRC * a.B + e) * dk, w[j], l, dim, dk);
      }
      float sc = group_sum<GL>(acc[j]);
      if (MODEL == MAR_MODEL_TRANSE) {
        const float sd = group_sum<GL>(nd[j]), ss = group_sum<GL>(ns[j]);
        sc = -sqrtf(sc);
        if (l == 0 && valid) { qq[(size_t)MAR_SIDE_DST * a.B + e] = sd; qq[(size_t)MAR_SIDE_SRC * a.B + e] = ss; }
      }
      if (l == 0 && valid) {
        pos[e] = sc;
        if (pos_user) pos_user[e] = sc;
        if (rank_dst) { rank_dst[e] = 1; rank_src[e] = 1; }
      }
    }
    return;
  }
  {
    const int blk = block - nbB;
    const int cs = IMG ? blk / wpc_n : 0;                        // 2 * chunk + side
    const int r0 = (IMG ? blk % wpc_n : blk) * RN + grp * P;     // first row: in its chunk-side, or among the 2*cn negatives
    const int nr = IMG ? a.N : 2 * a.cn;
    if (IMG) { if (r0 - grp * P >= ((nr + SP_TY - 1) & ~(SP_TY - 1))) return; }     // uniform over the workgroup
    else if (r0 >= nr) return;
    float4 x[P][NV];
    size_t krow[P];
#pragma unroll
    for (int j = 0; j < P; ++j) {
      const int rr = min(r0 + j, nr - 1);
      const int side = IMG ? cs & 1 : (rr >= a.cn ? MAR_SIDE_DST : MAR_SIDE_SRC);
      const size_t cj = IMG ? (size_t)(cs >> 1) * a.N + rr : (size_t)(rr - (side == MAR_SIDE_DST ? a.cn : 0));    // chunk*N + j
      const int32_t id = side == MAR_SIDE_DST ? a.neg_dst[cj] : a.neg_src[cj];
      const float* row = a.node_emb + (size_t)id * dim;
      krow[j] = (size_t)side * a.C * a.N + cj;
      if (j == 0) fetch_shift();
#pragma unroll
      for (int v = 0; v < NV; ++v) {
        x[j][v] = load_cols<GL, VEC, false>(row, l, v, dim);
      }
    }
    if constexpr (SHIFT) {
      take_shift();
#pragma unroll
      for (int j = 0; j < P; ++j) {
#pragma unroll
        for (int v = 0; v < NV; ++v) x[j][v] = sub4(x[j][v], shift[v]);
      }
    }
    float scale = 1.f;
    if (IMG && F16) {
      float mx = 0.f, norm2[P];
      bool bad = false;
#pragma unroll
      for (int j = 0; j < P; ++j) {
#pragma unroll
        for (int v = 0; v < NV; ++v) {
          if (r0 + j < nr) { mx = finite_max4(mx, x[j][v]); bad |= !finite4(x[j][v]); }
        }
      }
      put_max(0, grp * P, mx, bad);
      if (eval) {
#pragma unroll
        for (int j = 0; j < P; ++j) {
          float n2 = 0.f;
#pragma unroll
          for (int v = 0; v < NV; ++v) add_dot<VEC, false>(n2, x[j][v], x[j][v]);
          norm2[j] = group_sum<GL>(n2);
          if (l == 0 && r0 + j < nr) atomicMax(&s_n2[grp * P / SP_EB], __float_as_int(fabsf(norm2[j])));
        }
      }
      __syncthreads();
      const int e = sp_exponent(s_max[0][grp * P / SP_EB]);
      scale = ldexpf(1.f, e);
      if (l == 0 && r0 % SP_EB == 0 && r0 / SP_TY < ki.tiles)
        ki.exps[(size_t)cs * ki.tiles * 2 + r0 / SP_EB] = (float)e + (s_bad[0][grp * P / SP_EB] ? SP_NONFINITE : 0.f);
      if (eval && r0 / SP_TY < ki.tiles) {
        // bounds of the scaled rows' norms: from the norm (a square that underflows is below 1e-25), or where its square
        // leaves the range, from the scale
        const float most = s_max[0][grp * P / SP_EB] ? sqrtf((float)dk) * 0x1p15f : 0.f;
        auto bound = [&](float n2) { return n2 < 1e37f ? fminf(most, 1.001f * sqrtf(fmaxf(n2, 1e-25f)) * scale) : most; };
        float* norms = ki.norms + ((size_t)cs * ki.tiles + r0 / SP_TY) * SP_NORMS;
        if (l == 0 && r0 % SP_EB == 0) norms[r0 % SP_TY / SP_EB] = bound(__int_as_float(s_n2[grp * P / SP_EB]));
#pragma unroll
        for (int j = 0; j < P; ++j) {
          float m = 0.f;
#pragma unroll
          for (int v = 0; v < NV; ++v) m = finite_max4(m, x[j][v]);
          m = group_max<GL>(m);
          if (l == 0) norms[2 + r0 % SP_TY + j] = m > 0.f ? bound(norm2[j]) : -1.f;
        }
      }
    }
#pragma unroll
    for (int j = 0; j < P; ++j) {
      const bool valid = r0 + j < nr;
      if (IMG) {
        if ((r0 + j) / SP_TY < ki.tiles) {
          if (!valid) {
#pragma unroll
            for (int v = 0; v < NV; ++v) x[j][v] = make_float4(0.f, 0.f, 0.f, 0.f);
          }
          store_image_row<GL, NV, VEC, false, F16>(ki, sp_row(ki, cs, r0 + j), x[j], scale, l, dim);
        }
      } else if (valid) {
        store_dense_row<GL, NV, VEC, false>(Km + krow[j] * dk, x[j], l, dim, dk);
      }
      if (MODEL == MAR_MODEL_TRANSE) {
        float nn = 0.f;
#pragma unroll
        for (int v = 0; v < NV; ++v) add_dot<VEC, false>(nn, x[j][v], x[j][v]);
        nn = group_sum<GL>(nn);
        if (l == 0 && valid) kk[krow[j]] = nn;
      }
    }
  }
}

// ------------------------------------------------------------------ chain rule -----
// From the gradients w.r.t. the two edge-side operands (gq_dst w.r.t. the DST-side q, gq_src
// w.r.t. the SRC-side q) and the positive term -2 f(e) to gradient rows of s, r, d, written at
// the occurrences' fixed places.  Also the per-edge loss terms, summed per block in a fixed order.
//
// Pass 1 leaves, per part p of a stripe, the softmax reference m_p, the sum l_p and the unnormalised
// O_p = sum_j exp(a_j - m_p) n_j.  merge_parts turns them into the log-sum-exp and one factor per part,
// fac_p = exp(m_p - m) / l with m = max m_p and l = sum_p l_p exp(m_p - m), so that gq = sum_p fac_p O_p.

__device__ __forceinline__ float merge_parts(const float* __restrict__ ml, size_t row, size_t part_rows, int sy1, float ml_log2,
                                             float (&fac)[MAR_MAX_PARTS]) {
  const float2* __restrict__ p2 = reinterpret_cast<const float2*>(ml) + row;
  float2 v[MAR_MAX_PARTS];
#pragma unroll
  for (int p = 0; p < MAR_MAX_PARTS; ++p) v[p] = p < sy1 ? p2[p * part_rows] : make_float2(-3.0e38f, 0.f);
  float mx = v[0].x;
#pragma unroll
  for (int p = 1; p < MAR_MAX_PARTS; ++p) mx = fmaxf(mx, v[p].x);
  float ls = 0.f;
#pragma unroll
  for (int p = 0; p < MAR_MAX_PARTS; ++p) { fac[p] = __expf((v[p].x - mx) * ml_log2); ls += fac[p] * v[p].y; }
  const float il = 1.f / ls;
#pragma unroll
  for (int p = 0; p < MAR_MAX_PARTS; ++p) fac[p] *= il;
  return mx * ml_log2 + logf(ls);
}

// Chain rule of one element: from s, r, d, the merged operand gradients u (DST side) and w (SRC side).
template <int MODEL>
__device__ __forceinline__ void chain1(float s, float r, float d, float u, float w, float inv2, float& gs, float& gd, float& gr) {
  if (MODEL == MAR_MODEL_DISTMULT) {
    gs = r * (u - 2.f * d); gd = r * (w - 2.f * s); gr = s * u + d * w - 2.f * s * d;
  } else if (MODEL == MAR_MODEL_DOT) {
    gs = u - 2.f * d; gd = w - 2.f * s; gr = 0.f;
  } else {                                               // TransE: inv2 = 2 / distance (0 at distance 0)
    const float dl = (s + r - d) * inv2;                 // 2 * unit(s + r - d)
    gs = u + dl; gr = u - w + dl; gd = w - dl;
  }
}

// ComplEx, one complex element: g_s = conj(r) (gU - 2 d), g_d = r (gW - 2 s), g_r = conj(s) gU + conj(gW) d - 2 conj(s) d.
__device__ __forceinline__ void chain_complex(float sr, float si, float rr, float ri, float dr, float di, float ure, float uim,
                                              float wre, float wim, float& gsr, float& gsi, float& gdr, float& gdi,
                                              float& grr, float& gri) {
  const float zr = ure - 2.f * dr, zi = uim - 2.f * di;
  gsr = rr * zr + ri * zi;  gsi = rr * zi - ri * zr;
  const float yr = wre - 2.f * sr, yi = wim - 2.f * si;
  gdr = rr * yr - ri * yi;  gdi = rr * yi + ri * yr;
  grr = sr * ure + si * uim + wre * dr + wim * di - 2.f * (sr * dr + si * di);
  gri = sr * uim - si * ure + wre * di - wim * dr - 2.f * (sr * di - si * dr);
}

// Columns col .. col + 3 of a table row (col a multiple of 4 below dim), zeros from dim on.  Rows of no whole 16 bytes lie at any multiple
// of 4 bytes, which the memory pipeline takes 16 bytes at a time all the same (the type says so).  A row's last columns are read
// with those before them and moved down.  (In place of one column a lane and step, each waiting for the last one's loads: the chain rule of
// 1,000 edges of 50 floats 11 -> 6 us.  In the reduce, which has no such chain, four single loads are faster: 15 against 18.)
typedef float RowCols __attribute__((ext_vector_type(4), aligned(4)));
template <bool VEC> __device__ __forceinline__ float4 load_any4(const float* __restrict__ row, int col, int dim) {
  if (VEC) return *reinterpret_cast<const float4*>(row + col);
  float4 v = make_float4(0.f, 0.f, 0.f, 0.f);
  if (dim < 4) {                                           // uniform
    v.x = row[0];
    if (dim > 1) v.y = row[1];
    if (dim > 2) v.z = row[2];
    return v;
  }
  const int at = min(col, dim - 4);
  const RowCols r = *reinterpret_cast<const RowCols*>(row + at);
  const bool m1 = ((col - at) & 1) != 0, m2 = ((col - at) & 2) != 0;
  const float x = m1 ? r.y : r.x, y = m1 ? r.z : r.y, z = m1 ? r.w : r.z, w = m1 ? 0.f : r.w;
  v.x = m2 ? z : x; v.y = m2 ? w : y; v.z = m2 ? 0.f : z; v.w = m2 ? 0.f : w;
  return v;
}
// One group of GL lanes per edge.  VEC (dim % 4 == 0): a lane moves NV float4s per row (for ComplEx NV float2s of
// the real half and the matching float2s of the imaginary half), every load of the edge is issued before the
// first use; SY1 > 0: pass 1 was split into exactly SY1 parts (1 for the large batch shapes), SY1 = 0: a.sy1 parts.
template <int GL, int NV, int MODEL, bool VEC, int SY1, bool CARRY>
__global__ void __launch_bounds__(256)
k_chain(RowArgs a, int carried, const float* __restrict__ gQ, const float* __restrict__ ml, const float* __restrict__ pos,
        float* __restrict__ lse_dst, float* __restrict__ lse_src, float* __restrict__ G, float* __restrict__ loss_part, MarSortJob job) {
  extern __shared__ uint32_t sort_lds[];
  if (CARRY && (int)blockIdx.x < carried) { sort_job<MAR_SORT_SCATTER>(job, sort_lds); return; }
  const int block = CARRY ? (int)blockIdx.x - carried : (int)blockIdx.x;
  constexpr int GPB = 256 / GL;
  constexpr int P = SY1 ? SY1 : MAR_MAX_PARTS;
  __shared__ float lsum[GPB];
  const int grp = threadIdx.x / GL, l = threadIdx.x % GL;
  const int e = block * GPB + grp;
  const int dim = a.dim, dk = a.dk;
  const int sy1 = SY1 ? SY1 : a.sy1;
  const size_t part_rows = (size_t)2 * a.B;
  float le = 0.f;
  if (e < a.n) {
    // every lane of the group merges the parts of both sides (same addresses: one broadcast load each)
    float facu[MAR_MAX_PARTS], facw[MAR_MAX_PARTS];
    const size_t row_u = (size_t)MAR_SIDE_DST * a.B + e, row_w = (size_t)MAR_SIDE_SRC * a.B + e;
    const float lse_u = merge_parts(ml, row_u, part_rows, sy1, a.ml_log2, facu);
    const float lse_w = merge_parts(ml, row_w, part_rows, sy1, a.ml_log2, facw);
    const float pe = pos[e];
    if (l == 0 && lse_dst) lse_dst[e] = lse_u;             // where the caller asks for them
    if (l == 0 && lse_src) lse_src[e] = lse_w;
    le = -2.f * pe + lse_u + lse_w;
    const float* gu0 = gQ + row_u * dk;
    const float* gw0 = gQ + row_w * dk;
    const size_t pstride = part_rows * dk;
    const float* s_row = a.node_emb + (size_t)a.src[e] * dim;
    const float* r_row = a.rel_emb + (size_t)(MODEL == MAR_MODEL_DOT ? 0 : a.rel[e]) * dim;
    const float* d_row = a.node_emb + (size_t)a.dst[e] * dim;
    float* gs = G + (size_t)e * dk;                              // gradient row of occurrence k is row k
    float* gd = G + ((size_t)a.n + e) * dk;
    float* gr = G + (2 * (size_t)a.n + e) * dk;
    float inv2 = 0.f;
    if (MODEL == MAR_MODEL_TRANSE) { const float dist = -pe; inv2 = dist > 0.f ? 2.f / dist : 0.f; }
    if (VEC && MODEL == MAR_MODEL_COMPLEX) {
      const int h = dim >> 1;
      float2 sr[NV], si[NV], rr[NV], ri[NV], dr[NV], di[NV], ur[NV], ui[NV], wr[NV], wi[NV];
#pragma unroll
      for (int v = 0; v < NV; ++v) {
        const int k = 2 * (l + GL * v);
        if (k < h) {
          sr[v] = *reinterpret_cast<const float2*>(s_row + k); si[v] = *reinterpret_cast<const float2*>(s_row + h + k);
          rr[v] = *reinterpret_cast<const float2*>(r_row + k); ri[v] = *reinterpret_cast<const float2*>(r_row + h + k);
          dr[v] = *reinterpret_cast<const float2*>(d_row + k); di[v] = *reinterpret_cast<const float2*>(d_row + h + k);
          ur[v] = ui[v] = wr[v] = wi[v] = make_float2(0.f, 0.f);
#pragma unroll
          for (int p = 0; p < P; ++p) {
            if (SY1 || p < sy1) {
              const float2 a0 = *reinterpret_cast<const float2*>(gu0 + p * pstride + k), a1 = *reinterpret_cast<const float2*>(gu0 + p * pstride + h + k);
              const float2 b0 = *reinterpret_cast<const float2*>(gw0 + p * pstride + k), b1 = *reinterpret_cast<const float2*>(gw0 + p * pstride + h + k);
              ur[v].x += facu[p] * a0.x; ur[v].y += facu[p] * a0.y; ui[v].x += facu[p] * a1.x; ui[v].y += facu[p] * a1.y;
              wr[v].x += facw[p] * b0.x; wr[v].y += facw[p] * b0.y; wi[v].x += facw[p] * b1.x; wi[v].y += facw[p] * b1.y;
            }
          }
        }
      }
#pragma unroll
      for (int v = 0; v < NV; ++v) {
        const int k = 2 * (l + GL * v);
        if (k < h) {
          float2 osr, osi, odr, odi, orr, ori;
          chain_complex(sr[v].x, si[v].x, rr[v].x, ri[v].x, dr[v].x, di[v].x, ur[v].x, ui[v].x, wr[v].x, wi[v].x, osr.x, osi.x, odr.x, odi.x, orr.x, ori.x);
          chain_complex(sr[v].y, si[v].y, rr[v].y, ri[v].y, dr[v].y, di[v].y, ur[v].y, ui[v].y, wr[v].y, wi[v].y, osr.y, osi.y, odr.y, odi.y, orr.y, ori.y);
          *reinterpret_cast<float2*>(gs + k) = osr; *reinterpret_cast<float2*>(gs + h + k) = osi;
          *reinterpret_cast<float2*>(gd + k) = odr; *reinterpret_cast<float2*>(gd + h + k) = odi;
          *reinterpret_cast<float2*>(gr + k) = orr; *reinterpret_cast<float2*>(gr + h + k) = ori;
        }
      }
    } else if (MODEL != MAR_MODEL_COMPLEX) {
      float4 s4[NV], r4[NV], d4[NV], u4[NV], w4[NV];
#pragma unroll
      for (int v = 0; v < NV; ++v) {
        const int k = 4 * (l + GL * v);
        if (k < dim) {
          s4[v] = load_any4<VEC>(s_row, k, dim); d4[v] = load_any4<VEC>(d_row, k, dim);
          r4[v] = MODEL == MAR_MODEL_DOT ? make_float4(0.f, 0.f, 0.f, 0.f) : load_any4<VEC>(r_row, k, dim);
          u4[v] = w4[v] = make_float4(0.f, 0.f, 0.f, 0.f);
#pragma unroll
          for (int p = 0; p < P; ++p) {
            if (SY1 || p < sy1) {
              const float4 a0 = *reinterpret_cast<const float4*>(gu0 + p * pstride + k), b0 = *reinterpret_cast<const float4*>(gw0 + p * pstride + k);
              u4[v].x += facu[p] * a0.x; u4[v].y += facu[p] * a0.y; u4[v].z += facu[p] * a0.z; u4[v].w += facu[p] * a0.w;
              w4[v].x += facw[p] * b0.x; w4[v].y += facw[p] * b0.y; w4[v].z += facw[p] * b0.z; w4[v].w += facw[p] * b0.w;
            }
          }
        }
      }
#pragma unroll
      for (int v = 0; v < NV; ++v) {
        const int k = 4 * (l + GL * v);
        if (k < dim) {
          float4 os, od, og;
          chain1<MODEL>(s4[v].x, r4[v].x, d4[v].x, u4[v].x, w4[v].x, inv2, os.x, od.x, og.x);
          chain1<MODEL>(s4[v].y, r4[v].y, d4[v].y, u4[v].y, w4[v].y, inv2, os.y, od.y, og.y);
          chain1<MODEL>(s4[v].z, r4[v].z, d4[v].z, u4[v].z, w4[v].z, inv2, os.z, od.z, og.z);
          chain1<MODEL>(s4[v].w, r4[v].w, d4[v].w, u4[v].w, w4[v].w, inv2, os.w, od.w, og.w);
          *reinterpret_cast<float4*>(gs + k) = os; *reinterpret_cast<float4*>(gd + k) = od;
          if (MODEL != MAR_MODEL_DOT) *reinterpret_cast<float4*>(gr + k) = og;
        }
      }
    } else {
      // ComplEx of any width: one complex element per lane and step
      auto merged = [&](const float* base, const float (&f)[MAR_MAX_PARTS], int k) {
        float v = 0.f;
#pragma unroll
        for (int p = 0; p < P; ++p) if (SY1 || p < sy1) v += f[p] * base[p * pstride + k];
        return v;
      };
      const int h = dim >> 1;
      for (int k = l; k < h; k += GL) {
        chain_complex(s_row[k], s_row[h + k], r_row[k], r_row[h + k], d_row[k], d_row[h + k], merged(gu0, facu, k), merged(gu0, facu, h + k),
                      merged(gw0, facw, k), merged(gw0, facw, h + k), gs[k], gs[h + k], gd[k], gd[h + k], gr[k], gr[h + k]);
      }
      for (int k = dim + l; k < dk; k += GL) { gs[k] = 0.f; gd[k] = 0.f; gr[k] = 0.f; }
    }
  }
  if (l == 0) lsum[grp] = le;
  __syncthreads();
  if (threadIdx.x == 0) {
    float t = 0.f;
    for (int i = 0; i < GPB; ++i) t += lsum[i];
    loss_part[block] = t;
  }
}

// ------------------------------------------------------------ filtered evaluation -----
// One lane group per (edge, corrupted side): takes the listed true candidates that outscore the edge out of its rank.
// The edge's rows are read once; candidates are taken FILT at a time, their ids and then their rows all in flight, in
// lists of one or two one at a time (20,000 edges, both sides, always one / always FILT / so: lists of 1 row of 400 floats
// 27 / 33 / 27 us, of 2: 39 / 37 / 38, of 16: 253 / 158 / 163, of 16 rows of 100 floats 114 / 59 / 60).  Scores are
// formed in the operation order of the positive score above.
#define FILT 4
template <int GL, int NV, bool VEC, int MODEL>
__global__ void __launch_bounds__(256)
k_filter(RowArgs a, const int64_t* __restrict__ dst_off, const int32_t* __restrict__ dst_ids,
         const int64_t* __restrict__ src_off, const int32_t* __restrict__ src_ids, const float* __restrict__ pos,
         int32_t* __restrict__ rank_dst, int32_t* __restrict__ rank_src) {
  constexpr bool CPLX = MODEL == MAR_MODEL_COMPLEX;
  constexpr int GPB = 256 / GL;
  const int grp = threadIdx.x / GL, l = threadIdx.x % GL;
  const int idx = blockIdx.x * GPB + grp;
  if (idx >= 2 * a.n) return;
  const int side = idx >= a.n ? MAR_SIDE_DST : MAR_SIDE_SRC;
  const int e = side == MAR_SIDE_DST ? idx - a.n : idx;
  const int dim = a.dim;
  const int64_t* off = side == MAR_SIDE_DST ? dst_off : src_off;
  const int32_t* ids = side == MAR_SIDE_DST ? dst_ids : src_ids;
  const int64_t k0 = off[e], k1 = off[e + 1];
  if (k0 >= k1) return;
  const float p = pos[e];
  const float* kept_row = a.node_emb + (size_t)(side == MAR_SIDE_DST ? a.src[e] : a.dst[e]) * dim;   // the endpoint that stays
  const float* r_row = a.rel_emb + (size_t)(MODEL == MAR_MODEL_DOT ? 0 : a.rel[e]) * dim;
  float4 kept[NV], r[NV];
#pragma unroll
  for (int v = 0; v < NV; ++v) {
    kept[v] = load_cols<GL, VEC, CPLX>(kept_row, l, v, dim);
    r[v] = MODEL == MAR_MODEL_DOT ? make_float4(0.f, 0.f, 0.f, 0.f) : load_cols<GL, VEC, CPLX>(r_row, l, v, dim);
  }
  int better = 0;
  // N candidates from k on, the list's last one again where there are fewer
  auto take = [&](int64_t k, auto count) __attribute__((always_inline)) {
    constexpr int N = decltype(count)::value;
    float4 c[N][NV];
#pragma unroll
    for (int j = 0; j < N; ++j) {
      const float* c_row = a.node_emb + (size_t)ids[k + j < k1 ? k + j : k1 - 1] * dim;
#pragma unroll
      for (int v = 0; v < NV; ++v) c[j][v] = load_cols<GL, VEC, CPLX>(c_row, l, v, dim);
    }
#pragma unroll
    for (int j = 0; j < N; ++j) {
      float acc = 0.f;
#pragma unroll
      for (int v = 0; v < NV; ++v) {
        const float4 s = side == MAR_SIDE_DST ? kept[v] : c[j][v], d = side == MAR_SIDE_DST ? c[j][v] : kept[v];
        const float4 u = dst_operand<MODEL>(s, r[v]);
        if (MODEL == MAR_MODEL_TRANSE) { const float4 df = sub4(u, d); add_dot<VEC, false>(acc, df, df); }
        else add_dot<VEC, CPLX>(acc, u, d);
      }
      acc = group_sum<GL>(acc);
      const float f = MODEL == MAR_MODEL_TRANSE ? -sqrtf(acc) : acc;
      better += k + j < k1 && f > p ? 1 : 0;
    }
  };
  if (k1 - k0 <= 2) {
    for (int64_t k = k0; k < k1; ++k) take(k, std::integral_constant<int, 1>());
  } else {
    for (int64_t k = k0; k < k1; k += FILT) take(k, std::integral_constant<int, FILT>());
  }
  // The unfiltered rank comes from the matrix cores, this count from the vector ALU: a candidate within rounding
  // of the edge's score can be counted here and not there, so the difference is kept at 1 or above.
  if (l == 0 && better) {
    int32_t* rk = (side == MAR_SIDE_DST ? rank_dst : rank_src) + e;
    const int32_t v = *rk - better;
    *rk = v < 1 ? 1 : v;
  }
}

// ------------------------------------------------- per-row reduce + Adagrad scatter -----
// The gradient rows are summed per table row over the row-sorted order (a stable sort, so a row's
// occurrences are always added in the same order and the sums are bit-reproducible) and the Adagrad
// update (Sec. 5.1; one update per touched row and step) is applied where the sum becomes complete.
struct ReduceArgs {
  float *node_emb, *node_state, *rel_emb, *rel_state;
  const float* G;            // [n_rows][dk] gradient rows
  float* carry;              // [blocks][2][dk] partial sums of segments that cross block borders
  const uint32_t* ids;       // position in row-sorted order -> unified id
  const int32_t* perm;       // position -> gradient row
  const int32_t* rank_sorted;   // position -> rank among the unique rows; only with dbg_grad or defer_grad, else NULL
  int32_t* scalars;          // [2] = number of entries in `owners`
  int32_t* owners;           // blocks in which a segment begins that continues into later blocks
  float* dbg_grad;           // [unique rows][dim] summed gradients (debug output), or NULL
  float* defer_grad;         // [unique rows][dk], or NULL: if set, a node row's summed gradient is stored here and the row is
                             // left alone (its update is applied later, by k_stage_apply); relation rows are updated as usual
  int64_t n_rows;
  int32_t block;             // positions per workgroup
  int32_t num_nodes, dim, dk;
  float lr, eps;
};

__device__ __forceinline__ void add4(float4& a, const float4& b) { a.x += b.x; a.y += b.y; a.z += b.z; a.w += b.w; }

// Four consecutive floats of a table row starting at column `col`.  VEC: rows are 16-byte aligned (dim % 4 == 0).

template <bool VEC> __device__ __forceinline__ float4 load_row4(const float* __restrict__ row, int col, int dim) {
  if (VEC) return *reinterpret_cast<const float4*>(row + col);
  float4 v;
  v.x = col + 0 < dim ? row[col + 0] : 0.f; v.y = col + 1 < dim ? row[col + 1] : 0.f;
  v.z = col + 2 < dim ? row[col + 2] : 0.f; v.w = col + 3 < dim ? row[col + 3] : 0.f;
  return v;
}

template <bool VEC> __device__ __forceinline__ void store_row4(float* __restrict__ row, int col, int dim, const float4& v) {
  if (VEC) { *reinterpret_cast<float4*>(row + col) = v; return; }
  if (col + 0 < dim) row[col + 0] = v.x;
  if (col + 1 < dim) row[col + 1] = v.y;
  if (col + 2 < dim) row[col + 2] = v.z;
  if (col + 3 < dim) row[col + 3] = v.w;
}

__device__ __forceinline__ void table_rows(const ReduceArgs& a, int32_t id, float*& emb, float*& st) {
  if (id < a.num_nodes) { emb = a.node_emb + (size_t)id * a.dim; st = a.node_state + (size_t)id * a.dim; }
  else { emb = a.rel_emb + (size_t)(id - a.num_nodes) * a.dim; st = a.rel_state + (size_t)(id - a.num_nodes) * a.dim; }
}

// state += g^2; theta -= lr * g / (sqrt(state) + eps) on four columns whose old values are th, s0 (Sec. 5.1: Adagrad).
// The one place where the update is spelled out: every kernel that applies it goes through here.
__device__ __forceinline__ void adagrad_math(const float4& g, const float4& th, const float4& s0, float lr, float eps, float4& e1, float4& s1) {
  s1.x = s0.x + g.x * g.x; s1.y = s0.y + g.y * g.y; s1.z = s0.z + g.z * g.z; s1.w = s0.w + g.w * g.w;
  e1.x = th.x - lr * g.x / (sqrtf(s1.x) + eps); e1.y = th.y - lr * g.y / (sqrtf(s1.y) + eps);
  e1.z = th.z - lr * g.z / (sqrtf(s1.z) + eps); e1.w = th.w - lr * g.w / (sqrtf(s1.w) + eps);
}

__device__ __forceinline__ bool row_deferred(const ReduceArgs& a, int32_t id) { return a.defer_grad != nullptr && id < a.num_nodes; }

// Finishes a table row whose summed gradient over four columns is g: Adagrad on the row (old values th, s0), or,
// for a deferred node row, the gradient goes to defer_grad and the table is not touched.
template <bool VEC>
__device__ __forceinline__ void adagrad4(const ReduceArgs& a, int32_t id, float* __restrict__ emb, float* __restrict__ st, int rank, int col,
                                         const float4& g, const float4& th, const float4& s0) {
  if (a.dbg_grad) store_row4<VEC>(a.dbg_grad + (size_t)rank * a.dim, col, a.dim, g);
  if (row_deferred(a, id)) { *reinterpret_cast<float4*>(a.defer_grad + (size_t)rank * a.dk + col) = g; return; }
  float4 s1, e1;
  adagrad_math(g, th, s0, a.lr, a.eps, e1, s1);
  store_row4<VEC>(st, col, a.dim, s1);
  store_row4<VEC>(emb, col, a.dim, e1);
}

// Old values of four columns of a table row; a deferred row is not read.
template <bool VEC>
__device__ __forceinline__ void load_old4(const ReduceArgs& a, int32_t id, const float* emb, const float* st, int col, float4& th, float4& s0) {
  if (row_deferred(a, id)) { th = s0 = make_float4(0.f, 0.f, 0.f, 0.f); return; }
  th = load_row4<VEC>(emb, col, a.dim); s0 = load_row4<VEC>(st, col, a.dim);
}

// A workgroup takes 256 / GL tasks of PPT consecutive positions, one per group of GL lanes (the lanes of a group move one
// row as float4s, NV per lane).  PPT = GL (256 positions per workgroup) for large batches, which are bound by memory;
// 8 or 4 (BATCH or twice that) for small ones, which are bound by the latency of the batches a group works
// through one after the other and of too few workgroups.  Each lane first fetches the id and the gradient row of one
// position of its task, and the group the ids on either side of it: equal neighbours are one segment, so the segments'
// borders follow without further loads and no later load depends on another.
// The task's rows are then fetched BATCH at a time -- together with the table row and accumulator row of
// every position at which a segment ends that also began inside the task -- and added up in position
// order; such a segment is finished by the Adagrad update right there.  A segment that crosses the task's
// borders leaves a partial sum in LDS (head: began earlier, tail: continues); the workgroup then chains the
// partials of its tasks in order, finishes the segments that lie inside the workgroup, and writes those
// that cross its own borders to `carry` (slot 0: began in an earlier workgroup, slot 1: continues into the
// next; a workgroup with a slot-1 partial appends itself to `owners`).
template <int GL, int NV, int BATCH, bool VEC, int PPT>
__global__ void __launch_bounds__(256) k_reduce_apply(ReduceArgs a) {
  constexpr int GPB = 256 / GL;
  __shared__ float4 s_head[GPB][GL * NV], s_tail[GPB][GL * NV];
  __shared__ int s_hs[GPB], s_tf[GPB];       // head: 0 none, 1 ends inside the task, 2 runs through it; tail: 0 / 1
  __shared__ int s_fin[GPB];                 // the head slot of this task holds a finished sum (set by the chaining step)
  const int grp = threadIdx.x / GL, l = threadIdx.x % GL;
  const int64_t p0 = (int64_t)blockIdx.x * (GPB * PPT) + (int64_t)grp * PPT;
  const int64_t left = a.n_rows - p0;
  const int cnt = left < 0 ? 0 : (left < PPT ? (int)left : PPT);
  const int64_t p1 = p0 + cnt;
  const int nq = a.dk >> 2;

  int my_rank = 0, my_row = 0, my_id = -1;
  int id_before = -2, id_after = -2;                       // ids of the positions before and behind the task (-2: none)
  if (l < cnt) {
    my_id = (int)a.ids[p0 + l];
    my_row = a.perm[p0 + l];
    if (a.rank_sorted) my_rank = a.rank_sorted[p0 + l];
    if (p0 > 0) id_before = (int)a.ids[p0 - 1];
    if (p1 < a.n_rows) id_after = (int)a.ids[p1];
  }
  id_before = __shfl(id_before, 0, GL); id_after = __shfl(id_after, 0, GL);
  const int id_first = __shfl(my_id, 0, GL), id_last = __shfl(my_id, cnt > 0 ? cnt - 1 : 0, GL);
  const bool from_before = cnt > 0 && id_first == id_before;   // the first position's segment began before the task
  const bool goes_on = cnt > 0 && id_last == id_after;         // the last position's segment continues behind it
  int my_kind = 0;                                         // 0 no segment end, 1 end of a segment that began inside the task,
  {                                                        // 2 end of a segment that began before it
    const int right = __shfl_down(my_id, 1, GL);
    const int next = l == cnt - 1 ? id_after : right;
    if (l < cnt && next != my_id) my_kind = from_before && my_id == id_first ? 2 : 1;
  }
  float4 acc[NV];
#pragma unroll
  for (int v = 0; v < NV; ++v) acc[v] = make_float4(0.f, 0.f, 0.f, 0.f);

  for (int i0 = 0; i0 < cnt; i0 += BATCH) {
    float4 g[BATCH][NV], th[BATCH][NV], s0[BATCH][NV];
    int kind[BATCH];
#pragma unroll
    for (int j = 0; j < BATCH; ++j) {
      const int pj = (i0 + j) & (GL - 1);
      const bool valid = i0 + j < cnt;
      const int row = __shfl(my_row, pj, GL);
      const int id = __shfl(my_id, pj, GL);
      kind[j] = valid ? __shfl(my_kind, pj, GL) : 0;
      const float* grow = a.G + (size_t)row * a.dk;
#pragma unroll
      for (int v = 0; v < NV; ++v) {
        const int q = l + GL * v;
        g[j][v] = (valid && q < nq) ? *reinterpret_cast<const float4*>(grow + 4 * q) : make_float4(0.f, 0.f, 0.f, 0.f);
      }
      if (kind[j] == 1) {
        float *emb, *st;
        table_rows(a, id, emb, st);
#pragma unroll
        for (int v = 0; v < NV; ++v) {
          const int q = l + GL * v;
          if (q < nq) load_old4<VEC>(a, id, emb, st, 4 * q, th[j][v], s0[j][v]);
        }
      }
    }
#pragma unroll
    for (int j = 0; j < BATCH; ++j) {
      if (i0 + j < cnt) {
#pragma unroll
        for (int v = 0; v < NV; ++v) add4(acc[v], g[j][v]);
        if (kind[j] != 0) {
          const int pj = (i0 + j) & (GL - 1);
          if (kind[j] == 1) {
            float *emb, *st;
            const int32_t fid = __shfl(my_id, pj, GL);
            table_rows(a, fid, emb, st);
            const int rank = __shfl(my_rank, pj, GL);
#pragma unroll
            for (int v = 0; v < NV; ++v) {
              const int q = l + GL * v;
              if (q < nq) adagrad4<VEC>(a, fid, emb, st, rank, 4 * q, acc[v], th[j][v], s0[j][v]);
            }
          } else {
#pragma unroll
            for (int v = 0; v < NV; ++v) s_head[grp][l + GL * v] = acc[v];
          }
#pragma unroll
          for (int v = 0; v < NV; ++v) acc[v] = make_float4(0.f, 0.f, 0.f, 0.f);
        }
      }
    }
  }
  // what is left in acc belongs to the segment of the task's last position, if that segment continues
  int hs = 0, tf = 0;
  if (from_before) hs = (id_last == id_first && goes_on) ? 2 : 1;
  if (goes_on) {
    if (!(from_before && id_last == id_first)) tf = 1;
#pragma unroll
    for (int v = 0; v < NV; ++v) (tf ? s_tail : s_head)[grp][l + GL * v] = acc[v];
  }
  if (l == 0) { s_hs[grp] = hs; s_tf[grp] = tf; s_fin[grp] = 0; }
  __syncthreads();

  // Chain the tasks' partial sums in task order: thread q owns column block q and walks the tasks (LDS only).
  // A segment that ends inside the workgroup and also began inside it leaves its sum in the head slot of the
  // task it ends in (s_fin marks it); those sums are then turned into Adagrad updates by all lane groups at
  // once -- group g takes task g -- so that their table reads do not queue up behind one another.
  const int q = threadIdx.x;
  float4 run = make_float4(0.f, 0.f, 0.f, 0.f);
  bool active = false, inside = false;                     // a segment is open / it began inside this workgroup
  for (int gi = 0; gi < GPB; ++gi) {
    const int h = s_hs[gi];                                // uniform over the workgroup
    if (h) {
      const float4 hv = q < nq ? s_head[gi][q] : make_float4(0.f, 0.f, 0.f, 0.f);
      if (active) add4(run, hv); else { run = hv; active = true; inside = false; }
      if (h == 1) {
        if (inside) {
          if (q < nq) s_head[gi][q] = run;
          if (q == 0) s_fin[gi] = 1;
        } else if (q < nq) {
          *reinterpret_cast<float4*>(a.carry + ((size_t)blockIdx.x * 2 + 0) * a.dk + 4 * q) = run;
        }
        active = false;
      }
    }
    if (s_tf[gi]) {
      run = q < nq ? s_tail[gi][q] : make_float4(0.f, 0.f, 0.f, 0.f);
      active = true; inside = true;
    }
  }
  if (active) {
    if (q < nq) *reinterpret_cast<float4*>(a.carry + ((size_t)blockIdx.x * 2 + (inside ? 1 : 0)) * a.dk + 4 * q) = run;
    if (inside && threadIdx.x == 0) a.owners[atomicAdd(&a.scalars[2], 1)] = (int32_t)blockIdx.x;
  }
  __syncthreads();
  if (s_fin[grp]) {                                        // uniform over the lane group
    const int rank = __shfl(my_rank, 0, GL);               // the segment that ends in task grp is the one its first position belongs to
    float *emb, *st;
    const int32_t fid = __shfl(my_id, 0, GL);
    table_rows(a, fid, emb, st);
#pragma unroll
    for (int v = 0; v < NV; ++v) {
      const int qq = l + GL * v;
      if (qq < nq) {
        float4 th, s0;
        load_old4<VEC>(a, fid, emb, st, 4 * qq, th, s0);
        adagrad4<VEC>(a, fid, emb, st, rank, 4 * qq, s_head[grp][qq], th, s0);
      }
    }
  }
}

// Finishes the segments that span several workgroups of k_reduce_apply: a workgroup of SPAN_WAVES waves takes an
// entry of `owners` (in any order: every entry is a different table row), adds that block's slot-1 partial
// and the slot-0 partials of the following blocks up to the segment's end -- wave w takes every SPAN_WAVES-th,
// FB at a time, then the waves' sums are combined through LDS in wave order: a fixed tree -- and applies
// the Adagrad update.  Block 0 first adds up the per-block loss terms, also in a fixed order.
#define SPAN_WAVES 16
template <int NV, bool VEC>
__global__ void __launch_bounds__(64 * SPAN_WAVES)
k_span_apply(ReduceArgs a, const float* __restrict__ loss_part, int n_loss_part, float* __restrict__ loss_out) {
  constexpr int NT = 64 * SPAN_WAVES;
  __shared__ float4 part[SPAN_WAVES][64 * NV];
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  if (blockIdx.x == 0 && loss_out) {                        // uniform over the workgroup
    // thread t adds terms t, t + NT, ..., then lanes, then the waves in order
    __shared__ float wsum[SPAN_WAVES];
    float t = 0.f;
    for (int i = threadIdx.x; i < n_loss_part; i += NT) t += loss_part[i];
#pragma unroll
    for (int o = 32; o >= 1; o >>= 1) t += __shfl_xor(t, o);
    if (lane == 0) wsum[wave] = t;
    __syncthreads();
    if (threadIdx.x == 0) {
      float s = 0.f;
      for (int w = 0; w < SPAN_WAVES; ++w) s += wsum[w];
      *loss_out = s;
    }
  }
  const int nq = a.dk >> 2;
  const int n_owners = a.scalars[2];
  for (int o = blockIdx.x; o < n_owners; o += gridDim.x) {  // uniform over the workgroup
    const int64_t blk = a.owners[o];
    const int64_t pe = (blk + 1) * a.block < a.n_rows ? (blk + 1) * a.block : a.n_rows;
    const uint32_t seg_id = a.ids[pe - 1];
    const int rank = a.rank_sorted ? a.rank_sorted[pe - 1] : 0;
    // the last block whose first position belongs to the segment: blocks blk + 1 .. last_blk do, 64 probes at a time
    int64_t last_blk = blk, after = (a.n_rows + a.block - 1) / a.block;
    while (after - last_blk > 1) {
      const int64_t stepb = (after - last_blk + 63) / 64, t = last_blk + (lane + 1) * stepb;
      const bool in = t < after && a.ids[t * a.block] == seg_id;
      const int k = __popcll(__ballot(in));                // ids ascend: the first k probes are in
      const int64_t nxt = last_blk + (int64_t)(k + 1) * stepb;
      last_blk += k * stepb;
      if (nxt < after) after = nxt;
    }
    float4 acc[NV];
#pragma unroll
    for (int v = 0; v < NV; ++v) {
      const int q = lane + 64 * v;
      acc[v] = (wave == 0 && q < nq) ? *reinterpret_cast<const float4*>(a.carry + ((size_t)blk * 2 + 1) * a.dk + 4 * q)
                                     : make_float4(0.f, 0.f, 0.f, 0.f);
    }
    constexpr int FB = 4;                                   // partial rows in flight per wave
    for (int64_t t = blk + 1 + wave; t <= last_blk; t += SPAN_WAVES * FB) {
      float4 rows[FB][NV];
#pragma unroll
      for (int j = 0; j < FB; ++j) {
        const int64_t tt = t + SPAN_WAVES * j;
#pragma unroll
        for (int v = 0; v < NV; ++v) {
          const int q = lane + 64 * v;
          rows[j][v] = (tt <= last_blk && q < nq) ? *reinterpret_cast<const float4*>(a.carry + ((size_t)tt * 2) * a.dk + 4 * q)
                                                  : make_float4(0.f, 0.f, 0.f, 0.f);
        }
      }
#pragma unroll
      for (int j = 0; j < FB; ++j) {
#pragma unroll
        for (int v = 0; v < NV; ++v) add4(acc[v], rows[j][v]);
      }
    }
    __syncthreads();                                        // the previous entry's sums have been read
#pragma unroll
    for (int v = 0; v < NV; ++v) part[wave][lane + 64 * v] = acc[v];
    __syncthreads();
    if (wave == 0) {
      float *emb, *st;
      const int32_t fid = (int32_t)seg_id;
      table_rows(a, fid, emb, st);
#pragma unroll
      for (int v = 0; v < NV; ++v) {
        const int q = lane + 64 * v;
        if (q < nq) {
          float4 s = part[0][q], th, s0;
          for (int w = 1; w < SPAN_WAVES; ++w) add4(s, part[w][q]);
          load_old4<VEC>(a, fid, emb, st, 4 * q, th, s0);
          adagrad4<VEC>(a, fid, emb, st, rank, 4 * q, s, th, s0);
        }
      }
    }
  }
}

// ------------------------------------------------ staging for out-of-memory training -----
// Training with the node table outside device memory (Sec. 3: the table lives in CPU memory, batches move through
// gather / transfer / compute / transfer / update stages).  Here the table is pinned host memory that the GPU reads
// and writes directly; a batch's unique node rows are staged into a compact device table (row = rank of the node
// among the batch's unique rows), the step runs on that table with ids replaced by ranks, and the summed node
// gradients are applied to the host table afterwards.
struct StageArgs {
  const float* host_emb;     // [num_nodes][dim] pinned host memory, device-accessible
  float* host_state;         // [num_nodes][dim] (k_stage_apply)
  float* host_emb_rw;        // same table, writable (k_stage_apply)
  float* compact;            // [unique rows][dim] device
  const float* gsum;         // [unique rows][dk] summed gradients per unique row
  const int32_t* uniq;       // ascending unified ids of the batch's rows: the node ids come first
  const int32_t* scalars;    // [1] = number of unique nodes
  const uint32_t* keys0;     // gradient row -> rank
  int32_t *c_src, *c_dst, *c_neg_dst, *c_neg_src;   // ids replaced by ranks
  int32_t n, cn, roles, sy2, dim, dk;
  float lr, eps;
  const int32_t* prev_uniq[MAR_STAGE_PREV]; const int32_t* prev_scalars[MAR_STAGE_PREV];   // see MarStage
  int32_t num_prev;
  uint8_t* shared;
};

// Ranks in place of node ids, in the layout the step's entry arrays have.
__global__ void __launch_bounds__(256) k_stage_ids(StageArgs a) {
  const int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x;
  const int64_t n3 = (int64_t)a.roles * a.n;
  if (i < a.n) { a.c_src[i] = (int32_t)a.keys0[i]; a.c_dst[i] = (int32_t)a.keys0[a.n + i]; }
  if (i < a.cn) {
    a.c_neg_dst[i] = (int32_t)a.keys0[n3 + i * a.sy2];
    a.c_neg_src[i] = (int32_t)a.keys0[n3 + ((int64_t)a.cn + i) * a.sy2];
  }
}

#define STAGE_ROWS 4   // rows in flight per lane group
// Workgroups of a staging kernel.  A few keep the host link full (51 GB/s read; 20,000-row batches of 100 floats, three
// batches: 32 workgroups 3576 us, 64 3514, 128 3401 - 3434, one per 32 rows 3733): their outstanding host accesses hold
// up every other memory access of the CUs they sit on, and the step of the next batch runs on the others.
#define STAGE_WGS 128

// Whether `id` is in a batch's ascending unique list.
__device__ __forceinline__ bool in_list(const int32_t* __restrict__ uniq, int n, int32_t id) {
  int lo = 0, hi = n;
  while (lo < hi) { const int mid = (lo + hi) >> 1; if (uniq[mid] < id) lo = mid + 1; else hi = mid; }
  return lo < n && uniq[lo] == id;
}

// compact[rank] = host table row of the rank-th unique node; shared[rank] = whether a batch in flight, whose update is
// still to come, has the node too.  One lane group per STAGE_ROWS rows.
template <int GL, int NV, bool VEC>
__global__ void __launch_bounds__(256) k_stage_gather(StageArgs a) {
  constexpr int GPB = 256 / GL;
  const int grp = threadIdx.x / GL, l = threadIdx.x % GL;
  const int un = a.scalars[1];
  for (int r0 = (blockIdx.x * GPB + grp) * STAGE_ROWS; r0 < un; r0 += (int)gridDim.x * GPB * STAGE_ROWS) {
  if (l < STAGE_ROWS && r0 + l < un) {
    bool s = a.num_prev < 0;
    for (int p = 0; p < a.num_prev && !s; ++p) s = in_list(a.prev_uniq[p], a.prev_scalars[p][1], a.uniq[r0 + l]);
    a.shared[r0 + l] = s ? 1 : 0;
  }
  float4 v4[STAGE_ROWS][NV];
#pragma unroll
  for (int j = 0; j < STAGE_ROWS; ++j) {
    const float* row = a.host_emb + (size_t)a.uniq[min(r0 + j, un - 1)] * a.dim;
#pragma unroll
    for (int v = 0; v < NV; ++v) {
      const int k = 4 * (l + GL * v);
      if (k < a.dim) v4[j][v] = load_row4<VEC>(row, k, a.dim);
    }
  }
#pragma unroll
  for (int j = 0; j < STAGE_ROWS; ++j) {
    if (r0 + j < un) {
      float* out = a.compact + (size_t)(r0 + j) * a.dim;
#pragma unroll
      for (int v = 0; v < NV; ++v) {
        const int k = 4 * (l + GL * v);
        if (k < a.dim) store_row4<VEC>(out, k, a.dim, v4[j][v]);
      }
    }
  }
  }
}

// Adagrad on the host table rows of the batch's unique nodes with the summed gradients the step left in gsum
// (Sec. 3, last stage: the update is applied to whatever the table holds now, in batch order).  A row that no batch in
// flight shared still holds what was staged, so its embedding is taken from the compact table instead of over the link.
template <int GL, int NV, bool VEC>
__global__ void __launch_bounds__(256) k_stage_apply(StageArgs a) {
  constexpr int GPB = 256 / GL;
  const int grp = threadIdx.x / GL, l = threadIdx.x % GL;
  const int un = a.scalars[1];
  for (int r0 = (blockIdx.x * GPB + grp) * STAGE_ROWS; r0 < un; r0 += (int)gridDim.x * GPB * STAGE_ROWS) {
  float4 th[STAGE_ROWS][NV], s0[STAGE_ROWS][NV], g[STAGE_ROWS][NV];
  size_t off[STAGE_ROWS];
#pragma unroll
  for (int j = 0; j < STAGE_ROWS; ++j) {
    const int r = min(r0 + j, un - 1);
    off[j] = (size_t)a.uniq[r] * a.dim;
    const float* emb = !a.shared || a.shared[r] ? a.host_emb_rw + off[j] : a.compact + (size_t)r * a.dim;
#pragma unroll
    for (int v = 0; v < NV; ++v) {
      const int k = 4 * (l + GL * v);
      if (k < a.dim) {
        th[j][v] = load_row4<VEC>(emb, k, a.dim);
        s0[j][v] = load_row4<VEC>(a.host_state + off[j], k, a.dim);
        g[j][v] = *reinterpret_cast<const float4*>(a.gsum + (size_t)r * a.dk + k);
      }
    }
  }
#pragma unroll
  for (int j = 0; j < STAGE_ROWS; ++j) {
    if (r0 + j < un) {
#pragma unroll
      for (int v = 0; v < NV; ++v) {
        const int k = 4 * (l + GL * v);
        if (k < a.dim) {
          float4 e1, s1;
          adagrad_math(g[j][v], th[j][v], s0[j][v], a.lr, a.eps, e1, s1);
          store_row4<VEC>(a.host_state + off[j], k, a.dim, s1);
          store_row4<VEC>(a.host_emb_rw + off[j], k, a.dim, e1);
        }
      }
    }
  }
  }
}

// ------------------------------------------------------------------- launchers -----
static RowArgs row_args(const mar_ctx* c, const MarBatch& b) {
  const MarDims& d = c->dm;
  RowArgs a;
  a.node_emb = c->node_emb; a.rel_emb = c->rel_emb;
  a.src = b.src; a.rel = b.rel; a.dst = b.dst; a.neg_src = b.neg_src; a.neg_dst = b.neg_dst;
  a.n = b.n; a.cn = b.cn; a.B = d.B; a.C = d.C; a.N = d.N; a.S = d.S; a.dim = d.dim; a.dk = d.dk; a.model = c->cfg.model;
  a.num_nodes = (int32_t)d.num_nodes;
  a.sy1 = d.sy1; a.sy2 = d.sy2; a.roles = d.roles; a.ml_log2 = mar_on_images(d) ? MAR_LN2 : 1.f; a.shift = c->L.shift;
  return a;
}

template <int GL, int NV, int MODEL, int FORM>
static void launch_prep(const RowArgs& a, const MarLayout& L, float* pos_out, int32_t* rank_dst, int32_t* rank_src, const SplitImages& qi,
                        const SplitImages& ki, const MarSortJob& job, hipStream_t st) {
  constexpr bool img = FORM != PREP_DENSE;
  constexpr int gpb = 256 / GL, re = gpb * prep_edges(GL, img), rn = gpb * PREP_NEGS;
  const int wpc_e = (qi.tiles * SP_TY + re - 1) / re, wpc_n = (ki.tiles * SP_TY + rn - 1) / rn;
  const int nchunks = a.cn / a.N;
  const int nbB = img ? nchunks * wpc_e : (a.n + re - 1) / re;
  const int nbC = img ? 2 * nchunks * wpc_n : (2 * a.cn + rn - 1) / rn;
  const dim3 grid(nbB + nbC + job.blocks), blk(256);
  const unsigned lds = job.blocks ? 4u << MAR_SORT_MAX_BITS : 0u;
  // evaluation keeps the fp32 operands for close comparisons, or (dense) works on them: they lie in the gradients' places
  float* q = MODEL == MAR_MODEL_TRANSE ? L.Q : (rank_dst ? L.gQ : nullptr);
  float* km = MODEL == MAR_MODEL_TRANSE ? L.Km : L.G;
#define PREP_LAUNCH(V, CARRY) hipLaunchKernelGGL((k_prep<GL, NV, V, MODEL, FORM, CARRY>), grid, blk, lds, st, a, job.blocks, nbB, wpc_e, wpc_n, q, km, L.qq, L.kk, L.pos, pos_out, rank_dst, rank_src, qi, ki, job)
  if constexpr (img || MODEL == MAR_MODEL_TRANSE) {         // (the bilinear models' dense form is evaluation's: it carries nothing)
    if (job.blocks) { if (a.dim % 4 == 0) PREP_LAUNCH(true, true); else PREP_LAUNCH(false, true); return; }
  }
  if (a.dim % 4 == 0) PREP_LAUNCH(true, false); else PREP_LAUNCH(false, false);
#undef PREP_LAUNCH
}

hipError_t mar_launch_prep(const mar_ctx* c, const MarBatch& b, float* pos_out, int bf16, int32_t* rank_dst, int32_t* rank_src,
                           hipStream_t st, const MarSortJob* job) {
  const MarLayout& L = c->L;
  const MarSortJob jb = job ? *job : MarSortJob{};
  RowArgs a = row_args(c, b);
  const SplitImages qi = sp_images(L.Qimg, L.Qexp, nullptr, a.dk, c->dm.S), ki = sp_images(L.Kimg, L.Kexp, L.Knorm, a.dk, c->dm.N);
  const int GL = mar_lane_group(a.dk);
  const int form = rank_dst && mar_eval_dense(c->dm, b) ? PREP_DENSE : (bf16 ? PREP_BF16 : PREP_F16);
#define PREP3(GLV, NVV, M) do { \
    if (form == PREP_F16) launch_prep<GLV, NVV, M, PREP_F16>(a, L, pos_out, rank_dst, rank_src, qi, ki, jb, st); \
    else if (form == PREP_BF16) launch_prep<GLV, NVV, M, PREP_BF16>(a, L, pos_out, rank_dst, rank_src, qi, ki, jb, st); \
    else launch_prep<GLV, NVV, M, PREP_DENSE>(a, L, pos_out, rank_dst, rank_src, qi, ki, jb, st); } while (0)
#define PREP(GLV, NVV) do { switch (a.model) { \
    case MAR_MODEL_DISTMULT: PREP3(GLV, NVV, MAR_MODEL_DISTMULT); break; \
    case MAR_MODEL_COMPLEX: PREP3(GLV, NVV, MAR_MODEL_COMPLEX); break; \
    case MAR_MODEL_TRANSE: \
      if (c->dm.dist_img && !rank_dst) launch_prep<GLV, NVV, MAR_MODEL_TRANSE, PREP_F16>(a, L, pos_out, rank_dst, rank_src, qi, ki, jb, st); \
      else launch_prep<GLV, NVV, MAR_MODEL_TRANSE, PREP_DENSE>(a, L, pos_out, rank_dst, rank_src, qi, ki, jb, st); \
      break; \
    default: PREP3(GLV, NVV, MAR_MODEL_DOT); break; } } while (0)
  // lanes x float4s per lane cover a row (ComplEx: lanes x float2s cover half a row)
  if (GL == 16) PREP(16, 1); else if (GL == 32) PREP(32, 1); else if (a.dk <= 256) PREP(64, 1); else PREP(64, 2);
#undef PREP
#undef PREP3
  return hipGetLastError();
}

hipError_t mar_launch_filter(const mar_ctx* c, const MarBatch& b, const int64_t* dst_off, const int32_t* dst_ids,
                             const int64_t* src_off, const int32_t* src_ids, const float* pos, int32_t* rank_dst,
                             int32_t* rank_src, hipStream_t st) {
  RowArgs a = row_args(c, b);
  const int GL = mar_lane_group(a.dk), gpb = 256 / GL;
  const dim3 grid((2 * b.n + gpb - 1) / gpb), blk(256);
#define FILTER3(GLV, NVV, M) do { \
    if (a.dim % 4 == 0) hipLaunchKernelGGL((k_filter<GLV, NVV, true, M>), grid, blk, 0, st, a, dst_off, dst_ids, src_off, src_ids, pos, rank_dst, rank_src); \
    else hipLaunchKernelGGL((k_filter<GLV, NVV, false, M>), grid, blk, 0, st, a, dst_off, dst_ids, src_off, src_ids, pos, rank_dst, rank_src); } while (0)
#define FILTER(GLV, NVV) do { switch (a.model) { \
    case MAR_MODEL_DISTMULT: FILTER3(GLV, NVV, MAR_MODEL_DISTMULT); break; \
    case MAR_MODEL_COMPLEX: FILTER3(GLV, NVV, MAR_MODEL_COMPLEX); break; \
    case MAR_MODEL_TRANSE: FILTER3(GLV, NVV, MAR_MODEL_TRANSE); break; \
    default: FILTER3(GLV, NVV, MAR_MODEL_DOT); break; } } while (0)
  if (GL == 16) FILTER(16, 1); else if (GL == 32) FILTER(32, 1); else if (a.dk <= 256) FILTER(64, 1); else FILTER(64, 2);
#undef FILTER
#undef FILTER3
  return hipGetLastError();
}

template <int GL, int NV, int MODEL>
static void launch_chain(const RowArgs& a, const MarLayout& L, float* lse_dst, float* lse_src, dim3 grid, const MarSortJob& job, hipStream_t st) {
#define CHAIN2(V, S, CARRY) hipLaunchKernelGGL((k_chain<GL, NV, MODEL, V, S, CARRY>), grid, dim3(256), CARRY ? SORT_LDS_BYTES : 0, st, a, job.blocks, L.gQ, L.ml, L.pos, lse_dst, lse_src, L.G, L.loss_part, job)
#define CHAIN(V, S) do { if (job.blocks) CHAIN2(V, S, true); else CHAIN2(V, S, false); } while (0)
  if (a.dim % 4 == 0) { if (a.sy1 == 1) CHAIN(true, 1); else if (a.sy1 == 2) CHAIN(true, 2); else CHAIN(true, 0); }
  else CHAIN(false, 0);
#undef CHAIN
#undef CHAIN2
}

template <int GL, int NV>
static void launch_chain_model(const RowArgs& a, const MarLayout& L, float* lse_dst, float* lse_src, dim3 grid, const MarSortJob& job, hipStream_t st) {
  switch (a.model) {
    case MAR_MODEL_DISTMULT: launch_chain<GL, NV, MAR_MODEL_DISTMULT>(a, L, lse_dst, lse_src, grid, job, st); break;
    case MAR_MODEL_COMPLEX:  launch_chain<GL, NV, MAR_MODEL_COMPLEX>(a, L, lse_dst, lse_src, grid, job, st); break;
    case MAR_MODEL_TRANSE:   launch_chain<GL, NV, MAR_MODEL_TRANSE>(a, L, lse_dst, lse_src, grid, job, st); break;
    default:                 launch_chain<GL, NV, MAR_MODEL_DOT>(a, L, lse_dst, lse_src, grid, job, st); break;
  }
}

hipError_t mar_launch_chain(const mar_ctx* c, const MarBatch& b, const mar_debug_out* dbg, hipStream_t st, const MarSortJob* carried) {
  const MarLayout& L = c->L;
  RowArgs a = row_args(c, b);
  const int GL = mar_lane_group(a.dk), gpb = 256 / GL;
  const MarSortJob job = carried ? *carried : MarSortJob{};
  const dim3 grid((b.n + gpb - 1) / gpb + job.blocks);
  float *lse_dst = dbg ? dbg->lse_dst : nullptr, *lse_src = dbg ? dbg->lse_src : nullptr;
  // lanes x float4s per lane cover a row (ComplEx: lanes x float2s cover half a row)
  if (GL == 16) launch_chain_model<16, 1>(a, L, lse_dst, lse_src, grid, job, st);
  else if (GL == 32) launch_chain_model<32, 1>(a, L, lse_dst, lse_src, grid, job, st);
  else if (a.dk <= 256) launch_chain_model<64, 1>(a, L, lse_dst, lse_src, grid, job, st);
  else launch_chain_model<64, 2>(a, L, lse_dst, lse_src, grid, job, st);
  return hipGetLastError();
}

hipError_t mar_launch_reduce(const mar_ctx* c, const MarBatch& b, float* loss_out, float* dbg_grad, float* defer_grad, hipStream_t st) {
  const MarLayout& L = c->L;
  const MarDims& d = c->dm;
  ReduceArgs a;
  a.node_emb = c->node_emb; a.node_state = c->node_state; a.rel_emb = c->rel_emb; a.rel_state = c->rel_state;
  a.G = L.G; a.carry = L.carry; a.ids = L.ids_sorted; a.perm = L.perm; a.rank_sorted = dbg_grad || defer_grad ? L.rank_sorted : nullptr;
  a.scalars = L.scalars; a.owners = L.owners; a.dbg_grad = dbg_grad; a.defer_grad = defer_grad; a.n_rows = b.n_pos;
  a.num_nodes = (int32_t)d.num_nodes; a.dim = d.dim; a.dk = d.dk; a.lr = c->cfg.lr; a.eps = c->cfg.eps;
  a.block = mar_reduce_block(d);
  const int64_t blocks = (b.n_pos + a.block - 1) / a.block;
  const dim3 grid((unsigned)blocks), grids((unsigned)(blocks < 512 ? blocks : 512)), blk(256), blks(64 * SPAN_WAVES);
  const int GL = mar_lane_group(d.dk), gpb = 256 / GL;
  const int n_loss_part = (b.n + gpb - 1) / gpb;
  const bool vec = d.dim % 4 == 0;
#define RED2(GLV, NVV, BT, P) do { \
    if (vec) hipLaunchKernelGGL((k_reduce_apply<GLV, NVV, BT, true, P>), grid, blk, 0, st, a); \
    else hipLaunchKernelGGL((k_reduce_apply<GLV, NVV, BT, false, P>), grid, blk, 0, st, a); } while (0)
#define RED(GLV, NVV, BT) do { \
    if (d.reduce_small == 4) RED2(GLV, NVV, 4, 4); else if (d.reduce_small) RED2(GLV, NVV, BT, 8); else RED2(GLV, NVV, BT, GLV); } while (0)
  if (GL == 16) RED(16, 1, 8); else if (GL == 32) RED(32, 1, 8); else if (d.dk <= 256) RED(64, 1, 8); else RED(64, 2, 4);
#undef RED
#undef RED2
  if (d.dk <= 256) {
    if (vec) hipLaunchKernelGGL((k_span_apply<1, true>), grids, blks, 0, st, a, L.loss_part, n_loss_part, loss_out);
    else hipLaunchKernelGGL((k_span_apply<1, false>), grids, blks, 0, st, a, L.loss_part, n_loss_part, loss_out);
  } else {
    if (vec) hipLaunchKernelGGL((k_span_apply<2, true>), grids, blks, 0, st, a, L.loss_part, n_loss_part, loss_out);
    else hipLaunchKernelGGL((k_span_apply<2, false>), grids, blks, 0, st, a, L.loss_part, n_loss_part, loss_out);
  }
  return hipGetLastError();
}

static StageArgs stage_args(const mar_ctx* c, const MarBatch& b, const MarStage& sg) {
  const MarDims& d = c->dm;
  StageArgs a;
  a.host_emb = sg.host_emb; a.host_emb_rw = sg.host_emb; a.host_state = sg.host_state;
  a.compact = sg.compact; a.gsum = sg.gsum; a.uniq = c->L.uniq; a.scalars = c->L.scalars; a.keys0 = c->L.keys0;
  a.c_src = sg.c_src; a.c_dst = sg.c_dst; a.c_neg_dst = sg.c_neg_dst; a.c_neg_src = sg.c_neg_src;
  a.n = b.n; a.cn = b.cn; a.roles = d.roles; a.sy2 = d.sy2; a.dim = d.dim; a.dk = d.dk;
  a.lr = c->cfg.lr; a.eps = c->cfg.eps;
  for (int p = 0; p < MAR_STAGE_PREV; ++p) { a.prev_uniq[p] = sg.prev_uniq[p]; a.prev_scalars[p] = sg.prev_scalars[p]; }
  a.num_prev = sg.num_prev; a.shared = sg.shared;
  return a;
}

// most unique nodes a batch can have: the grids of the staging kernels are sized for it, the kernels read the count
static int64_t stage_rows_max(const mar_ctx* c, const MarBatch& b) {
  const int64_t occ = 2 * (int64_t)b.n + 2 * (int64_t)b.cn;
  return occ < c->dm.num_nodes ? occ : c->dm.num_nodes;
}

#define STAGE_LAUNCH(KERNEL) do { \
    const int GL = mar_lane_group(a.dk), gpb = 256 / GL; \
    const int64_t full = (stage_rows_max(c, b) + gpb * STAGE_ROWS - 1) / (gpb * STAGE_ROWS); \
    const dim3 grid((unsigned)(full < STAGE_WGS ? full : STAGE_WGS)), blk(256); \
    const bool vec = a.dim % 4 == 0; \
    if (GL == 16) { if (vec) hipLaunchKernelGGL((KERNEL<16, 1, true>), grid, blk, 0, st, a); else hipLaunchKernelGGL((KERNEL<16, 1, false>), grid, blk, 0, st, a); } \
    else if (GL == 32) { if (vec) hipLaunchKernelGGL((KERNEL<32, 1, true>), grid, blk, 0, st, a); else hipLaunchKernelGGL((KERNEL<32, 1, false>), grid, blk, 0, st, a); } \
    else if (a.dk <= 256) { if (vec) hipLaunchKernelGGL((KERNEL<64, 1, true>), grid, blk, 0, st, a); else hipLaunchKernelGGL((KERNEL<64, 1, false>), grid, blk, 0, st, a); } \
    else { if (vec) hipLaunchKernelGGL((KERNEL<64, 2, true>), grid, blk, 0, st, a); else hipLaunchKernelGGL((KERNEL<64, 2, false>), grid, blk, 0, st, a); } \
  } while (0)

hipError_t mar_launch_stage_in(const mar_ctx* c, const MarBatch& b, const MarStage& sg, hipStream_t st) {
  StageArgs a = stage_args(c, b, sg);
  const int64_t work = b.n > b.cn ? b.n : b.cn;
  hipLaunchKernelGGL(k_stage_ids, dim3((unsigned)((work + 255) / 256)), dim3(256), 0, st, a);
  STAGE_LAUNCH(k_stage_gather);
  return hipGetLastError();
}

hipError_t mar_launch_stage_out(const mar_ctx* c, const MarBatch& b, const MarStage& sg, hipStream_t st) {
  StageArgs a = stage_args(c, b, sg);
  STAGE_LAUNCH(k_stage_apply);
  return hipGetLastError();
}
