// Operand images of the contraction passes that split their operands (gfx950): geometry and the stores that build them.
//
// A matrix that takes part in a pass (the chunk's negatives, the chunk's edge-side operands) is kept as "images": per
// chunk-side and tile of 32 rows a plane of the rows' hi parts and a plane of their lo parts, each [32][PA bytes], a
// row = 16 NK 16-bit values: the dk columns and zeros up to the next multiple of 16 that an instantiation serves.  The
// 16-byte units of a row lie in an order of their own (sp_swizzle).  An image is one contiguous block of IMG bytes (a
// multiple of 1 KB).
//   fp32 precision:  v 2^e = hi + lo with hi = f16(v 2^e), lo = f16(v 2^e - hi), one exponent e per block of 16 rows,
//                    chosen so that the block's largest value lies in [2^14, 2^15); e is kept beside the images.
//   SPLIT_BF16:      v = hi + lo with hi = bf16(v), lo = bf16(v - hi).
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

#include "mar_common.h"

#ifdef __HIPCC__
#define MAR_HD __host__ __device__
#else
#define MAR_HD
#endif

// Row pitch of a plane whose rows hold 16 NK values, in 16-byte units: a multiple of 4.
constexpr int sp_units(int nk) { return (2 * nk + 3) / 4 * 4; }
constexpr int sp_pitch(int nk) { return 16 * sp_units(nk); }
// Unit u of row y lies at unit u ^ sp_swizzle(units, y) of the row, chosen so that the reads of the passes are free of bank
// conflicts (counted: none in evaluation and at 400 floats; 4.1e5 of 1.2e7 LDS cycles in the training passes at 100 floats, whose
// packed last block reads halves of its rows in two planes).  The LDS has 64 banks, 16 units; 16-byte reads are served in groups of 16 lanes -- 0-3, 12-15,
// 20-23, 24-27, then the other lanes of the first 32 -- and transpose reads of 8 bytes in groups of 32.  With the pitch alone
// rows y % 4 start 4 or 12 units apart (mod 16) where units % 16 is 4 or 12, 8 apart where it is 8, together where it is 0;
// the upper bits make up for what is missing, so that four consecutive rows lie in four different groups of 4 units.
// Score product: lane 16 g + i reads unit u + g of row i, u = 0 mod 4 (32 x 32 blocks: lane 32 h + m unit u + h of row m, u even).  Transpose reads: lanes 16 g + i read 32 bytes at an even
// unit of rows 4 g .. 4 g + 3.  So with L(q) the lower two bits for rows 4 q .. 4 q + 3: L(0), L(3), L(1) ^ 1, L(2) ^ 1 differ, and
// L(0), L(1) and L(2), L(3) differ in the upper bit: 0, 2, 3, 1.
constexpr int sp_group(int units) { return units % 16 == 0 ? 16 : (units % 16 == 8 ? 8 : 4); }   // units a swizzle permutes
MAR_HD constexpr int sp_swizzle(int units, int y) {
  return (units % 16 == 0 ? 4 * (y & 3) : (units % 16 == 8 ? 4 * ((y >> 1) & 1) : 0)) | (((y >> 1) ^ (y >> 2)) & 2) | ((y >> 3) & 1);
}
constexpr int SP_TY = MAR_SPLIT_TILE_ROWS;                 // rows per image
constexpr int SP_EB = 16;                                  // rows per exponent
constexpr int SP_SR = MAR_SPLIT_STRIPE_ROWS;               // stationary rows per workgroup: four waves of 32
// 16-column blocks (NK) of the instantiation that serves dk.
constexpr int sp_nk(int dk) { return dk <= 32 ? 2 : (dk <= 64 ? 4 : (dk <= 96 ? 6 : (dk <= 112 ? 7 : (dk <= 128 ? 8 : (dk <= 192 ? 12 : (dk <= 256 ? 16 : 25)))))); }
constexpr int sp_plane(int nk) { return SP_TY * sp_pitch(nk); }
constexpr int sp_image(int nk) { return (2 * sp_plane(nk) + 1023) / 1024 * 1024; }
constexpr int SP_NORMS = 2 + SP_TY;
// Where share q of all units' tiles begins: shares of `share` tiles, the first `rest` one more.  A border one tile off a unit's is
// moved there, for a piece of one tile costs its stationary rows all the same (units of at least three tiles: mar_plan_shares).
MAR_HD inline int64_t sp_share_border(int64_t share, int32_t rest, int ntiles, int q) {
  const int64_t b = q * share + (q < rest ? q : rest), in = b % ntiles;
  return in == 1 ? b - 1 : (in == ntiles - 1 ? b + 1 : b);
}
static inline int sp_tiles(int rows) { return (rows + SP_TY - 1) / SP_TY; }

// Where the gather writes an image set: [chunk-sides][tiles][IMG].
struct SplitImages {
  char* base;
  float* exps;          // [chunk-sides][2 tiles] exponent of every 16-row block (+ SP_NONFINITE)
  float* norms;         // evaluation: [chunk-sides][tiles][SP_NORMS] bounds of the scaled rows' norms: of the two blocks (0: all
                        // zero), then of the 32 rows (-1: a zero row)
  int32_t units, plane, img, tiles, dkp;
};
// Added to the exponent of a block that holds an infinity or a NaN (its exponent is that of its finite values).
#define SP_NONFINITE 1024.f
static inline SplitImages sp_images(char* base, float* exps, float* norms, int dk, int rows_per_chunk) {
  const int nk = sp_nk(dk);
  SplitImages g;
  g.base = base; g.exps = exps; g.norms = norms; g.units = sp_units(nk); g.plane = sp_plane(nk); g.img = sp_image(nk);
  g.tiles = sp_tiles(rows_per_chunk); g.dkp = 16 * nk;
  return g;
}

#ifdef __HIPCC__
// Row `row` of chunk-side `cs`: its start in the hi plane (the lo plane's is g.plane bytes further) and its swizzle in bytes.
struct SplitRow { char* hi; int plane, swz; };
__device__ __forceinline__ SplitRow sp_row(const SplitImages& g, int cs, int row) {
  SplitRow r;
  r.hi = g.base + ((size_t)cs * g.tiles + row / SP_TY) * g.img + (row % SP_TY) * g.units * 16;
  r.plane = g.plane; r.swz = 16 * sp_swizzle(g.units, row % SP_TY);
  return r;
}
// Exponent of a block whose largest finite magnitude has these float bits: 2^e max lies in [2^14, 2^15).  Clamped to
// what a float power of two and the sums of a pass can hold (a block of values below 2^-66 keeps fewer bits).  A block of
// zeros takes the largest exponent: the softmax reference follows score log2(e) - e, and such a block, whose rows carry
// nothing, must not move it away from the others, whose weights would lose bits to the f16 range (worst gradient row beside
// such a block, values of 1e-5: 9e-7 off, with exponent 0 9e-3).
#define SP_EMAX 80
__device__ __forceinline__ int sp_exponent(int max_bits) {
  const int e = 141 - (max_bits >> 23);
  return e > SP_EMAX ? SP_EMAX : e;
}
typedef _Float16 sp_h2 __attribute__((ext_vector_type(2)));
typedef _Float16 sp_h4 __attribute__((ext_vector_type(4)));
typedef __bf16 sp_bf2 __attribute__((ext_vector_type(2)));
typedef __bf16 sp_bf4 __attribute__((ext_vector_type(4)));

// hi and lo parts of a scaled value; an infinity or NaN is its hi part alone
__device__ __forceinline__ void sp_parts(float v, _Float16& h, _Float16& l) {
  h = (_Float16)v;
  l = (_Float16)(fabsf(v) <= 3.0e38f ? v - (float)h : 0.f);
}
__device__ __forceinline__ void sp_parts(float v, __bf16& h, __bf16& l) { h = (__bf16)v; l = (__bf16)(v - (float)h); }

template <bool F16> __device__ __forceinline__ void sp_store1(const SplitRow& row, int col, float v, float scale) {
  char* const at = row.hi + ((2 * col) ^ row.swz);
  if (F16) {
    _Float16 h, l;
    sp_parts(v * scale, h, l);
    *reinterpret_cast<_Float16*>(at) = h;
    *reinterpret_cast<_Float16*>(at + row.plane) = l;
  } else {
    __bf16 h, l;
    sp_parts(v, h, l);
    *reinterpret_cast<__bf16*>(at) = h;
    *reinterpret_cast<__bf16*>(at + row.plane) = l;
  }
}
template <bool F16> __device__ __forceinline__ void sp_store2(const SplitRow& row, int col, float2 v, float scale) {
  char* const at = row.hi + ((2 * col) ^ row.swz);
  if (F16) {
    _Float16 h[2], l[2];
    sp_parts(v.x * scale, h[0], l[0]); sp_parts(v.y * scale, h[1], l[1]);
    *reinterpret_cast<sp_h2*>(at) = (sp_h2){h[0], h[1]};
    *reinterpret_cast<sp_h2*>(at + row.plane) = (sp_h2){l[0], l[1]};
  } else {
    __bf16 h[2], l[2];
    sp_parts(v.x, h[0], l[0]); sp_parts(v.y, h[1], l[1]);
    *reinterpret_cast<sp_bf2*>(at) = (sp_bf2){h[0], h[1]};
    *reinterpret_cast<sp_bf2*>(at + row.plane) = (sp_bf2){l[0], l[1]};
  }
}
template <bool F16> __device__ __forceinline__ void sp_store4(const SplitRow& row, int col, float4 v, float scale) {
  char* const at = row.hi + ((2 * col) ^ row.swz);
  if (F16) {
    _Float16 h[4], l[4];
    sp_parts(v.x * scale, h[0], l[0]); sp_parts(v.y * scale, h[1], l[1]); sp_parts(v.z * scale, h[2], l[2]); sp_parts(v.w * scale, h[3], l[3]);
    *reinterpret_cast<sp_h4*>(at) = (sp_h4){h[0], h[1], h[2], h[3]};
    *reinterpret_cast<sp_h4*>(at + row.plane) = (sp_h4){l[0], l[1], l[2], l[3]};
  } else {
    __bf16 h[4], l[4];
    sp_parts(v.x, h[0], l[0]); sp_parts(v.y, h[1], l[1]); sp_parts(v.z, h[2], l[2]); sp_parts(v.w, h[3], l[3]);
    *reinterpret_cast<sp_bf4*>(at) = (sp_bf4){h[0], h[1], h[2], h[3]};
    *reinterpret_cast<sp_bf4*>(at + row.plane) = (sp_bf4){l[0], l[1], l[2], l[3]};
  }
}
#endif
