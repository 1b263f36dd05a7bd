// Device helpers shared by the kernels on the 16-bit matrix pipe (gfx950): matrix instruction, the hi/lo split of weights,
// LDS reads, geometry.
#pragma once
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

__device__ __forceinline__ v16f mfma32h(v8s a, v8s b, v16f c) {
  return __builtin_amdgcn_mfma_f32_32x32x16_f16(__builtin_bit_cast(v8h, a), __builtin_bit_cast(v8h, b), c, 0, 0, 0);
}
template <bool F16> __device__ __forceinline__ v4f mfma16h(v8s a, v8s b, v4f c) {
  if (F16) return __builtin_amdgcn_mfma_f32_16x16x32_f16(__builtin_bit_cast(v8h, a), __builtin_bit_cast(v8h, b), c, 0, 0, 0);
  return __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(v8b, a), __builtin_bit_cast(v8b, b), c, 0, 0, 0);
}

// v = hi + lo, two values per step: one packed conversion and two mixed-precision multiply-adds (f16; neg1 = -1 in a
// register the compiler cannot see through, or it would turn the multiply-add into a conversion and a subtraction),
// two packed conversions with the unpacking between them (bf16).
template <bool F16> __device__ __forceinline__ void split8(const float (&v)[8], float neg1, v8s& hi, v8s& lo) {
  v4i hw, lw;                                              // two 16-bit values per word
#pragma unroll
  for (int i = 0; i < 4; ++i) {
    const float p0 = v[2 * i], p1 = v[2 * i + 1];
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
__device__ __forceinline__ v8s lds_read16(unsigned address) {
  return *(__attribute__((address_space(3))) const v8s*)address;
}
__device__ __forceinline__ v4s lds_read_tr(const char* p) {
  return __builtin_amdgcn_ds_read_tr16_b64_v4i16((__attribute__((address_space(3))) v4s*)p);
}
__device__ __forceinline__ v8s join8(v4s a, v4s b) { return __builtin_shufflevector(a, b, 0, 1, 2, 3, 4, 5, 6, 7); }

#define SP_PEND 6                                          // candidates whose comparisons a lane of pass 3 keeps for the end (5 bits of a word each)
#define SP_FULL 8                                          // added to their number: this lane takes no more (above SP_PEND)
// Steps of 32 columns whose stationary fragments TransE's passes keep in LDS: 400 floats' sums and fragments leave too few registers
// for the weights (all in registers 62 and 73 spilled; one step in LDS 14 and 41, two 0 and 13).
constexpr int sp_dist_lds_steps(int nk) { return nk > 16 ? 3 : 0; }
template <int NK>
struct SplitGeom {
  static constexpr int UNITS = sp_units(NK);
  static constexpr int PA = sp_pitch(NK);
  static constexpr int PLANE = sp_plane(NK);
  static constexpr int IMG = sp_image(NK);
  static constexpr int NCH = IMG / 1024;                   // 1 KB pieces of an image
  static constexpr size_t LDS_TILES = 2 * (size_t)IMG + 4 * SP_TY * 4;
  static constexpr size_t LDS_BYTES = LDS_TILES < SORT_LDS_BYTES ? SORT_LDS_BYTES : LDS_TILES;   // two images, and (pass 2) the log-sum-exp of a tile's edges
  static constexpr size_t LDS_BYTES_DIST = LDS_BYTES + 2 * SP_TY * 4 + (size_t)sp_dist_lds_steps(NK) * 4 * 4096 + 3 * 2 * 256 * 4;   // TransE: and the squared norms of two tiles' rows, stationary fragments, close pairs
  static constexpr size_t LDS_BYTES3 = 2 * (size_t)IMG + 2 * SP_PEND * 256 * 4;   // two images, and the lanes' pending candidates: id, how often
};
