// Operand handling shared by the low-precision kernels: types, the lane roles
// of a wave's 64 complex columns, the turned operand, the partial branch
// weights, and the splitting of left vectors into operand planes.
#pragma once

#include "e2m3.h"

#include <hip/hip_runtime.h>
#include <stdint.h>

namespace mps {
namespace {

typedef float floatx16 __attribute__((ext_vector_type(16)));
typedef __bf16 bf16_t;
typedef _Float16 f16_t;
typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef _Float16 f16x8 __attribute__((ext_vector_type(8)));

template <typename T>
struct Vec8;
template <>
struct Vec8<bf16_t> {
  typedef bf16x8 type;
  static __device__ floatx16 mfma(type a, type b, floatx16 c) {
    return __builtin_amdgcn_mfma_f32_32x32x16_bf16(a, b, c, 0, 0, 0);
  }
};
template <>
struct Vec8<f16_t> {
  typedef f16x8 type;
  static __device__ floatx16 mfma(type a, type b, floatx16 c) {
    return __builtin_amdgcn_mfma_f32_32x32x16_f16(a, b, c, 0, 0, 0);
  }
};

// A wave's 64 complex columns as MFMA blocks: acc[rb][2 b] and acc[rb][2 b + 1]
// hold the real and imaginary parts of the 32 columns of block b, lane j the
// column wave_col(b, j).  This order keeps the partial weights' additions
// those of 16-column blocks taken in order (store_partials).
__device__ inline int wave_col(int b, int j) { return (j >> 4) * 32 + b * 16 + (j & 15); }

// The p = 1 row of the embedding from the p = 0 row, per lane: (x, y) ->
// (-y, x).  With the real parts of 4 complex in one half of a lane's 8 K
// values and the imaginary ones in the other (kblk_off) that is an exchange
// of the halves and two sign flips.
template <typename V8>
__device__ inline V8 turn(V8 v) {
  typedef unsigned uintx4 __attribute__((ext_vector_type(4)));
  const uintx4 w = __builtin_bit_cast(uintx4, v);
  return __builtin_bit_cast(V8, uintx4{w[2] ^ 0x80008000u, w[3] ^ 0x80008000u, w[0], w[1]});
}

// LDS rows are 32 bytes (16 K values = 2 chunks of 16 bytes).  The chunk is
// XOR-swizzled by row bits 2 and 3 so that the 16-byte reads of 8 or 16
// consecutive lanes (consecutive rows, same chunk) land in distinct banks.
__device__ inline int swz(int row) { return ((row >> 2) ^ (row >> 3)) & 1; }
__device__ inline int lds_off(int row, int chunk) { return row * 32 + ((chunk ^ swz(row)) << 4); }

typedef int intx4 __attribute__((ext_vector_type(4)));
typedef int intx8 __attribute__((ext_vector_type(8)));

// E8M0 scale codes of the FP8 products: 2^-19 on the left-vector operand
// (the common factor of both corrections), 2^0 on the site tensor's.
constexpr int kScale8L = 127 - 19;
constexpr int kScale8B = 127;

// turn (above) for a pair plane's E4M3 codes (groups of 8 bytes) and an E2M3
// record's codes (dwords 0..2 real, 3..5 imaginary parts; dword 6, the scale,
// is shared: the maximum is the same).
__device__ inline intx8 turn_e4m3(intx8 w) {
  intx8 o;
#pragma unroll
  for (int i = 0; i < 8; i += 2) {
    o[i] = w[i + 1] ^ (int)0x80808080u;
    o[i + 1] = w[i];
  }
  return o;
}
__device__ inline intx8 turn_e2m3(intx8 w) {
  return intx8{w[3] ^ 0x20820820, w[4] ^ 0x08208208, w[5] ^ (int)0x82082082u, w[0], w[1], w[2], w[6], 0};
}

// Partial branch weight of 64 complex columns (the granularity of every kernel
// and variant).  Per row and part (re, im) the sum runs over
// the columns 16 + t, t, 32 + t, 48 + t (fused multiply-adds in that order),
// then over t by an xor butterfly (8, 4, 2, 1), then re + im: the same order
// everywhere.
// Lane j of a 32-lane half holds columns t and 16 + t (j = t < 16) or 32 + t
// and 48 + t (j = 16 + t), both parts; swapping 16-lane rows between the two
// parts gives every lane one part's four columns (lanes t the real parts,
// 16 + t the imaginary ones), and after a rotate-add by 8 the values repeat
// with period 8, so that rotations by 4, 2 and 1 meet the butterfly's
// partners.  Registers and DPP only: no LDS permutes.
template <int R>
__device__ inline float add_ror(float s) {
  return s + __uint_as_float(__builtin_amdgcn_update_dpp(0, __float_as_uint(s), 0x120 + R, 0xF, 0xF, true));
}
__device__ inline float part_sum(float re0, float im0, float re1, float im1) {
  const auto p0 = __builtin_amdgcn_permlane16_swap(__float_as_uint(re0), __float_as_uint(im0), false, false);
  const auto p1 = __builtin_amdgcn_permlane16_swap(__float_as_uint(re1), __float_as_uint(im1), false, false);
  const float x0 = __uint_as_float(p0[0]), x1 = __uint_as_float(p1[0]);
  const float x2 = __uint_as_float(p0[1]), x3 = __uint_as_float(p1[1]);
  float s = __builtin_fmaf(x0, x0, x1 * x1);
  s = __builtin_fmaf(x2, x2, s);
  s = __builtin_fmaf(x3, x3, s);
  s = add_ror<8>(s);
  s = add_ror<4>(s);
  s = add_ror<2>(s);
  s = add_ror<1>(s);
  const auto q = __builtin_amdgcn_permlane16_swap(__float_as_uint(s), __float_as_uint(s), false, false);
  return __uint_as_float(q[0]) + __uint_as_float(q[1]);
}

// ---- left vectors to operand planes -----------------------------------------
// 4 complex (half a 16-K slice: real parts, then imaginary) as x = hi + lo,
// hi = T(x) (round to nearest even), lo = T(x - hi).
__device__ inline uint32_t pair16(uint16_t a, uint16_t b) { return (uint32_t)a | ((uint32_t)b << 16); }
template <typename T>
__device__ inline void split4(const float2 (&v)[4], uint32_t (&h)[4], uint32_t (&l)[4]) {
#pragma unroll
  for (int j = 0; j < 4; ++j) {
    const float x = j < 2 ? v[2 * j].x : v[2 * j - 4].y, y = j < 2 ? v[2 * j + 1].x : v[2 * j - 3].y;
    const T xh = (T)x, yh = (T)y;
    h[j] = pair16(__builtin_bit_cast(uint16_t, xh), __builtin_bit_cast(uint16_t, yh));
    const T xl = (T)(x - (float)xh), yl = (T)(y - (float)yh);
    l[j] = pair16(__builtin_bit_cast(uint16_t, xl), __builtin_bit_cast(uint16_t, yl));
  }
}

// The fp16 parts, and the E4M3 codes of hi * 2^8 and lo * 2^19 (8 bytes each).
__device__ inline void split4_e4m3(const float2 (&v)[4], uint32_t (&h)[4], uint32_t (&ch)[2], uint32_t (&cl)[2]) {
  unsigned a[4], b[4];
#pragma unroll
  for (int j = 0; j < 4; ++j) {
    const float x = j < 2 ? v[2 * j].x : v[2 * j - 4].y, y = j < 2 ? v[2 * j + 1].x : v[2 * j - 3].y;
    const f16_t xh = (f16_t)x, yh = (f16_t)y;
    h[j] = pair16(__builtin_bit_cast(uint16_t, xh), __builtin_bit_cast(uint16_t, yh));
    const float xf = (float)xh, yf = (float)yh;
    a[j] = (unsigned)__builtin_amdgcn_cvt_pk_fp8_f32(xf * 256.f, yf * 256.f, 0, false) & 0xFFFFu;
    b[j] = (unsigned)__builtin_amdgcn_cvt_pk_fp8_f32((x - xf) * 524288.f, (y - yf) * 524288.f, 0, false) & 0xFFFFu;
  }
  ch[0] = a[0] | (a[1] << 16);
  ch[1] = a[2] | (a[3] << 16);
  cl[0] = b[0] | (b[1] << 16);
  cl[1] = b[2] | (b[3] << 16);
}

// Four codes (first in the low 6 bits) of values divided by their record's
// scale and by 64: E4M3 has E2M3's 3 mantissa bits, and its smallest normal
// value is 2^-6 where E2M3's is 1, so the conversion instruction's code of
// x / 64 is e2m3_code(x) with the sign at bit 7 (equal for every float of
// magnitude <= 7.5: all bit patterns compared on the GPU).  About 4
// instructions a value against 14 for e2m3_code.
__device__ inline uint32_t e2m3x4(float a, float b, float c, float d) {
  uint32_t w = (uint32_t)__builtin_amdgcn_cvt_pk_fp8_f32(a, b, 0, false);
  w = (uint32_t)__builtin_amdgcn_cvt_pk_fp8_f32(c, d, (int)w, true);
  w = (w & 0x1F1F1F1Fu) | ((w >> 2) & 0x20202020u);
  w = (w & 0x003F003Fu) | ((w >> 2) & 0x0FC00FC0u);
  return (w & 0xFFFu) | ((w >> 4) & 0xFFF000u);
}

// A whole slice (8 complex): the fp16 parts and the E2M3 record.
__device__ inline void split8_e2m3(const float2 (&v)[8], uint32_t (&h)[8], uint32_t (&w)[8]) {
  float hv[16], lv[16];
  float m = 0.f;
#pragma unroll
  for (int j = 0; j < 8; ++j) {
    // word j of the plane: re 0 1, re 2 3, im 0 1, im 2 3, then the same of complex 4 .. 7
    const int e = 4 * (j >> 2) + 2 * (j & 1);
    const float x = j & 2 ? v[e].y : v[e].x, y = j & 2 ? v[e + 1].y : v[e + 1].x;
    const f16_t xh = (f16_t)x, yh = (f16_t)y;
    h[j] = pair16(__builtin_bit_cast(uint16_t, xh), __builtin_bit_cast(uint16_t, yh));
    const float xf = (float)xh, yf = (float)yh;
    const int t = (j & 2 ? 8 : 0) + e;  // 0..7 the real parts, 8..15 the imaginary ones
    hv[t] = xf * 256.f;
    hv[t + 1] = yf * 256.f;
    lv[t] = (x - xf) * 524288.f;
    lv[t + 1] = (y - yf) * 524288.f;
    m = fmaxf(m, fmaxf(fmaxf(fabsf(hv[t]), fabsf(hv[t + 1])), fmaxf(fabsf(lv[t]), fabsf(lv[t + 1]))));
  }
  const int k = e2m3_scale_exp(m);
  const float inv = ldexpf(1.f, -k - 6);
#pragma unroll
  for (int e = 0; e < 16; e += 8) {
    // 24 bits of 4 codes each: high parts, then low parts
    uint32_t g[4];
#pragma unroll
    for (int q = 0; q < 2; ++q) {
      const int i = e + 4 * q;
      g[q] = e2m3x4(hv[i] * inv, hv[i + 1] * inv, hv[i + 2] * inv, hv[i + 3] * inv);
      g[2 + q] = e2m3x4(lv[i] * inv, lv[i + 1] * inv, lv[i + 2] * inv, lv[i + 3] * inv);
    }
    uint32_t* const o = w + 3 * (e >> 3);
    o[0] = g[0] | (g[1] << 24);
    o[1] = (g[1] >> 8) | (g[2] << 16);
    o[2] = (g[2] >> 16) | (g[3] << 8);
  }
  w[6] = (uint32_t)(127 + k);
  w[7] = 0u;
}

}  // namespace
}  // namespace mps
