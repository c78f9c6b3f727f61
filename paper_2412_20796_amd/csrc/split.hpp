// fp32 operands as three bf16 parts for the bf16 matrix cores (see gemm.hpp).
#pragma once
#include <hip/hip_runtime.h>

namespace chg {

typedef float f32x16 __attribute__((ext_vector_type(16)));
typedef float f32x2 __attribute__((ext_vector_type(2)));
typedef __bf16 bf16x2 __attribute__((ext_vector_type(2)));
typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
// four floats of which only the first's alignment is known
struct __attribute__((packed, aligned(4))) f4u {
  float x, y, z, w;
};

struct Split8 {
  bf16x8 h, m, l;
};

// two values to bf16, and the rounded pair back as fp32
__device__ __forceinline__ unsigned bf16_pair(float a, float b, float& ra, float& rb) {
  const f32x2 v = {a, b};
  const unsigned u = __builtin_bit_cast(unsigned, __builtin_convertvector(v, bf16x2));
  ra = __uint_as_float(u << 16);
  rb = __uint_as_float(u & 0xffff0000u);
  return u;
}

// x = h + m + l: h = bf16(x), m = bf16(x - h), l = bf16(x - h - m). Exact for
// |x| from 2^-110 (below, l may be under 2^-126, which the matrix cores take
// as 0) up to the largest bf16 number, 3.39e38 (above, h is infinite and m is
// not a number).
__device__ __forceinline__ Split8 split8(const float (&x)[8]) {
  uint4 h, m, l;
  unsigned* hp = reinterpret_cast<unsigned*>(&h);
  unsigned* mp = reinterpret_cast<unsigned*>(&m);
  unsigned* lp = reinterpret_cast<unsigned*>(&l);
#pragma unroll
  for (int q = 0; q < 4; ++q) {
    float a, b;
    hp[q] = bf16_pair(x[2 * q], x[2 * q + 1], a, b);
    const float r0 = x[2 * q] - a, r1 = x[2 * q + 1] - b;
    mp[q] = bf16_pair(r0, r1, a, b);
    float c, d;
    lp[q] = bf16_pair(r0 - a, r1 - b, c, d);
  }
  return Split8{__builtin_bit_cast(bf16x8, h), __builtin_bit_cast(bf16x8, m), __builtin_bit_cast(bf16x8, l)};
}

// The same for operands laid out once (the weights), for which h is cut and not
// rounded where it would be infinite, and the other parts of an infinite value
// are 0: x = h + m + l up to the largest fp32 number, and for infinities.
__device__ __forceinline__ Split8 split8_all(const float (&x)[8]) {
  bool big = false;
#pragma unroll
  for (int q = 0; q < 8; ++q) big = big || !(fabsf(x[q]) < 3.39e38f);
  if (!big) return split8(x);
  uint4 h, m, l;
  unsigned short* hp = reinterpret_cast<unsigned short*>(&h);
  unsigned short* mp = reinterpret_cast<unsigned short*>(&m);
  unsigned short* lp = reinterpret_cast<unsigned short*>(&l);
#pragma unroll
  for (int q = 0; q < 8; ++q) {
    const float hv = __uint_as_float(__float_as_uint(x[q]) & 0xffff0000u);
    const float r = isinf(x[q]) ? 0.f : x[q] - hv;
    float mv, z0, z1;
    hp[q] = (unsigned short)(__float_as_uint(hv) >> 16);
    mp[q] = (unsigned short)bf16_pair(r, r, mv, z0);
    lp[q] = (unsigned short)bf16_pair(r - mv, r - mv, z0, z1);
  }
  return Split8{__builtin_bit_cast(bf16x8, h), __builtin_bit_cast(bf16x8, m), __builtin_bit_cast(bf16x8, l)};
}

// the values back from their parts
__device__ __forceinline__ void unsplit8(const Split8& p, float (&x)[8]) {
#pragma unroll
  for (int q = 0; q < 8; ++q) x[q] = ((float)p.h[q] + (float)p.m[q]) + (float)p.l[q];
}

// a lane's part of a packed tile: three planes of 64 16-byte pieces
__device__ __forceinline__ Split8 packed8(const uint4* p) {
  return Split8{__builtin_bit_cast(bf16x8, p[0]), __builtin_bit_cast(bf16x8, p[64]), __builtin_bit_cast(bf16x8, p[128])};
}
__device__ __forceinline__ Split8 as_split8(const uint4 (&p)[3]) {
  return Split8{__builtin_bit_cast(bf16x8, p[0]), __builtin_bit_cast(bf16x8, p[1]), __builtin_bit_cast(bf16x8, p[2])};
}

// hi + lo += x y over 16 k: the products of the leading parts, whose bits the
// sum keeps, and the others, small terms first (hi and lo may be one)
__device__ __forceinline__ void mfma_split(const Split8& x, const Split8& y, f32x16& hi, f32x16& lo) {
  lo = __builtin_amdgcn_mfma_f32_32x32x16_bf16(x.l, y.h, lo, 0, 0, 0);
  lo = __builtin_amdgcn_mfma_f32_32x32x16_bf16(x.h, y.l, lo, 0, 0, 0);
  lo = __builtin_amdgcn_mfma_f32_32x32x16_bf16(x.m, y.m, lo, 0, 0, 0);
  lo = __builtin_amdgcn_mfma_f32_32x32x16_bf16(x.m, y.h, lo, 0, 0, 0);
  lo = __builtin_amdgcn_mfma_f32_32x32x16_bf16(x.h, y.m, lo, 0, 0, 0);
  hi = __builtin_amdgcn_mfma_f32_32x32x16_bf16(x.h, y.h, hi, 0, 0, 0);
}

}  // namespace chg
