// Operands of the matrix-core products of the basis fit: pieces of feature rows, and Y in the layout of the back-projection.
#pragma once
#include "svdc_device.h"

namespace svdc {
namespace {

// Eight consecutive channels of one token as they are loaded, and as matrix-core operands.  bf16 features are the
// operand; float32 features are split into bf16 high + low parts when used (the products then take the high part
// against both parts of the other operand and the low part against its high part: about 16 significant bits).
template <typename T>
struct FPiece;
template <>
struct FPiece<bf16_t> {
  static constexpr bool kTwoParts = false;
  u32x4 w;
  __device__ __forceinline__ void load(const bf16_t* p) { w = *reinterpret_cast<const u32x4*>(p); }
  __device__ __forceinline__ void operands(u32x4* hi, u32x4* lo) const { *hi = w; *lo = w; }
  __device__ __forceinline__ float sumsq() const {
    float s = 0.f;
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      const float x0 = bf16_lo(w[i]), x1 = bf16_hi(w[i]);
      s += x0 * x0 + x1 * x1;
    }
    return s;
  }
};
template <>
struct FPiece<float> {
  static constexpr bool kTwoParts = true;
  f32x4 x[2];
  __device__ __forceinline__ void load(const float* p) {
    x[0] = *reinterpret_cast<const f32x4*>(p);
    x[1] = *reinterpret_cast<const f32x4*>(p + 4);
  }
  __device__ __forceinline__ void operands(u32x4* hi, u32x4* lo) const {
    const float c8[8] = {x[0][0], x[0][1], x[0][2], x[0][3], x[1][0], x[1][1], x[1][2], x[1][3]};
    split_operand(c8, hi, lo);
  }
  __device__ __forceinline__ float sumsq() const {
    float s = 0.f;
#pragma unroll
    for (int i = 0; i < 4; ++i) s += x[0][i] * x[0][i] + x[1][i] * x[1][i];
    return s;
  }
};

// Packed Y for the back-projection: Y rounded to bf16, already in the layout of its MFMA operand, so that the
// back-projection fetches an operand with one 16-byte load per lane instead of 8 scalar loads and 4 conversions.
// A 32-row step s and coefficient tile jt form one 1 KB word; lane (r, g), element e holds
//   Y[32 s + 16 (e / 4) + 4 g + e % 4][16 jt + r]      (0 for rows >= N),
// i.e. the lane's four accumulator rows of the step's first 16-row tile followed by those of the second.  The
// back-projection contracts over the rows of a step in this same order.  Index: ((b nsteps + s) KT + jt) 64 + lane.
// float32 features: the same words in two parts, bf16 high then low, word ((b nsteps + s) KT + jt) 2 + part.
// A projection stores them by halves: the four accumulator rows of one 16-row tile are 8 bytes.
__device__ __forceinline__ f32x4 rows_inside(const f32x4& t, int row, int N) {
  f32x4 a = t;
#pragma unroll
  for (int i = 0; i < 4; ++i)
    if (row + i >= N) a[i] = 0.f;
  return a;
}
__device__ __forceinline__ void store_y_half(FPiece<bf16_t>, u32x4* Yp, int64_t word, int half, const f32x4& t, int row, int N) {
  const f32x4 a = rows_inside(t, row, N);
  reinterpret_cast<uint2*>(Yp + word * 64 + (threadIdx.x & 63))[half] = make_uint2(pack_bf16(a[0], a[1]), pack_bf16(a[2], a[3]));
}
__device__ __forceinline__ void store_y_half(FPiece<float>, u32x4* Yp, int64_t word, int half, const f32x4& t, int row, int N) {
  const f32x4 a = rows_inside(t, row, N);
  const uint32_t h0 = pack_bf16(a[0], a[1]), h1 = pack_bf16(a[2], a[3]);
  const uint32_t l0 = pack_bf16(a[0] - bf16_lo(h0), a[1] - bf16_hi(h0)), l1 = pack_bf16(a[2] - bf16_lo(h1), a[3] - bf16_hi(h1));
  uint2* out = reinterpret_cast<uint2*>(Yp + word * 2 * 64 + (threadIdx.x & 63)) + half;
  out[0] = make_uint2(h0, h1);
  out[2 * 64] = make_uint2(l0, l1);
}

}  // namespace
}  // namespace svdc
