// Tiles of the float32 matrix instructions, shared by the kernels that serve any shape (general steps, products of the fit).
//
// v_mfma_f32_16x16x4_f32: lane (r = lane % 16, g = lane / 16) holds A[m = r][kk = g], B[kk = g][n = r] and the four
// results D[m = 4 g + i][n = r].
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

#include "svdc_device.h"

namespace svdc {
namespace {

__device__ __forceinline__ f32x4 mfma_f32(float a, float b, const f32x4& c) {
  return __builtin_amdgcn_mfma_f32_16x16x4f32(a, b, c, 0, 0, 0);
}

// Eight consecutive channels d .. d + 7 of a token row; channels at or beyond D read as zero (D is a multiple of 8 for
// bf16 and of 4 for float32, d of 8).
template <typename T>
struct Piece;
template <>
struct Piece<bf16_t> {
  u32x4 w;
  __device__ __forceinline__ void load(const bf16_t* row, int d, int D) {
    w = u32x4{0u, 0u, 0u, 0u};
    if (d < D) w = *reinterpret_cast<const u32x4*>(row + d);
  }
  __device__ __forceinline__ float get(int e) const { return e & 1 ? bf16_hi(w[e >> 1]) : bf16_lo(w[e >> 1]); }
  static __device__ __forceinline__ void store(bf16_t* row, int d, int D, const f32x4 (&x)[2]) {
    if (d < D)
      *reinterpret_cast<u32x4*>(row + d) = u32x4{pack_bf16(x[0][0], x[0][1]), pack_bf16(x[0][2], x[0][3]),
                                                 pack_bf16(x[1][0], x[1][1]), pack_bf16(x[1][2], x[1][3])};
  }
};
template <>
struct Piece<float> {
  f32x4 x[2];
  __device__ __forceinline__ void load(const float* row, int d, int D) {
#pragma unroll
    for (int t = 0; t < 2; ++t) {
      x[t] = f32x4{0.f, 0.f, 0.f, 0.f};
      if (d + 4 * t < D) x[t] = *reinterpret_cast<const f32x4*>(row + d + 4 * t);
    }
  }
  __device__ __forceinline__ float get(int e) const { return x[e >> 2][e & 3]; }
  static __device__ __forceinline__ void store(float* row, int d, int D, const f32x4 (&y)[2]) {
#pragma unroll
    for (int t = 0; t < 2; ++t)
      if (d + 4 * t < D) *reinterpret_cast<f32x4*>(row + d + 4 * t) = y[t];
  }
};

// A piece of V, 32 channels from chunk c x KW = 16 KT coefficients from j0, on its way to the wave that uses it: loads
// of whole row segments requested a piece ahead, then LDS, from where both phases read it in the lane layout that they
// need.  (Loaded in that layout directly, an instruction touches 16 rows: twice the time.)  The LDS area belongs to one
// wave, so no barrier is needed: the LDS executes a wave's accesses in order.  The loads are bounds-checked buffer
// loads over the chunk's rows: rows beyond D and, with an offset past the end, columns beyond k read as zero.
template <int KT>
struct VPiece {
  static constexpr int KW = 16 * KT, RPL = 64 / KW, NL = 32 / RPL, KS = KW + 4;
  static constexpr int kFloats = 32 * KS;
  float x[NL];
  __device__ __forceinline__ void load(const float* v, int D, int k, int c, int j0) {
    const int lane = threadIdx.x & 63, row = lane / KW, col = j0 + lane % KW;
    const auto rows = __builtin_amdgcn_make_buffer_rsrc(const_cast<float*>(v + (int64_t)32 * c * k), 0,
                                                        min(32, D - 32 * c) * k * 4, 0x00027000);
    const uint32_t off = col < k ? (uint32_t)(row * k + col) * 4u : 0x80000000u;
#pragma unroll
    for (int i = 0; i < NL; ++i)
      x[i] = __builtin_bit_cast(float, __builtin_amdgcn_raw_buffer_load_b32(rows, off + (uint32_t)(RPL * i * k) * 4u, 0, 0));
  }
  __device__ __forceinline__ void to_lds(float* lds) const {
    const int lane = threadIdx.x & 63, row = lane / KW, col = lane % KW;
    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
#pragma unroll
    for (int i = 0; i < NL; ++i) lds[(RPL * i + row) * KS + col] = x[i];
    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
  }
};

}  // namespace
}  // namespace svdc
