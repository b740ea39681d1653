// General (any shape, any k <= 1024) kernels for the full-compute step and the cached step, for either storage type.  They serve
// the shapes that the packed-basis kernels do not cover (hidden sizes that are not one of the instantiated multiples of 128, ranks
// above 128 or not a multiple of 4) and calls without a packed basis.  There are two kinds of each, between which step_tiling.h
// decides: on the float32 matrix cores (v_mfma_f32_16x16x4_f32: float32 operands as they are, float32 accumulation), and, further
// down, on the bf16 ones with float32 values in three parts, for larger calls of ranks 17 to 128.  This is about the first.
//
// The layout of the instruction is in f32_tiles.h.  The contraction index is permuted so that loads are wide: a lane loads eight
// consecutive channels 32 c + 8 g + e of its token row, and step e of eight contracts the channels {32 c + 8 g + e}.
//
// What bounds them: the matrix pipe (256 flop per clock and compute unit; busy 44 % of a unit's time in the cached step and
// 48 % in the full step below by its counter, which at rank 50, padded to 64, and with the units that wait for the last
// ones is 30 % of the rate over the whole launch) behind the
// latency of V, which has no packed form here and comes from L2 as it is.  A workgroup holds 16 token rows, so V is
// read once per 16 rows and not once per row, and the operands of the next 32 channels are requested before the current
// ones are multiplied.  Measured at 4 x 2173 x 1408 bf16, rank 50: full step 904 -> 68 us, cached step 290 -> 33 us; at
// 22848 x 2136, rank 21: 1454 -> 108 and 490 -> 67 us, against one wave per token row on the vector units, which read
// all of V for every row.  Tiles of 32 rows were no faster with these instructions (half as many waves to hide the latency).
#include <algorithm>
#include <type_traits>

#include "f32_tiles.h"
#include "step_tiling.h"
#include "svdc_device.h"
#include "svdc_internal.h"

namespace svdc {

namespace {

// Coefficients of the workgroup's 16 rows in LDS: row stride 16 ceil(k / 16) + 4 floats (rows fall into different
// banks for the 16-byte reads below), zeros beyond k.
__host__ __device__ inline int coef_stride(int k) { return (k + 15) / 16 * 16 + 4; }

// For the chunks c0, c0 + cstep, ... < nchunk of 32 channels: P = C V^T of the workgroup's 16 rows (C in LDS), handed to
// `emit(c, P)` as the lane's eight channels 32 c + 8 g .. of row r; `fetch(c)` is called before the products so that the
// caller can request what it combines P with.  Lane (r, g) takes, for the two halves t of the chunk,
// V[32 c + 8 (r / 4) + 4 t + r % 4][j0 + 16 s + 4 g + e] as the operand of step (s, e): with its rows permuted like this
// the result of half t is the lane's channels 32 c + 8 g + 4 t + i of token row r.
template <int KT, typename Fetch, typename Emit>
__device__ __forceinline__ void reconstruct(const float* v, const float* cs, float* vlds, int D, int k, int c0, int cstep,
                                            int nchunk, Fetch fetch, Emit emit) {
  const int lane = threadIdx.x & 63, r = lane & 15, g = lane >> 4, CS = coef_stride(k);
  constexpr int KS = VPiece<KT>::KS;
  if (c0 >= nchunk) return;
  VPiece<KT> vp;
  vp.load(v, D, k, c0, 0);
  for (int c = c0; c < nchunk; c += cstep) {
    fetch(c);
    f32x4 acc[2][4];      // four accumulators per result tile: short chains of additions
#pragma unroll
    for (int t = 0; t < 2; ++t)
#pragma unroll
      for (int h = 0; h < 4; ++h) acc[t][h] = f32x4{0.f, 0.f, 0.f, 0.f};
    for (int j0 = 0; j0 < k; j0 += 16 * KT) {
      vp.to_lds(vlds);
      const bool more = j0 + 16 * KT < k;
      const int cn = more ? c : c + cstep;
      if (cn < nchunk) vp.load(v, D, k, cn, more ? j0 + 16 * KT : 0);
#pragma unroll
      for (int s = 0; s < KT; ++s) {
        if (j0 + 16 * s >= k) break;
        const f32x4 b = *reinterpret_cast<const f32x4*>(cs + r * CS + j0 + 16 * s + 4 * g);
        f32x4 a[2];
#pragma unroll
        for (int t = 0; t < 2; ++t)
          a[t] = *reinterpret_cast<const f32x4*>(vlds + (8 * (r >> 2) + 4 * t + (r & 3)) * KS + 16 * s + 4 * g);
#pragma unroll
        for (int e = 0; e < 4; ++e)
#pragma unroll
          for (int t = 0; t < 2; ++t) acc[t][e] = mfma_f32(a[t][e], b[e], acc[t][e]);
      }
    }
    f32x4 p[2];
#pragma unroll
    for (int t = 0; t < 2; ++t)
#pragma unroll
      for (int i = 0; i < 4; ++i) p[t][i] = (acc[t][0][i] + acc[t][1][i]) + (acc[t][2][i] + acc[t][3][i]);
    emit(c, p);
  }
}

// Full-compute step (Eq. 8-11): C = F V, R = F - C V^T, EMA update of S.  A workgroup takes 16 token rows; its eight
// waves take every eighth chunk of 32 channels.  Phase 1 projects, 16 KT coefficients at a time, with four accumulators per
// result tile, which leaves registers for two workgroups per compute unit; the waves' partial sums meet in LDS.  The
// accumulators are added up every two chunks, so that no chain of float32 additions is longer than 16 products, and float64
// joins what is left.  Without that the chains grow with the channels: C of 2040 channels was off by 1.5e-7 of its norm,
// 1.25e-7 with one chain per lane and a tree over 64 lanes, 0.95e-7 like this.  It costs nothing to 5 %, 9 % at
// 256 rows and ranks of several passes.
// Phase 2 forms the residual chunk by chunk.  F and R may alias, R and Rp too: phase 1 has read all of the workgroup's
// rows before the barrier, and phase 2 reads every element in the lane that overwrites it.
constexpr int kStepWaves = 8;
template <typename T, int KT>
__global__ __launch_bounds__(64 * kStepWaves, 4) void full_step_general_kernel(const T* F, const float* __restrict__ V, T* R,
                                                                            const T* Rp, float alpha_r, float* S,
                                                                            float* C, int N, int D, int k,
                                                                            int64_t ldf, int64_t bstride,
                                                                            float alpha, int init) {
  // per wave: its piece of V; between the phases its partial sums
  __shared__ __align__(16) float vstage[kStepWaves][VPiece<KT>::kFloats];
  static_assert(VPiece<KT>::kFloats >= KT * 256, "partial sums fit");
  extern __shared__ __align__(16) float cs[];        // [16][coef_stride(k)]
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), lane = threadIdx.x & 63, r = lane & 15, g = lane >> 4;
  const int b = blockIdx.y, row0 = blockIdx.x * 16, CS = coef_stride(k);
  const int nchunk = (D + 31) / 32;
  const float* v = V + (int64_t)b * D * k;
  float* vlds = vstage[wave];
  struct alignas(4 * KT) RowVec { float v[KT]; };
  const int64_t roff = (int64_t)b * bstride + (int64_t)min(row0 + r, N - 1) * ldf;

  for (int j0 = 0; j0 < k; j0 += 16 * KT) {
    f32x4 acc[KT][4], tot[KT];
#pragma unroll
    for (int jt = 0; jt < KT; ++jt) {
      tot[jt] = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
      for (int h = 0; h < 4; ++h) acc[jt][h] = f32x4{0.f, 0.f, 0.f, 0.f};
    }
    Piece<T> fn;
    VPiece<KT> vp;
    if (wave < nchunk) {
      fn.load(F + roff, 32 * wave + 8 * g, D);
      vp.load(v, D, k, wave, j0);
    }
    for (int c = wave; c < nchunk; c += kStepWaves) {
      const Piece<T> f = fn;
      vp.to_lds(vlds);
      if (c + kStepWaves < nchunk) {
        fn.load(F + roff, 32 * (c + kStepWaves) + 8 * g, D);
        vp.load(v, D, k, c + kStepWaves, j0);
      }
      if (c >= 2 * kStepWaves && (c / kStepWaves) % 2 == 0) {
#pragma unroll
        for (int jt = 0; jt < KT; ++jt) {
          tot[jt] += (acc[jt][0] + acc[jt][1]) + (acc[jt][2] + acc[jt][3]);
#pragma unroll
          for (int h = 0; h < 4; ++h) acc[jt][h] = f32x4{0.f, 0.f, 0.f, 0.f};
        }
      }
#pragma unroll
      for (int e = 0; e < 8; ++e) {
        // columns of the result tile jt: j0 + KT r + jt, so that one wide LDS read brings the operands of all tiles
        const float x = f.get(e);
        const RowVec vv = *reinterpret_cast<const RowVec*>(vlds + (8 * g + e) * VPiece<KT>::KS + KT * r);
#pragma unroll
        for (int jt = 0; jt < KT; ++jt) acc[jt][e & 3] = mfma_f32(x, vv.v[jt], acc[jt][e & 3]);
      }
    }
    f32x4* part = reinterpret_cast<f32x4*>(vlds);
    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
#pragma unroll
    for (int jt = 0; jt < KT; ++jt) {
      f32x4 s;
#pragma unroll
      for (int i = 0; i < 4; ++i)
        s[i] = (float)((((double)acc[jt][0][i] + acc[jt][1][i]) + ((double)acc[jt][2][i] + acc[jt][3][i])) + tot[jt][i]);
      part[jt * 64 + lane] = s;
    }
    __syncthreads();
    // D[m = 4 g + i][n = r]: row 4 g + i, coefficient j0 + KT r + jt
    if (wave < KT) {
      const int j = j0 + KT * r + wave;
      double c[4] = {0.0, 0.0, 0.0, 0.0};
#pragma unroll
      for (int w = 0; w < kStepWaves; ++w) {
        const f32x4 p = reinterpret_cast<const f32x4*>(vstage[w])[wave * 64 + lane];
#pragma unroll
        for (int i = 0; i < 4; ++i) c[i] += (double)p[i];
      }
      if (j < CS - 4) {
#pragma unroll
        for (int i = 0; i < 4; ++i) cs[(4 * g + i) * CS + j] = j < k ? (float)c[i] : 0.f;
      }
    }
    __syncthreads();
  }

  // EMA update of the coefficient state (Eq. 11 with alpha = 1 - beta); the rows of a tile are contiguous in S and C
  const int nrow = min(16, N - row0);
  const int64_t soff = ((int64_t)b * N + row0) * k;
  for (int e = threadIdx.x; e < nrow * k; e += 64 * kStepWaves) {
    const int row = e / k, j = e - row * k;
    const float c = cs[row * CS + j];
    const float s = init ? c : (1.f - alpha) * S[soff + e] + alpha * c;
    S[soff + e] = s;
    if (C) C[soff + e] = c;
  }

  // residual R = F - C V^T (Eq. 10)
  Piece<T> f, rp;
  auto fetch = [&](int c) {
    f.load(F + roff, 32 * c + 8 * g, D);
    if (Rp) rp.load(Rp + roff, 32 * c + 8 * g, D);
  };
  reconstruct<KT>(v, cs, vlds, D, k, wave, kStepWaves, nchunk, fetch, [&](int c, const f32x4 (&p)[2]) {
    f32x4 x[2];
#pragma unroll
    for (int t = 0; t < 2; ++t)
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        x[t][i] = f.get(4 * t + i) - p[t][i];
        // optional smoothing of the residual state (Rp: previous residual, may be the buffer R itself)
        if (Rp) x[t][i] = (1.f - alpha_r) * rp.get(4 * t + i) + alpha_r * x[t][i];
      }
    if (row0 + r < N) Piece<T>::store(R + roff, 32 * c + 8 * g, D, x);
  });
}

// Cached step (Sec. 3.5): Fhat = C_hat V^T + R [+ X] with the coefficient forecast C_hat = sum_m w_m S_m
// (one state with weight one is the paper's EMA forecast).  X is nullable; Fhat may alias R or X.  A workgroup of four
// waves takes 16 rows and, of the chunks of 32 channels, the blockIdx.z-th of gridDim.z shares (small problems would
// leave compute units idle otherwise).
constexpr int kCachedWaves = 4;
template <typename T, int KT>
__global__ __launch_bounds__(64 * kCachedWaves, 4) void forecast_general_kernel(const CoefStates st,
                                                                             const float* __restrict__ V, const T* R,
                                                                             const T* X, T* Fh, int N, int D, int k,
                                                                             int64_t ldf, int64_t bstride) {
  __shared__ __align__(16) float vstage[kCachedWaves][VPiece<KT>::kFloats];
  extern __shared__ __align__(16) float cs[];        // [16][coef_stride(k)]
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), lane = threadIdx.x & 63, r = lane & 15, g = lane >> 4;
  const int b = blockIdx.y, row0 = blockIdx.x * 16, CS = coef_stride(k), kpad = CS - 4;
  const int nchunk = (D + 31) / 32;
  // the coefficients of the tile, zeros beyond N and k; 16 threads per row
  const int64_t soff = ((int64_t)b * N + row0) * k;
  {
    const int row = threadIdx.x >> 4;
    for (int j = threadIdx.x & 15; j < kpad; j += 16) {
      float c = 0.f;
      if (row0 + row < N && j < k) {
        const int64_t at = soff + (int64_t)row * k + j;
        c = st.w[0] * st.s[0][at];
        for (int m = 1; m < st.m; ++m) c = __builtin_fmaf(st.w[m], st.s[m][at], c);
      }
      cs[row * CS + j] = c;
    }
  }
  __syncthreads();
  const int64_t roff = (int64_t)b * bstride + (int64_t)min(row0 + r, N - 1) * ldf;
  Piece<T> f, xp;
  auto fetch = [&](int c) {
    f.load(R + roff, 32 * c + 8 * g, D);
    if (X) xp.load(X + roff, 32 * c + 8 * g, D);
  };
  reconstruct<KT>(V + (int64_t)b * D * k, cs, vstage[wave], D, k, blockIdx.z * kCachedWaves + wave,
                  kCachedWaves * gridDim.z, nchunk, fetch, [&](int c, const f32x4 (&p)[2]) {
    f32x4 x[2];
#pragma unroll
    for (int t = 0; t < 2; ++t)
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        x[t][i] = f.get(4 * t + i);
        if (X) x[t][i] += xp.get(4 * t + i);
        x[t][i] += p[t][i];
      }
    if (row0 + r < N) Piece<T>::store(Fh + roff, 32 * c + 8 * g, D, x);
  });
}

// ---------------------------------------------------------------------------
// The same two steps with the products on the bf16 matrix cores, for ranks of 17 to 128 where step_tiling.h says so: a float32
// is the exact sum of three bf16 parts (8 significant bits each), a product of two keeps six of the nine products of parts,
// and a bf16 feature is one part already, whose products with V are whole.  The three that are dropped are at most 2^-24 of the
// product, half a unit of a float32 in the last place (parts are up to 2^-8 and 2^-17 of what is split), and 2^-27.5 in the mean.
// An instruction contracts 32 channels or coefficients at 16 times the rate of the float32 one, so six cost less than half of it;
// what bounds the kernels instead are the vector instructions (13 for every pair of elements of V that is split, 74 for every row
// tile and chunk that is put together), which is why 32 or 48 rows share a piece of V.  The leading products of every chunk are
// added up in float64: C is within 2.8e-8 of its norm of the float64 product at 1408 and 2.8e-8 at 3304 channels, 3.4e-8 with
// float32 instructions.
// Measured at 4 x 2173 x 1408 bf16, rank 50: full step 68 -> 46 us, cached step 31 -> 23 us (44 and 22.5 with parts that do not
// reach the whole range); 22848 x 2136 at rank 21: 110 -> 73 and 67 -> 47 us.
// ---------------------------------------------------------------------------
// What is split is multiplied by 2^24 first, so that the third part of the smallest normal float32 is a normal bf16 too: the sum
// of the parts is exact for everything below 2^104 in magnitude.  Beyond that, at an infinity or a NaN the parts hold an infinity
// or a NaN and so does every result that they are part of; those results are formed once more on the float32 matrix cores
// (the second pass of the full step, reconstruct_parts), as the kernels above do.
constexpr float kPartScale = 0x1p24f;
constexpr float kPartProduct = 0x1p-48f;      // of a product whose factors were both split
constexpr float kMaxFinite = 3.402823466e38f;
struct Parts { u32x4 p[3]; };
__device__ __forceinline__ Parts split_parts(const float (&x)[8]) {
  Parts out;
  float rem[8];
#pragma unroll
  for (int e = 0; e < 8; ++e) rem[e] = x[e] * kPartScale;
#pragma unroll
  for (int n = 0; n < 3; ++n)
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      const uint32_t w = pack_bf16(rem[2 * i], rem[2 * i + 1]);
      out.p[n][i] = w;
      if (n < 2) {
        rem[2 * i] -= bf16_lo(w);
        rem[2 * i + 1] -= bf16_hi(w);
      }
    }
  return out;
}
__device__ __forceinline__ f32x4 mfma_parts(const u32x4& a, const u32x4& b, const f32x4& c) {
  return __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8, a), __builtin_bit_cast(bf16x8, b), c, 0, 0, 0);
}
// The products of a feature's parts with those of V: the leading one into `lead`, the others, 2^-8 of it and less, into `rest`.
__device__ __forceinline__ void feature_product(const Piece<bf16_t>& f, const Parts& v, f32x4& lead, f32x4& rest) {
  lead = mfma_parts(f.w, v.p[0], lead);
  rest = mfma_parts(f.w, v.p[2], rest);
  rest = mfma_parts(f.w, v.p[1], rest);
}
__device__ __forceinline__ void feature_product(const Parts& f, const Parts& v, f32x4& lead, f32x4& rest) {
  lead = mfma_parts(f.p[0], v.p[0], lead);
  rest = mfma_parts(f.p[0], v.p[2], rest);
  rest = mfma_parts(f.p[2], v.p[0], rest);
  rest = mfma_parts(f.p[1], v.p[1], rest);
  rest = mfma_parts(f.p[0], v.p[1], rest);
  rest = mfma_parts(f.p[1], v.p[0], rest);
}
__device__ __forceinline__ const Piece<bf16_t>& feature_parts(const Piece<bf16_t>& f) { return f; }
__device__ __forceinline__ Parts feature_parts(const Piece<float>& f) {
  const float x[8] = {f.x[0][0], f.x[0][1], f.x[0][2], f.x[0][3], f.x[1][0], f.x[1][1], f.x[1][2], f.x[1][3]};
  return split_parts(x);
}

// i-th chunk of 32 channels of a wave among `waves`: pairs of neighbours, whose rows share lines of 128 bytes
__device__ __forceinline__ int pair_chunk(int i, int wave, int waves) { return 2 * (wave + (i >> 1) * waves) + (i & 1); }
__device__ __forceinline__ int pair_chunks(int nchunk, int wave, int waves) {
  const int pairs = (nchunk + 1) / 2, mine = wave < pairs ? (pairs - wave + waves - 1) / waves : 0;
  // the last pair of all may be a single chunk
  return 2 * mine - (mine > 0 && (nchunk & 1) && (pairs - 1) % waves == wave ? 1 : 0);
}

// A piece of V in LDS times 32 coefficients of 16 RT rows, as operand words `cw` of the piece's first row tile, `tiles` row tiles apart.
template <int RT>
__device__ __forceinline__ void piece_products(const float* vlds, const u32x4* cw, int tiles, f32x4 (&lead)[RT][2], f32x4 (&rest)[RT][2]) {
  const int lane = threadIdx.x & 63, r = lane & 15, g = lane >> 4;
  Parts a[2];
#pragma unroll
  for (int t = 0; t < 2; ++t) {
    const float* row = vlds + (8 * (r >> 2) + 4 * t + (r & 3)) * VPiece<2>::KS + 8 * g;
    const f32x4 x0 = *reinterpret_cast<const f32x4*>(row), x1 = *reinterpret_cast<const f32x4*>(row + 4);
    const float x[8] = {x0[0], x0[1], x0[2], x0[3], x1[0], x1[1], x1[2], x1[3]};
    a[t] = split_parts(x);
  }
#pragma unroll
  for (int rt = 0; rt < RT; ++rt) {
    Parts b;
#pragma unroll
    for (int n = 0; n < 3; ++n) b.p[n] = cw[(rt * tiles * 3 + n) * 64 + lane];
#pragma unroll
    for (int t = 0; t < 2; ++t) feature_product(a[t], b, lead[rt][t], rest[rt][t]);
  }
}
template <int RT>
__device__ __forceinline__ void clear_products(f32x4 (&lead)[RT][2], f32x4 (&rest)[RT][2]) {
#pragma unroll
  for (int rt = 0; rt < RT; ++rt)
#pragma unroll
    for (int t = 0; t < 2; ++t) lead[rt][t] = rest[rt][t] = f32x4{0.f, 0.f, 0.f, 0.f};
}
// lead += rest; whether all of the wave's results are finite
template <int RT>
__device__ __forceinline__ bool finish_products(f32x4 (&lead)[RT][2], const f32x4 (&rest)[RT][2]) {
  float top = 0.f;
#pragma unroll
  for (int rt = 0; rt < RT; ++rt)
#pragma unroll
    for (int t = 0; t < 2; ++t) {
      lead[rt][t] += rest[rt][t];
#pragma unroll
      for (int q = 0; q < 4; ++q) top = __builtin_elementwise_maximum(top, __builtin_fabsf(lead[rt][t][q]));   // a NaN stays
    }
  return __builtin_amdgcn_ballot_w64(!(top <= kMaxFinite)) == 0;
}

// P = C V^T of 16 RT rows for the wave's chunks, C as operand words in LDS: cw[(rt kt2 + kt) 3 + part][lane], lane (r, g), e ->
// C[row r][32 kt + 8 g + e].  Like `reconstruct` above, a pair of chunks at a time: `fetch(c, rows)` requests what P is combined
// with, a pair ahead; `emit(c, rt, piece of rows, P, scale)` gets the results, P times a scale.  Stops before the first chunk whose
// results are not all finite and returns its index, the number of chunks if there is none: what a result is combined with may be
// overwritten by it, so that nothing can be formed again afterwards, and to do it in this loop costs registers (40 spilled).
template <int RT, typename Rows, typename Fetch, typename Emit>
__device__ __forceinline__ int reconstruct_parts(const float* v, const u32x4* cw, float* vlds, int D, int k, int kt2, int wave,
                                                 int waves, int nchunk, Fetch fetch, Emit emit) {
  const int mine = pair_chunks(nchunk, wave, waves);
  if (mine <= 0) return mine;
  VPiece<2> vp;
  vp.load(v, D, k, pair_chunk(0, wave, waves), 0);
  Rows next[2];
#pragma unroll
  for (int h = 0; h < 2; ++h) fetch(pair_chunk(h, wave, waves), next[h]);
  for (int i0 = 0; i0 < mine; i0 += 2) {
    Rows rows[2];
#pragma unroll
    for (int h = 0; h < 2; ++h) {
      rows[h] = next[h];
      if (i0 + 2 < mine) fetch(pair_chunk(i0 + 2 + h, wave, waves), next[h]);
    }
#pragma unroll
    for (int h = 0; h < 2; ++h) {
      const int i = i0 + h;
      if (i >= mine) break;
      const int c = pair_chunk(i, wave, waves);
      f32x4 lead[RT][2], rest[RT][2];
      clear_products<RT>(lead, rest);
      for (int kt = 0; kt < kt2; ++kt) {
        vp.to_lds(vlds);
        const bool more = kt + 1 < kt2;
        if (more || i + 1 < mine) vp.load(v, D, k, more ? c : pair_chunk(i + 1, wave, waves), more ? 32 * (kt + 1) : 0);
        piece_products<RT>(vlds, cw + kt * 3 * 64, kt2, lead, rest);
      }
      if (!finish_products<RT>(lead, rest)) return i;
#pragma unroll
      for (int rt = 0; rt < RT; ++rt) emit(c, rt, rows[h], lead[rt], kPartProduct);
    }
  }
  return mine;
}

// The same from the wave's chunk i on, with results that are not finite replaced by those of the float32 instructions, formed as in
// `reconstruct`; `coef(rt, j)` gives C[row 16 rt + r][j .. j + 3].
template <int RT, typename Rows, typename Fetch, typename Coef, typename Emit>
__device__ __forceinline__ void reconstruct_rest(int i, const float* v, const u32x4* cw, float* vlds, int D, int k, int kt2, int wave,
                                                 int waves, int nchunk, Fetch fetch, Coef coef, Emit emit) {
  const int lane = threadIdx.x & 63, r = lane & 15, g = lane >> 4, mine = pair_chunks(nchunk, wave, waves);
#pragma nounroll
  for (; i < mine; ++i) {
    const int c = pair_chunk(i, wave, waves);
    f32x4 lead[RT][2], rest[RT][2];
    clear_products<RT>(lead, rest);
#pragma nounroll
    for (int kt = 0; kt < kt2; ++kt) {
      VPiece<2> vp;
      vp.load(v, D, k, c, 32 * kt);
      vp.to_lds(vlds);
      piece_products<RT>(vlds, cw + kt * 3 * 64, kt2, lead, rest);
    }
    finish_products<RT>(lead, rest);
#pragma unroll
    for (int rt = 0; rt < RT; ++rt) {
      f32x4 acc[2][4];
#pragma unroll
      for (int t = 0; t < 2; ++t)
#pragma unroll
        for (int e = 0; e < 4; ++e) acc[t][e] = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma nounroll
      for (int j0 = 0; j0 < k; j0 += 16) {
        VPiece<1> vp;
        vp.load(v, D, k, c, j0);
        vp.to_lds(vlds);
        const f32x4 b = coef(rt, j0 + 4 * g);
#pragma unroll
        for (int t = 0; t < 2; ++t) {
          const f32x4 a = *reinterpret_cast<const f32x4*>(vlds + (8 * (r >> 2) + 4 * t + (r & 3)) * VPiece<1>::KS + 4 * g);
#pragma unroll
          for (int e = 0; e < 4; ++e) acc[t][e] = mfma_f32(a[e], b[e], acc[t][e]);
        }
      }
#pragma unroll
      for (int t = 0; t < 2; ++t)
#pragma unroll
        for (int q = 0; q < 4; ++q) {
          const float x = lead[rt][t][q], plain = (acc[t][0][q] + acc[t][1][q]) + (acc[t][2][q] + acc[t][3][q]);
          lead[rt][t][q] = __builtin_fabsf(x) <= kMaxFinite ? x * kPartProduct : plain;
        }
    }
    Rows rows;
    fetch(c, rows);
#pragma unroll
    for (int rt = 0; rt < RT; ++rt) emit(c, rt, rows, lead[rt], 1.f);
  }
}

// What full_step_general_kernel leaves in its stage for a wave's chunks and 16 KT coefficients of the lane's row: the same sums in the
// same order.
template <typename T, int KT>
__device__ __forceinline__ void project_plain(const T* frow, const float* v, float* vlds, int D, int k, int j0, int wave, int nchunk) {
  const int lane = threadIdx.x & 63, r = lane & 15, g = lane >> 4;
  f32x4 acc[KT][4], tot[KT];
#pragma unroll
  for (int jt = 0; jt < KT; ++jt) {
    tot[jt] = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int h = 0; h < 4; ++h) acc[jt][h] = f32x4{0.f, 0.f, 0.f, 0.f};
  }
#pragma nounroll
  for (int c = wave; c < nchunk; c += kStepWaves) {
    Piece<T> f;
    f.load(frow, 32 * c + 8 * g, D);
    VPiece<KT> vp;
    vp.load(v, D, k, c, j0);
    vp.to_lds(vlds);
    if (c >= 2 * kStepWaves && (c / kStepWaves) % 2 == 0) {
#pragma unroll
      for (int jt = 0; jt < KT; ++jt) {
        tot[jt] += (acc[jt][0] + acc[jt][1]) + (acc[jt][2] + acc[jt][3]);
#pragma unroll
        for (int h = 0; h < 4; ++h) acc[jt][h] = f32x4{0.f, 0.f, 0.f, 0.f};
      }
    }
#pragma unroll
    for (int e = 0; e < 8; ++e) {
      const float x = f.get(e);
#pragma unroll
      for (int jt = 0; jt < KT; ++jt)
        acc[jt][e & 3] = mfma_f32(x, vlds[(8 * g + e) * VPiece<KT>::KS + KT * r + jt], acc[jt][e & 3]);
    }
  }
  __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
#pragma unroll
  for (int jt = 0; jt < KT; ++jt)
#pragma unroll
    for (int i = 0; i < 4; ++i)
      reinterpret_cast<f32x4*>(vlds)[jt * 64 + lane][i] =
          (float)((((double)acc[jt][0][i] + acc[jt][1][i]) + ((double)acc[jt][2][i] + acc[jt][3][i])) + tot[jt][i]);
}
// The sum of the waves' results of a tile, `stage` floats apart.
__device__ __forceinline__ f32x4 sum_waves(const float* part, int stage, int tile) {
  double c[4] = {0.0, 0.0, 0.0, 0.0};
#pragma unroll
  for (int w = 0; w < kStepWaves; ++w) {
    const f32x4 p = reinterpret_cast<const f32x4*>(part + w * stage)[tile * 64 + (threadIdx.x & 63)];
#pragma unroll
    for (int i = 0; i < 4; ++i) c[i] += (double)p[i];
  }
  return f32x4{(float)c[0], (float)c[1], (float)c[2], (float)c[3]};
}

// Full step on 16 RT rows: the structure of full_step_general_kernel, 32 coefficients of phase 1 at a time.  Two registers spill for
// three tiles of float32 rows.
template <typename T, int RT, bool REMA>
__global__ __launch_bounds__(64 * kStepWaves, 2) void full_step_parts_kernel(const T* F, const float* __restrict__ V, T* R,
                                                                          const T* Rp, float alpha_r, float* S, float* C,
                                                                          int N, int D, int k, int64_t ldf, int64_t bstride,
                                                                          float alpha, int init) {
  constexpr int KT = 2, ROWS = 16 * RT;
  using Stage = VPiece<KT>;
  // per wave: its piece of V; between the phases its partial sums
  constexpr int kStage = Stage::kFloats > KT * RT * 256 ? Stage::kFloats : KT * RT * 256;
  __shared__ __align__(16) float vstage[kStepWaves][kStage];
  __shared__ int s_redo;                 // 1 + the first coefficient of the pass that left sums that are not finite
  extern __shared__ __align__(16) char dyn[];
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), lane = threadIdx.x & 63, r = lane & 15, g = lane >> 4;
  const int b = blockIdx.y, row0 = blockIdx.x * ROWS, kt2 = (k + 31) / 32, CS = 32 * kt2 + 4;
  u32x4* cw = reinterpret_cast<u32x4*>(dyn);                                        // [RT][kt2][3][64]
  float* cs = reinterpret_cast<float*>(dyn + (size_t)RT * kt2 * 3 * 1024);          // [ROWS][CS]
  const int nchunk = (D + 31) / 32, mine = pair_chunks(nchunk, wave, kStepWaves);
  const float* v = V + (int64_t)b * D * k;
  float* vlds = vstage[wave];
  int64_t roff[RT];
#pragma unroll
  for (int rt = 0; rt < RT; ++rt) roff[rt] = (int64_t)b * bstride + (int64_t)min(row0 + 16 * rt + r, N - 1) * ldf;

  if (threadIdx.x == 0) s_redo = 0;      // ahead of the barriers of the first pass
  constexpr double kProduct = sizeof(T) == 2 ? 1.0 / kPartScale : (double)kPartProduct;
  for (int j0 = 0; j0 < k; j0 += 16 * KT) {
    f32x4 rest[RT][KT];
    f64x4 tot[RT][KT];
#pragma unroll
    for (int rt = 0; rt < RT; ++rt)
#pragma unroll
      for (int jt = 0; jt < KT; ++jt) {
        rest[rt][jt] = f32x4{0.f, 0.f, 0.f, 0.f};
        tot[rt][jt] = f64x4{0.0, 0.0, 0.0, 0.0};
      }
    Piece<T> fn[2][RT];
    Stage vp;
    auto load_rows = [&](int i, Piece<T> (&to)[RT]) {
      const int c = pair_chunk(i, wave, kStepWaves);
#pragma unroll
      for (int rt = 0; rt < RT; ++rt) to[rt].load(F + roff[rt], 32 * c + 8 * g, D);
    };
    if (mine > 0) {
      load_rows(0, fn[0]);
      vp.load(v, D, k, pair_chunk(0, wave, kStepWaves), j0);
      if (mine > 1) load_rows(1, fn[1]);
    }
    for (int i = 0; i < mine; ++i) {
      Piece<T> f[RT];
#pragma unroll
      for (int rt = 0; rt < RT; ++rt) {
        f[rt] = fn[0][rt];
        fn[0][rt] = fn[1][rt];
      }
      vp.to_lds(vlds);
      if (i + 1 < mine) vp.load(v, D, k, pair_chunk(i + 1, wave, kStepWaves), j0);
      if (i + 2 < mine) load_rows(i + 2, fn[1]);
      // columns of the result tile jt: j0 + 2 r + jt
      float x[KT][8];
#pragma unroll
      for (int e = 0; e < 8; ++e) {
        const float2 w = *reinterpret_cast<const float2*>(vlds + (8 * g + e) * Stage::KS + KT * r);
        x[0][e] = w.x;
        x[1][e] = w.y;
      }
      Parts vv[KT];
#pragma unroll
      for (int jt = 0; jt < KT; ++jt) vv[jt] = split_parts(x[jt]);
#pragma unroll
      for (int rt = 0; rt < RT; ++rt) {
        const auto fp = feature_parts(f[rt]);
#pragma unroll
        for (int jt = 0; jt < KT; ++jt) {
          f32x4 lead = f32x4{0.f, 0.f, 0.f, 0.f};
          feature_product(fp, vv[jt], lead, rest[rt][jt]);
#pragma unroll
          for (int q = 0; q < 4; ++q) tot[rt][jt][q] += (double)lead[q];
        }
      }
    }
    f32x4* part = reinterpret_cast<f32x4*>(vlds);
    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
#pragma unroll
    for (int rt = 0; rt < RT; ++rt)
#pragma unroll
      for (int jt = 0; jt < KT; ++jt) {
#pragma unroll
        for (int q = 0; q < 4; ++q) part[(rt * KT + jt) * 64 + lane][q] = (float)((tot[rt][jt][q] + (double)rest[rt][jt][q]) * kProduct);
      }
    __syncthreads();
    // D[m = 4 g + i][n = r]: row 4 g + i, coefficient j0 + 2 r + jt
    if (wave < RT * KT) {
      static_assert(RT * KT <= kStepWaves, "one sum per wave");
      const int rt = wave / KT, j = j0 + KT * r + wave % KT;
      const f32x4 c = sum_waves(vstage[0], kStage, wave);
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        const float x = j < k ? c[i] : 0.f;
        cs[(16 * rt + 4 * g + i) * CS + j] = x;
        if (!(__builtin_fabsf(x) <= kMaxFinite)) s_redo = j0 + 1;
      }
    }
    __syncthreads();
    if (__builtin_amdgcn_readfirstlane(s_redo) == j0 + 1) {
#pragma nounroll
      for (int rt = 0; rt < RT; ++rt) {
        project_plain<T, KT>(F + (int64_t)b * bstride + (int64_t)min(row0 + 16 * rt + r, N - 1) * ldf, v, vlds, D, k, j0, wave, nchunk);
        __syncthreads();
        const int j = j0 + KT * r + wave;
        if (wave < KT && j < k) {
          const f32x4 c = sum_waves(vstage[0], kStage, wave);
#pragma unroll
          for (int i = 0; i < 4; ++i) {
            float& x = cs[(16 * rt + 4 * g + i) * CS + j];
            if (!(__builtin_fabsf(x) <= kMaxFinite)) x = c[i];
          }
        }
        __syncthreads();
      }
    }
  }

  // operand words of the coefficients; the EMA update of the state (Eq. 11 with alpha = 1 - beta)
  for (int n = wave; n < RT * kt2; n += kStepWaves) {
    const float* c = cs + (16 * (n / kt2) + r) * CS + 32 * (n % kt2) + 8 * g;
    const float x[8] = {c[0], c[1], c[2], c[3], c[4], c[5], c[6], c[7]};
    const Parts p = split_parts(x);
#pragma unroll
    for (int m = 0; m < 3; ++m) cw[(n * 3 + m) * 64 + lane] = p.p[m];
  }
  const int nrow = min(ROWS, N - row0);
  const int64_t soff = ((int64_t)b * N + row0) * k;
  for (int e = threadIdx.x; e < nrow * k; e += 64 * kStepWaves) {
    const int row = e / k, j = e - row * k;
    const float c = cs[row * CS + j];
    const float s = init ? c : (1.f - alpha) * S[soff + e] + alpha * c;
    S[soff + e] = s;
    if (C) C[soff + e] = c;
  }
  __syncthreads();

  // residual R = F - C V^T (Eq. 10)
  struct Rows { Piece<T> f[RT], rp[REMA ? RT : 1]; };
  auto fetch = [&](int c, Rows& to) {
#pragma unroll
    for (int rt = 0; rt < RT; ++rt) {
      to.f[rt].load(F + roff[rt], 32 * c + 8 * g, D);
      if constexpr (REMA) to.rp[rt].load(Rp + roff[rt], 32 * c + 8 * g, D);
    }
  };
  auto emit = [&](int c, int rt, const Rows& rows, const f32x4 (&p)[2], float scale) {
    f32x4 x[2];
#pragma unroll
    for (int t = 0; t < 2; ++t)
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        x[t][i] = __builtin_fmaf(-p[t][i], scale, rows.f[rt].get(4 * t + i));
        if constexpr (REMA) x[t][i] = (1.f - alpha_r) * rows.rp[rt].get(4 * t + i) + alpha_r * x[t][i];
      }
    if (row0 + 16 * rt + r < N) Piece<T>::store(R + roff[rt], 32 * c + 8 * g, D, x);
  };
  const int done = reconstruct_parts<RT, Rows>(v, cw, vlds, D, k, kt2, wave, kStepWaves, nchunk, fetch, emit);
  if (done < mine)
    reconstruct_rest<RT, Rows>(done, v, cw, vlds, D, k, kt2, wave, kStepWaves, nchunk, fetch,
                               [&](int rt, int j) { return *reinterpret_cast<const f32x4*>(cs + (16 * rt + r) * CS + j); }, emit);
}

// Cached step on 16 RT rows; the blockIdx.z-th of gridDim.z shares of the channels.  Bounded to the registers of three workgroups
// per compute unit, of which float32 rows spill 14 and bf16 rows none.
template <typename T, int RT>
__global__ __launch_bounds__(64 * kCachedWaves, 3) void forecast_parts_kernel(const CoefStates st, const float* __restrict__ V,
                                                                           const T* R, T* Fh, int N, int D, int k,
                                                                           int64_t ldf, int64_t bstride) {
  __shared__ __align__(16) float vstage[kCachedWaves][VPiece<2>::kFloats];
  extern __shared__ __align__(16) char dyn[];
  u32x4* cw = reinterpret_cast<u32x4*>(dyn);                                        // [RT][kt2][3][64]
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), lane = threadIdx.x & 63, r = lane & 15, g = lane >> 4;
  const int b = blockIdx.y, row0 = blockIdx.x * 16 * RT, kt2 = (k + 31) / 32;
  const int nchunk = (D + 31) / 32;
  auto coefficient = [&](int rt, int j) {              // of row 16 rt + r, zero beyond k
    const int64_t a = ((int64_t)b * N + min(row0 + 16 * rt + r, N - 1)) * k + min(j, k - 1);
    float c = st.w[0] * st.s[0][a];
    for (int m = 1; m < st.m; ++m) c = __builtin_fmaf(st.w[m], st.s[m][a], c);
    return j < k ? c : 0.f;
  };
  for (int n = wave; n < RT * kt2; n += kCachedWaves) {
    float x[8];
#pragma unroll
    for (int e = 0; e < 8; ++e) x[e] = coefficient(n / kt2, 32 * (n % kt2) + 8 * g + e);
    const Parts p = split_parts(x);
#pragma unroll
    for (int m = 0; m < 3; ++m) cw[(n * 3 + m) * 64 + lane] = p.p[m];
  }
  __syncthreads();
  int64_t roff[RT];
#pragma unroll
  for (int rt = 0; rt < RT; ++rt) roff[rt] = (int64_t)b * bstride + (int64_t)min(row0 + 16 * rt + r, N - 1) * ldf;
  struct Rows { Piece<T> f[RT]; };
  auto fetch = [&](int c, Rows& to) {
#pragma unroll
    for (int rt = 0; rt < RT; ++rt) to.f[rt].load(R + roff[rt], 32 * c + 8 * g, D);
  };
  auto emit = [&](int c, int rt, const Rows& rows, const f32x4 (&p)[2], float scale) {
    f32x4 x[2];
#pragma unroll
    for (int t = 0; t < 2; ++t)
#pragma unroll
      for (int i = 0; i < 4; ++i) x[t][i] = __builtin_fmaf(p[t][i], scale, rows.f[rt].get(4 * t + i));
    if (row0 + 16 * rt + r < N) Piece<T>::store(Fh + roff[rt], 32 * c + 8 * g, D, x);
  };
  const float* v = V + (int64_t)b * D * k;
  const int share = blockIdx.z * kCachedWaves + wave, shares = kCachedWaves * gridDim.z;
  const int done = reconstruct_parts<RT, Rows>(v, cw, vstage[wave], D, k, kt2, share, shares, nchunk, fetch, emit);
  if (done < pair_chunks(nchunk, share, shares))
    reconstruct_rest<RT, Rows>(done, v, cw, vstage[wave], D, k, kt2, share, shares, nchunk, fetch,
                               [&](int rt, int j) {
                                 return f32x4{coefficient(rt, j), coefficient(rt, j + 1), coefficient(rt, j + 2), coefficient(rt, j + 3)};
                               }, emit);
}

constexpr int kCachedPartsRows = 2;   // row tiles of the cached step above
// calls fn(KT) with the coefficient tiles that a piece of V holds, as a compile-time constant.  The full step stops at
// two (32 coefficients at a time, ranks above 32 in several passes over the rows): with four its accumulators leave one
// or, spilled, two workgroups per compute unit (93 against 67 us at rank 50).
template <int kMaxTiles, typename Fn>
int32_t general_dispatch(const svdc_shape& s, Fn fn) {
  if (s.k <= 16) return fn(std::integral_constant<int, 1>{});
  if constexpr (kMaxTiles > 2) {
    if (s.k > 32) return fn(std::integral_constant<int, 4>{});
  }
  return fn(std::integral_constant<int, 2>{});
}

// the coefficients take up to 66 KB of LDS (rank 1024) beside the pieces of V
template <typename K>
int32_t allow_lds(K kernel, size_t bytes) {
  if (bytes <= 8 * 1024) return SVDC_OK;
  return hipFuncSetAttribute((const void*)kernel, hipFuncAttributeMaxDynamicSharedMemorySize, (int)bytes) == hipSuccess
             ? SVDC_OK : SVDC_E_HIP;
}

template <typename T>
int32_t full_step_general_typed(const svdc_shape& s, const void* F, const float* V, void* R, float* S, float* C,
                                float alpha, int init, ResidualEma re, hipStream_t st) {
  constexpr bool kF32 = sizeof(T) == 4;
  const int rt = full_step_may_take_parts(s.D, s.k, kF32, re.prev != nullptr)
                     ? full_step_parts_rows(s.N, s.B, s.D, s.k, kF32, re.prev != nullptr, num_compute_units()) : 0;
  if (rt > 0) {
    auto go = [&](auto tiles) -> int32_t {
      constexpr int RT = decltype(tiles)::value;
      constexpr bool kRema = !kF32 && RT > 1;       // the others are not asked for
      const auto kernel = kRema && re.prev ? full_step_parts_kernel<T, RT, kRema> : full_step_parts_kernel<T, RT, false>;
      const int kt2 = (s.k + 31) / 32;
      const size_t lds = (size_t)RT * kt2 * 3 * 1024 + (size_t)16 * RT * (32 * kt2 + 4) * sizeof(float);
      if (allow_lds(kernel, lds) != SVDC_OK) return SVDC_E_HIP;
      kernel<<<dim3((s.N + 16 * RT - 1) / (16 * RT), s.B), 64 * kStepWaves, lds, st>>>(
          (const T*)F, V, (T*)R, (const T*)re.prev, re.alpha_r, S, C, s.N, s.D, s.k, s.ldf, s.block_stride, alpha, init);
      return launch_status();
    };
    if constexpr (!kF32) {
      if (rt == 1) return go(std::integral_constant<int, 1>{});
    }
    if (rt == 2) return go(std::integral_constant<int, 2>{});
    return go(std::integral_constant<int, 3>{});
  }
  return general_dispatch<2>(s, [&](auto kt) -> int32_t {
    auto kernel = full_step_general_kernel<T, decltype(kt)::value>;
    const size_t lds = (size_t)16 * coef_stride(s.k) * sizeof(float);
    if (allow_lds(kernel, lds) != SVDC_OK) return SVDC_E_HIP;
    kernel<<<dim3((s.N + 15) / 16, s.B), 64 * kStepWaves, lds, st>>>((const T*)F, V, (T*)R, (const T*)re.prev, re.alpha_r,
                                                                     S, C, s.N, s.D, s.k, s.ldf, s.block_stride, alpha,
                                                                     init);
    return launch_status();
  });
}

template <typename T>
int32_t forecast_general_typed(const svdc_shape& s, const CoefStates& cs, const float* V, const void* R, const void* X,
                               void* Out, hipStream_t st) {
  constexpr bool kF32 = sizeof(T) == 4;
  if (cached_step_may_take_parts(s.D, s.k, kF32, cs.m, X != nullptr) &&
      cached_step_takes_parts(s.N, s.B, s.D, s.k, kF32, cs.m, num_compute_units())) {
    auto kernel = forecast_parts_kernel<T, kCachedPartsRows>;
    const size_t lds = (size_t)kCachedPartsRows * ((s.k + 31) / 32) * 3 * 1024;
    if (allow_lds(kernel, lds) != SVDC_OK) return SVDC_E_HIP;
    const int64_t tiles = (s.N + 16 * kCachedPartsRows - 1) / (16 * kCachedPartsRows);
    kernel<<<dim3((unsigned)tiles, s.B, cached_shares(tiles, s.B, s.D, true, num_compute_units())), 64 * kCachedWaves, lds, st>>>(
        cs, V, (const T*)R, (T*)Out, s.N, s.D, s.k, s.ldf, s.block_stride);
    return launch_status();
  }
  return general_dispatch<4>(s, [&](auto kt) -> int32_t {
    auto kernel = forecast_general_kernel<T, decltype(kt)::value>;
    const size_t lds = (size_t)16 * coef_stride(s.k) * sizeof(float);
    if (allow_lds(kernel, lds) != SVDC_OK) return SVDC_E_HIP;
    const int64_t tiles = (s.N + 15) / 16;
    // few channels have one share only, whatever the device: its query is a fiftieth of the smallest calls
    const int shares = s.D > 32 * (4 * kCachedWaves - 1) ? cached_shares(tiles, s.B, s.D, false, num_compute_units()) : 1;
    kernel<<<dim3((unsigned)tiles, s.B, shares), 64 * kCachedWaves, lds, st>>>(cs, V, (const T*)R, (const T*)X, (T*)Out,
                                                                               s.N, s.D, s.k, s.ldf, s.block_stride);
    return launch_status();
  });
}

}  // namespace

int32_t launch_full_step_general(const svdc_shape& s, const void* F, const float* V, void* R, float* S,
                                 float* C, float alpha, int init, ResidualEma re, hipStream_t st) {
  if (s.dtype == SVDC_BF16) return full_step_general_typed<bf16_t>(s, F, V, R, S, C, alpha, init, re, st);
  return full_step_general_typed<float>(s, F, V, R, S, C, alpha, init, re, st);
}

int32_t launch_forecast_general(const svdc_shape& s, const CoefStates& cs, const float* V, const void* R,
                                const void* X, void* Out, hipStream_t st) {
  if (s.dtype == SVDC_BF16) return forecast_general_typed<bf16_t>(s, cs, V, R, X, Out, st);
  return forecast_general_typed<float>(s, cs, V, R, X, Out, st);
}

// ---------------------------------------------------------------------------
// Rank selection by retained energy (Eq. 6) from the leading singular values and ||F||_F^2:
// k* = smallest count whose squared singular values sum to at least tau * ||F||_F^2, in float64, summed left to
// right.  One thread per block (k <= 1024 values).
// ---------------------------------------------------------------------------
__global__ void select_rank_kernel(const float* __restrict__ sigma, const float* __restrict__ fro2, float tau,
                                   int32_t* k_star, int32_t* reached, int B, int k) {
  const int b = blockIdx.x * blockDim.x + threadIdx.x;
  if (b >= B) return;
  const double thr = (double)tau * (double)fro2[b];
  double acc = 0.0;
  int ks = k, ok = 0;
  for (int i = 0; i < k; ++i) {
    const double s = (double)sigma[(int64_t)b * k + i];
    acc = acc + s * s;
    if (acc >= thr) {
      ks = i + 1;
      ok = 1;
      break;
    }
  }
  k_star[b] = ks;
  if (reached) reached[b] = ok;
}

// zero the columns j >= k_star[b] of V[b] (and of sigma[b])
__global__ __launch_bounds__(256) void truncate_basis_kernel(float* V, float* sigma, const int32_t* __restrict__ k_star,
                                                             int D, int k) {
  const int b = blockIdx.y;
  const int ks = k_star[b];
  const int64_t n = (int64_t)D * k;
  const int64_t idx = (int64_t)blockIdx.x * 256 + threadIdx.x;
  if (idx < n && (int)(idx % k) >= ks) V[(int64_t)b * n + idx] = 0.f;
  if (sigma && idx < k && idx >= ks) sigma[(int64_t)b * k + idx] = 0.f;
}

int32_t launch_select_rank(int B, int k, const float* sigma, const float* fro2, float tau, int32_t* k_star,
                           int32_t* reached, hipStream_t st) {
  select_rank_kernel<<<(B + 63) / 64, 64, 0, st>>>(sigma, fro2, tau, k_star, reached, B, k);
  return launch_status();
}

int32_t launch_truncate_basis(const svdc_shape& s, float* V, float* sigma, const int32_t* k_star, hipStream_t st) {
  const int64_t n = (int64_t)s.D * s.k;
  dim3 grid((unsigned)((n + 255) / 256), s.B);
  truncate_basis_kernel<<<grid, 256, 0, st>>>(V, sigma, k_star, s.D, s.k);
  return launch_status();
}

}  // namespace svdc
