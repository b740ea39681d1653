// Basis fit (Sec. 3.2, Eq. 4-5): the k leading right singular vectors of F by
// randomized subspace iteration followed by a Rayleigh-Ritz step.
//
//   Q <- Omega                             Omega: D x l Gaussian, l = k + p
//   repeat q times:  Y = F Q;  Z = F^T Y;  Q <- orth(Z)       (one application of F^T F)
//   Y = F Q;  H = Y^T Y = L L^T;  L = W diag(sigma) X^T       (one-sided Jacobi on L, fp64: H = W diag(sigma^2) W^T)
//   V_k = Q W[:, :k],  sigma_k = sigma[:k]
//
// orth() is CholeskyQR applied twice; every l x l object (Gram matrices, Cholesky
// factors, Jacobi rotations) is float64 because Z = F^T F Q has the squared
// condition number of F's leading part and its Gram matrix squares it again.
// The tall matrices Q, Z (D x l) and Y (N x l) are float32.
//
// This file holds the small-matrix kernels, the host orchestration and the versions of the two products with F for any
// hidden size; those for multiples of 128 are in fit_mfma_kernels.hip.
#include <algorithm>
#include <utility>

#include <type_traits>

#include "chol_kernels.h"
#include "f32_tiles.h"
#include "step_tiling.h"
#include "svdc_device.h"
#include "svdc_internal.h"

namespace svdc {

// ---------------------------------------------------------------------------
// counter-based Gaussian test matrix
// ---------------------------------------------------------------------------
__device__ __forceinline__ uint64_t mix64(uint64_t x) {
  // 64-bit finaliser (xor-shift-multiply rounds); statistically adequate for a sketch matrix
  x ^= x >> 30; x *= 0xbf58476d1ce4e5b9ull;
  x ^= x >> 27; x *= 0x94d049bb133111ebull;
  x ^= x >> 31;
  return x;
}

// element i of the Gaussian test matrix
__device__ __forceinline__ float omega(int64_t i, uint64_t seed) {
  const uint64_t h = mix64(seed * 0x9e3779b97f4a7c15ull + (uint64_t)i + 1);
  const uint32_t a = (uint32_t)h, c = (uint32_t)(h >> 32);
  const float u1 = ((float)(a >> 8) + 0.5f) * (1.0f / 16777216.0f);   // (0,1)
  const float u2 = ((float)(c >> 8) + 0.5f) * (1.0f / 16777216.0f);
  return sqrtf(-2.0f * __logf(u1)) * __cosf(6.283185307179586f * u2);  // Box-Muller
}
__global__ void init_omega_kernel(float* Q, int64_t total, uint64_t seed) {
  const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (i < total) Q[i] = omega(i, seed);
}

// Start of a fit with power iterations on the matrix cores: the test matrix [B, D, l] as operand words of the projection (layout: see
// PackedQ; low parts where the first product takes them), the accumulators and status words (`misc`) cleared, and Z where it has to be.
// One launch instead of four (one block of 4608 x 3072, rank 32: 18 -> 5 us).
__global__ __launch_bounds__(256) void init_sketch_kernel(PackedQ pq, int B, int D, int l, bool low_parts, uint64_t seed, double* misc, int64_t nmisc,
                                                          float* Z, int64_t nz) {
  const int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x;
  if (i < nmisc) misc[i] = 0.0;
  if (4 * i + 3 < nz) *reinterpret_cast<float4*>(Z + 4 * i) = make_float4(0.f, 0.f, 0.f, 0.f);
  else
    for (int64_t j = 4 * i; j < nz; ++j) Z[j] = 0.f;
  const int kts = pq.kt[0] + (pq.ranges > 1 ? pq.kt[1] : 0), lane = (int)(i & 63), r = lane & 15, g = lane >> 4;
  const int64_t word = i >> 6;
  const int jt = (int)(word % kts), cg = (int)(word / kts % (D / 32)), h = jt >= pq.kt[0] ? 1 : 0;
  const int64_t b = word / kts / (D / 32);
  if (b >= B) return;
  const int KT = pq.kt[h], tile = jt - (h ? pq.kt[0] : 0), col = 128 * h + 16 * tile + r;
  const int64_t per = (int64_t)D * KT * 16;                     // elements of one part of one block
  float x[8];
#pragma unroll
  for (int e = 0; e < 8; ++e) x[e] = col < l ? omega((b * D + 32 * cg + 8 * g + e) * l + col, seed) : 0.f;
  u32x4 hi, lo;
  split_operand(x, &hi, &lo);
  u32x4* p = reinterpret_cast<u32x4*>(pq.p + pq.offset[h]) + b * 2 * (per / 8) + ((int64_t)cg * KT + tile) * 64 + lane;
  p[0] = hi;
  if (low_parts) p[per / 8] = lo;
}

__global__ void fill_zero_kernel(double* p, int64_t n) {
  const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (i < n) p[i] = 0.0;
}
__global__ void fill_zero_f32_kernel(float* p, int64_t n) {
  const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (i < n) p[i] = 0.f;
}

// ---------------------------------------------------------------------------
// Products with F for hidden sizes that are not multiples of 128, on the float32 matrix cores: Y = F Q and Z = F^T Y.
// Bound by the matrix rate at wide sketches (256 flop per clock and compute unit, columns padded to 16, 32 or 64) and by the
// latency of their loads at narrow ones.  One block of 15752 x 1440 bf16, 8 columns: 14 us (Y) and 16 us (Z), 1905 x 1312 with
// 192 columns: 20 and 23 us, against 160 and 112, 153 and 111 us on the vector units with both operands staged in LDS an
// element at a time.
// ---------------------------------------------------------------------------

// Y[N x l] = F[N x D] Q[D x l], 16 KT columns of Y.  A wave has 16 RT token rows and walks over chunks of 32 channels: a lane's
// eight channels 32 c + 8 g + e of its row are one (bf16) or two loads, step e of eight contracts the channels
// {32 c + 8 g + e}, and the rows of Q pass through the wave's own LDS area a chunk ahead (VPiece).  The four waves of a
// workgroup take WK shares of the chunks each for 4 / WK row groups; with WK = 4 their sums meet in LDS.
constexpr int kFitWaves = 4;
template <typename T, int KT, int RT, int WK>
__global__ __launch_bounds__(64 * kFitWaves) void fit_rows_general_kernel(const T* __restrict__ F, const float* __restrict__ Q,
                                                                          float* __restrict__ Y, int N, int D, int l,
                                                                          int64_t ldf, int64_t bstride) {
  using Stage = VPiece<KT>;
  static_assert(WK == 1 || WK == kFitWaves, "a wave alone, or all four on the same rows");
  static_assert(Stage::kFloats >= RT * KT * 256, "partial sums fit");
  __shared__ __align__(16) float stage[kFitWaves][Stage::kFloats];
  struct alignas(4 * KT) RowVec { float v[KT]; };
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), lane = threadIdx.x & 63, r = lane & 15, g = lane >> 4;
  const int b = blockIdx.z, j0 = blockIdx.y * 16 * KT, nchunk = (D + 31) / 32;
  const int row0 = (blockIdx.x * (kFitWaves / WK) + (WK == 1 ? wave : 0)) * 16 * RT;
  if (WK == 1 && row0 >= N) return;
  const float* q = Q + (int64_t)b * D * l;
  float* lds = stage[wave];
  const T* frow[RT];
#pragma unroll
  for (int rt = 0; rt < RT; ++rt) frow[rt] = F + (int64_t)b * bstride + (int64_t)min(row0 + 16 * rt + r, N - 1) * ldf;

  constexpr int NH = KT * RT >= 4 ? 1 : 4 / (KT * RT);   // accumulators per result tile: four chains at least
  f32x4 acc[RT][KT][NH];
#pragma unroll
  for (int rt = 0; rt < RT; ++rt)
#pragma unroll
    for (int jt = 0; jt < KT; ++jt)
#pragma unroll
      for (int h = 0; h < NH; ++h) acc[rt][jt][h] = f32x4{0.f, 0.f, 0.f, 0.f};
  const int c0 = WK == 1 ? 0 : wave;
  Piece<T> fn[RT];
  Stage vp;
  if (c0 < nchunk) {
#pragma unroll
    for (int rt = 0; rt < RT; ++rt) fn[rt].load(frow[rt], 32 * c0 + 8 * g, D);
    vp.load(q, D, l, c0, j0);
  }
  for (int c = c0; c < nchunk; c += WK) {
    Piece<T> f[RT];
#pragma unroll
    for (int rt = 0; rt < RT; ++rt) f[rt] = fn[rt];
    vp.to_lds(lds);
    if (c + WK < nchunk) {
#pragma unroll
      for (int rt = 0; rt < RT; ++rt) fn[rt].load(frow[rt], 32 * (c + WK) + 8 * g, D);
      vp.load(q, D, l, c + WK, j0);
    }
#pragma unroll
    for (int e = 0; e < 8; ++e) {
      // columns of the result tile jt: j0 + KT r + jt, so that one wide LDS read brings the operands of all tiles
      const RowVec qv = *reinterpret_cast<const RowVec*>(lds + (8 * g + e) * Stage::KS + KT * r);
#pragma unroll
      for (int rt = 0; rt < RT; ++rt) {
        const float x = f[rt].get(e);
#pragma unroll
        for (int jt = 0; jt < KT; ++jt) acc[rt][jt][e % NH] = mfma_f32(x, qv.v[jt], acc[rt][jt][e % NH]);
      }
    }
  }
#pragma unroll
  for (int rt = 0; rt < RT; ++rt)
#pragma unroll
    for (int jt = 0; jt < KT; ++jt)
#pragma unroll
      for (int h = 1; h < NH; ++h) acc[rt][jt][0] += acc[rt][jt][h];
  // D[m = 4 g + i][n = r]: row 4 g + i, column j0 + KT r + jt
  auto store = [&](int rt, int jt, const f32x4& x) {
    const int j = j0 + KT * r + jt;
    if (j >= l) return;
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      const int row = row0 + 16 * rt + 4 * g + i;
      if (row < N) Y[((int64_t)b * N + row) * l + j] = x[i];
    }
  };
  if constexpr (WK == 1) {
#pragma unroll
    for (int rt = 0; rt < RT; ++rt)
#pragma unroll
      for (int jt = 0; jt < KT; ++jt) store(rt, jt, acc[rt][jt][0]);
  } else {
    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
    f32x4* mine = reinterpret_cast<f32x4*>(lds);
#pragma unroll
    for (int rt = 0; rt < RT; ++rt)
#pragma unroll
      for (int jt = 0; jt < KT; ++jt) mine[(rt * KT + jt) * 64 + lane] = acc[rt][jt][0];
    __syncthreads();
#pragma unroll
    for (int n = 0; n < RT * KT; ++n) {
      if (n % kFitWaves != wave) continue;
      f32x4 x = reinterpret_cast<const f32x4*>(stage[0])[n * 64 + lane];
#pragma unroll
      for (int w = 1; w < kFitWaves; ++w) x += reinterpret_cast<const f32x4*>(stage[w])[n * 64 + lane];
      store(n / KT, n % KT, x);
    }
  }
}

// Z[D x l] (+)= F^T Y over the token rows of one share, 128 channels x 16 KT columns.  A lane holds the eight channels
// d0 + 8 r .. of token n + g, element e of which is the operand of the tile of channels {d0 + 8 m + e}, and the
// columns j0 + 16 t + r of the same token: both come straight from memory, whole lines at a time.  The waves take every
// fourth group of four tokens, their sums meet in LDS in a fixed order, those of several shares in float atomics.
template <typename T, int KT>
__global__ __launch_bounds__(64 * kFitWaves) void fit_cols_general_kernel(const T* __restrict__ F, const float* __restrict__ Y,
                                                                          float* __restrict__ Z, int N, int D, int l,
                                                                          int64_t ldf, int64_t bstride, int share, int nshare) {
  constexpr int UN = KT >= 4 ? 2 : 4;               // token groups requested at a time, one such set ahead
  __shared__ __align__(16) f32x4 part[kFitWaves][2 * KT][64];
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), lane = threadIdx.x & 63, r = lane & 15, g = lane >> 4;
  const int b = blockIdx.z / nshare, d0 = blockIdx.x * 128, j0 = blockIdx.y * 16 * KT;
  const int n0 = (blockIdx.z % nshare) * share, n1 = min(N, n0 + share);
  const T* f = F + (int64_t)b * bstride;
  const float* y = Y + (int64_t)b * N * l + j0 + r;
  f32x4 acc[8][KT];
#pragma unroll
  for (int e = 0; e < 8; ++e)
#pragma unroll
    for (int t = 0; t < KT; ++t) acc[e][t] = f32x4{0.f, 0.f, 0.f, 0.f};
  Piece<T> fp[UN];
  float yp[UN][KT];
  auto load = [&](int n) {                          // the wave's groups of the UN x 16 tokens from n
#pragma unroll
    for (int u = 0; u < UN; ++u) {
      const int tok = n + 16 * u + 4 * wave + g, at = min(tok, n1 - 1);
      fp[u].load(f + (int64_t)at * ldf, d0 + 8 * r, tok < n1 ? D : 0);
#pragma unroll
      for (int t = 0; t < KT; ++t) {
        const bool in = tok < n1 && j0 + 16 * t + r < l;
        yp[u][t] = in ? y[(int64_t)at * l + 16 * t] : 0.f;
      }
    }
  };
  load(n0);
  for (int n = n0; n < n1; n += 16 * UN) {
    Piece<T> fc[UN];
    float yc[UN][KT];
#pragma unroll
    for (int u = 0; u < UN; ++u) {
      fc[u] = fp[u];
#pragma unroll
      for (int t = 0; t < KT; ++t) yc[u][t] = yp[u][t];
    }
    if (n + 16 * UN < n1) load(n + 16 * UN);
#pragma unroll
    for (int u = 0; u < UN; ++u)
#pragma unroll
      for (int e = 0; e < 8; ++e) {
        const float x = fc[u].get(e);
#pragma unroll
        for (int t = 0; t < KT; ++t) acc[e][t] = mfma_f32(x, yc[u][t], acc[e][t]);
      }
  }
#pragma unroll
  for (int e = 0; e < 8; e += 2) {                  // two channel tiles at a time through LDS
#pragma unroll
    for (int s = 0; s < 2; ++s)
#pragma unroll
      for (int t = 0; t < KT; ++t) part[wave][s * KT + t][lane] = acc[e + s][t];
    __syncthreads();
#pragma unroll
    for (int n = 0; n < 2 * KT; ++n) {
      if (n % kFitWaves != wave) continue;
      f32x4 x = part[0][n][lane];
#pragma unroll
      for (int w = 1; w < kFitWaves; ++w) x += part[w][n][lane];
      const int j = j0 + 16 * (n % KT) + r;
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        const int d = d0 + 8 * (4 * g + i) + e + n / KT;
        if (d >= D || j >= l) continue;
        float* z = Z + ((int64_t)b * D + d) * l + j;
        if (nshare > 1) atomicAdd(z, x[i]);
        else *z = x[i];
      }
    }
    __syncthreads();
  }
}

// ---------------------------------------------------------------------------
// 64 x 64 x (4 K4) float64 product on the matrix cores (v_mfma_f64_16x16x4_f64), shared by the Gram matrices and the
// small tile products below.  Both operands sit in LDS with the contraction index as the row:
//   As[k][i] (row stride LDA), Bs[k][j] (row stride LDB),  acc += sum_k As[k][i] * Bs[k][j].
// Wave w of four takes the 32 x 32 quadrant (w / 2, w % 2) as 2 x 2 tiles of 16 x 16.  Lane layout of the
// instruction (checked on the device with one-hot operands):
//   A operand: lane -> A[i = lane % 16][k = lane / 16]        B operand: lane -> B[k = lane / 16][j = lane % 16]
//   D: lane, v  -> D[i = 4 v + lane / 16][j = lane % 16]
// so a lane reads As[4 k4 + lane / 16][i0 + lane % 16]: 16 consecutive doubles per group of 16 lanes, and with a row
// stride of 80 doubles the two groups of a half wave fall into different halves of the LDS banks.
// ---------------------------------------------------------------------------
constexpr int kM64Stride = 80;

struct Quadrant {
  int i0, j0, m, kq;   // first row / column of the wave's quadrant, lane % 16, lane / 16
  __device__ __forceinline__ Quadrant() {
    const int wave = threadIdx.x >> 6, lane = threadIdx.x & 63;
    i0 = 32 * (wave >> 1); j0 = 32 * (wave & 1); m = lane & 15; kq = lane >> 4;
  }
  // row and column (inside the 64 x 64 tile) of element v of accumulator tile (a, b)
  __device__ __forceinline__ int row(int a, int v) const { return i0 + 16 * a + 4 * v + kq; }
  __device__ __forceinline__ int col(int b) const { return j0 + 16 * b + m; }
};

template <int K4>
__device__ __forceinline__ void mfma64_accumulate(const double* As, const double* Bs, const Quadrant& q,
                                                  f64x4 (&acc)[2][2]) {
#pragma unroll
  for (int k4 = 0; k4 < K4; ++k4) {
    const double* ar = As + (4 * k4 + q.kq) * kM64Stride + q.i0 + q.m;
    const double* br = Bs + (4 * k4 + q.kq) * kM64Stride + q.j0 + q.m;
    const double a0 = ar[0], a1 = ar[16], b0 = br[0], b1 = br[16];
    acc[0][0] = __builtin_amdgcn_mfma_f64_16x16x4f64(a0, b0, acc[0][0], 0, 0, 0);
    acc[0][1] = __builtin_amdgcn_mfma_f64_16x16x4f64(a0, b1, acc[0][1], 0, 0, 0);
    acc[1][0] = __builtin_amdgcn_mfma_f64_16x16x4f64(a1, b0, acc[1][0], 0, 0, 0);
    acc[1][1] = __builtin_amdgcn_mfma_f64_16x16x4f64(a1, b1, acc[1][1], 0, 0, 0);
  }
}

// ---------------------------------------------------------------------------
// Partial Gram matrices A^T A in float64, A float32 [rows x l]; rows split over grid.x, 64 x 64 tiles of the lower
// block triangle (tile row >= tile column) over grid.y: the factorisation that follows never reads the rest.
// Four rows of A are one step of the matrix instruction, and a lane's operand A[row 4 k + lane / 16][column lane % 16] is
// a coalesced load, so nothing is staged: each of the four waves takes every fourth group of four rows, requests the
// next ones ahead, and multiplies the 16 x 16 tiles on or below the diagonal (10 of 16 in a diagonal tile); the waves'
// sums meet in LDS.  27 us for 57 blocks of 3072 x 64 (the float64 matrix rate
// allows 11), 8.2 us for one, against 40 and 14 us with all 16 tiles and the rows staged in LDS as float64, two barriers
// per 16 rows.
// ---------------------------------------------------------------------------
template <bool DIAGONAL>
__device__ __forceinline__ void gram_tile(const float* a, double* g, f64x4 (*part)[DIAGONAL ? 10 : 16][64], int rows, int l, int ti, int tj,
                                          int rbeg, int rend) {
  constexpr int NI = 4, U = 4;         // column tiles per side; groups of four rows in flight
  const int wave = threadIdx.x >> 6, lane = threadIdx.x & 63, m = lane & 15, kq = lane >> 4;
  int ci[NI], cj[NI];
  bool ini[NI], inj[NI];
#pragma unroll
  for (int x = 0; x < NI; ++x) {
    ini[x] = 64 * ti + 16 * x + m < l;
    inj[x] = 64 * tj + 16 * x + m < l;
    ci[x] = min(64 * ti + 16 * x + m, l - 1);
    cj[x] = min(64 * tj + 16 * x + m, l - 1);
  }
  f64x4 acc[NI][NI];
#pragma unroll
  for (int x = 0; x < NI; ++x)
#pragma unroll
    for (int y = 0; y < NI; ++y) acc[x][y] = f64x4{0.0, 0.0, 0.0, 0.0};
  // loaded from clamped addresses; what lies outside is made zero when it is used, so that no load is waited for early
  float vi[U][NI], vj[U][NI];
  auto fetch = [&](int u, int r0) {
    const float* row = a + (int64_t)min(r0 + kq, rows - 1) * l;
#pragma unroll
    for (int x = 0; x < NI; ++x) {
      vi[u][x] = row[ci[x]];
      if constexpr (!DIAGONAL) vj[u][x] = row[cj[x]];
    }
  };
#pragma unroll
  for (int u = 0; u < U; ++u) fetch(u, rbeg + 4 * wave + 16 * u);
  for (int r0 = rbeg + 4 * wave; r0 < rend; r0 += 16 * U) {
#pragma unroll
    for (int u = 0; u < U; ++u) {
      const bool in = r0 + 16 * u + kq < rend;
      double di[NI], dj[NI];
#pragma unroll
      for (int x = 0; x < NI; ++x) {
        di[x] = (double)(in && ini[x] ? vi[u][x] : 0.f);
        if constexpr (!DIAGONAL) dj[x] = (double)(in && inj[x] ? vj[u][x] : 0.f);
      }
      fetch(u, r0 + 16 * (u + U));
#pragma unroll
      for (int x = 0; x < NI; ++x)
#pragma unroll
        for (int y = 0; y < NI; ++y) {
          if (DIAGONAL && y > x) continue;
          acc[x][y] = __builtin_amdgcn_mfma_f64_16x16x4f64(di[x], DIAGONAL ? di[y] : dj[y], acc[x][y], 0, 0, 0);
        }
      __builtin_amdgcn_sched_barrier(0);
    }
  }
  // sum over the waves, two at a time (a wave's 16 tiles are 32 KB)
  const auto tile = [](int x, int y) { return DIAGONAL ? x * (x + 1) / 2 + y : 4 * x + y; };
#pragma unroll
  for (int half = 2; half >= 1; half >>= 1) {
    if (wave >= half && wave < 2 * half) {
#pragma unroll
      for (int x = 0; x < NI; ++x)
#pragma unroll
        for (int y = 0; y < NI; ++y)
          if (!(DIAGONAL && y > x)) part[wave - half][tile(x, y)][lane] = acc[x][y];
    }
    __syncthreads();
    if (wave < half) {
#pragma unroll
      for (int x = 0; x < NI; ++x)
#pragma unroll
        for (int y = 0; y < NI; ++y)
          if (!(DIAGONAL && y > x)) acc[x][y] += part[wave][tile(x, y)][lane];
    }
    __syncthreads();
  }
  if (wave != 0) return;
  // D[i = 4 v + lane / 16][j = lane % 16]; the tiles above the diagonal are the mirror images of those below
#pragma unroll
  for (int x = 0; x < NI; ++x)
#pragma unroll
    for (int y = 0; y < NI; ++y) {
      if (DIAGONAL && y > x) continue;
#pragma unroll
      for (int v = 0; v < 4; ++v) {
        const int gi = 64 * ti + 16 * x + 4 * v + kq, gj = 64 * tj + 16 * y + m;
        if (gi >= l || gj >= l) continue;
        g[(int64_t)gi * l + gj] = acc[x][y][v];
        if (DIAGONAL && y < x) g[(int64_t)gj * l + gi] = acc[x][y][v];
      }
    }
}

// Where the partial Gram matrices (l x l doubles each) lie: the first end[0] in p[0], up to end[1] in p[1], the others in p[2].
struct GramParts {
  double* p[3];
  int64_t end[2];
  __device__ __forceinline__ double* at(int64_t i, int64_t ll) const {
    return i < end[0] ? p[0] + i * ll : (i < end[1] ? p[1] + (i - end[0]) * ll : p[2] + (i - end[1]) * ll);
  }
};

// ONE_TILE: l <= 64, a single tile on the diagonal (a kernel of its own: 150 instead of 330 registers)
template <bool ONE_TILE>
__global__ __launch_bounds__(256, ONE_TILE ? 3 : 1) void gram_f64_kernel(const float* __restrict__ A, GramParts parts, int rows, int l,
                                                       int rows_per_slice) {
  __shared__ f64x4 part[2 * (ONE_TILE ? 10 : 16) * 64];
  const int b = blockIdx.z;
  int ti = 0;
  while ((ti + 1) * (ti + 2) / 2 <= (int)blockIdx.y) ++ti;
  const int tj = blockIdx.y - ti * (ti + 1) / 2;
  const float* a = A + (int64_t)b * rows * l;
  double* g = parts.at((int64_t)b * gridDim.x + blockIdx.x, (int64_t)l * l);   // partial Gram matrix of this row slice
  const int rbeg = blockIdx.x * rows_per_slice, rend = min(rows, rbeg + rows_per_slice);
  if (ONE_TILE || ti == tj) gram_tile<true>(a, g, reinterpret_cast<f64x4(*)[10][64]>(part), rows, l, ti, tj, rbeg, rend);
  else if constexpr (!ONE_TILE) gram_tile<false>(a, g, reinterpret_cast<f64x4(*)[16][64]>(part), rows, l, ti, tj, rbeg, rend);
}

// G[b] = sum over the row slices of the partial Gram matrices, in a fixed order (no atomics: the same bits every run);
// lower block triangle only, like the partial matrices.  64 elements per workgroup, the slices in four shares with
// several loads in flight each (one thread per element walking over 16 slices took 6.2 us at any size, this 3 us).
__global__ __launch_bounds__(256) void gram_reduce_kernel(GramParts parts, double* G, int nslice, int l) {
  __shared__ double share[3][64];
  const int b = blockIdx.y, lane = threadIdx.x & 63, q = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int64_t ll = (int64_t)l * l;
  const int64_t e = (int64_t)blockIdx.x * 64 + lane;
  const bool in = e < ll && (e % l) / 64 <= (e / l) / 64;
  double s = 0.0;
  if (in) {
#pragma unroll 6
    for (int i = q; i < nslice; i += 4) s += parts.at((int64_t)b * nslice + i, ll)[e];
  }
  if (q > 0) share[q - 1][lane] = s;
  __syncthreads();
  if (q == 0 && in) G[(int64_t)b * ll + e] = (s + share[0][lane]) + (share[1][lane] + share[2][lane]);
}

// ---------------------------------------------------------------------------
// 64 x 64 tile of a product A[64 x K] (rows of type TA) * Bm[K x 64] (float64), accumulated in float64 on the matrix
// cores by one workgroup of 256 threads (mfma64_accumulate).  The inner dimension is walked in chunks of 32 staged in
// LDS as float64, A transposed to [k][r]; the next chunk's elements are fetched into registers before the current one
// is multiplied, so their latency is hidden behind the arithmetic.
//   load_a(r, k)  element (r, k) of A, 0 outside        load_b(k, j)  element (k, j) of Bm, 0 outside
//   emit(r, j, x) called for every element (r, j) of the tile that this lane holds
// ---------------------------------------------------------------------------
constexpr int kTileK = 32;
struct TileGemmLds {
  double Bs[kTileK * kM64Stride];          // [k][j]
  double As[kTileK * (kM64Stride + 1)];    // [k][r], odd stride: the transposing stores of a wave spread over the banks
};

template <typename TA, typename LoadA, typename LoadB, typename Emit>
__device__ __forceinline__ void tile_gemm_64x64(int K, LoadA load_a, LoadB load_b, TileGemmLds& lds, Emit emit) {
  constexpr int LA = kM64Stride + 1;
  const int t = threadIdx.x;
  // staging role of this thread: 8 elements of each operand per chunk
  const int ar = t >> 5, ak = t & 31;          // A: rows ar + 8 e, column ak
  const int bk = t >> 6, bj = t & 63;          // B: rows bk + 4 e, column bj
  TA ra[8];
  double rb[8];
  auto fetch = [&](int k0) {
#pragma unroll
    for (int e = 0; e < 8; ++e) {
      ra[e] = load_a(ar + 8 * e, k0 + ak);
      rb[e] = load_b(k0 + bk + 4 * e, bj);
    }
  };
  const Quadrant q;
  f64x4 acc[2][2];
#pragma unroll
  for (int x = 0; x < 2; ++x)
#pragma unroll
    for (int y = 0; y < 2; ++y) acc[x][y] = f64x4{0.0, 0.0, 0.0, 0.0};
  fetch(0);
  for (int k0 = 0; k0 < K; k0 += kTileK) {
    if (k0 > 0) __syncthreads();               // the previous chunk has been read by everybody
#pragma unroll
    for (int e = 0; e < 8; ++e) {
      lds.As[ak * LA + ar + 8 * e] = (double)ra[e];
      lds.Bs[(bk + 4 * e) * kM64Stride + bj] = rb[e];
    }
    __syncthreads();
    if (k0 + kTileK < K) fetch(k0 + kTileK);
#pragma unroll
    for (int k4 = 0; k4 < kTileK / 4; ++k4) {
      const double* arow = lds.As + (4 * k4 + q.kq) * LA + q.i0 + q.m;
      const double* brow = lds.Bs + (4 * k4 + q.kq) * kM64Stride + q.j0 + q.m;
      const double a0 = arow[0], a1 = arow[16], b0 = brow[0], b1 = brow[16];
      acc[0][0] = __builtin_amdgcn_mfma_f64_16x16x4f64(a0, b0, acc[0][0], 0, 0, 0);
      acc[0][1] = __builtin_amdgcn_mfma_f64_16x16x4f64(a0, b1, acc[0][1], 0, 0, 0);
      acc[1][0] = __builtin_amdgcn_mfma_f64_16x16x4f64(a1, b0, acc[1][0], 0, 0, 0);
      acc[1][1] = __builtin_amdgcn_mfma_f64_16x16x4f64(a1, b1, acc[1][1], 0, 0, 0);
    }
  }
#pragma unroll
  for (int x = 0; x < 2; ++x)
#pragma unroll
    for (int v = 0; v < 4; ++v)
#pragma unroll
      for (int y = 0; y < 2; ++y) emit(q.row(x, v), q.col(y), acc[x][y][v]);
}

// ---------------------------------------------------------------------------
// Out[rows x m] (float32) = In[rows x l] (float32) * M[l x m] (float64, row stride ldm), 64 x 64 tiles.
// ---------------------------------------------------------------------------
__global__ __launch_bounds__(256) void rows_times_small_kernel(const float* __restrict__ In,
                                                               const double* __restrict__ M, float* Out,
                                                               int rows, int l, int m, int ldm) {
  __shared__ TileGemmLds lds;
  const int b = blockIdx.z;
  const float* in = In + (int64_t)b * rows * l;
  const double* mm = M + (int64_t)b * l * ldm;
  float* out = Out + (int64_t)b * rows * m;
  const int r0 = blockIdx.x * 64, j0 = blockIdx.y * 64;
  tile_gemm_64x64<float>(
      l, [&](int r, int k) { return (r0 + r < rows && k < l) ? in[(int64_t)(r0 + r) * l + k] : 0.f; },
      [&](int k, int j) { return (k < l && j0 + j < m) ? mm[(int64_t)k * ldm + j0 + j] : 0.0; }, lds,
      [&](int r, int j, double x) {
        if (r0 + r < rows && j0 + j < m) out[(int64_t)(r0 + r) * m + j0 + j] = (float)x;
      });
}

// ---------------------------------------------------------------------------
// Blocked Cholesky factorisation for l > 128, left-looking over column blocks of 64: for block k at columns c0..c0+63
//   L_kk = chol(A_kk - sum_{c < c0} L[k, c] L[k, c]^T), and L_kk^-T              (chol_tiles_kernel)
//   L_ik = (A_ik - sum_{c < c0} L[i, c] L[k, c]^T) L_kk^-T  for rows i below      (this kernel, 64 rows per workgroup)
// The finished columns are kept twice, as L in the lower triangle and as L^T in the upper one (G[c][r] = L[r][c]).
// The sum runs on the float64 matrix cores; the solve goes by panels of 16 columns, a wave for 16 rows: a substitution (see
// `substitute` for why not a product with the inverse), and a product of the finished panel with the rows of L_kk below.  256
// columns, one block: 15.1 us a launch on average, 14.7 us as one product with the inverse; a substitution row by row took twice that.
// ---------------------------------------------------------------------------
constexpr int kTileLd = kM64Stride + 1;   // row stride of a transposed 64 x 64 float64 tile in LDS

__global__ __launch_bounds__(256) void chol_panel_kernel(double* G, int l, int c0) {
  constexpr int H = kCholBlock, LD = H + 1, LT = 20;
  __shared__ TileGemmLds lds;
  __shared__ double Tt[H * kTileLd];     // [column][row]
  static_assert(sizeof(TileGemmLds) >= H * LD * sizeof(double), "L_kk fits");
  const int b = blockIdx.y, t = threadIdx.x, lane = t & 63, m = lane & 15, kq = lane >> 4;
  const int wave = __builtin_amdgcn_readfirstlane(t >> 6);
  double* g = G + (int64_t)b * l * l;
  const int r0 = c0 + H + blockIdx.x * H;          // first row of this workgroup
  double ld[H * H / 256];                          // L_kk on its way to LDS
#pragma unroll
  for (int e = 0; e < H * H / 256; ++e) ld[e] = g[(int64_t)(c0 + wave + 4 * e) * l + c0 + lane];
  if (c0 > 0) {
    tile_gemm_64x64<double>(
        c0, [&](int r, int k) { return r0 + r < l ? g[(int64_t)(r0 + r) * l + k] : 0.0; },
        [&](int k, int j) { return g[(int64_t)k * l + c0 + j]; }, lds,
        [&](int r, int j, double x) { Tt[j * kTileLd + r] = (r0 + r < l ? g[(int64_t)(r0 + r) * l + c0 + j] : 0.0) - x; });
  } else {
    for (int e = t; e < H * H; e += 256) {
      const int r = e / H, j = e % H;
      Tt[j * kTileLd + r] = r0 + r < l ? g[(int64_t)(r0 + r) * l + c0 + j] : 0.0;
    }
  }
  __syncthreads();                                 // Tt is complete, the operands of the product have been read
  double* L = reinterpret_cast<double*>(&lds);     // [64][LD]
#pragma unroll
  for (int e = 0; e < H * H / 256; ++e) L[(wave + 4 * e) * LD + lane] = ld[e];
  f64x4 x[4];                                      // the wave's 16 rows, 16 columns each
#pragma unroll
  for (int q = 0; q < 4; ++q)
#pragma unroll
    for (int v = 0; v < 4; ++v) x[q][v] = Tt[(16 * q + m) * kTileLd + 16 * wave + 4 * v + kq];
  __syncthreads();
  double* own = Tt + wave * 16 * LT;               // the finished panel on its way from the result layout to the operand layout
#pragma unroll
  for (int q = 0; q < 4; ++q) {
    const double* lrow = L + (16 * q + m) * LD + 16 * q;
    const double rinv = 1.0 / lrow[m];
    double lo[8], hi[8];
#pragma unroll
    for (int j = 0; j < 8; ++j) {
      lo[j] = j < m ? lrow[j] : 0.0;
      hi[j] = j + 8 < m ? lrow[j + 8] : 0.0;
    }
    unit_columns<0>(lo, rinv);
    unit_columns<8>(hi, rinv);
    substitute<0>(x[q], lo);
    substitute<8>(x[q], hi);
    x[q] = x[q] * rinv;
#pragma unroll
    for (int v = 0; v < 4; ++v) {
      const int r = r0 + 16 * wave + 4 * v + kq, c = c0 + 16 * q + m;
      own[(4 * v + kq) * LT + m] = x[q][v];
      if (r < l) {
        g[(int64_t)r * l + c] = x[q][v];
        g[(int64_t)c * l + r] = x[q][v];
      }
    }
    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");   // a wave's own LDS area
#pragma unroll
    for (int k4 = 0; k4 < 4; ++k4) {
      const double av = -own[m * LT + 4 * k4 + kq];
#pragma unroll
      for (int n = q + 1; n < 4; ++n)
        x[n] = __builtin_amdgcn_mfma_f64_16x16x4f64(av, L[(16 * n + m) * LD + 16 * q + 4 * k4 + kq], x[n], 0, 0, 0);
    }
    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
  }
}

// ---------------------------------------------------------------------------
// Out = In L^-T for 64 rows per workgroup, all columns: by column blocks of 64,
//   Out_j = (In_j - sum_{i < j} Out_i L_ji^T) L_jj^-T
// with the inverses of the diagonal blocks (chol_tiles_kernel) and L^T from the upper triangle of G, every product on the
// float64 matrix cores.  A wave has 16 rows to itself: its rows of In and the small matrices (which all workgroups
// share, so they come from L2) are loaded in operand layout straight into registers, and of the 16 x 16 tiles of the
// triangular L_jj^-T only the ten that are not zero are used.  The contraction index of step (s, e) is
// 16 s + 4 (lane / 16) + e, so that a lane's four steps are one 16-byte piece of a float32 row.
// The result leaves as float32 rows (out, nullable) and/or as the operand words of the projection (pq.p, nullable; see
// PackedQ), so that an iteration that goes on with the projection writes nothing else.  zero_in: the rows of In are
// cleared once they have been read (the next back-projection accumulates into them).  Bound by the float64 matrix rate
// (11 us for 57 blocks of 3072 x 64) and the latency of its loads: 38 us there and 8.4 us for one block, against 57 + 20 and 26 + 5 us for a
// forward substitution per row followed by a packing kernel.
// ---------------------------------------------------------------------------
__device__ __forceinline__ void pack_rows(const float* ot, int ldo, int row0, int D, int b, int l, PackedQ pq);

// NT: 16-column tiles of the only column block, 1 (l <= 16) or 4 (l <= 64); 0: several blocks of 64 columns.
template <int NT>
__global__ __launch_bounds__(256, NT == 1 ? 6 : (NT == 4 ? 3 : 1)) void apply_factor_kernel(float* In, const double* __restrict__ G,
                                                           const double* __restrict__ Minv, int64_t m_bstride, float* out,
                                                           PackedQ pq, int rows, int l, int zero_in) {
  constexpr bool ONE_BLOCK = NT > 0;
  constexpr int H = kCholBlock, LT = H + 2, TY = ONE_BLOCK ? NT : 4;
  extern __shared__ __align__(16) char dyn[];
  const int nb = ONE_BLOCK ? 1 : (l + H - 1) / H, ldo = ONE_BLOCK ? 16 * TY + 4 : nb * H + 4;
  float* ot = reinterpret_cast<float*>(dyn);                                             // [64][ldo]
  const int wave = threadIdx.x >> 6, lane = threadIdx.x & 63, m = lane & 15, kq = lane >> 4;
  // the wave's right-hand sides on their way from the result layout to the operand layout, [16][LT]
  double* tt = reinterpret_cast<double*>(dyn + (size_t)H * ldo * sizeof(float)) + wave * 16 * LT;
  const int b = blockIdx.y, r0 = blockIdx.x * H, rw = r0 + 16 * wave;
  float* in = In + (int64_t)b * rows * l;
  const double* g = G + (int64_t)b * l * l;
  for (int j0 = 0; j0 < l; j0 += H) {
    const int w = min(H, l - j0), ldm = l <= H ? l : H;
    const double* mi = Minv + (int64_t)b * m_bstride + (int64_t)(j0 / H) * H * H;
    double bm[TY][4][TY];                        // [s][e][y], y >= s: L_jj^-T[16 s + 4 kq + e][16 y + m]
    auto load_b = [&](int s) {
#pragma unroll
      for (int e = 0; e < 4; ++e)
#pragma unroll
        for (int y = s; y < TY; ++y) {
          const int k = 16 * s + 4 * kq + e, j = 16 * y + m;
          bm[s][e][y] = mi[min(k, w - 1) * ldm + min(j, w - 1)];     // columns beyond w are not used
        }
    };
    load_b(0);
    double a[TY][4];
    if (j0 == 0) {
      const float* row = in + (int64_t)min(rw + m, rows - 1) * l;
#pragma unroll
      for (int s = 0; s < TY; ++s) {
        const int k = 16 * s + 4 * kq;
        if ((l & 3) == 0) {
          float4 x = make_float4(0.f, 0.f, 0.f, 0.f);
          if (k < w) x = *reinterpret_cast<const float4*>(row + k);
          a[s][0] = x.x; a[s][1] = x.y; a[s][2] = x.z; a[s][3] = x.w;
        } else {
#pragma unroll
          for (int e = 0; e < 4; ++e) a[s][e] = k + e < w ? (double)row[k + e] : 0.0;
        }
      }
    } else if constexpr (!ONE_BLOCK) {
      f64x4 up[4];
      float rhs[4][4];
#pragma unroll
      for (int y = 0; y < 4; ++y) {
        up[y] = f64x4{0.0, 0.0, 0.0, 0.0};
#pragma unroll
        for (int v = 0; v < 4; ++v) {
          const int r = rw + 4 * v + kq, j = 16 * y + m;
          rhs[y][v] = (r < rows && j < w) ? in[(int64_t)r * l + j0 + j] : 0.f;
        }
      }
      double gb[4][4], gn[4][4];               // [e][y]: L^T[k0 + 4 kq + e][j0 + 16 y + m]
      auto fetch = [&](int k0) {
#pragma unroll
        for (int e = 0; e < 4; ++e)
#pragma unroll
          for (int y = 0; y < 4; ++y) {
            const int j = 16 * y + m;
            gn[e][y] = j < w ? g[(int64_t)(k0 + 4 * kq + e) * l + j0 + j] : 0.0;
          }
      };
      fetch(0);
      for (int k0 = 0; k0 < j0; k0 += 16) {
#pragma unroll
        for (int e = 0; e < 4; ++e)
#pragma unroll
          for (int y = 0; y < 4; ++y) gb[e][y] = gn[e][y];
        if (k0 + 16 < j0) fetch(k0 + 16);
        const float4 o = *reinterpret_cast<const float4*>(ot + (16 * wave + m) * ldo + k0 + 4 * kq);
        const double oa[4] = {o.x, o.y, o.z, o.w};
#pragma unroll
        for (int e = 0; e < 4; ++e)
#pragma unroll
          for (int y = 0; y < 4; ++y) up[y] = __builtin_amdgcn_mfma_f64_16x16x4f64(oa[e], gb[e][y], up[y], 0, 0, 0);
      }
      __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
#pragma unroll
      for (int y = 0; y < 4; ++y)
#pragma unroll
        for (int v = 0; v < 4; ++v) tt[(4 * v + kq) * LT + 16 * y + m] = (double)rhs[y][v] - up[y][v];
      __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
#pragma unroll
      for (int s = 0; s < 4; ++s)
#pragma unroll
        for (int e = 0; e < 4; ++e) a[s][e] = tt[m * LT + 16 * s + 4 * kq + e];
    }
    f64x4 acc[TY];
#pragma unroll
    for (int y = 0; y < TY; ++y) acc[y] = f64x4{0.0, 0.0, 0.0, 0.0};
#pragma unroll
    for (int s = 0; s < TY; ++s) {
      if (s < TY - 1) load_b(s + 1);                // one step ahead
#pragma unroll
      for (int e = 0; e < 4; ++e)
#pragma unroll
        for (int y = s; y < TY; ++y) {
          const double bv = w < 16 * TY && 16 * s + 4 * kq + e >= w ? 0.0 : bm[s][e][y];
          acc[y] = __builtin_amdgcn_mfma_f64_16x16x4f64(a[s][e], bv, acc[y], 0, 0, 0);
        }
      __builtin_amdgcn_sched_barrier(0);
    }
    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
#pragma unroll
    for (int y = 0; y < TY; ++y)
#pragma unroll
      for (int v = 0; v < 4; ++v) ot[(16 * wave + 4 * v + kq) * ldo + j0 + 16 * y + m] = (float)acc[y][v];
    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");   // a wave reads back only its own rows until here
  }
  __syncthreads();
  const int nrow = min(H, rows - r0);
  float* irow = in + (int64_t)r0 * l;
  float* orow = out ? out + ((int64_t)b * rows + r0) * l : nullptr;
  if (orow || zero_in) {
    int r = threadIdx.x / l, j = threadIdx.x % l;        // element e = r l + j, advanced by 256 without divisions
    const int dr = 256 / l, dj = 256 % l;
    for (int e = threadIdx.x; e < nrow * l; e += 256) {
      if (orow) orow[e] = ot[r * ldo + j];
      if (zero_in) irow[e] = 0.f;
      r += dr; j += dj;
      if (j >= l) { j -= l; ++r; }
    }
  }
  if (pq.p) pack_rows(ot, ldo, r0, rows, b, l, pq);
}

// The 64 rows of Q in `ot` as operand words of the projection: tile (cg, jt) of 64 lanes x 8 bf16, lane (r, g), e ->
// Q[32 cg + 8 g + e][16 jt + r], high and low parts; sketches wider than 128 as two column ranges.
__device__ __forceinline__ void pack_rows(const float* ot, int ldo, int row0, int D, int b, int l, PackedQ pq) {
  const int wave = threadIdx.x >> 6, lane = threadIdx.x & 63, r = lane & 15, g = lane >> 4;
#pragma unroll
  for (int h = 0; h < 2; ++h) {
    if (h >= pq.ranges) break;
    const int KT = pq.kt[h];
    const int64_t per = (int64_t)D * KT * 16;                     // elements of one part of one block
    u32x4* p = reinterpret_cast<u32x4*>(pq.p + pq.offset[h]) + (int64_t)b * 2 * (per / 8);
    for (int q = wave; q < 2 * KT; q += 4) {
      const int c = q / KT, jt = q % KT, cg = row0 / 32 + c;
      if (32 * cg >= D) continue;
      const int col = 128 * h + 16 * jt + r;
      float x[8];
#pragma unroll
      for (int e = 0; e < 8; ++e) x[e] = col < l ? ot[(32 * c + 8 * g + e) * ldo + col] : 0.f;
      u32x4 hi, lo;
      split_operand(x, &hi, &lo);
      const int64_t at = ((int64_t)cg * KT + jt) * 64 + lane;
      p[at] = hi;
      p[per / 8 + at] = lo;
    }
  }
}

// ---------------------------------------------------------------------------
// Eigenvectors of H = L L^T by a one-sided (Hestenes) Jacobi SVD of the Cholesky factor L itself (l x l, float64),
// one workgroup per block: plane rotations on column pairs until all columns are orthogonal, with a round-robin
// ordering so that l/2 disjoint pairs are rotated concurrently.  L J_1 J_2 ... = U diag(sigma): the final columns,
// normalised, are the LEFT singular vectors of L, which are the eigenvectors of H -- so the rotations are never
// accumulated (half the work and half the storage of a Jacobi on L^T that tracks its right vectors), and working on
// the columns of L instead of those of L^T means diagonalising L^T L, which is one step of the Cholesky-LR iteration
// closer to diagonal than H = L L^T: fewer sweeps.
//   Lfac  in   [l x l] lower-triangular Cholesky factor of H = Y^T Y
//   Wout  out  [l x l] row-major, column r = eigenvector of H of rank r (descending eigenvalue)
//   sigma out  [k] leading singular values of Y = square roots of the eigenvalues
// Columns whose norm is at round-off level (a rank-deficient sketch, kept factorisable by the diagonal shift) are
// still orthogonalised relative to their own norm, so the normalised set stays orthonormal.
// ---------------------------------------------------------------------------
// x from the lane that the DPP control word selects (both halves of the double)
template <int CTRL>
__device__ __forceinline__ double dpp_move(double x) {
  const int lo = __double2loint(x), hi = __double2hiint(x);
  return __hiloint2double(__builtin_amdgcn_update_dpp(hi, hi, CTRL, 0xf, 0xf, true),
                          __builtin_amdgcn_update_dpp(lo, lo, CTRL, 0xf, 0xf, true));
}
// Sum over aligned groups of min(width, 16) lanes (width a power of two); every lane of a group gets the sum.
// Lane i adds lane i^1, then i^2 (quad permutations); once the quads are uniform, mirroring a half row (i <-> 7-i)
// and then a row (i <-> 15-i) brings in the other quads.
template <int WIDTH>
__device__ __forceinline__ double row_sum(double x) {
  if constexpr (WIDTH >= 2) x += dpp_move<0xB1>(x);    // quad_perm [1,0,3,2]
  if constexpr (WIDTH >= 4) x += dpp_move<0x4E>(x);    // quad_perm [2,3,0,1]
  if constexpr (WIDTH >= 8) x += dpp_move<0x141>(x);   // row_half_mirror
  if constexpr (WIDTH >= 16) x += dpp_move<0x140>(x);  // row_mirror
  return x;
}

// x and y from lane i ^ (8 S), S = 1, 2 or 4: rows of 16 lanes rotated by 8, then neighbouring rows or halves of the wave
// swapped.  v_permlane16_swap exchanges the odd rows of its first operand with the even rows of its second,
// v_permlane32_swap the upper half with the lower one: applied to a word of x and one of y and then to the same two in the other
// order, it moves both and leaves each in the other's register, so that a double costs two instructions and no copy.
template <int S>
__device__ __forceinline__ void xor_rows(double& x, double& y) {
  if constexpr (S == 1) {     // row_ror:8
    x = dpp_move<0x128>(x);
    y = dpp_move<0x128>(y);
  } else if constexpr (S == 2 || S == 4) {
    auto swap = [](uint32_t u, uint32_t v) {
      if constexpr (S == 2) {
        const auto r = __builtin_amdgcn_permlane16_swap(u, v, false, false);
        return __builtin_amdgcn_permlane16_swap(r[1], r[0], false, false);
      } else {
        const auto r = __builtin_amdgcn_permlane32_swap(u, v, false, false);
        return __builtin_amdgcn_permlane32_swap(r[1], r[0], false, false);
      }
    };
    const auto lo = swap((uint32_t)__double2loint(x), (uint32_t)__double2loint(y));
    const auto hi = swap((uint32_t)__double2hiint(x), (uint32_t)__double2hiint(y));
    x = __hiloint2double((int)hi[0], (int)lo[0]);
    y = __hiloint2double((int)hi[1], (int)lo[1]);
  } else {                    // several bits, one after the other
    if constexpr (S & 1) xor_rows<1>(x, y);
    if constexpr (S & 2) xor_rows<2>(x, y);
    if constexpr (S & 4) xor_rows<4>(x, y);
  }
}

// The rotation that makes two columns with squared norms al, be and inner product ga orthogonal: x' = cs x - sn y,
// y' = sn x + cs y.  False (and nothing set) when they are orthogonal to 1e-7 already (compared in squares, no sqrt): the
// outputs are float32, and a sweep that finds nothing above the threshold ends the iteration.  *big is set when the cosine of
// the angle between the columns was above 3.2e-5.
// The ANGLE only steers convergence, so tan(theta) = sign(z) / (|z| + sqrt(1 + z^2)) comes from the float32 reciprocal and
// square root of the hardware (each good to an ulp; the exact division and square root were a third of the dependent
// chain of a rotation).  cos and sin belong to exactly that tangent in float64: 1 / sqrt(1 + t^2) from the float32
// estimate (1e-7) and one step of third order.  jacobi_wave_kernel hands over norms that followed the rotations since their
// columns were loaded (al - t ga, be + t ga) and not sums over the elements.  For columns that are nearly parallel the error of
// t, some 3e-7 of be, can exceed the norm that is left or make it negative; the test below then rotates a pair that needs no
// rotation, or by a wrong angle.  That costs rotations and no accuracy: the rotation is orthogonal whatever its angle, such
// a pair sets *big, so that another sweep follows, and the norms are summed anew at every load and again for sigma.
__device__ __forceinline__ bool jacobi_angle(double al, double be, double ga, double* tt, double* cs, double* sn, int* big) {
  const double g2 = ga * ga, ab = al * be;
  if (!(g2 > 1e-14 * ab)) return false;
  const float z = (float)((be - al) * 0.5 * __builtin_amdgcn_rcp(ga));
  const float az = fabsf(z), am = fminf(az, 1e9f);     // the root is |z| to the last bit from there on (and z^2 may overflow)
  const float tf = __builtin_copysignf(__builtin_amdgcn_rcpf(az + fmaxf(__builtin_amdgcn_sqrtf(fmaf(am, am, 1.f)), az)), z);
  *tt = (double)tf;
  const double n2 = fma(*tt, *tt, 1.0);
  const double c0 = (double)__builtin_amdgcn_rsqf(fmaf(tf, tf, 1.f));
  const double e1 = fma(-(n2 * c0), c0, 1.0);
  *cs = fma(c0 * e1, fma(0.375, e1, 0.5), c0);
  *sn = *cs * *tt;
  if (g2 > 1e-9 * ab) *big = 1;
  return true;
}

// One plane rotation of the one-sided Jacobi on columns in LDS: the TP lanes of a pair (lane gl of TP, a compile-time
// power of two <= 16: with a run-time width every level of the sums below is a branch) make columns ap and aq (length l)
// orthogonal.  A lane handles exactly NE elements of a column, NE >= ceil(l / tp), so the element loops
// unroll with a fixed trip count, their LDS loads are issued together, and the elements stay in registers between
// the dot products and the rotation.  A rotation above the threshold of jacobi_angle sets *big (a flag in a register:
// the caller publishes it once per sweep).
template <int NE, int TP>
__device__ __forceinline__ void jacobi_rotate(double* ap, double* aq, int l, int gl, int* big) {
  static_assert(TP <= 16, "sums inside a row of 16 lanes");
  double al = 0.0, be = 0.0, ga = 0.0;
  double xs[NE], ys[NE];
#pragma unroll
  for (int e = 0; e < NE; ++e) {
    const int r = gl + e * TP;
    xs[e] = r < l ? ap[r] : 0.0;
    ys[e] = r < l ? aq[r] : 0.0;
  }
#pragma unroll
  for (int e = 0; e < NE; ++e) {
    al += xs[e] * xs[e]; be += ys[e] * ys[e]; ga += xs[e] * ys[e];
  }
  al = row_sum<TP>(al); be = row_sum<TP>(be); ga = row_sum<TP>(ga);
  double tt, cs, sn;
  if (jacobi_angle(al, be, ga, &tt, &cs, &sn, big)) {
#pragma unroll
    for (int e = 0; e < NE; ++e) {
      const int r = gl + e * TP;
      if (r < l) {
        ap[r] = cs * xs[e] - sn * ys[e];
        aq[r] = sn * xs[e] + cs * ys[e];
      }
    }
  }
}

// players p, q of pair `group` in step `step` of a round-robin over `le` players (le even): le - 1 steps pair
// everybody with everybody once
__device__ __forceinline__ void round_robin_pair(int le, int step, int group, int* p, int* q) {
  if (group == 0) { *p = le - 1; *q = step % (le - 1); }
  else { *p = (step + group) % (le - 1); *q = (step + (le - 1) - group) % (le - 1); }
}

// The same pairing followed step by step without divisions (a remainder by a run-time divisor costs about as many
// instructions as the rest of a rotation): start(le, group) gives the pair of step 0, next() that of the step after.
struct RoundRobin {
  int p, q, m;
  bool fixed;   // group 0 keeps player le - 1
  __device__ __forceinline__ void start(int le, int group) {
    m = le - 1;
    fixed = group == 0;
    p = fixed ? le - 1 : group;      // group <= le / 2 - 1 < m
    q = fixed ? 0 : m - group;
  }
  __device__ __forceinline__ void next() {
    if (!fixed) p = p + 1 == m ? 0 : p + 1;
    q = q + 1 == m ? 0 : q + 1;
  }
};

// Singular values, rank order and normalised columns from the orthogonal columns A (LDS, column stride la) of an
// l <= 138 Jacobi, for a workgroup of nt threads.  The squared norms are ranked by their bit patterns (the sign of a NaN
// removed): the order of the values, and a total one where features with an infinity or a NaN leave norms that compare
// with nothing, so that the ranks are a permutation and every entry of `order` that is read below has been written.
struct JacobiOrder { double nrm[138], inv[138]; int order[138]; };
__device__ __forceinline__ void jacobi_output(const double* A, int la, int l, int k, int nt, JacobiOrder& o, double* wo,
                                              float* sigma) {
  const int t = threadIdx.x;
  for (int j = t >> 3; j < l; j += nt / 8) {
    double s = 0.0;
    for (int r = t & 7; r < l; r += 8) s += A[j * la + r] * A[j * la + r];
    s = row_sum<8>(s);
    if ((t & 7) == 0) o.nrm[j] = fabs(s);
  }
  __syncthreads();
  for (int j = t; j < l; j += nt) {
    const double nj = o.nrm[j];
    const long long kj = __double_as_longlong(nj);
    int rank = 0;
#pragma unroll 8
    for (int i = 0; i < l; ++i) {
      const long long ki = __double_as_longlong(o.nrm[i]);
      rank += (ki > kj || (ki == kj && i < j)) ? 1 : 0;
    }
    if (rank < k) sigma[rank] = (float)sqrt(nj);
    o.order[rank] = j;
    o.inv[rank] = nj > 0.0 ? 1.0 / sqrt(nj) : 0.0;
  }
  __syncthreads();
  for (int i = t >> 6; i < l; i += nt >> 6)            // a row per wave: no division by a run-time length
    for (int r = t & 63; r < l; r += kWave) wo[i * l + r] = A[o.order[r] * la + i] * o.inv[r];
}

// Two blocks of eight columns in a wave's registers, 8 lanes per column: row g of the wave (lanes 8 g .. 8 g + 7) holds a column
// x of the first block and a column y of the second, elements gl + 8 e.  A column is its elements times a scale d (id = 1 / d), n
// its squared norm.  The rotation x <- cs (x - t y), y <- cs (y + t x) of the columns is, of the elements, x <- x - (t dy / dx) y and
// then, with the new x, y <- y + (t cs^2 dx / dy) x, and dx <- cs dx, dy <- dy / cs: two operations in place per pair of elements
// instead of four and copies.
template <int NE>
struct ColumnPairs {
  static_assert(NE % 2 == 0, "elements move by pairs");
  struct Scale { double n, d, id; };
  double x[NE], y[NE];
  Scale sx, sy;
  int big;
  static __device__ __forceinline__ Scale unit_scale(const double (&v)[NE]) {
    double n0 = 0.0, n1 = 0.0;
#pragma unroll
    for (int e = 0; e < NE; e += 2) { n0 = fma(v[e], v[e], n0); n1 = fma(v[e + 1], v[e + 1], n1); }
    return Scale{row_sum<8>(n0 + n1), 1.0, 1.0};
  }
  static __device__ __forceinline__ Scale load(double (&v)[NE], const double* p) {
#pragma unroll
    for (int e = 0; e < NE; ++e) v[e] = p[8 * e];
    return unit_scale(v);
  }
  static __device__ __forceinline__ void store(const double (&v)[NE], const Scale& s, double* p) {
#pragma unroll
    for (int e = 0; e < NE; ++e) p[8 * e] = v[e] * s.d;
  }
  // every row rotates its x with its y
  __device__ __forceinline__ void rotate() {
    double g0 = 0.0, g1 = 0.0;
#pragma unroll
    for (int e = 0; e < NE; e += 2) { g0 = fma(x[e], y[e], g0); g1 = fma(x[e + 1], y[e + 1], g1); }
    const double ga = row_sum<8>(g0 + g1) * (sx.d * sy.d);
    double tt, cs, sn;
    if (jacobi_angle(sx.n, sy.n, ga, &tt, &cs, &sn, &big)) {
      const double a = -tt * (sy.d * sx.id), c = (sn * cs) * (sx.d * sy.id), ics = cs * fma(tt, tt, 1.0);
#pragma unroll
      for (int e = 0; e < NE; ++e) {
        x[e] = fma(a, y[e], x[e]);
        y[e] = fma(c, x[e], y[e]);
      }
      sx = Scale{fma(-tt, ga, sx.n), sx.d * cs, sx.id * ics};
      sy = Scale{fma(tt, ga, sy.n), sy.d * ics, sy.id * cs};
    }
  }
  // columns (and scales) from the row with the exclusive-or of the number
  template <int S>
  static __device__ __forceinline__ void move(double (&v)[NE], Scale& s) {
#pragma unroll
    for (int e = 0; e < NE; e += 2) xor_rows<S>(v[e], v[e + 1]);
    double twin = s.id;
    xor_rows<S>(s.n, s.d);
    xor_rows<S>(s.id, twin);
  }
  template <int S>
  __device__ __forceinline__ void rotate_next() {
    move<S>(y, sy);
    rotate();
  }
  // every column of the first block with every one of the second; row g ends with the y of row g ^ 4
  __device__ __forceinline__ void rotate_across() {
    rotate();
    rotate_next<1>();      // rows of y now hold column g ^ 1
    rotate_next<2>();      // 3
    rotate_next<1>();      // 2
    rotate_next<4>();      // 6
    rotate_next<1>();      // 7
    rotate_next<2>();      // 5
    rotate_next<1>();      // 4
  }
  // x of the rows with bit S and y of the rows without it change places
  template <int S>
  __device__ __forceinline__ void exchange() {
    auto swap = [](double& u, double& v) {
      if constexpr (S == 1) {
        const bool odd = (threadIdx.x & 8) != 0;
        const double um = dpp_move<0x128>(u), vm = dpp_move<0x128>(v);
        u = odd ? vm : u;
        v = odd ? v : um;
      } else {
        auto word = [](uint32_t p, uint32_t q) {
          if constexpr (S == 2) return __builtin_amdgcn_permlane16_swap(p, q, false, false);
          else return __builtin_amdgcn_permlane32_swap(p, q, false, false);
        };
        const auto l = word((uint32_t)__double2loint(u), (uint32_t)__double2loint(v));
        const auto h = word((uint32_t)__double2hiint(u), (uint32_t)__double2hiint(v));
        u = __hiloint2double((int)h[0], (int)l[0]);
        v = __hiloint2double((int)h[1], (int)l[1]);
      }
    };
#pragma unroll
    for (int e = 0; e < NE; ++e) swap(x[e], y[e]);
    swap(sx.n, sy.n);
    swap(sx.d, sy.d);
    swap(sx.id, sy.id);
  }
  // The pairs inside both blocks side by side, in seven rounds: with the upper half of x and the lower one of y exchanged, rows
  // pair columns of the lower and upper half of the same block, and so on with quarters and eighths.  The x and y that start in
  // rows 0 .. 7 are left in the order of `inside_column`.
  __device__ __forceinline__ void rotate_inside() {
    exchange<4>();         // (x0 x1 x2 x3 | y0 ..), (x4 x5 x6 x7 | y4 ..)
    rotate();
    rotate_next<1>();
    rotate_next<2>();
    rotate_next<1>();      // second: (x6 x7 x4 x5 | ..)
    exchange<2>();         // (x0 x1 x6 x7 | ..), (x2 x3 x4 x5 | ..)
    rotate();
    rotate_next<1>();      // second: (x3 x2 x5 x4 | ..)
    exchange<1>();         // (x0 x3 x6 x5 | ..), (x1 x2 x7 x4 | ..)
    rotate();
    exchange<4>();         // (x0 x3 x6 x5 x1 x2 x7 x4), (y0 y3 y6 y5 y1 y2 y7 y4)
  }
  static __device__ __forceinline__ int inside_column(int g) { return (0x47215630 >> (4 * g)) & 7; }
};

// l <= 128, one workgroup per block.  The columns form blocks of 8, and a wave takes two blocks at a time into registers: 8
// lanes per column (ColumnPairs).  Eight rounds pair every column of the first with every one of the second, the second block moving
// by exclusive-or of the row number (in Gray code order, one bit per round) through lane permutations: no LDS, no
// barrier.  A round-robin over the blocks, LDS in between, pairs every block with every other once per sweep; in its first
// step the columns inside each block are paired too.  Per sweep of 64 columns that is 7 trips through LDS and 7
// barriers instead of 63 -- with a trip per rotation the LDS reads, writes and the barrier were half of a round at 64
// columns and the LDS bandwidth bound 128 columns.  The squared norms are formed once per trip and follow the rotations
// (al - t ga, be + t ga), so that a rotation sums one inner product over the lanes.
// What bounds it: the dependent chain of a rotation at 64 columns (one wave per SIMD), the number of instructions at 128 (two):
// 16 multiply-adds for an inner product, 32 to rotate, 32 to 40 to move 16 elements, 45 for sums and angle, each 5 clocks.
// Measured inside the fit of one block of 4608 x 3072 bf16, rank 32: 106 us (64 columns); of 18432 x 3072 float32, rank 64:
// 528 us (128 columns); against 116 and 570 us with 14 rounds for the pairs inside blocks, 154 and 762 us also with four
// operations per rotated pair of elements, copies and selections where columns move and a branch in the angle, 254 and 1106 us with 16 lanes per pair, every rotation from and to LDS.
template <int NE>
__global__ __launch_bounds__(512) void jacobi_wave_kernel(const double* __restrict__ Lfac, double* Wout, float* sigma, int l,
                                                          int k, const double* fro_acc, float* fro2, int max_sweeps,
                                                          int32_t* info) {
  constexpr int la = 8 * NE + 8;        // 8 columns that lie 8 doubles past a multiple of 32 apart: no bank conflicts
  extern __shared__ double A[];         // [nbe 8][la], column-major, zeros beyond l
  __shared__ JacobiOrder ord;
  __shared__ int s_big[2];
  const int b = blockIdx.x, t = threadIdx.x, nt = blockDim.x, wave = t >> 6, g = (t & 63) >> 3, gl = t & 7;
  const double* Lf = Lfac + (int64_t)b * l * l;
  const int nbe = nt / 32;              // blocks of 8 columns, even: two per wave
  for (int idx = t; idx < 8 * nbe * 8 * NE; idx += nt) {
    const int c = idx / (8 * NE), r = idx % (8 * NE);
    if (r >= l || c >= l || c > r) A[c * la + r] = 0.0;
  }
  for (int r = wave; r < l; r += nt >> 6)
    for (int c = t & 63; c <= r; c += kWave) A[c * la + r] = Lf[r * l + c];   // A = L
  if (t == 0 && fro2) fro2[b] = (float)fro_acc[b];
  if (t == 0) s_big[0] = 0;
  __syncthreads();

  ColumnPairs<NE> cp;
  // Up to 16 columns (NE = 2) most of a block may be zeros: there, pairs inside a block are looked at one by one (3 columns:
  // 15.6 -> 6.9 us with 14 rounds for both blocks).
  constexpr bool kFull = NE > 2;
  using Scale = typename ColumnPairs<NE>::Scale;
  // rotate column g with column g ^ S of the same block: both rows form the rotation, each keeps its own column
  auto rotate_inside = [&](auto s, double (&xv)[NE], Scale& sv) {
    constexpr int S = decltype(s)::value;
    constexpr int kTop = S >= 4 ? 4 : (S >= 2 ? 2 : 1);
    const bool lower = (g & kTop) == 0;                 // which of the two plays x: they differ in the highest bit of S
    double pv[NE], g0 = 0.0, g1 = 0.0;
    Scale sp = sv;
#pragma unroll
    for (int e = 0; e < NE; ++e) pv[e] = xv[e];
    ColumnPairs<NE>::template move<S>(pv, sp);
#pragma unroll
    for (int e = 0; e < NE; e += 2) { g0 = fma(xv[e], pv[e], g0); g1 = fma(xv[e + 1], pv[e + 1], g1); }
    const double ga = row_sum<8>(g0 + g1) * (sv.d * sp.d);
    double tt, cs, sn;
    if (jacobi_angle(lower ? sv.n : sp.n, lower ? sp.n : sv.n, ga, &tt, &cs, &sn, &cp.big)) {
      if (lower) tt = -tt;
      const double a = tt * (sp.d * sv.id), ics = cs * fma(tt, tt, 1.0);
#pragma unroll
      for (int e = 0; e < NE; ++e) xv[e] = fma(a, pv[e], xv[e]);
      sv = Scale{fma(tt, ga, sv.n), sv.d * cs, sv.id * ics};
    }
  };
  auto rotate_first_inside = [&](int n, double (&xv)[NE], Scale& sv) {      // every pair of the block's first n columns
    if (n > 1) rotate_inside(std::integral_constant<int, 1>{}, xv, sv);
    if (n > 2) { rotate_inside(std::integral_constant<int, 2>{}, xv, sv); rotate_inside(std::integral_constant<int, 3>{}, xv, sv); }
    if (n > 4) {
      rotate_inside(std::integral_constant<int, 4>{}, xv, sv);
      rotate_inside(std::integral_constant<int, 5>{}, xv, sv);
      rotate_inside(std::integral_constant<int, 6>{}, xv, sv);
      rotate_inside(std::integral_constant<int, 7>{}, xv, sv);
    }
  };

  bool converged = false;
  for (int sweep = 0; sweep < max_sweeps; ++sweep) {
    cp.big = 0;
    RoundRobin rr;
    rr.start(nbe, wave);
    for (int step = 0; step < nbe - 1; ++step) {
      double* bx = A + 8 * rr.p * la + gl;
      double* by = A + 8 * rr.q * la + gl;
      int cx = g, cy = g;
      cp.sx = cp.load(cp.x, bx + cx * la);
      cp.sy = cp.load(cp.y, by + cy * la);
      if (step == 0) {
        if constexpr (kFull) {
          cp.rotate_inside();
          cx = cp.inside_column(g);
          cy = cx;
        } else {
          rotate_first_inside(l - 8 * rr.p, cp.x, cp.sx);
          rotate_first_inside(l - 8 * rr.q, cp.y, cp.sy);
        }
      }
      if (kFull || (8 * rr.p < l && 8 * rr.q < l)) {   // both blocks have columns (l is the same for the whole wave)
        cp.rotate_across();
        cy = kFull && step == 0 ? cp.inside_column(g ^ 4) : g ^ 4;
      }
      cp.store(cp.x, cp.sx, bx + cx * la);
      cp.store(cp.y, cp.sy, by + cy * la);
      rr.next();
      __syncthreads();
    }
    if (cp.big && gl == 0) atomicOr(&s_big[sweep & 1], 1);
    if (t == 0) s_big[(sweep + 1) & 1] = 0;
    __syncthreads();
    // Done when a sweep rotated nothing, or only pairs whose cosine was below 3.2e-5: cyclic Jacobi converges
    // quadratically, so what such a sweep leaves behind is of the order of the square of that, far below the 1e-7
    // threshold, and the sweep that would merely confirm it (a seventh of the kernel's time) is not run.
    if (s_big[sweep & 1] == 0) { converged = true; break; }
  }
  if (t == 0 && !converged && info) atomicOr(info + b, SVDC_FIT_JACOBI_CAPPED);
  jacobi_output(A, la, l, k, nt, ord, Wout + (int64_t)b * l * l, sigma + (int64_t)b * k);
}

// 128 < l <= 138: the whole matrix still fits the LDS, but not padded; every rotation from and to LDS.
template <int NE, int NT, int TP>
__global__ __launch_bounds__(NT) void jacobi_kernel(const double* __restrict__ Lfac, double* Wout, float* sigma,
                                                    int l, int k, const double* fro_acc, float* fro2,
                                                    int max_sweeps, int32_t* info) {
  extern __shared__ double A[];         // column-major
  __shared__ JacobiOrder ord;
  __shared__ int s_big[2];
  const int b = blockIdx.x, t = threadIdx.x;
  const double* Lf = Lfac + (int64_t)b * l * l;
  const int la = l | 1;                 // odd column stride: concurrently rotated columns spread over the LDS banks
  for (int idx = t; idx < l * l; idx += NT) {
    const int r = idx / l, c = idx % l;
    A[c * la + r] = (c <= r) ? Lf[idx] : 0.0;   // A = L
  }
  if (t == 0 && fro2) fro2[b] = (float)fro_acc[b];
  if (t == 0) s_big[0] = 0;
  __syncthreads();
  const int le = (l + 1) & ~1;         // players in the round-robin (one dummy if l is odd)
  const int npairs = le / 2;           // <= 69; the host picks TP with TP * npairs <= NT
  const int group = t / TP, gl = t % TP;
  const bool active = group < npairs;
  bool converged = false;
  for (int sweep = 0; sweep < max_sweeps; ++sweep) {
    int my_big = 0;
    RoundRobin rr;
    rr.start(le, active ? group : 0);
    for (int step = 0; step < le - 1; ++step) {
      if (active && rr.p < l && rr.q < l) jacobi_rotate<NE, TP>(A + rr.p * la, A + rr.q * la, l, gl, &my_big);
      rr.next();
      __syncthreads();
    }
    if (my_big && gl == 0) atomicOr(&s_big[sweep & 1], 1);
    if (t == 0) s_big[(sweep + 1) & 1] = 0;
    __syncthreads();
    if (s_big[sweep & 1] == 0) { converged = true; break; }
  }
  if (t == 0 && !converged && info) atomicOr(info + b, SVDC_FIT_JACOBI_CAPPED);
  jacobi_output(A, la, l, k, NT, ord, Wout + (int64_t)b * l * l, sigma + (int64_t)b * k);
}

// ---------------------------------------------------------------------------
// The same Jacobi for 138 < l <= 256, where the matrix (l x l float64) no longer fits the LDS of one workgroup: by
// column blocks.  The columns form nb = ceil(l / 32) blocks; a round-robin over the blocks pairs every block with
// every other once per sweep, and the pairs of one round-robin step are disjoint, so one launch handles a step with
// one workgroup per block pair: it brings the pair's 64 columns into LDS, rotates every pair across the two blocks
// (four waves on 8-column blocks in registers, ColumnPairs, 32 rounds; in the first step of a sweep every pair among the 64
// columns, 63 rounds, which covers the pairs inside the blocks) and writes them back: each pair of columns once per sweep.
// 192 columns, 9 sweeps: 1.1 ms, against 2.3 with 16 lanes per pair and every rotation from and to LDS; half of the rest of
// the time were divisions by l where columns are loaded and stored, now a column per wave.
// The working matrix A lives in global memory column by column (A[c * l + r]); the very first launch reads its
// columns from the Cholesky factor instead.  Convergence is tracked per block in three rotating counters cnt[b][0..2]: the launches of sweep s count
// the rotations with a cosine above 3.2e-5 in cnt[s % 3], return at once when cnt[(s - 1) % 3] is zero (the previous
// sweep found nothing: converged, and it stays so because nothing is counted any more), and the first launch of the
// sweep clears cnt[(s + 1) % 3] for the next one.  jacobi_finish_kernel then sorts and normalises.
// ---------------------------------------------------------------------------
constexpr int kJbCols = 32, kJbThreads = 256;

template <int NE>
__global__ __launch_bounds__(kJbThreads) void jacobi_block_kernel(const double* __restrict__ Lfac, double* gA, int l, int step,
                                                                  int sweep, int first, int* cnt) {
  extern __shared__ double A[];                         // [NC][la], column-major, zeros beyond l
  __shared__ int s_big;
  constexpr int NT = kJbThreads, NC = 2 * kJbCols, NB = NC / 8, la = 8 * NE + 8;
  static_assert(NB == 2 * (NT / kWave), "a wave per pair of 8-column blocks");
  const int b = blockIdx.y, t = threadIdx.x, wave = t >> 6, g = (t & 63) >> 3, gl = t & 7;
  int* c3 = cnt + 4 * b;
  if (blockIdx.x == 0 && step == 0 && t == 0) c3[(sweep + 1) % 3] = 0;
  if (sweep > 0 && c3[(sweep + 2) % 3] == 0) return;   // uniform over the workgroup
  const int nb = (l + kJbCols - 1) / kJbCols, nbe = (nb + 1) & ~1;
  int bi, bj;
  round_robin_pair(nbe, step, blockIdx.x, &bi, &bj);
  double* ga = gA + (int64_t)b * l * l;
  // global column of local column c (>= l: none)
  auto gcol = [&](int c) { const int blk = c < kJbCols ? bi : bj; return blk < nb ? blk * kJbCols + (c & (kJbCols - 1)) : l; };
  if (first) {
    const double* Lf = Lfac + (int64_t)b * l * l;
    for (int idx = t; idx < 8 * NE * NC; idx += NT) {
      const int r = idx / NC, c = idx % NC, gc = gcol(c);
      A[c * la + r] = r < l && gc <= r ? Lf[(int64_t)r * l + gc] : 0.0;
    }
  } else {
    const int lane = t & 63;
#pragma unroll 4
    for (int c = wave; c < NC; c += NT / kWave) {       // a column per wave: no division by a run-time length
      const int gc = gcol(c);
      const double* col = ga + (int64_t)min(gc, l - 1) * l;
      double v[(8 * NE + 63) / 64];
#pragma unroll
      for (int i = 0; i < (8 * NE + 63) / 64; ++i) v[i] = col[min(lane + 64 * i, l - 1)];
#pragma unroll
      for (int i = 0; i < (8 * NE + 63) / 64; ++i) {
        const int r = lane + 64 * i;
        if (8 * NE % 64 == 0 || r < 8 * NE) A[c * la + r] = r < l && gc < l ? v[i] : 0.0;
      }
    }
  }
  if (t == 0) s_big = 0;
  __syncthreads();
  ColumnPairs<NE> cp;
  cp.big = 0;
  auto block = [&](int q) { return A + 8 * q * la + gl; };
  if (step == 0) {
    // first step of a sweep: every pair among the 64 columns, i.e. also the pairs inside each block (every block is
    // in exactly one pair of step 0)
    RoundRobin rr;
    rr.start(NB, wave);
    for (int st = 0; st < NB - 1; ++st) {
      double* bx = block(rr.p);
      double* by = block(rr.q);
      int cx = g, cy = g ^ 4;
      cp.sx = cp.load(cp.x, bx + g * la);
      cp.sy = cp.load(cp.y, by + g * la);
      if (st == 0) {
        cp.rotate_inside();
        cx = cp.inside_column(g);
        cy = cp.inside_column(g ^ 4);
      }
      cp.rotate_across();
      cp.store(cp.x, cp.sx, bx + cx * la);
      cp.store(cp.y, cp.sy, by + cy * la);
      rr.next();
      __syncthreads();
    }
  } else {
    // later steps: only the pairs across the two blocks; a wave keeps its columns of the first one
    cp.sx = cp.load(cp.x, block(wave) + g * la);
    for (int st = 0; st < NB / 2; ++st) {
      double* by = block(NB / 2 + ((wave + st) & (NB / 2 - 1)));
      cp.sy = cp.load(cp.y, by + g * la);
      cp.rotate_across();
      cp.store(cp.y, cp.sy, by + (g ^ 4) * la);
      __syncthreads();
    }
    cp.store(cp.x, cp.sx, block(wave) + g * la);
    __syncthreads();
  }
  if (cp.big && gl == 0) atomicAdd(&s_big, 1);
  __syncthreads();
#pragma unroll 4
  for (int c = wave; c < NC; c += NT / kWave) {
    const int gc = gcol(c);
    if (gc >= l) continue;
#pragma unroll
    for (int i = 0; i < (8 * NE + 63) / 64; ++i) {
      const int r = (t & 63) + 64 * i;
      if (r < l) ga[(int64_t)gc * l + r] = A[c * la + r];
    }
  }
  if (t == 0 && s_big > 0) atomicAdd(&c3[sweep % 3], s_big);
}

// Column norms -> singular values, rank order, normalised eigenvectors (same outputs as jacobi_kernel), one
// workgroup per block, one wave per column at a time.
__global__ __launch_bounds__(1024) void jacobi_finish_kernel(const double* __restrict__ gA, double* Wout, float* sigma,
                                                            int l, int k, const double* fro_acc, float* fro2,
                                                            int max_sweeps, const int* cnt, int32_t* info) {
  __shared__ double nrm[256];
  const int b = blockIdx.x, t = threadIdx.x, wave = t >> 6, lane = t & 63;
  const double* A = gA + (int64_t)b * l * l;
  if (t == 0) {
    if (fro2) fro2[b] = (float)fro_acc[b];
    // the last sweep still found rotations to do
    if (info && cnt[4 * b + (max_sweeps - 1) % 3] != 0) atomicOr(info + b, SVDC_FIT_JACOBI_CAPPED);
  }
  for (int j = wave; j < l; j += 16) {
    double s = 0.0;
    for (int r = lane; r < l; r += kWave) s += A[(int64_t)j * l + r] * A[(int64_t)j * l + r];
    s = wave_sum(s);
    if (lane == 0) nrm[j] = fabs(s);
  }
  __syncthreads();
  double* wo = Wout + (int64_t)b * l * l;
  for (int j = wave; j < l; j += 16) {
    const double nj = nrm[j];
    const long long kj = __double_as_longlong(nj);       // ranked by bit pattern, as in jacobi_output
    int rank = 0;
    for (int i = lane; i < l; i += kWave) {
      const long long ki = __double_as_longlong(nrm[i]);
      rank += (ki > kj || (ki == kj && i < j)) ? 1 : 0;
    }
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) rank += __shfl_xor(rank, o, kWave);
    if (lane == 0 && rank < k) sigma[(int64_t)b * k + rank] = (float)sqrt(nj);
    const double inv = nj > 0.0 ? 1.0 / sqrt(nj) : 0.0;
    for (int i = lane; i < l; i += kWave) wo[(int64_t)i * l + rank] = A[(int64_t)j * l + i] * inv;
  }
}

// ---------------------------------------------------------------------------
// sum of squares of F[b] in float64 (||F||_F^2 for the energy rule, Eq. 6)
// ---------------------------------------------------------------------------
// Eight channels per lane and load, four loads in flight; a workgroup takes every gridDim.x-th group of 256 pieces.
template <typename T>
__global__ __launch_bounds__(256) void sumsq_kernel(const T* __restrict__ F, double* acc, int N, int D,
                                                    int64_t ldf, int64_t bstride) {
  __shared__ double part[4];
  const int b = blockIdx.y, t = threadIdx.x, per_row = (D + 7) / 8;
  const T* f = F + (int64_t)b * bstride;
  const int64_t total = (int64_t)N * per_row, step = (int64_t)gridDim.x * 256;
  double s0 = 0.0, s1 = 0.0;
  for (int64_t i = (int64_t)blockIdx.x * 256 + t; i < total; i += 4 * step) {
    Piece<T> p[4];
#pragma unroll
    for (int u = 0; u < 4; ++u) {
      const int64_t at = min(i + u * step, total - 1), row = at / per_row;
      p[u].load(f + row * ldf, i + u * step < total ? 8 * (int)(at - row * per_row) : D, D);
    }
#pragma unroll
    for (int u = 0; u < 4; ++u)
#pragma unroll
      for (int e = 0; e < 8; e += 2) {
        const double x = (double)p[u].get(e), y = (double)p[u].get(e + 1);
        s0 = fma(x, x, s0);
        s1 = fma(y, y, s1);
      }
  }
  const double s = wave_sum(s0 + s1);
  if ((t & 63) == 0) part[t >> 6] = s;
  __syncthreads();
  if (t == 0) atomicAdd(&acc[b], part[0] + part[1] + part[2] + part[3]);
}

// ---------------------------------------------------------------------------
// host orchestration
// ---------------------------------------------------------------------------
static size_t align_up(size_t x, size_t a) { return (x + a - 1) / a * a; }

constexpr size_t kLdsBudget = 150 * 1024;  // dynamic LDS a single workgroup may take (160 KB per CU)
constexpr int kGramSlices = 16;   // row slices whose partial Gram matrices are summed in a fixed order

bool make_fit_plan(const svdc_shape& s, const svdc_fit_params* p, FitPlan* plan) {
  int pp = p ? p->oversample_p : 0;
  int q = p ? p->power_iters_q : 0;
  if (pp < -1 || q < -1 || pp > 4096 || q > 64) return false;
  if (pp == 0) pp = s.k;
  if (pp == -1) pp = 0;
  if (q == 0) q = (s.dtype == SVDC_BF16) ? 3 : 5;
  if (q == -1) q = 0;
  int l = s.k + pp;
  l = std::min(l, std::min(s.N, s.D));
  l = std::min(l, 256);
  if (l < s.k) return false;  // k > 256 is not supported by the fit
  plan->l = l;
  plan->q = q;
  plan->seed = p ? p->seed : 0;
  const int sweeps = p ? p->jacobi_max_sweeps : 0;
  if (sweeps < 0 || sweeps > 1000) return false;
  // default cap: 40 sweeps; 20 for the Jacobi by column blocks (l > 138), which takes 8-9 and whose launches are
  // issued up to the cap (those after convergence return at once, but are not free)
  plan->max_sweeps = sweeps == 0 ? ((size_t)l * (l + 1) * sizeof(double) <= kLdsBudget ? 40 : 20) : sweeps;
  size_t off = 0;
  const size_t B = s.B;
  plan->off_Q = off; off = align_up(off + B * s.D * l * sizeof(float), 256);
  plan->off_Z = off; off = align_up(off + B * s.D * l * sizeof(float), 256);
  // Y as float32 rows; the matrix-core path also keeps its packed bf16 form there between a projection and the
  // back-projection that follows (never both at once)
  size_t y_bytes = B * (size_t)s.N * l * sizeof(float);
  if (fit_mfma_supported(s, l)) y_bytes = std::max(y_bytes, fit_mfma_packed_y_bytes(s, l, 1));
  plan->off_Y = off; off = align_up(off + y_bytes, 256);
  plan->off_G = off; off = align_up(off + B * l * l * sizeof(double), 256);
  plan->off_Gp = off; off = align_up(off + B * kGramSlices * (size_t)l * l * sizeof(double), 256);
  plan->off_M = off; off = align_up(off + B * l * l * sizeof(double), 256);
  plan->off_W = off; off = align_up(off + B * l * l * sizeof(double), 256);   // Jacobi matrix when l > 138
  // ||F||_F^2 accumulators (B doubles) followed by the status words (B int32, see svdcache_fit_status_offset)
  plan->off_misc = off; off = align_up(off + B * sizeof(double), 256);
  plan->off_info = off; off = align_up(off + B * sizeof(int32_t), 256);
  // convergence counters of the Jacobi by column blocks (4 int32 per block); cleared together with the two above
  plan->off_jcnt = off; off = align_up(off + B * 4 * sizeof(int32_t), 256);
  plan->mfma = fit_mfma_supported(s, l);
  plan->off_Qp = off;
  if (plan->mfma) off = align_up(off + fit_mfma_packed_q_bytes(s, l), 256);
  plan->total = off;
  return true;
}

namespace {


int32_t set_dyn_lds(const void* fn, size_t bytes) {
  if (bytes <= 48 * 1024) return SVDC_OK;
  return hipFuncSetAttribute(fn, hipFuncAttributeMaxDynamicSharedMemorySize, (int)bytes) == hipSuccess
             ? SVDC_OK : SVDC_E_HIP;
}

void zero_f64(double* p, int64_t n, hipStream_t st) {
  fill_zero_kernel<<<(unsigned)((n + 255) / 256), 256, 0, st>>>(p, n);
}
void zero_f32(float* p, int64_t n, hipStream_t st) {
  fill_zero_f32_kernel<<<(unsigned)((n + 255) / 256), 256, 0, st>>>(p, n);
}

template <typename T>
void gemm_fq(const svdc_shape& s, int l, const T* F, const float* Q, float* Y, hipStream_t st) {
  auto launch = [&](auto kernel, int rows, int cols) {
    kernel<<<dim3((s.N + rows - 1) / rows, (l + cols - 1) / cols, s.B), 64 * kFitWaves, 0, st>>>(F, Q, Y, s.N, s.D, l, s.ldf,
                                                                                                s.block_stride);
  };
  // 128 rows per workgroup read Q once for eight tiles; 32 (four waves on the same rows) while those would be fewer than two
  // workgroups per compute unit, 16 while even those of 32 would be
  auto by_rows = [&](auto kt) {
    constexpr int KT = decltype(kt)::value;
    const int64_t tiles = (int64_t)((s.N + 15) / 16) * ((l + 16 * KT - 1) / (16 * KT)) * s.B, cus = num_compute_units();
    if (tiles >= 16 * cus) launch(fit_rows_general_kernel<T, KT, 2, 1>, 128, 16 * KT);
    else if (tiles >= 4 * cus) launch(fit_rows_general_kernel<T, KT, 2, kFitWaves>, 32, 16 * KT);
    else launch(fit_rows_general_kernel<T, KT, 1, kFitWaves>, 16, 16 * KT);
  };
  if (l <= 16) by_rows(std::integral_constant<int, 1>{});
  else if (l <= 32) by_rows(std::integral_constant<int, 2>{});
  else by_rows(std::integral_constant<int, 4>{});
}
template <typename T>
void gemm_fty(const svdc_shape& s, int l, const T* F, const float* Y, float* Z, hipStream_t st) {
  auto launch = [&](auto kernel, int kt) {
    const int slabs = (s.D + 127) / 128, cols = (l + 16 * kt - 1) / (16 * kt);
    // shares of the tokens: two workgroups per compute unit, at least 64 tokens each
    const int64_t want = std::max<int64_t>(1, 2 * (int64_t)num_compute_units() / ((int64_t)slabs * cols * s.B));
    const int share = (int)std::max<int64_t>(64, (((s.N + want - 1) / want) + 15) / 16 * 16), nshare = (s.N + share - 1) / share;
    if (nshare > 1) zero_f32(Z, (int64_t)s.B * s.D * l, st);
    kernel<<<dim3(slabs, cols, s.B * nshare), 64 * kFitWaves, 0, st>>>(F, Y, Z, s.N, s.D, l, s.ldf, s.block_stride, share, nshare);
  };
  if (l <= 16) launch(fit_cols_general_kernel<T, 1>, 1);
  else if (l <= 32) launch(fit_cols_general_kernel<T, 2>, 2);
  else launch(fit_cols_general_kernel<T, 4>, 4);
}

// Scratch for partial Gram matrices: areas of float64 values.
struct GramScratch { double* p[3]; int64_t doubles[3]; };

void gram(const float* A, double* G, GramScratch sc, int B, int rows, int l, hipStream_t st) {
  const int ntile = (l + 63) / 64, tiles = ntile * (ntile + 1) / 2;
  const int64_t ll = (int64_t)l * l;
  const int64_t held[3] = {sc.doubles[0] / ll, sc.doubles[1] / ll, sc.doubles[2] / ll};
  const int rows_per_slice = gram_slice_rows(rows, l, (int64_t)tiles * B, (held[0] + held[1] + held[2]) / B, num_compute_units());
  const GramParts parts{{sc.p[0], sc.p[1], sc.p[2]}, {held[0], held[0] + held[1]}};
  const int nslice = (rows + rows_per_slice - 1) / rows_per_slice;
  const dim3 grid(nslice, tiles, B);
  if (l <= 64) gram_f64_kernel<true><<<grid, 256, 0, st>>>(A, parts, rows, l, rows_per_slice);
  else gram_f64_kernel<false><<<grid, 256, 0, st>>>(A, parts, rows, l, rows_per_slice);
  gram_reduce_kernel<<<dim3((unsigned)((ll + 63) / 64), B), 256, 0, st>>>(parts, G, nslice, l);
}

// Cholesky factor of G + shift I in place, l <= 256: L in the lower triangle; for l > 64 the strict upper triangle
// holds L^T outside the 64 x 64 diagonal blocks (whose upper halves are zeroed).  M (block stride l * l doubles)
// receives the transposed inverses of the diagonal blocks: row stride l for the only one of l <= 64, otherwise 64 and
// 64 * 64 doubles apart; with l > 128 its last entry carries the shift from the first block to the later ones.
// want_inv = false (the factor is all that is asked for): the inverses are not formed.
void chol_factor(double* G, int B, int l, int32_t* info, hipStream_t st, double* M, bool want_inv) {
  const int64_t ll = (int64_t)l * l;
  constexpr int H = kCholBlock;
  auto factor = [&](auto kernel, int tiles, int c0, int w, double* slot, bool inverse) {
    kernel<<<B, tiles == 1 ? 64 : 128 * tiles, 0, st>>>(G, l, c0, w, M + (int64_t)(c0 / H) * H * H, ll, l <= H ? l : H, inverse ? 1 : 0, slot, ll,
                                     1e-14, info);
  };
  if (l <= 16) return factor(chol_tiles_kernel<1>, 1, 0, l, nullptr, want_inv);
  if (l <= H) return factor(chol_tiles_kernel<4>, 4, 0, l, nullptr, want_inv);
  if (l <= 2 * H) return factor(chol_tiles_kernel<8>, 8, 0, l, nullptr, want_inv);
  for (int c0 = 0; c0 < l; c0 += H) {
    const int w = std::min(H, l - c0);
    const bool last = c0 + w >= l;
    factor(chol_tiles_kernel<4>, 4, c0, w, M + ll - 1, want_inv);
    if (!last) chol_panel_kernel<<<dim3((l - c0 - w + H - 1) / H, B), 256, 0, st>>>(G, l, c0);
  }
}

// Out[rows x m] = In[rows x l] * M[l x m]
void rows_times_small(const float* In, const double* M, float* Out, int B, int rows, int l, int m, int ldm,
                      hipStream_t st) {
  dim3 grid((rows + 63) / 64, (m + 63) / 64, B);
  rows_times_small_kernel<<<grid, 256, 0, st>>>(In, M, Out, rows, l, m, ldm);
}

// Out = In * L^-T with L and the inverses of its diagonal blocks in G and M (chol_factor)
int32_t apply_factor(float* In, float* out, PackedQ pq, const double* G, const double* M, int B, int rows, int l,
                     bool zero_in, hipStream_t st) {
  constexpr int H = kCholBlock;
  const int nb = (l + H - 1) / H;
  const size_t lds = (size_t)H * ((l <= 16 ? 16 : nb * H) + 4) * sizeof(float) + (nb > 1 ? (size_t)H * (H + 2) * sizeof(double) : 0);
  const dim3 grid((rows + H - 1) / H, B);
  auto launch = [&](auto kernel) -> int32_t {
    if (set_dyn_lds((const void*)kernel, lds) != SVDC_OK) return SVDC_E_HIP;
    kernel<<<grid, 256, lds, st>>>(In, G, M, (int64_t)l * l, out, pq, rows, l, zero_in ? 1 : 0);
    return SVDC_OK;
  };
  if (l <= 16) return launch(apply_factor_kernel<1>);
  return nb == 1 ? launch(apply_factor_kernel<4>) : launch(apply_factor_kernel<0>);
}

// Orthonormalise the columns of Zin by CholeskyQR (Gram matrix, Cholesky factor and products with it in float64).
// One pass is accurate to about eps32 * cond(Zin), enough to keep the power iteration well conditioned: the result leaves
// as the projection's operand words where there is a packed form (pq.p), else as float32 rows in Qout.  two_pass repeats
// the step on the result (CholeskyQR2), giving orthonormality at float32 round-off; the result is then back in Zin, as
// float32 rows, and in the packed form.
int32_t orth(float* Zin, float* Qout, double* G, GramScratch sc, double* M, int B, int rows, int l, bool two_pass,
             PackedQ pq, bool zero_in, int32_t* info, hipStream_t st) {
  gram(Zin, G, sc, B, rows, l, st);
  chol_factor(G, B, l, info, st, M, true);
  const PackedQ none{};
  if (!two_pass) return apply_factor(Zin, pq.p ? nullptr : Qout, pq, G, M, B, rows, l, zero_in, st);
  if (apply_factor(Zin, Qout, none, G, M, B, rows, l, false, st) != SVDC_OK) return SVDC_E_HIP;
  // the second pass factors a matrix that is already orthonormal to float32 round-off: only the first one can
  // meet a dependent column
  gram(Qout, G, sc, B, rows, l, st);
  chol_factor(G, B, l, nullptr, st, M, true);
  return apply_factor(Qout, Zin, pq, G, M, B, rows, l, false, st);
}

template <typename T>
int32_t run_fit_typed(const svdc_shape& s, const FitPlan& pl, const T* F, float* V, float* sigma, float* fro2,
                      char* ws, hipStream_t st) {
  const int l = pl.l, B = s.B;
  float* Q = (float*)(ws + pl.off_Q);
  float* Z = (float*)(ws + pl.off_Z);
  float* Y = (float*)(ws + pl.off_Y);
  double* G = (double*)(ws + pl.off_G);
  double* Gp = (double*)(ws + pl.off_Gp);
  double* M = (double*)(ws + pl.off_M);
  double* Wg = (double*)(ws + pl.off_W);
  double* misc = (double*)(ws + pl.off_misc);
  int32_t* info = (int32_t*)(ws + pl.off_info);

  const int64_t nq = (int64_t)B * s.D * l;
  // fro accumulators, status words and Jacobi counters are adjacent 256-byte aligned areas: one fill clears them all
  const int64_t nmisc = (int64_t)((pl.off_jcnt - pl.off_misc) + align_up((size_t)B * 4 * sizeof(int32_t), 8)) / 8;
  void* Qp = ws + pl.off_Qp;
  // Partial Gram matrices go into their own area, into whichever of Y and Z is not in use and into the operand words of Q, which the
  // last product has read and apply_factor writes again.
  auto scratch = [&](void* other, int64_t rows) {
    return GramScratch{{(double*)other, Gp, (double*)Qp},
                       {(int64_t)B * rows * l / 2, (int64_t)B * kGramSlices * l * l, (int64_t)((pl.total - pl.off_Qp) / sizeof(double))}};
  };
  const PackedQ pq = pl.mfma ? fit_mfma_packed_q(s, l, Qp) : PackedQ{};
  // Between the two products Y has its packed form, which for float32 features is in two parts as large as the float32 rows
  // themselves, up to the padding of N and l: it may run on into the Gram matrices' areas, not in use at that time, and
  // stays float32 rows where even that is too small.
  constexpr bool kF32 = std::is_same<T, float>::value;
  void* Yp = kF32 && fit_mfma_packed_y_bytes(s, l, 2) > pl.off_M - pl.off_Y ? nullptr : (void*)Y;
  // several row groups accumulate Z with atomics: it has to be clear beforehand
  const bool zero_z = pl.mfma && fit_mfma_backproject_accumulates(s, l, Yp != nullptr);
  bool z_clear = false;
  // With power iterations the Gaussian test matrix (D x l) is used as it is: its columns are well conditioned
  // and every product F^T F Q is re-orthonormalised afterwards.  With none, the sketch is Z = F^T Omega with a
  // Gaussian Omega (N x l) -- the plain randomized range finder, exact when rank(F) <= l -- and Q <- orth(Z), two
  // passes, goes straight into the Rayleigh-Ritz step.
  if (pl.q == 0) {
    const int64_t ny = (int64_t)B * s.N * l;
    zero_f64(misc, nmisc, st);
    init_omega_kernel<<<(unsigned)((ny + 255) / 256), 256, 0, st>>>(Y, ny, pl.seed);
    if (pl.mfma) fit_mfma_backproject(s, l, F, Y, nullptr, Z, false, st);
    else gemm_fty<T>(s, l, F, Y, Z, st);
    if (orth(Z, Q, G, scratch(Y, s.N), M, B, s.D, l, true, pq, false, info, st) != SVDC_OK) return SVDC_E_HIP;
    std::swap(Q, Z);
  } else if (pl.mfma) {
    // one launch: the test matrix as operand words, the cleared words, and Z where several row groups accumulate in it
    const int64_t nz = zero_z ? nq : 0, nw = (int64_t)B * (s.D / 32) * (pq.kt[0] + (pq.ranges > 1 ? pq.kt[1] : 0)) * 64;
    const int64_t n = std::max(std::max((nz + 3) / 4, nmisc), nw);
    init_sketch_kernel<<<(unsigned)((n + 255) / 256), 256, 0, st>>>(pq, B, s.D, l, kF32, pl.seed, misc, nmisc, Z, nz);
    z_clear = zero_z;
  } else {
    zero_f64(misc, nmisc, st);
    init_omega_kernel<<<(unsigned)((nq + 255) / 256), 256, 0, st>>>(Q, nq, pl.seed);
  }

  const bool want_fro = fro2 != nullptr;
  bool fro_done = false;
  // Y = F Q.  The last product feeds the Rayleigh-Ritz step and uses the full-precision operand split.
  // float32 features: every product splits both operands.
  auto project = [&](bool last) {
    if (pl.mfma) {
      fit_mfma_project(s, l, F, Qp, Y, last ? nullptr : Yp, (last && want_fro) ? misc : nullptr,
                       last || kF32, st);
      if (last && want_fro) fro_done = true;
    } else {
      gemm_fq<T>(s, l, F, Q, Y, st);
    }
  };
  for (int it = 0; it < pl.q; ++it) {
    project(false);
    if (pl.mfma) {
      fit_mfma_backproject(s, l, F, Y, Yp, Z, z_clear, st);
    } else {
      gemm_fty<T>(s, l, F, Y, Z, st);
    }
    const bool last_it = it + 1 == pl.q;
    if (orth(Z, Q, G, scratch(Y, s.N), M, B, s.D, l, last_it, pq, zero_z && !last_it, info, st) != SVDC_OK)
      return SVDC_E_HIP;
    z_clear = zero_z;
    if (last_it) std::swap(Q, Z);
  }

  // Rayleigh-Ritz on span(Q)
  project(true);
  gram(Y, G, scratch(Z, s.D), B, s.N, l, st);
  chol_factor(G, B, l, info, st, M, false);   // M: scratch until the Jacobi writes it
  if (want_fro && !fro_done) {
    // at most four workgroups per compute unit, at least 8192 elements each: all of a block's add to one word
    const int64_t pieces = (int64_t)s.N * ((s.D + 7) / 8);
    const int64_t groups = std::min<int64_t>((pieces + 1023) / 1024, std::max<int64_t>(1, 4 * (int64_t)num_compute_units() / B));
    sumsq_kernel<T><<<dim3((unsigned)groups, B), 256, 0, st>>>(F, misc, s.N, s.D, s.ldf, s.block_stride);
  }
  int32_t jrc = SVDC_OK;
  if ((size_t)l * (l + 1) * sizeof(double) <= kLdsBudget) {   // l <= 138: the whole matrix in the LDS of one workgroup
    auto launch = [&](auto kernel, int nt, size_t lds) -> int32_t {
      if (set_dyn_lds((const void*)kernel, lds) != SVDC_OK) return SVDC_E_HIP;
      kernel<<<B, nt, lds, st>>>(G, M, sigma, l, s.k, misc, fro2, pl.max_sweeps, info);
      return SVDC_OK;
    };
    // a wave per pair of 8-column blocks, columns of 8 lanes x NE elements
    auto by_waves = [&](auto ne) -> int32_t {
      constexpr int NE = decltype(ne)::value;
      const int waves = (l + 15) / 16;
      return launch(jacobi_wave_kernel<NE>, 64 * waves, (size_t)16 * waves * (8 * NE + 8) * sizeof(double));
    };
    if (l <= 16) jrc = by_waves(std::integral_constant<int, 2>{});
    else if (l <= 32) jrc = by_waves(std::integral_constant<int, 4>{});
    else if (l <= 64) jrc = by_waves(std::integral_constant<int, 8>{});
    else if (l <= 128) jrc = by_waves(std::integral_constant<int, 16>{});
    else jrc = launch(jacobi_kernel<18, 1024, 8>, 1024, (size_t)l * (l | 1) * sizeof(double));
  } else {                                          // by column blocks, one launch per round-robin step
    const int nb = (l + kJbCols - 1) / kJbCols, nbe = (nb + 1) & ~1;
    const size_t lds = (size_t)2 * kJbCols * ((l <= 192 ? 192 : 256) + 8) * sizeof(double);   // columns of 8 lanes x 24 or 32
    int* cnt = (int*)(ws + pl.off_jcnt);
    auto sweeps = [&](auto kernel) -> int32_t {
      if (set_dyn_lds((const void*)kernel, lds) != SVDC_OK) return SVDC_E_HIP;
      for (int sweep = 0; sweep < pl.max_sweeps; ++sweep)
        for (int step = 0; step < nbe - 1; ++step)
          kernel<<<dim3(nbe / 2, B), kJbThreads, lds, st>>>(G, Wg, l, step, sweep, sweep == 0 && step == 0, cnt);
      return SVDC_OK;
    };
    jrc = l <= 192 ? sweeps(jacobi_block_kernel<24>) : sweeps(jacobi_block_kernel<32>);
    jacobi_finish_kernel<<<B, 1024, 0, st>>>(Wg, M, sigma, l, s.k, misc, fro2, pl.max_sweeps, cnt, info);
  }
  if (jrc != SVDC_OK) return jrc;
  rows_times_small(Q, M, V, B, s.D, l, s.k, l, st);
  return launch_status();
}

}  // namespace

int32_t run_fit(const svdc_shape& s, const FitPlan& plan, const void* F, float* V, float* sigma, float* fro2,
                void* workspace, hipStream_t st) {
  if (s.dtype == SVDC_BF16)
    return run_fit_typed<bf16_t>(s, plan, (const bf16_t*)F, V, sigma, fro2, (char*)workspace, st);
  return run_fit_typed<float>(s, plan, (const float*)F, V, sigma, fro2, (char*)workspace, st);
}

}  // namespace svdc
