// Matrix-core versions of the two products with F in the basis fit (bf16 features as they are; float32 features
// split into bf16 high + low parts on the fly, see FPiece and fit_backproject_f32_kernel):
//   project      Y[N x l] = F * Q           both operands streamed through registers (project_stream.h); in large bf16 calls with
//                                           wide sketches Q shared through LDS by waves that split the rows
//                                           (fit_project_rows_kernel), or with narrow ones stationary in registers for the last
//                                           product (fit_project_mfma_kernel)
//   backproject  Z[D x l] += F[rows, :]^T * Y[rows, :]         (Z accumulators stationary in registers)
// Both stream F exactly once per column range of the sketch (one range up to width 128, two up to 256), in 16- or
// 32-row tiles, on v_mfma_f32_16x16x32_bf16 (operand layouts: see mfma_kernels.hip).  A projection that is followed by a back-projection hands Y over as
// packed bf16 operand words (store_y_half) instead of float32 rows; the last projection of a fit writes float32 rows
// for the Gram matrix.  backproject stores Z directly when one workgroup covers all rows of a block and otherwise
// combines the partial results of its row groups with float atomics (into a Z that its caller cleared, or that it clears itself).
#include <algorithm>
#include <type_traits>

#include "fit_operands.h"
#include "step_tiling.h"
#include "svdc_device.h"
#include "svdc_internal.h"

namespace svdc {

namespace {

constexpr int kWaves = 4;

// ---------------------------------------------------------------------------
// project: Y = F Q for a group of TG 16-row tiles per workgroup, no atomics.
// The workgroup walks over the channel slabs (128 * NCW channels each); for one
// slab wave w keeps the Q operands of its NCW chunks (all KT coefficient tiles)
// in registers and streams the group's row tiles of that slab past them.  The
// partial products of all slabs accumulate in registers (TG x KT accumulators per
// wave); at the end the four waves' partial sums are added through LDS in a
// fixed order and stored once.
//   A operand = F tile   (m = token row, kk = channel)   -- the natural 16-byte row pieces
//   B operand = Q tile   (kk = channel, n = coefficient)
//   D[m = 4 g + i][n = r]  ->  Y[row 16 tile + 4 g + i][16 jt + r]
// For the last product of large calls with sketches of up to 32 columns, in bf16 with both parts of Q: 57 x 4608 x 3072, width 16
// 305 us, 328 streamed (project_stream_kernel); 32 356 and 366.  Also accumulates sum F^2 (for ||F||_F^2, fro_acc nullable).
// ---------------------------------------------------------------------------
template <int NCW, int KT, int TG>
__global__ __launch_bounds__(256) void fit_project_mfma_kernel(const bf16_t* __restrict__ F,
                                                               const uint16_t* __restrict__ Qp, float* Y,
                                                               double* fro_acc, int N, int D, int l,
                                                               int64_t ldf, int64_t bstride, int NS,
                                                               int groups_per_block, int ldy) {
  constexpr int PD = 2;
  static_assert(TG % PD == 0, "prefetch ring must divide the tile group");
  __shared__ f32x4 part[kWaves][2][KT][64];
  const int b = blockIdx.x / groups_per_block, rg = blockIdx.x % groups_per_block;
  const int wave = threadIdx.x >> 6, lane = threadIdx.x & 63, r = lane & 15, g = lane >> 4;
  const int64_t per = (int64_t)D * KT * 16;
  const u32x4* Qhi = reinterpret_cast<const u32x4*>(Qp + (int64_t)b * 2 * per);
  const u32x4* Qlo = reinterpret_cast<const u32x4*>(Qp + (int64_t)b * 2 * per + per);
  const bf16_t* fbase = F + (int64_t)b * bstride + 8 * g;
  const int tile0 = rg * TG;
  const int ntiles = min(TG, (N + 15) / 16 - tile0);

  f32x4 acc[TG][KT];
#pragma unroll
  for (int t = 0; t < TG; ++t)
#pragma unroll
    for (int jt = 0; jt < KT; ++jt) acc[t][jt] = f32x4{0.f, 0.f, 0.f, 0.f};

  FPiece<bf16_t> fin[PD][NCW];
  auto load_tile = [&](int slab, int t, FPiece<bf16_t>(&fi)[NCW]) {
    const int row = min((tile0 + t) * 16 + r, N - 1);
    const int cg0 = (slab * kWaves + wave) * NCW;
#pragma unroll
    for (int c = 0; c < NCW; ++c) fi[c].load(fbase + (int64_t)row * ldf + 32 * (cg0 + c));
  };
#pragma unroll
  for (int u = 0; u < PD; ++u) load_tile(0, u, fin[u]);

  float ssq = 0.f;
  for (int slab = 0; slab < NS; ++slab) {
    const int cg0 = (slab * kWaves + wave) * NCW;
    u32x4 q_hi[NCW][KT], q_lo[NCW][KT];
#pragma unroll
    for (int c = 0; c < NCW; ++c)
#pragma unroll
      for (int jt = 0; jt < KT; ++jt) {
        const int64_t ti = (int64_t)(cg0 + c) * KT + jt;
        q_hi[c][jt] = Qhi[ti * 64 + lane];
        q_lo[c][jt] = Qlo[ti * 64 + lane];
      }
#pragma unroll
    for (int t = 0; t < TG; ++t) {
      const int u = t % PD;
      if (t < ntiles) {
#pragma unroll
        for (int c = 0; c < NCW; ++c) {
          const u32x4 fh = fin[u][c].w;
#pragma unroll
          for (int jt = 0; jt < KT; ++jt) {
            acc[t][jt] = mfma16(fh, q_hi[c][jt], acc[t][jt]);
            acc[t][jt] = mfma16(fh, q_lo[c][jt], acc[t][jt]);
          }
          if ((tile0 + t) * 16 + r < N) ssq += fin[u][c].sumsq();
        }
      }
      // refill this ring slot with the tile PD steps ahead (possibly in the next slab)
      if (t + PD < TG) {
        if (t + PD < ntiles) load_tile(slab, t + PD, fin[u]);
      } else if (slab + 1 < NS) {
        load_tile(slab + 1, t + PD - TG, fin[u]);
      }
    }
  }
  if (fro_acc) {
    const double s = wave_sum((double)ssq);
    if (lane == 0) atomicAdd(fro_acc + b, s);
  }

  // add the four waves' partial sums, two row tiles per round
  float* ybase = Y + (int64_t)b * N * ldy;
#pragma unroll
  for (int rd = 0; rd < TG / 2; ++rd) {
#pragma unroll
    for (int tt = 0; tt < 2; ++tt)
#pragma unroll
      for (int jt = 0; jt < KT; ++jt) part[wave][tt][jt][lane] = acc[2 * rd + tt][jt];
    __syncthreads();
#pragma unroll
    for (int item = 0; item < 2 * KT; ++item) {
      if ((item % kWaves) != wave) continue;
      const int tt = item / KT, jt = item % KT;
      f32x4 s = part[0][tt][jt][lane];
#pragma unroll
      for (int w = 1; w < kWaves; ++w) {
        const f32x4 p = part[w][tt][jt][lane];
        s[0] += p[0]; s[1] += p[1]; s[2] += p[2]; s[3] += p[3];
      }
      const int j = 16 * jt + r;
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        const int row = (tile0 + 2 * rd + tt) * 16 + 4 * g + i;
        if (row < N && j < l) ybase[(int64_t)row * ldy + j] = s[i];
      }
    }
    __syncthreads();
  }
}

// ---------------------------------------------------------------------------
// project, row-split version for large bf16 calls with wide sketches: the four waves of a workgroup take different row tiles
// (RTW each) and all channels, so no partial sums have to be combined, and they share the Q operands through LDS:
// the operand words of a slab of SC 32-channel chunks are fetched once per workgroup (registers -> LDS, double
// buffered, one barrier per slab) and every wave reads them from there.  Per token row the packed sketch is then
// read from L2 once per 64 RTW rows and from LDS once per 16 RTW rows, against once per 16 to 96 rows when both operands are
// streamed (project_stream_kernel), at the price of a memory latency and a barrier per slab, which only several workgroups on a
// compute unit hide.  57 x 4608 x 3072, this and streamed: split operands, width 64 394 and 447 us alone (435 in a traced refit), width 128 575 and 587; plain
// ones, width 128 431 and 457 us.  20 blocks: 146 and 164, 225 and 216, 166 and 170; 8 blocks: 92 and 72, 118 and 95, 88 and 76.
//   A operand = F tile   (m = token row, kk = channel)   -- the natural 16-byte row pieces
//   B operand = Q tile   (kk = channel, n = coefficient)
//   D[m = 4 g + i][n = r]  ->  Y[row 16 tile + 4 g + i][16 jt + r]
// SPLIT (the last product of a fit): both parts of Q, float32 rows of Y and sum F^2 (fro_acc nullable); otherwise the
// words of the back-projection.
// ---------------------------------------------------------------------------
template <int KT, int RTW, int SC, bool SPLIT>
__global__ __launch_bounds__(256, KT == 8 ? 2 : 1) void fit_project_rows_kernel(const bf16_t* __restrict__ F,
                                                               const uint16_t* __restrict__ Qp, float* Y,
                                                               u32x4* Yp, double* fro_acc, int N, int D, int l,
                                                               int64_t ldf, int64_t bstride,
                                                               int groups_per_block, int ldy) {
  // With split operands the chunks of F are requested two at a time: the two 64-byte
  // pieces of a 128-byte line belong to neighbouring chunks, and asked for a whole chunk's work apart the line comes
  // from L2 twice (4 % slower).  With plain operands a slot is refilled as soon as its chunk is done (two chunks
  // in flight instead of four: 3 % slower at width 128).
  constexpr bool PAIRED = SPLIT;
  constexpr int PD = 4;                       // chunks of F in flight per wave
  static_assert(SC == 2 || SC == 4, "slab of 2 or 4 chunks");
  static_assert(PAIRED || SC == PD, "without pairing the ring slot of a chunk is its index in the slab");
  constexpr int NP = SPLIT ? 2 : 1;           // operand parts (high, low)
  constexpr int WPW = SC * KT / kWaves;       // operand words a wave stages per slab and part
  static_assert(SC * KT % kWaves == 0, "staging must divide among the waves");
  const int b = blockIdx.x / groups_per_block, rg = blockIdx.x % groups_per_block;
  const int lane = threadIdx.x & 63, r = lane & 15, g = lane >> 4;
  const int wave = threadIdx.x >> 6;
  __shared__ u32x4 qs[2][NP][SC * KT][64];
  const int64_t per = (int64_t)D * KT * 16;
  const int NS = D / (32 * SC), NC = NS * SC;
  const u32x4* Qhi = reinterpret_cast<const u32x4*>(Qp + (int64_t)b * 2 * per);
  const u32x4* Qlo = reinterpret_cast<const u32x4*>(Qp + (int64_t)b * 2 * per + per);
  const bf16_t* fbase = F + (int64_t)b * bstride + 8 * g;
  const int tile0 = (rg * kWaves + wave) * RTW;

  f32x4 acc[RTW][KT];
#pragma unroll
  for (int t = 0; t < RTW; ++t)
#pragma unroll
    for (int jt = 0; jt < KT; ++jt) acc[t][jt] = f32x4{0.f, 0.f, 0.f, 0.f};

  int64_t rowoff[RTW];
#pragma unroll
  for (int t = 0; t < RTW; ++t) rowoff[t] = (int64_t)min((tile0 + t) * 16 + r, N - 1) * ldf;
  FPiece<bf16_t> fin[PD][RTW];
  auto load_chunk = [&](int chunk, FPiece<bf16_t>(&fi)[RTW]) {
#pragma unroll
    for (int t = 0; t < RTW; ++t) fi[t].load(fbase + rowoff[t] + 32 * chunk);
  };
  u32x4 stg[NP][WPW];
  auto load_stage = [&](int slab) {
#pragma unroll
    for (int i = 0; i < WPW; ++i) {
      const int64_t w = (int64_t)slab * SC * KT + wave * WPW + i;
      stg[0][i] = Qhi[w * 64 + lane];
      if (SPLIT) stg[NP - 1][i] = Qlo[w * 64 + lane];
    }
  };
  auto store_stage = [&](int buf) {
#pragma unroll
    for (int i = 0; i < WPW; ++i)
#pragma unroll
      for (int p = 0; p < NP; ++p) qs[buf][p][wave * WPW + i][lane] = stg[p][i];
  };
  load_stage(0);
#pragma unroll
  for (int u = 0; u < PD; ++u)
    if (u < NC) load_chunk(u, fin[u]);
  store_stage(0);
  __syncthreads();

  float ssq = 0.f;
  // one slab; with paired requests PAR = slab % 2 is a compile-time value, so that the ring slots are static
  static_assert(!PAIRED || 2 * SC % PD == 0, "the ring repeats with every second slab");
  auto do_slab = [&](int slab, auto par) {
    constexpr int PAR = decltype(par)::value;
    const int buf = PAIRED ? (PAR & 1) : (slab & 1);
    if (slab + 1 < NS) load_stage(slab + 1);
#pragma unroll
    for (int c = 0; c < SC; ++c) {
      const int chunk = slab * SC + c;
      constexpr int kSlotBase = (PAR * SC) % PD;
      const int u = (kSlotBase + c) % PD;     // = chunk % PD
      u32x4 fh[RTW];
#pragma unroll
      for (int t = 0; t < RTW; ++t) fh[t] = fin[u][t].w;
#pragma unroll
      for (int jt = 0; jt < KT; ++jt) {
        const u32x4 bh = qs[buf][0][c * KT + jt][lane];
        u32x4 bl;
        if (SPLIT) bl = qs[buf][NP - 1][c * KT + jt][lane];
#pragma unroll
        for (int t = 0; t < RTW; ++t) {
          acc[t][jt] = mfma16(fh[t], bh, acc[t][jt]);
          if (SPLIT) acc[t][jt] = mfma16(fh[t], bl, acc[t][jt]);
        }
      }
      if (SPLIT) {
#pragma unroll
        for (int t = 0; t < RTW; ++t)
          if ((tile0 + t) * 16 + r < N) ssq += fin[u][t].sumsq();
      }
      if constexpr (PAIRED) {
        if (c % 2 == 1) {                     // chunks c - 1 and c are done: refill both slots together
          if (chunk - 1 + PD < NC) load_chunk(chunk - 1 + PD, fin[(kSlotBase + c - 1) % PD]);
          if (chunk + PD < NC) load_chunk(chunk + PD, fin[u]);
        }
      } else {
        if (chunk + PD < NC) load_chunk(chunk + PD, fin[u]);
      }
    }
    if (slab + 1 < NS) store_stage(buf ^ 1);
    __syncthreads();
  };
  if constexpr (PAIRED) {
    for (int slab = 0; slab < NS; slab += 2) {
      do_slab(slab, std::integral_constant<int, 0>{});
      if (slab + 1 < NS) do_slab(slab + 1, std::integral_constant<int, 1>{});
    }
  } else {
    for (int slab = 0; slab < NS; ++slab) do_slab(slab, std::integral_constant<int, 0>{});
  }
  if (SPLIT && fro_acc) {
    const double s = wave_sum((double)ssq);
    if (lane == 0) atomicAdd(fro_acc + b, s);
  }
  if constexpr (!SPLIT) {   // the wave's two tiles are one 32-row step
    static_assert(RTW == 2, "two tiles");
    const int nsteps = (N + 31) / 32, step = tile0 / 2;
    if (step < nsteps) {
#pragma unroll
      for (int jt = 0; jt < KT; ++jt)
#pragma unroll
        for (int t = 0; t < 2; ++t)
          store_y_half(FPiece<bf16_t>{}, Yp, ((int64_t)b * nsteps + step) * KT + jt, t, acc[t][jt], 16 * (tile0 + t) + 4 * g, N);
    }
    return;
  }
  float* ybase = Y + (int64_t)b * N * ldy;
#pragma unroll
  for (int t = 0; t < RTW; ++t)
#pragma unroll
    for (int jt = 0; jt < KT; ++jt) {
      const int j = 16 * jt + r;
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        const int row = (tile0 + t) * 16 + 4 * g + i;
        if (row < N && j < l) ybase[(int64_t)row * ldy + j] = acc[t][jt][i];
      }
    }
}

// The CW x RS waves of a workgroup, RS of which took different rows of the same channels, add their TILES accumulator tiles: tile t ends up in
// the wave of share t % RS.
template <int TILES, int CW, int RS>
__device__ __forceinline__ void sum_row_shares(f32x4* acc, int wave, int lane) {
  extern __shared__ u32x4 lds_words[];
  f32x4* part = reinterpret_cast<f32x4*>(lds_words);
  const int share = wave / CW;
#pragma unroll
  for (int t = 0; t < TILES; ++t)
    if (t % RS != share) part[(wave * TILES + t) * 64 + lane] = acc[t];
  __syncthreads();
#pragma unroll
  for (int t = 0; t < TILES; ++t)
    if (t % RS == share) {
#pragma unroll
      for (int o = 1; o < RS; ++o) acc[t] += part[(((wave + o * CW) % (CW * RS)) * TILES + t) * 64 + lane];
    }
}

// ---------------------------------------------------------------------------
// backproject: Z[d][j] += sum_rows F[row][d] Y[row][j] over the workgroup's rows.
// The contraction runs over token rows, so both operands need 8 consecutive
// rows per lane:
//   A operand (m = channel, kk = row): a lane loads, for each of its 8 rows, the
//       32-bit word holding channels (2 r, 2 r + 1) of a 32-channel chunk and
//       regroups the low / high halves with v_perm into the operands of the
//       "even" (d = 2 r) and "odd" (d = 2 r + 1) channel tiles;
//   B operand (kk = row, n = coefficient): Y[row 8 g + e][16 jt + r] converted to bf16.
//   D[m = 4 g + i][n = r]  ->  Z[32 chunk + 2 (4 g + i) + parity][16 jt + r]
// Accumulators (NCW chunks x 2 parities x KT tiles) stay in registers over all rows.
// ---------------------------------------------------------------------------
// PACKED: Y comes as the operand words that the projection wrote (store_y_half); the rows of a 32-row step are then
// contracted in that word's order, kk = 8 g + e  <->  row 16 (e / 4) + 4 g + e % 4.
// RS: waves that take every RS-th step of the same channels (backproject_plan).
template <int NCW, int KT, bool PACKED, int RS>
__global__ __launch_bounds__(256) void fit_backproject_mfma_kernel(const bf16_t* __restrict__ F,
                                                                   const float* __restrict__ Y,
                                                                   const u32x4* __restrict__ Yp, float* Z, int N,
                                                                   int D, int l, int64_t ldf, int64_t bstride,
                                                                   int NS, int groups_per_block,
                                                                   int rows_per_group, int ldy, int ldz) {
  const int slab = blockIdx.x % NS;
  const int rgb = blockIdx.x / NS;
  const int b = rgb / groups_per_block, rg = rgb % groups_per_block;
  constexpr int CW = kWaves / RS;          // waves that take different channels
  const int wave = threadIdx.x >> 6, lane = threadIdx.x & 63, r = lane & 15, g = lane >> 4;
  const int share = RS == 1 ? 0 : __builtin_amdgcn_readfirstlane(wave / CW);
  const int cg0 = (slab * CW + (RS == 1 ? wave : wave % CW)) * NCW;
  const uint32_t* fbase = reinterpret_cast<const uint32_t*>(F + (int64_t)b * bstride + 32 * cg0) + r;
  const int64_t ldw = ldf / 2;   // row stride in 32-bit words
  const float* ybase = Y + (int64_t)b * N * ldy;
  const int row_end = min(N, (rg + 1) * rows_per_group), row_begin = rg * rows_per_group + 32 * share;

  f32x4 acc[NCW][2][KT];
#pragma unroll
  for (int c = 0; c < NCW; ++c)
#pragma unroll
    for (int p = 0; p < 2; ++p)
#pragma unroll
      for (int jt = 0; jt < KT; ++jt) acc[c][p][jt] = f32x4{0.f, 0.f, 0.f, 0.f};

  uint32_t fw[NCW][8];
  float yv[PACKED ? 1 : KT][8];
  u32x4 yw[PACKED ? KT : 1];
  const int nsteps = (N + 31) / 32;
  auto load_step = [&](int row0) {
#pragma unroll
    for (int e = 0; e < 8; ++e) {
      const int row = PACKED ? row0 + 16 * (e / 4) + 4 * g + e % 4 : row0 + 8 * g + e;
      const int rowc = min(row, N - 1);
#pragma unroll
      for (int c = 0; c < NCW; ++c) fw[c][e] = fbase[(int64_t)rowc * ldw + 16 * c];
      if constexpr (!PACKED) {
#pragma unroll
        for (int jt = 0; jt < KT; ++jt) {
          const int j = 16 * jt + r;
          yv[jt][e] = (row < row_end && j < l) ? ybase[(int64_t)row * ldy + j] : 0.f;
        }
      }
    }
    if constexpr (PACKED) {   // row groups start at multiples of 32 rows; rows >= N are zero in the packed words
#pragma unroll
      for (int jt = 0; jt < KT; ++jt) yw[jt] = Yp[(((int64_t)b * nsteps + row0 / 32) * KT + jt) * 64 + lane];
    }
  };
  if (row_begin < row_end) load_step(row_begin);
  for (int row0 = row_begin; row0 < row_end; row0 += 32 * RS) {
    u32x4 yop[KT];
#pragma unroll
    for (int jt = 0; jt < KT; ++jt) {
      if constexpr (PACKED)
        yop[jt] = yw[jt];
      else
        yop[jt] = u32x4{pack_bf16(yv[jt][0], yv[jt][1]), pack_bf16(yv[jt][2], yv[jt][3]),
                        pack_bf16(yv[jt][4], yv[jt][5]), pack_bf16(yv[jt][6], yv[jt][7])};
    }
    u32x4 fop[NCW][2];
#pragma unroll
    for (int c = 0; c < NCW; ++c)
#pragma unroll
      for (int w = 0; w < 4; ++w) {
        fop[c][0][w] = __builtin_amdgcn_perm(fw[c][2 * w + 1], fw[c][2 * w], 0x05040100u);
        fop[c][1][w] = __builtin_amdgcn_perm(fw[c][2 * w + 1], fw[c][2 * w], 0x07060302u);
      }
    if (row0 + 32 * RS < row_end) load_step(row0 + 32 * RS);
#pragma unroll
    for (int c = 0; c < NCW; ++c)
#pragma unroll
      for (int p = 0; p < 2; ++p)
#pragma unroll
        for (int jt = 0; jt < KT; ++jt) acc[c][p][jt] = mfma16(fop[c][p], yop[jt], acc[c][p][jt]);
  }

  if constexpr (RS > 1) sum_row_shares<NCW * 2 * KT, CW, RS>(&acc[0][0][0], wave, lane);

  float* zbase = Z + (int64_t)b * D * ldz;
#pragma unroll
  for (int c = 0; c < NCW; ++c)
#pragma unroll
    for (int p = 0; p < 2; ++p)
#pragma unroll
      for (int jt = 0; jt < KT; ++jt) {
        const int j = 16 * jt + r;
        if (j >= l || (RS > 1 && ((c * 2 + p) * KT + jt) % RS != share)) continue;
#pragma unroll
        for (int i = 0; i < 4; ++i) {
          const int d = 32 * (cg0 + c) + 2 * (4 * g + i) + p;
          // one row group per block: every element has a single writer
          if (groups_per_block == 1) zbase[(int64_t)d * ldz + j] = acc[c][p][jt][i];
          else atomicAdd(zbase + (int64_t)d * ldz + j, acc[c][p][jt][i]);
        }
      }
}

// ---------------------------------------------------------------------------
// backproject for float32 features: the same contraction, Z[d][j] += sum_rows F[row][d] Y[row][j], with both
// operands split into bf16 high + low parts (F_hi Y_hi + F_lo Y_hi + F_hi Y_lo).  A lane loads, for each
// of its 8 rows, the two float32 channels (2 r, 2 r + 1) of a chunk and splits them.  PACKED: Y comes as the two-part
// operand words that the projection wrote (store_y_half), with the rows of a step in that word's order; otherwise as
// float32 rows, 8 scalar loads and a split per operand in every wave, which bounded the kernel (18432 x 3072, sketch 128:
// 134 us, 75 us with the words, 55 with the waves on different rows).  Same output mapping and row-group scheme as the bf16 kernel.
// ---------------------------------------------------------------------------
template <int NCW, int KT, bool PACKED, int RS>
__global__ __launch_bounds__(256) void fit_backproject_f32_kernel(const float* __restrict__ F,
                                                                  const float* __restrict__ Y,
                                                                  const u32x4* __restrict__ Yp, float* Z, int N,
                                                                  int D, int l, int64_t ldf, int64_t bstride,
                                                                  int NS, int groups_per_block, int rows_per_group,
                                                                  int ldy, int ldz) {
  const int slab = blockIdx.x % NS;
  const int rgb = blockIdx.x / NS;
  const int b = rgb / groups_per_block, rg = rgb % groups_per_block;
  constexpr int CW = kWaves / RS;          // waves that take different channels
  const int wave = threadIdx.x >> 6, lane = threadIdx.x & 63, r = lane & 15, g = lane >> 4;
  const int share = RS == 1 ? 0 : __builtin_amdgcn_readfirstlane(wave / CW);
  const int cg0 = (slab * CW + (RS == 1 ? wave : wave % CW)) * NCW;
  const f32x2* fbase = reinterpret_cast<const f32x2*>(F + (int64_t)b * bstride + 32 * cg0) + r;
  const int64_t ldw = ldf / 2;   // row stride in channel pairs
  const float* ybase = Y + (int64_t)b * N * ldy;
  const int row_end = min(N, (rg + 1) * rows_per_group), row_begin = rg * rows_per_group + 32 * share;
  const int nsteps = (N + 31) / 32;

  f32x4 acc[NCW][2][KT];
#pragma unroll
  for (int c = 0; c < NCW; ++c)
#pragma unroll
    for (int p = 0; p < 2; ++p)
#pragma unroll
      for (int jt = 0; jt < KT; ++jt) acc[c][p][jt] = f32x4{0.f, 0.f, 0.f, 0.f};

  f32x2 fw[NCW][8];
  float yv[PACKED ? 1 : KT][8];
  u32x4 yw[PACKED ? KT : 1][2];
  auto load_step = [&](int row0) {
#pragma unroll
    for (int e = 0; e < 8; ++e) {
      const int row = PACKED ? row0 + 16 * (e / 4) + 4 * g + e % 4 : row0 + 8 * g + e;
      const int rowc = min(row, N - 1);
#pragma unroll
      for (int c = 0; c < NCW; ++c) {
        fw[c][e] = fbase[(int64_t)rowc * ldw + 16 * c];
        if constexpr (!PACKED) {
          if (row >= row_end) fw[c][e] = f32x2{0.f, 0.f};
        }
      }
      if constexpr (!PACKED) {
#pragma unroll
        for (int jt = 0; jt < KT; ++jt) {
          const int j = 16 * jt + r;
          yv[jt][e] = (row < row_end && j < l) ? ybase[(int64_t)row * ldy + j] : 0.f;
        }
      }
    }
    if constexpr (PACKED) {   // row groups start at multiples of 32 rows; rows >= N are zero in the packed words
#pragma unroll
      for (int jt = 0; jt < KT; ++jt)
#pragma unroll
        for (int p = 0; p < 2; ++p) yw[jt][p] = Yp[((((int64_t)b * nsteps + row0 / 32) * KT + jt) * 2 + p) * 64 + lane];
    }
  };
  if (row_begin < row_end) load_step(row_begin);
  for (int row0 = row_begin; row0 < row_end; row0 += 32 * RS) {
    u32x4 yhi[KT], ylo[KT];
#pragma unroll
    for (int jt = 0; jt < KT; ++jt) {
      if constexpr (PACKED) { yhi[jt] = yw[jt][0]; ylo[jt] = yw[jt][1]; }
      else split_operand(yv[jt], &yhi[jt], &ylo[jt]);
    }
    u32x4 fhi[NCW][2], flo[NCW][2];
#pragma unroll
    for (int c = 0; c < NCW; ++c)
#pragma unroll
      for (int p = 0; p < 2; ++p) {
        float c8[8];
#pragma unroll
        for (int e = 0; e < 8; ++e) c8[e] = fw[c][e][p];
        split_operand(c8, &fhi[c][p], &flo[c][p]);
      }
    if (row0 + 32 * RS < row_end) load_step(row0 + 32 * RS);
#pragma unroll
    for (int c = 0; c < NCW; ++c)
#pragma unroll
      for (int p = 0; p < 2; ++p)
#pragma unroll
        for (int jt = 0; jt < KT; ++jt) {
          acc[c][p][jt] = mfma16(fhi[c][p], yhi[jt], acc[c][p][jt]);
          acc[c][p][jt] = mfma16(flo[c][p], yhi[jt], acc[c][p][jt]);
          acc[c][p][jt] = mfma16(fhi[c][p], ylo[jt], acc[c][p][jt]);
        }
  }

  if constexpr (RS > 1) sum_row_shares<NCW * 2 * KT, CW, RS>(&acc[0][0][0], wave, lane);

  float* zbase = Z + (int64_t)b * D * ldz;
#pragma unroll
  for (int c = 0; c < NCW; ++c)
#pragma unroll
    for (int p = 0; p < 2; ++p)
#pragma unroll
      for (int jt = 0; jt < KT; ++jt) {
        const int j = 16 * jt + r;
        if (j >= l || (RS > 1 && ((c * 2 + p) * KT + jt) % RS != share)) continue;
#pragma unroll
        for (int i = 0; i < 4; ++i) {
          const int d = 32 * (cg0 + c) + 2 * (4 * g + i) + p;
          if (groups_per_block == 1) zbase[(int64_t)d * ldz + j] = acc[c][p][jt][i];
          else atomicAdd(zbase + (int64_t)d * ldz + j, acc[c][p][jt][i]);
        }
      }
}

template <int KT>
constexpr int width_for() { return KT <= 2 ? 12 : (KT == 4 ? 6 : 3); }

// Row strides of the whole Y / Z matrices when a call covers only a range of their columns (sketches wider than 128
// are multiplied as two column ranges), and whether Z has been cleared for atomic accumulation already.
struct Strides {
  int ldy, ldz;
  bool z_cleared;
};

template <typename T, int NCW, int KT, int RS>
void backproject_launch(const svdc_shape& s, int l, const void* F, const float* Y, const u32x4* Yp, float* Z, int gpb, int rows,
                        Strides ld, hipStream_t st) {
  const int NS = s.D / (32 * NCW * (kWaves / RS));
  const unsigned grid = (unsigned)((int64_t)NS * gpb * s.B);
  constexpr int lds = RS > 1 ? kWaves * NCW * 2 * KT * 1024 : 0;
  static_assert(lds <= 160 * 1024, "partial sums");
  auto go = [&](auto kernel, auto f) {
    // beyond what a launch may ask for by itself; without it the launch fails, which the caller's check reports
    if constexpr (lds > 64 * 1024) (void)hipFuncSetAttribute((const void*)kernel, hipFuncAttributeMaxDynamicSharedMemorySize, lds);
    kernel<<<grid, 256, lds, st>>>(f, Y, Yp, Z, s.N, s.D, l, s.ldf, s.block_stride, NS, gpb, rows, ld.ldy, ld.ldz);
  };
  if constexpr (std::is_same<T, float>::value) {
    if (RS > 1 || Yp) go(fit_backproject_f32_kernel<NCW, KT, true, RS>, (const float*)F);
    else if constexpr (RS == 1) go(fit_backproject_f32_kernel<NCW, KT, false, 1>, (const float*)F);
  } else {
    if (RS > 1 || Yp) go(fit_backproject_mfma_kernel<NCW, KT, true, RS>, (const bf16_t*)F);
    else if constexpr (RS == 1) go(fit_backproject_mfma_kernel<NCW, KT, false, 1>, (const bf16_t*)F);
  }
}

__global__ void clear_f32_kernel(float* p, int64_t n) {
  const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (i < n) p[i] = 0.0f;
}

// How a back-projection runs: whether the waves of a workgroup take different rows of 64 channels (backproject_plan), row groups
// per block and their rows.
struct BackPlan {
  bool shares;
  int gpb, rows;
};
inline BackPlan backproject_rows(const svdc_shape& s, bool shares, int64_t groups) {
  const int64_t g = std::max<int64_t>(1, groups);
  const int r = (int)std::max<int64_t>(32, ((s.N + g - 1) / g + 31) / 32 * 32);
  return {shares, (s.N + r - 1) / r, r};
}
// Partial sums of different row groups meet in float atomics (about 250 G/s), which cost more than the parallelism they buy:
// one group per block as soon as the slabs of all blocks give about one workgroup per compute unit, otherwise just enough
// groups to reach that.  Then the four waves of a workgroup had better take different rows of 64 channels than different channels
// of 128 NCW: their sums meet in LDS, and with narrower slabs there are fewer groups and atomics.  One block of 4608 x 3072
// (18432 x 3072): bf16 width 64 15 -> 12 us (37 -> 25), 128 23 -> 17 (55 -> 33); float32 width 64 29 -> 16 (55 -> 41), 128 45 -> 24
// (74 -> 55).  Eight waves on 64 channels of 32 each: 10, 25, 15, 36 us for the bf16 figures, 15, 41, 23, 63 for the float32 ones, no better.
// - Only while the slabs are one round of workgroups (float32, width 64, 6 blocks of 4608 x 3072: 24 us slower), or at width 128,
//   where few workgroups fit on a compute unit, instead of three or more groups (8 blocks: float32 45 us faster, bf16 78 -> 67 us;
//   16 bf16 blocks, 2 groups: 125 -> 141 us).
// - From 512 rows on: with fewer the waves have hardly a step each (300 x 1024, bf16, width 64: a fit takes 329 us and 331 us).
// - As many groups as fit into one round (float32, width 64, 2 blocks of 4608 x 3072: 3 groups in a little more than one round
//   7 us slower than 2), rounded up where several workgroups fit on a compute unit (bf16, 2 blocks of 9000 x 4224: 12 us faster), and
//   so that each wave has a step.
template <typename T, int NCW, int KT>
BackPlan backproject_plan(const svdc_shape& s, bool packed) {
  const int64_t cus = num_compute_units(), slabs = (int64_t)(s.D / (128 * NCW)) * s.B, narrow = (int64_t)(s.D / 64) * s.B;
  const BackPlan wide = backproject_rows(s, false, (cus + slabs / 2) / slabs);
  if (!packed || wide.gpb == 1 || s.N < 512 || (narrow > cus && !(KT == 8 && wide.gpb >= 3))) return wide;
  constexpr bool kSeveral = std::is_same<T, bf16_t>::value && KT <= 4;    // workgroups on a compute unit
  return backproject_rows(s, true, std::min<int64_t>((kSeveral ? cus + narrow / 2 : cus) / narrow, (s.N + 127) / 128));
}

// largest instantiated slab width (chunks per wave) that divides D / 128 and is at most `cap` (compile time: what
// the registers hold) and `maxw` (run time)
template <int cap, typename Fn12, typename Fn6, typename Fn4, typename Fn3, typename Fn2, typename Fn1>
void by_width(int m, int maxw, Fn12 f12, Fn6 f6, Fn4 f4, Fn3 f3, Fn2 f2, Fn1 f1) {
  if constexpr (cap >= 12) { if (maxw >= 12 && m % 12 == 0) return f12(); }
  if constexpr (cap >= 6) { if (maxw >= 6 && m % 6 == 0) return f6(); }
  if constexpr (cap >= 4) { if (maxw >= 4 && m % 4 == 0) return f4(); }
  if constexpr (cap >= 3) { if (maxw >= 3 && m % 3 == 0) return f3(); }
  if (maxw >= 2 && m % 2 == 0) return f2();
  return f1();
}

template <int KT>
void project_kt(const svdc_shape& s, int l, const void* F, const void* Qp, float* Y, u32x4* Yp, double* fro_acc, bool split,
                Strides ld, hipStream_t st) {
  const int ntile = (s.N + 15) / 16;
  const bool large = projection_is_large(ntile, s.B, KT, s.D, num_compute_units());
  // Plain bf16 operands of width 64 have two workgroups on a compute unit up to 5 tiles, which evens out the rounds of large calls: over 60 of them whole
  // fits take 3.3 % less time with 5 tiles than with the height of stream_rows, 1.7 % more at worst, 13 % less at best.
  const int rt = KT == 4 && !split && large ? 5 : stream_rows(ntile, s.B, num_compute_units());
  if (s.dtype == SVDC_F32) return fit_project_stream_f32(KT, rt, s, l, ld.ldy, F, Qp, Y, Yp, fro_acc != nullptr, fro_acc, st);
  // large bf16 calls with both parts of Q, or wide plain ones, have kernels of their own
  if (!large || !(split || KT == 8)) return fit_project_stream_bf16(KT, rt, s, l, ld.ldy, F, Qp, Y, Yp, split, fro_acc, st);
  const bf16_t* f = (const bf16_t*)F;
  const uint16_t* q = (const uint16_t*)Qp;
  if constexpr (KT >= 4) {
    auto rows = [&](auto rtw, auto sc, auto sp) {
      constexpr int R = decltype(rtw)::value;
      const int g = (ntile + kWaves * R - 1) / (kWaves * R);
      fit_project_rows_kernel<KT, R, decltype(sc)::value, decltype(sp)::value>
          <<<(unsigned)((int64_t)g * s.B), 256, 0, st>>>(f, q, Y, Yp, fro_acc, s.N, s.D, l, s.ldf, s.block_stride, g, ld.ldy);
    };
    using Two = std::integral_constant<int, 2>;
    using Three = std::integral_constant<int, 3>;
    using Four = std::integral_constant<int, 4>;
    if constexpr (KT == 8) {
      if (split) rows(Two{}, Two{}, std::true_type{});
      else rows(Two{}, Four{}, std::false_type{});
    } else {
      rows(Three{}, Four{}, std::true_type{});
    }
  } else {
    // the widest slab of channels that divides them and whose two parts the registers hold
    constexpr int cap = KT == 1 ? 12 : 6, TG = 8;
    auto stationary = [&](auto ncw) {
      constexpr int NCW = decltype(ncw)::value;
      const int gpb = (ntile + TG - 1) / TG;
      fit_project_mfma_kernel<NCW, KT, TG><<<(unsigned)((int64_t)gpb * s.B), 256, 0, st>>>(
          f, q, Y, fro_acc, s.N, s.D, l, s.ldf, s.block_stride, s.D / (128 * NCW), gpb, ld.ldy);
    };
    by_width<cap>(
        s.D / 128, cap, [&] { stationary(std::integral_constant<int, (cap >= 12 ? 12 : 1)>{}); },
        [&] { stationary(std::integral_constant<int, 6>{}); }, [&] { stationary(std::integral_constant<int, 4>{}); },
        [&] { stationary(std::integral_constant<int, 3>{}); }, [&] { stationary(std::integral_constant<int, 2>{}); },
        [&] { stationary(std::integral_constant<int, 1>{}); });
  }
}

template <typename T, int NCW, int KT>
void backproject_one(const svdc_shape& s, int l, const void* F, const float* Y, const u32x4* Yp, float* Z,
                     Strides ld, hipStream_t st) {
  const BackPlan plan = backproject_plan<T, NCW, KT>(s, Yp != nullptr);
  if (plan.gpb > 1 && !ld.z_cleared) {   // atomics accumulate into Z (a single column range: Z is contiguous)
    const int64_t n = (int64_t)s.B * s.D * l;
    clear_f32_kernel<<<(unsigned)((n + 255) / 256), 256, 0, st>>>(Z, n);
  }
  if (plan.shares) backproject_launch<T, 2, KT, kWaves>(s, l, F, Y, Yp, Z, plan.gpb, plan.rows, ld, st);
  else backproject_launch<T, NCW, KT, 1>(s, l, F, Y, Yp, Z, plan.gpb, plan.rows, ld, st);
}

// slab widths of the float32 back-projection (twice the registers per loaded row, two operand parts on each side)
template <int KT>
constexpr int width_for_f32() { return KT <= 2 ? 6 : (KT == 4 ? 3 : 2); }

// Widest slab (chunks per wave) that the back-projection of this shape may take.
// Small batches: narrower slabs give more workgroups without more row groups, whose partial sums meet in float
// atomics (one per element and row group): the widest slab that still gives 64 slabs over all blocks, if any.
// Measured at 4608 x 3072, width 64: 42 -> 15 us for one block, 55 -> 36 us for 4, 72 -> 53 us for 8; from 28
// blocks on the widest slab is the fastest again.  Not for float32 features: their slabs are narrow already (2 chunks at
// width 128, 3 at 64), and every further slab loads the two-part words of Y again (one block of 18432 x 3072, width 128,
// slabs of one chunk: 74 -> 100 us; 4 of 4608, width 64: 54 -> 61 us).
template <typename T, int KT>
constexpr int backproject_cap() { return std::is_same<T, float>::value ? width_for_f32<KT>() : width_for<KT>(); }
template <typename T, int KT>
int backproject_max_width(const svdc_shape& s, bool packed) {
  constexpr int cap = backproject_cap<T, KT>();
  constexpr int64_t kMinSlabs = 64;
  const int m = s.D / 128;
  int maxw = cap;
  if (!std::is_same<T, float>::value && packed) {   // packed Y only: float32 rows of Y cost the same once per slab
    maxw = 1;
    for (int w : {2, 3, 4, 6, 12})
      if (w <= cap && m % w == 0 && (int64_t)(m / w) * s.B >= kMinSlabs) maxw = w;
  }
  return maxw;
}

// calls fn(NCW) with the slab width of this shape as a compile-time constant
template <typename T, int KT, typename Fn>
void backproject_by_width(const svdc_shape& s, bool packed, Fn fn) {
  constexpr int cap = backproject_cap<T, KT>();
  by_width<cap>(
      s.D / 128, backproject_max_width<T, KT>(s, packed), [&] { fn(std::integral_constant<int, (cap >= 12 ? 12 : 1)>{}); },
      [&] { fn(std::integral_constant<int, (cap >= 6 ? 6 : 1)>{}); },
      [&] { fn(std::integral_constant<int, (cap >= 4 ? 4 : 1)>{}); },
      [&] { fn(std::integral_constant<int, (cap >= 3 ? 3 : 1)>{}); }, [&] { fn(std::integral_constant<int, 2>{}); },
      [&] { fn(std::integral_constant<int, 1>{}); });
}

template <typename T, int KT>
void backproject_kt(const svdc_shape& s, int l, const void* F, const float* Y, const u32x4* Yp, float* Z,
                    Strides ld, hipStream_t st) {
  backproject_by_width<T, KT>(s, Yp != nullptr, [&](auto ncw) {
    backproject_one<T, decltype(ncw)::value, KT>(s, l, F, Y, Yp, Z, ld, st);
  });
}

// Sketches wider than 128 are handled as two column ranges (128 and the rest), each with the kernels of its own
// width: F is then read twice per product.
struct ColRange { int j0, l; };
inline int col_ranges(int l, ColRange (&r)[2]) {
  if (l <= 128) { r[0] = {0, l}; return 1; }
  r[0] = {0, 128};
  r[1] = {128, l - 128};
  return 2;
}
inline int kt_for(int l) { return l <= 16 ? 1 : (l <= 32 ? 2 : (l <= 64 ? 4 : 8)); }
inline size_t packed_q_bytes_one(const svdc_shape& s, int l) { return (size_t)s.B * 2 * s.D * kt_for(l) * 16 * sizeof(uint16_t); }
// parts: 1 (bf16 features) or 2 (float32 features: high and low)
inline size_t packed_y_bytes_one(const svdc_shape& s, int l, int parts) {
  return (size_t)s.B * (((size_t)s.N + 31) / 32) * kt_for(l) * parts * 1024;
}

template <typename Fn>
void by_kt(int l, Fn fn) {
  if (l <= 16) fn(std::integral_constant<int, 1>{});
  else if (l <= 32) fn(std::integral_constant<int, 2>{});
  else if (l <= 64) fn(std::integral_constant<int, 4>{});
  else fn(std::integral_constant<int, 8>{});
}

}  // namespace

bool fit_mfma_supported(const svdc_shape& s, int l) {
  return (s.dtype == SVDC_BF16 || s.dtype == SVDC_F32) && s.D % 128 == 0 && l <= 256;
}

size_t fit_mfma_packed_q_bytes(const svdc_shape& s, int l) {
  ColRange r[2];
  const int n = col_ranges(l, r);
  size_t bytes = 0;
  for (int h = 0; h < n; ++h) bytes += packed_q_bytes_one(s, r[h].l);
  return bytes;
}

size_t fit_mfma_packed_y_bytes(const svdc_shape& s, int l, int parts) {
  ColRange r[2];
  const int n = col_ranges(l, r);
  size_t bytes = 0;
  for (int h = 0; h < n; ++h) bytes += packed_y_bytes_one(s, r[h].l, parts);
  return bytes;
}

void fit_mfma_project(const svdc_shape& s, int l, const void* F, const void* Qp, float* Y, void* Ypacked, double* fro_acc,
                      bool split, hipStream_t st) {
  ColRange r[2];
  const int n = col_ranges(l, r);
  const char* qp = static_cast<const char*>(Qp);
  char* yp = static_cast<char*>(Ypacked);
  for (int h = 0; h < n; ++h) {
    const Strides ld{l, l, false};
    by_kt(r[h].l, [&](auto kt) {
      constexpr int KT = decltype(kt)::value;
      project_kt<KT>(s, r[h].l, F, qp, Y + r[h].j0, (u32x4*)yp, h == 0 ? fro_acc : nullptr, split, ld, st);
    });
    qp += packed_q_bytes_one(s, r[h].l);
    if (yp) yp += packed_y_bytes_one(s, r[h].l, s.dtype == SVDC_F32 ? 2 : 1);
  }
}

PackedQ fit_mfma_packed_q(const svdc_shape& s, int l, void* Qp) {
  ColRange r[2];
  PackedQ q;
  q.p = static_cast<char*>(Qp);
  q.ranges = col_ranges(l, r);
  int64_t off = 0;
  for (int h = 0; h < q.ranges; ++h) {
    q.kt[h] = kt_for(r[h].l);
    q.offset[h] = off;
    off += (int64_t)packed_q_bytes_one(s, r[h].l);
  }
  return q;
}

bool fit_mfma_backproject_accumulates(const svdc_shape& s, int l, bool packed) {
  ColRange r[2];
  const int n = col_ranges(l, r);
  bool any = false;
  for (int h = 0; h < n; ++h)
    by_kt(r[h].l, [&](auto kt) {
      constexpr int KT = decltype(kt)::value;
      auto asks = [&](auto elem) {
        using T = decltype(elem);
        backproject_by_width<T, KT>(s, packed, [&](auto ncw) { any = any || backproject_plan<T, decltype(ncw)::value, KT>(s, packed).gpb > 1; });
      };
      if (s.dtype == SVDC_F32) asks(float{});
      else asks(bf16_t{});
    });
  return any;
}

void fit_mfma_backproject(const svdc_shape& s, int l, const void* F, const float* Y, const void* Ypacked, float* Z,
                          bool z_clear, hipStream_t st) {
  ColRange r[2];
  const int n = col_ranges(l, r);
  const char* yp = static_cast<const char*>(Ypacked);
  bool cleared = z_clear;
  if (n > 1 && !cleared) {   // the column ranges interleave in memory: clear all of Z once, for whichever range accumulates
    const int64_t cnt = (int64_t)s.B * s.D * l;
    clear_f32_kernel<<<(unsigned)((cnt + 255) / 256), 256, 0, st>>>(Z, cnt);
    cleared = true;
  }
  for (int h = 0; h < n; ++h) {
    const Strides ld{l, l, cleared};
    by_kt(r[h].l, [&](auto kt) {
      constexpr int KT = decltype(kt)::value;
      if (s.dtype == SVDC_F32)
        backproject_kt<float, KT>(s, r[h].l, F, Y ? Y + r[h].j0 : nullptr, (const u32x4*)yp, Z + r[h].j0, ld, st);
      else
        backproject_kt<bf16_t, KT>(s, r[h].l, F, Y ? Y + r[h].j0 : nullptr, (const u32x4*)yp, Z + r[h].j0, ld, st);
    });
    if (yp) yp += packed_y_bytes_one(s, r[h].l, s.dtype == SVDC_F32 ? 2 : 1);
  }
}

}  // namespace svdc
