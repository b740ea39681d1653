// Matrix-core (MFMA) kernels for bf16 and float32 features on gfx950 (float32 operands are split into bf16 parts).
//
// All contractions go through v_mfma_f32_16x16x32_bf16 (wave64):
//     D[m][n] += sum_kk A[m][kk] * B[kk][n],   m, n in 0..15, kk in 0..31
// operand layout per lane l (r = l % 16, g = l / 16):
//     A: 8 bf16 = A[m = r][kk = 8g .. 8g+7]        B: 8 bf16 = B[kk = 8g .. 8g+7][n = r]
//     D: 4 f32  = D[m = 4g .. 4g+3][n = r]
// The contraction index kk may be any fixed permutation of the mathematical
// index as long as A and B use the same one, and the rows of A (columns of B)
// may be any permutation of the output index.  The kernels below choose those
// permutations so that
//   * a lane's 16-byte piece of a feature row (8 consecutive hidden channels
//     of one token) is at once a global-memory vector load, an MFMA operand
//     and the position of the MFMA result it must be combined with, and
//   * the accumulators of the projection are, after conversion to bf16,
//     directly the operand of the reconstruction,
// so no value ever moves between lanes.
//
// Basis operands are pre-packed once per fitted basis (svdcache_pack_basis)
// as bf16 "high" and "low" parts (V = hi + lo to ~16 significant bits) in
// per-wavefront tiles of 64 lanes x 16 bytes.
#include <algorithm>
#include <type_traits>

#include "step_tiling.h"
#include "svdc_device.h"
#include "svdc_internal.h"

namespace svdc {

namespace {

constexpr int kWavesPerGroup = 4;

// Direct global-to-LDS load of 16 bytes per lane: lane l's bytes land at lds_wave_base + 16 l.  Counts in vmcnt
// like any other vector memory load; lds_wave_base must be the same in all lanes of the wave.
__device__ __forceinline__ void load_to_lds16(const void* gsrc_lane, void* lds_wave_base) {
  __builtin_amdgcn_global_load_lds(gsrc_lane, lds_wave_base, 16, 0, 0);
}

// rank padded to 32, 64 or 128 (one reconstruction MFMA contracts 32 coefficients)
__host__ __device__ inline int padded_rank(int k) { return k <= 32 ? 32 : (k <= 64 ? 64 : 128); }

// ---------------------------------------------------------------------------
// Packed basis.  Per block, four arrays of D * KP bf16 each (KP = padded rank):
//   P1hi, P1lo : projection operand.      tile (cg, jt) of 64 lanes x 8 bf16:
//                lane (r, g), e  ->  V[d = 32 cg + 8 g + e][j = 16 jt + r]
//   P2hi, P2lo : reconstruction operand, NEGATED.   tile (cg, t, kt):
//                lane (r, g), e  -> -V[d = 32 cg + 8 (r / 4) + 4 t + r % 4][j = 32 kt + 16 (e / 4) + 4 g + e % 4]
// with cg = d / 32 the 32-channel chunk, jt the 16-coefficient tile, t the
// half of the chunk, kt the 32-coefficient group.  Entries with j >= k are 0.
// ---------------------------------------------------------------------------
__global__ __launch_bounds__(256) void pack_basis_kernel(const float* __restrict__ V, uint16_t* __restrict__ P,
                                                         int D, int k, int KP) {
  const int b = blockIdx.y;
  const int64_t per = (int64_t)D * KP;           // elements per array
  const int64_t idx = (int64_t)blockIdx.x * 256 + threadIdx.x;
  if (idx >= per) return;
  const float* v = V + (int64_t)b * D * k;
  uint16_t* p = P + (int64_t)b * 4 * per;
  const int e = idx & 7, lane = (idx >> 3) & 63, r = lane & 15, g = lane >> 4;
  const int64_t tile = idx >> 9;
  {  // projection operand
    const int KT = KP / 16;
    const int jt = tile % KT, cg = tile / KT;
    const int d = 32 * cg + 8 * g + e, j = 16 * jt + r;
    const float x = j < k ? v[(int64_t)d * k + j] : 0.f;
    const bf16_t hi = (bf16_t)x;
    const bf16_t lo = (bf16_t)(x - (float)hi);
    p[idx] = __builtin_bit_cast(uint16_t, hi);
    p[per + idx] = __builtin_bit_cast(uint16_t, lo);
  }
  {  // reconstruction operand (negated so that the MFMA computes F - V C^T)
    const int KT2 = KP / 32;
    const int kt = tile % KT2, t = (tile / KT2) & 1, cg = tile / (2 * KT2);
    const int d = 32 * cg + 8 * (r >> 2) + 4 * t + (r & 3);
    const int j = 32 * kt + 16 * (e >> 2) + 4 * g + (e & 3);
    const float x = j < k ? -v[(int64_t)d * k + j] : 0.f;
    const bf16_t hi = (bf16_t)x;
    const bf16_t lo = (bf16_t)(x - (float)hi);
    p[2 * per + idx] = __builtin_bit_cast(uint16_t, hi);
    p[3 * per + idx] = __builtin_bit_cast(uint16_t, lo);
  }
}

// ---------------------------------------------------------------------------
// Packed coefficient state: S [B, N, k] float32 as the operand words of the cached step.  Per block, 16-row tile and
// group kt of 32 coefficients two words of 64 lanes x 16 bytes (bf16 high part, then low part) of -S:
//   lane (r, g), e  ->  -S[row = 16 tile + r][j = 32 kt + 16 (e / 4) + 4 g + e % 4]     (0 for row >= N, j >= k)
// word index ((b ntile + tile) KT2 + kt) 2 + part.  The full step writes the same words next to S when asked.
// ---------------------------------------------------------------------------
__global__ __launch_bounds__(256) void pack_state_kernel(const float* __restrict__ S, u32x4* __restrict__ Sp, int N,
                                                         int k, int KT2, int64_t words_per_block) {
  const int b = blockIdx.y;
  const int64_t w = (int64_t)blockIdx.x * kWavesPerGroup + (threadIdx.x >> 6);   // (tile, kt)
  if (w >= words_per_block) return;
  const int lane = threadIdx.x & 63, r = lane & 15, g = lane >> 4;
  const int kt = (int)(w % KT2);
  const int64_t tile = w / KT2;
  const int64_t row = tile * 16 + r;
  float c8[8];
#pragma unroll
  for (int t = 0; t < 2; ++t) {
    const int j = 32 * kt + 16 * t + 4 * g;
    f32x4 x = {0.f, 0.f, 0.f, 0.f};
    if (row < N && j < k) x = *reinterpret_cast<const f32x4*>(S + ((int64_t)b * N + row) * k + j);
#pragma unroll
    for (int i = 0; i < 4; ++i) c8[4 * t + i] = -x[i];
  }
  u32x4 hi, lo;
  split_operand(c8, &hi, &lo);
  u32x4* out = Sp + ((int64_t)b * words_per_block + w) * 2 * 64 + lane;
  out[0] = hi;
  out[64] = lo;
}

// Eight consecutive channels of one token as they sit in memory and in registers.  bf16: 16 bytes,
// exact as an MFMA operand.  float32: 32 bytes; as an MFMA operand it is split into bf16 high + low parts.
template <typename T>
struct RowPiece;
template <>
struct RowPiece<bf16_t> {
  u32x4 w;
  __device__ __forceinline__ void load(const bf16_t* p) { w = *reinterpret_cast<const u32x4*>(p); }
  __device__ __forceinline__ f32x4 half(int t) const {
    return f32x4{bf16_lo(w[2 * t]), bf16_hi(w[2 * t]), bf16_lo(w[2 * t + 1]), bf16_hi(w[2 * t + 1])};
  }
  static __device__ __forceinline__ void store(bf16_t* p, const f32x4& x0, const f32x4& x1) {
    *reinterpret_cast<u32x4*>(p) =
        u32x4{pack_bf16(x0[0], x0[1]), pack_bf16(x0[2], x0[3]), pack_bf16(x1[0], x1[1]), pack_bf16(x1[2], x1[3])};
  }
};
template <>
struct RowPiece<float> {
  f32x4 x[2];
  __device__ __forceinline__ void load(const float* p) {
    x[0] = *reinterpret_cast<const f32x4*>(p);
    x[1] = *reinterpret_cast<const f32x4*>(p + 4);
  }
  __device__ __forceinline__ f32x4 half(int t) const { return x[t]; }
  static __device__ __forceinline__ void store(float* p, const f32x4& x0, const f32x4& x1) {
    *reinterpret_cast<f32x4*>(p) = x0;
    *reinterpret_cast<f32x4*>(p + 4) = x1;
  }
};

// ---------------------------------------------------------------------------
// Cached step (Sec. 3.5):  Fhat = S V^T + R   for bf16 R / Fhat.
//
// Basis-stationary: a wave keeps the (negated) reconstruction operands of NCW
// consecutive 32-channel chunks in registers and streams 16-row tiles of R past
// them, so the basis is read from L2 once per workgroup, not once per tile.
// A workgroup of 4 waves covers 4*NCW chunks (a "slab" of 128*NCW channels) and
// tiles_per_group row tiles; adjacent workgroup ids are adjacent slabs of the same
// rows.  Per tile and chunk: two MFMAs per 32 coefficients whose accumulator
// starts at R; the coefficient operand is -S (bf16 high + low parts), so the
// MFMA computes Fhat^T = R^T + (-V)(-S)^T.  PD tiles are kept in flight.
// EXT: the coefficient operand is sum_m w_m S_m over up to kMaxStates stored states (forecasters that are linear
// in them, Sec. 5.3) and a tensor X may be added to the result (Out = C_hat V^T + R + X).
// ---------------------------------------------------------------------------

// PS: the coefficient state comes as packed operand words (packed_state_kernel / the full step's second state
// output) instead of float32 rows: nothing is converted per tile.
// MSX, HX (EXT only): registers are held for MSX coefficient states per tile in flight, and for the added tensor only
// with HX -- a forecaster of two states that adds nothing should not pay for four states and a second row tile.
// SHARED: each wave loads (and combines, and converts) a quarter of a tile's coefficients and the four pass the operand words to each
// other through LDS, one barrier per tile; otherwise every wave loads all of them, at rank 64 a third of what the workgroup asks for with bf16
// rows, at rank 128 a half, and holds them in registers.  What those cost most, requests or registers, was not separated; with the registers that sharing
// frees, two workgroups per compute unit run where the table (forecast_variant) says so.  us, every wave and shared, inputs in turn: 2 x 119056 x
// 3072 bf16 rank 64 695 -> 611, 16 x 4608 rank 64 218 -> 195, rank 128 299 -> 256, single operands 193 -> 185 and 236 -> 202; 18432 rows of float32,
// rank 32, 64, 128 95 -> 90, 97 -> 93, 111 -> 103; two states and an added tensor, 19 x 4608 bf16 rank 16 322 -> 318, 16 blocks rank 64 359 -> 281, 8
// blocks rank 128 515 -> 181.  Not for plain bf16 calls up to rank 32 (57 x 4608, the same buffers again: 606 and 610 us).
template <typename T, int NCW, int KT2, bool SPLIT, int PD, bool EXT, bool PS, int MSX, bool HX, bool SHARED, int WPE>
__global__ __launch_bounds__(256, WPE) void forecast_mfma_kernel(const CoefStates cs, const uint16_t* __restrict__ P,
                                                            const T* R, const T* X, T* Fh, int N, int D, int k,
                                                            int64_t ldf, int64_t bstride, int NS,
                                                            int groups_per_block, int tiles_per_group) {
  static_assert(!(PS && EXT), "the packed state serves the plain cached step");
  const int slab = blockIdx.x % NS;
  const int rgb = blockIdx.x / NS;
  const int b = rgb / groups_per_block, rg = rgb % groups_per_block;
  const int wave = SHARED ? __builtin_amdgcn_readfirstlane(threadIdx.x >> 6) : threadIdx.x >> 6, lane = threadIdx.x & 63, r = lane & 15, g = lane >> 4;
  constexpr int KP = KT2 * 32, NP = SPLIT ? 2 : 1;
  // coefficients of a tile as items: 16 of the rank for all rows (half an operand word), or a packed word; the first, how many and in which
  // steps a wave loads them
  constexpr int ITEMS = PS ? KT2 * NP : KT2 * 2, MINE = SHARED ? (ITEMS + kWavesPerGroup - 1) / kWavesPerGroup : ITEMS;
  const int item0 = SHARED ? wave : 0;
  constexpr int kItemStep = SHARED ? kWavesPerGroup : 1;
  __shared__ u32x4 shared_words[SHARED ? 2 : 1][SHARED ? KT2 : 1][NP][SHARED ? 64 : 1];   // two buffers: one barrier per tile
  const int64_t per = (int64_t)D * KP;
  const u32x4* P2hi = reinterpret_cast<const u32x4*>(P + (int64_t)b * 4 * per + 2 * per);
  const u32x4* P2lo = reinterpret_cast<const u32x4*>(P + (int64_t)b * 4 * per + 3 * per);
  const int cg0 = (slab * kWavesPerGroup + wave) * NCW;
  const T* rbase = R + (int64_t)b * bstride + 32 * cg0 + 8 * g;
  T* obase = Fh + (int64_t)b * bstride + 32 * cg0 + 8 * g;
  // EXT: the coefficient forecast is sum_m w_m S_m over up to kMaxStates stored states, and a tensor X
  // (nullable) is added to the result; otherwise the single state cs.s[0] with weight 1, or -1 for a residual (R - S V^T).
  constexpr int MS = EXT ? MSX : 1;
  const int ntile_block = (N + 15) / 16;
  const bool has_x = EXT && HX && X != nullptr;
  const T* xbase = has_x ? X + (int64_t)b * bstride + 32 * cg0 + 8 * g : nullptr;
  const int64_t soff = (int64_t)b * N * k;
  // Row tiles rg, rg + groups_per_block, ...: the workgroups of a block advance through its rows side by
  // side, which keeps the addresses in flight close together (measurably kinder to HBM than giving each
  // workgroup a contiguous range of tiles).
  const int ntiles = min(tiles_per_group, (ntile_block - rg + groups_per_block - 1) / groups_per_block);

  RowPiece<T> rin[PD][NCW];
  RowPiece<T> xin[PD][(EXT && HX) ? NCW : 1];
  f32x4 sraw[PD][PS ? 1 : MS][PS ? 1 : MINE];
  u32x4 spk[PD][PS ? MINE : 1];   // packed state
  const u32x4* spbase = PS ? reinterpret_cast<const u32x4*>(cs.s[0]) + (int64_t)b * ntile_block * KT2 * 2 * 64 + lane : nullptr;
  // lane (r, g) needs S[row][j = 16 item + 4 g + i], i = 0..3 (zero beyond k)
  auto load_tile = [&](int tile, int u) {
    const int row = min(tile * 16 + r, N - 1);
    if constexpr (PS) {
#pragma unroll
      for (int q = 0; q < MINE; ++q) {
        const int item = item0 + kItemStep * q;
        if (SHARED && item >= ITEMS) break;
        spk[u][q] = spbase[(((int64_t)tile * KT2 + item / NP) * 2 + item % NP) * 64];
      }
    } else {
      // states outside: one branch on their number for all items (one per item took 1 x 1065 x 512 bf16, rank 4, three states 3.0 -> 3.2 us)
#pragma unroll
      for (int ms = 0; ms < MS; ++ms) {
        if (ms >= cs.m) break;
#pragma unroll
        for (int q = 0; q < MINE; ++q) {
          const int item = item0 + kItemStep * q, j = 16 * item + 4 * g;
          if (SHARED && item >= ITEMS) break;
          sraw[u][ms][q] = (j < k) ? *reinterpret_cast<const f32x4*>(cs.s[ms] + soff + (int64_t)row * k + j) : f32x4{0.f, 0.f, 0.f, 0.f};
        }
      }
    }
#pragma unroll
    for (int c = 0; c < NCW; ++c) rin[u][c].load(rbase + (int64_t)row * ldf + 32 * c);
    if constexpr (EXT && HX) {
      if (has_x) {
#pragma unroll
        for (int c = 0; c < NCW; ++c) xin[u][c].load(xbase + (int64_t)row * ldf + 32 * c);
      }
    }
  };
#pragma unroll
  for (int u = 0; u < PD; ++u)
    if (u < ntiles) load_tile(rg + u * groups_per_block, u);

  u32x4 a_hi[NCW][2][KT2], a_lo[NCW][2][KT2];
#pragma unroll
  for (int c = 0; c < NCW; ++c)
#pragma unroll
    for (int t = 0; t < 2; ++t)
#pragma unroll
      for (int kt = 0; kt < KT2; ++kt) {
        const int64_t ti = ((int64_t)(cg0 + c) * 2 + t) * KT2 + kt;
        a_hi[c][t][kt] = P2hi[ti * 64 + lane];
        if (SPLIT) a_lo[c][t][kt] = P2lo[ti * 64 + lane];
      }

  for (int it = 0; it < ntiles; it += PD) {
#pragma unroll
    for (int u = 0; u < PD; ++u) {
      if (it + u >= ntiles) continue;
      const int tile = rg + (it + u) * groups_per_block;
      u32x4 words[KT2][NP];
      auto at = [&](int kt, int part) -> u32x4& {
        if constexpr (SHARED) return shared_words[(it + u) & 1][kt][part][lane];
        else return words[kt][part];
      };
#pragma unroll
      for (int q = 0; q < MINE; ++q) {
        const int item = item0 + kItemStep * q;
        if (SHARED && item >= ITEMS) break;
        if constexpr (PS) {
          at(item / NP, item % NP) = spk[u][q];
        } else {
          float c4[4];
#pragma unroll
          for (int i = 0; i < 4; ++i) {
            if constexpr (EXT) {
              float x = cs.w[0] * sraw[u][0][q][i];
#pragma unroll
              for (int ms = 1; ms < MS; ++ms)
                if (ms < cs.m) x = __builtin_fmaf(cs.w[ms], sraw[u][ms][q][i], x);
              c4[i] = -x;
            } else {
              c4[i] = -cs.w[0] * sraw[u][0][q][i];
            }
          }
          const uint32_t h0 = pack_bf16(c4[0], c4[1]), h1 = pack_bf16(c4[2], c4[3]);
          auto put = [&](int part, uint32_t a, uint32_t c) {
            if constexpr (SHARED) {
              reinterpret_cast<uint2*>(&at(item / 2, part))[item % 2] = make_uint2(a, c);
            } else {
              words[item / 2][part][2 * (item % 2)] = a;
              words[item / 2][part][2 * (item % 2) + 1] = c;
            }
          };
          put(0, h0, h1);
          if (SPLIT)
            put(NP - 1, pack_bf16(c4[0] - bf16_lo(h0), c4[1] - bf16_hi(h0)), pack_bf16(c4[2] - bf16_lo(h1), c4[3] - bf16_hi(h1)));
        }
      }
      if constexpr (SHARED) {
        // only LDS has to be in order here: loads and stores of rows stay in flight
        __builtin_amdgcn_fence(__ATOMIC_RELEASE, "workgroup", "local");
        __builtin_amdgcn_s_barrier();
        __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "workgroup", "local");
#pragma unroll
        for (int kt = 0; kt < KT2; ++kt)
#pragma unroll
          for (int part = 0; part < NP; ++part) words[kt][part] = at(kt, part);
      }
      const int row = tile * 16 + r;
#pragma unroll
      for (int c = 0; c < NCW; ++c) {
        f32x4 res[2];
#pragma unroll
        for (int t = 0; t < 2; ++t) {
          f32x4 acc = rin[u][c].half(t);
          if constexpr (EXT && HX) {
            if (has_x) {
              const f32x4 xa = xin[u][c].half(t);
              acc[0] += xa[0]; acc[1] += xa[1]; acc[2] += xa[2]; acc[3] += xa[3];
            }
          }
#pragma unroll
          for (int kt = 0; kt < KT2; ++kt) {
            acc = mfma16(a_hi[c][t][kt], words[kt][0], acc);
            if (SPLIT) {
              acc = mfma16(a_hi[c][t][kt], words[kt][NP - 1], acc);
              acc = mfma16(a_lo[c][t][kt], words[kt][0], acc);
            }
          }
          res[t] = acc;
        }
        if (row < N) RowPiece<T>::store(obase + (int64_t)row * ldf + 32 * c, res[0], res[1]);
      }
      if (it + u + PD < ntiles) load_tile(tile + PD * groups_per_block, u);
    }
  }
}

// ---------------------------------------------------------------------------
// Full-compute step (Eq. 8-11) for bf16 F / R, one pass over F.
// Persistent workgroups (one per compute unit) walk over row tiles; a workgroup
// of 4 waves holds a tile of 16*RT token rows x D channels in registers: wave w
// keeps the channels [w D/4, (w+1) D/4) of all rows as packed bf16
// (RT * CH * 4 VGPRs, CH = D / 128 chunks of 32 channels).
//   phase 1  C^T partial = V^T F^T over the wave's channels (MFMA); the basis
//            operands stream from L2 through a ring of RD operand words so that
//            their latency is covered; partials of the 4 waves are summed through
//            LDS in a fixed order
//   EMA      wave w updates S (and writes C) for row tile w, w+4, ...
//   phase 2  R^T = F^T - V C^T per chunk: accumulator starts at F, A operand
//            is the negated basis, B operand is C (bf16 high [+ low] parts)
//   then     the next tile's rows are requested in one burst, so the loads are
//            in flight while nothing else of this wave waits behind them
// S1 / S2: use the low parts of the basis (and of C) in phase 1 / phase 2.
// REMA: the residual state is smoothed as well (ablation of Sec. 4.5): R = (1 - alpha_r) Rp + alpha_r (F - C V^T),
// with the previous residual Rp read chunk by chunk a few chunks ahead; Rp may be the buffer R.
// LT = 1 (bf16 only): one more row tile per workgroup tile lives in LDS, as an image of the registers it would
// occupy (96 KB at 3072 channels).  It arrives by direct global-to-LDS loads (lane l's 16 bytes land at
// base + 16 l), each wave reads back only what it loaded itself, and every basis operand then serves RT + 1
// row tiles: a third less basis traffic from L2 per token row at RT = 2.
// F and R may alias: a tile is completely on chip (registers, LDS) before it is overwritten.
// ---------------------------------------------------------------------------
template <typename T, int CH, int RT, int KT2, bool S1, bool S2, int RD, bool REMA, int LT = 0>
__global__ __launch_bounds__(256) void full_step_mfma_kernel(const T* F, const uint16_t* __restrict__ P,
                                                             T* R, const T* Rp, float alpha_r, float* S, float* C,
                                                             int N, int k, int64_t ldf, int64_t bstride,
                                                             float alpha, int init, int tiles_per_block,
                                                             int total, u32x4* Sp) {
  constexpr int KP = KT2 * 32, KT = KT2 * 2, D = CH * 128;
  constexpr int M = CH * KT;   // basis operand items per wave and phase (a high + a low 16-byte word per lane each)
  constexpr int RA = RT + LT;  // row tiles per workgroup tile: RT in registers, LT in LDS
  static_assert(LT == 0 || (LT == 1 && !REMA && sizeof(T) == 2), "the LDS row tile is for bf16 features, plain residual");
  __shared__ f32x4 part[kWavesPerGroup][KT][RA][64];
  __shared__ u32x4 ftile[LT ? kWavesPerGroup : 1][LT ? CH : 1][LT ? 64 : 1];
  const int wave = threadIdx.x >> 6, lane = threadIdx.x & 63, r = lane & 15, g = lane >> 4;
  const int64_t per = (int64_t)D * KP;
  const int cg0 = wave * CH;
  int v = blockIdx.x;
  if (v >= total) return;

  // the wave's slab of the tile: 8 channels per lane per (row tile, chunk)
  constexpr bool kF32 = sizeof(T) == 4;
  RowPiece<T> f[RT][CH];
  auto load_f_chunk = [&](int vv, int c) {
    const int b = vv / tiles_per_block, tile = vv % tiles_per_block;
    const T* fbase = F + (int64_t)b * bstride + 32 * (cg0 + c) + 8 * g;
#pragma unroll
    for (int rt = 0; rt < RT; ++rt) {
      const int row = min(tile * 16 * RA + 16 * rt + r, N - 1);
      f[rt][c].load(fbase + (int64_t)row * ldf);
    }
    if constexpr (LT > 0) {
      const int row = min(tile * 16 * RA + 16 * RT + r, N - 1);
      load_to_lds16(fbase + (int64_t)row * ldf, &ftile[wave][c][0]);
    }
  };
#pragma unroll
  for (int c = 0; c < CH; ++c) load_f_chunk(v, c);

  for (; v < total; v += gridDim.x) {
    const int b = v / tiles_per_block, tile = v % tiles_per_block;
    const u32x4* P1hi = reinterpret_cast<const u32x4*>(P + (int64_t)b * 4 * per) + lane;
    const u32x4* P1lo = reinterpret_cast<const u32x4*>(P + (int64_t)b * 4 * per + per) + lane;
    const u32x4* P2hi = reinterpret_cast<const u32x4*>(P + (int64_t)b * 4 * per + 2 * per) + lane;
    const u32x4* P2lo = reinterpret_cast<const u32x4*>(P + (int64_t)b * 4 * per + 3 * per) + lane;
    const int row0 = tile * 16 * RA;
    T* obase = R + (int64_t)b * bstride + 8 * g;

    // ---- phase 1: acc[jt][rt] = C^T[j = 16 jt + 4 g + i][row = 16 rt + r] over this wave's channels.
    // Operand item m = (chunk c, coefficient tile jt), consecutive in the packed basis; RD items in flight.
    const u32x4* p1h = P1hi + (int64_t)cg0 * KT * 64;
    const u32x4* p1l = P1lo + (int64_t)cg0 * KT * 64;
    u32x4 rh[RD], rl[RD];
#pragma unroll
    for (int m = 0; m < RD; ++m)
      if (m < M) {
        rh[m] = p1h[m * 64];
        if (S1) rl[m] = p1l[m * 64];
      }
    f32x4 acc[KT][RA];
#pragma unroll
    for (int jt = 0; jt < KT; ++jt)
#pragma unroll
      for (int rt = 0; rt < RA; ++rt) acc[jt][rt] = f32x4{0.f, 0.f, 0.f, 0.f};
    u32x4 lnext;            // the LDS row tile's piece of the next chunk, read one chunk ahead
    if constexpr (LT > 0) lnext = ftile[wave][0][lane];
    __builtin_amdgcn_sched_barrier(0);
    u32x4 bh[RA], bl[RA];   // feature operand of the current chunk: exact for bf16; high + low parts for float32
#pragma unroll
    for (int m = 0; m < M; ++m) {
      const int c = m / KT, jt = m % KT, slot = m % RD;
      if (jt == 0) {
        if constexpr (LT > 0) {
          bh[RT] = lnext;
          if (c + 1 < CH) lnext = ftile[wave][c + 1][lane];
        }
#pragma unroll
        for (int rt = 0; rt < RT; ++rt) {
          if constexpr (kF32) {
            const f32x4 x0 = f[rt][c].half(0), x1 = f[rt][c].half(1);
            const float x8[8] = {x0[0], x0[1], x0[2], x0[3], x1[0], x1[1], x1[2], x1[3]};
            split_operand(x8, &bh[rt], &bl[rt]);
          } else {
            bh[rt] = f[rt][c].w;
          }
        }
      }
#pragma unroll
      for (int rt = 0; rt < RA; ++rt) {
        acc[jt][rt] = mfma16(rh[slot], bh[rt], acc[jt][rt]);
        if (kF32) acc[jt][rt] = mfma16(rh[slot], bl[rt], acc[jt][rt]);
        if (S1) acc[jt][rt] = mfma16(rl[slot], bh[rt], acc[jt][rt]);
      }
      if (m + RD < M) {
        rh[slot] = p1h[(m + RD) * 64];
        if (S1) rl[slot] = p1l[(m + RD) * 64];
      }
      __builtin_amdgcn_sched_barrier(0);
    }

    // REMA: the residual state is smoothed too, R = (1 - alpha_r) R_prev + alpha_r (F - C V^T); PR chunks of the
    // previous residual are kept in flight
    constexpr int PR = 4;
    RowPiece<T> rp[REMA ? PR : 1][REMA ? RT : 1];
    const T* pbase = REMA ? Rp + (int64_t)b * bstride + 8 * g : nullptr;
    auto load_prev = [&](int c) {
      if constexpr (REMA) {
#pragma unroll
        for (int rt = 0; rt < RT; ++rt) {
          const int row = min(row0 + 16 * rt + r, N - 1);
          rp[c % PR][rt].load(pbase + (int64_t)row * ldf + 32 * (cg0 + c));
        }
      }
    };
    if constexpr (REMA) {
#pragma unroll
      for (int c = 0; c < PR; ++c)
        if (c < CH) load_prev(c);
    }

    // the first reconstruction operands are requested before the reduction so they arrive during it;
    // item n = (chunk c, half t, coefficient tile kt), again consecutive in memory
    const u32x4* p2h = P2hi + (int64_t)cg0 * 2 * KT2 * 64;
    const u32x4* p2l = P2lo + (int64_t)cg0 * 2 * KT2 * 64;
    u32x4 qh[RD], ql[RD];
#pragma unroll
    for (int n = 0; n < RD; ++n)
      if (n < M) {
        qh[n] = p2h[n * 64];
        if (S2) ql[n] = p2l[n * 64];
      }
    __builtin_amdgcn_sched_barrier(0);

    // sum the four partial products through LDS, same order in every wave
#pragma unroll
    for (int jt = 0; jt < KT; ++jt)
#pragma unroll
      for (int rt = 0; rt < RA; ++rt) part[wave][jt][rt][lane] = acc[jt][rt];
    __syncthreads();
#pragma unroll
    for (int jt = 0; jt < KT; ++jt)
#pragma unroll
      for (int rt = 0; rt < RA; ++rt) {
        f32x4 s = part[0][jt][rt][lane];
#pragma unroll
        for (int w = 1; w < kWavesPerGroup; ++w) {
          const f32x4 p = part[w][jt][rt][lane];
          s[0] += p[0]; s[1] += p[1]; s[2] += p[2]; s[3] += p[3];
        }
        acc[jt][rt] = s;
      }
    __syncthreads();   // the next tile reuses `part`

    // EMA update (Eq. 11, alpha = 1 - beta) and coefficient output, one wave per row tile.  Sp (nullable): the new
    // state also leaves as the cached step's operand words (negated, bf16 high + low parts; zeros beyond N and k).
    const int ntile_block = (N + 15) / 16;
#pragma unroll
    for (int rt = 0; rt < RA; ++rt) {
      if ((rt % kWavesPerGroup) != wave) continue;
      const int row = row0 + 16 * rt + r;
      const int tile16 = tile * RA + rt;
      if (tile16 >= ntile_block) continue;
      const int64_t srow = ((int64_t)b * N + min(row, N - 1)) * k;
      f32x4 snew[KT];
#pragma unroll
      for (int jt = 0; jt < KT; ++jt) {
        const int j = 16 * jt + 4 * g;
        snew[jt] = f32x4{0.f, 0.f, 0.f, 0.f};
        if (j >= k || row >= N) continue;   // k is a multiple of 4: a group of four is all inside or all outside
        const f32x4 c4 = acc[jt][rt];
        f32x4 s4 = c4;
        if (!init) {
          const f32x4 old = *reinterpret_cast<const f32x4*>(S + srow + j);
#pragma unroll
          for (int i = 0; i < 4; ++i) s4[i] = ema(old[i], c4[i], alpha);
        }
        *reinterpret_cast<f32x4*>(S + srow + j) = s4;
        if (C) *reinterpret_cast<f32x4*>(C + srow + j) = c4;
        snew[jt] = s4;
      }
      if (Sp) {
#pragma unroll
        for (int kt = 0; kt < KT2; ++kt) {
          float c8[8];
#pragma unroll
          for (int t = 0; t < 2; ++t)
#pragma unroll
            for (int i = 0; i < 4; ++i) c8[4 * t + i] = -snew[2 * kt + t][i];
          u32x4 hi, lo;
          split_operand(c8, &hi, &lo);
          u32x4* w = Sp + ((((int64_t)b * ntile_block + tile16) * KT2 + kt) * 2) * 64 + lane;
          w[0] = hi;
          w[64] = lo;
        }
      }
    }

    // coefficient operand of the reconstruction: kk = 8 g + 4 t + i  <->  j = 32 kt + 16 t + 4 g + i
    u32x4 chi[RA][KT2], clo[RA][KT2];
#pragma unroll
    for (int rt = 0; rt < RA; ++rt)
#pragma unroll
      for (int kt = 0; kt < KT2; ++kt) {
        float c8[8];
#pragma unroll
        for (int t = 0; t < 2; ++t)
#pragma unroll
          for (int i = 0; i < 4; ++i) c8[4 * t + i] = acc[2 * kt + t][rt][i];
        split_operand(c8, &chi[rt][kt], &clo[rt][kt]);
      }
    if constexpr (LT > 0) lnext = ftile[wave][0][lane];
    __builtin_amdgcn_sched_barrier(0);

    // ---- phase 2: residual, chunk by chunk
#pragma unroll
    for (int c = 0; c < CH; ++c) {
      f32x4 x[RA][2];
#pragma unroll
      for (int rt = 0; rt < RT; ++rt)
#pragma unroll
        for (int t = 0; t < 2; ++t) x[rt][t] = f[rt][c].half(t);
      if constexpr (LT > 0) {
        RowPiece<bf16_t> piece;
        piece.w = lnext;
        if (c + 1 < CH) lnext = ftile[wave][c + 1][lane];
#pragma unroll
        for (int t = 0; t < 2; ++t) x[RT][t] = piece.half(t);
      }
#pragma unroll
      for (int tk = 0; tk < 2 * KT2; ++tk) {
        const int t = tk / KT2, kt = tk % KT2, n = c * 2 * KT2 + tk, slot = n % RD;
#pragma unroll
        for (int rt = 0; rt < RA; ++rt) {
          x[rt][t] = mfma16(qh[slot], chi[rt][kt], x[rt][t]);
          if (S2) {
            x[rt][t] = mfma16(qh[slot], clo[rt][kt], x[rt][t]);
            x[rt][t] = mfma16(ql[slot], chi[rt][kt], x[rt][t]);
          }
        }
        if (n + RD < M) {
          qh[slot] = p2h[(n + RD) * 64];
          if (S2) ql[slot] = p2l[(n + RD) * 64];
        }
      }
#pragma unroll
      for (int rt = 0; rt < RA; ++rt) {
        if constexpr (REMA) {
#pragma unroll
          for (int t = 0; t < 2; ++t) {
            const f32x4 old = rp[c % PR][rt].half(t);
#pragma unroll
            for (int i = 0; i < 4; ++i) x[rt][t][i] = (1.f - alpha_r) * old[i] + alpha_r * x[rt][t][i];
          }
        }
        const int row = row0 + 16 * rt + r;
        if (row < N) RowPiece<T>::store(obase + (int64_t)row * ldf + 32 * (cg0 + c), x[rt][0], x[rt][1]);
      }
      if constexpr (REMA) {
        if (c + PR < CH) load_prev(c + PR);
      }
      __builtin_amdgcn_sched_barrier(0);
    }

    // request the next tile
    const int vn = v + (int)gridDim.x;
    if (vn < total) {
#pragma unroll
      for (int c = 0; c < CH; ++c) load_f_chunk(vn, c);
    }
  }
}


}  // namespace

bool mfma_shape_supported(const svdc_shape& s) {
  if (s.D % 128 != 0 || s.k > 128 || s.k % 4 != 0) return false;
  // hidden sizes 256, 512, 1024, 1152, 1536, 1920, 2048, 2560, 3072, 4096, 5120 (the full step is instantiated per width)
  switch (s.D / 128) {
    case 2: case 4: case 8: case 9: case 12: case 15: case 16: case 20: case 24: case 32: case 40: return true;
    default: return false;
  }
}

size_t mfma_packed_bytes(const svdc_shape& s) {
  return (size_t)s.B * 4 * s.D * padded_rank(s.k) * sizeof(uint16_t);
}

int32_t launch_pack_basis(const svdc_shape& s, const float* V, void* packed, hipStream_t st) {
  const int KP = padded_rank(s.k);
  const int64_t per = (int64_t)s.D * KP;
  dim3 grid((unsigned)((per + 255) / 256), s.B);
  pack_basis_kernel<<<grid, 256, 0, st>>>(V, (uint16_t*)packed, s.D, s.k, KP);
  return launch_status();
}

namespace {

// Whether a kind of call shares the coefficients among the waves of a workgroup, where they are a fair part of what it loads, and whether only
// calls of more than one workgroup per compute unit do: one that has only a few row tiles does not win back the barriers.  Shared
// against not, in such short calls, inputs in turn: several states of rank <= 32 in float32 5 % slower on average (290 sampled calls, up to 16 %; 12 x 691 x 512:
// 12.7 and 13.2 us), in bf16 without an added tensor 11 % (113 calls); packed states of rank 64 and 128 the same on average, -7 to +8 % (4 x 703 x 1920, rank 112:
// 13.6 and 14.4 us); all others 1 to 40 % faster.
enum class Share { kNever, kLongCalls, kAlways };
template <typename T, int NCW, int KT2, bool EXT, bool PS, bool HX, int MSX>
constexpr Share forecast_share() {
  constexpr bool kF32 = sizeof(T) == 4;
  if (NCW == 12 && KT2 == 1 && HX) return Share::kNever;   // adding_takes_wide_slabs
  // three and four states and a tensor in float32, slabs of 6: the barriers cost 2 to 4 % in calls of every length and rank (130 sampled calls;
  // 10 x 11383 x 3072 rank 8 760 -> 793 us), narrower slabs gain as the other kinds do
  if (kF32 && NCW == 6 && KT2 == 1 && HX && MSX > 2) return Share::kNever;
  if (KT2 == 1 && !EXT) return kF32 ? Share::kLongCalls : Share::kNever;
  if (PS || (KT2 == 1 && (kF32 || !HX))) return Share::kLongCalls;
  return Share::kAlways;
}

// Row tiles in flight (PD) and waves per SIMD that the registers are cut for, by the chunks of a slab.  Shared: the fastest, or
// within 3 % of it, of 5 to 8 variants timed per kind at 3072 channels with 6 to 16 tiles per workgroup (kernel comment); the others keep
// one workgroup per compute unit.  NARROW: a slab that cached_tiling chose instead of the widest one.  Of 6000 calls of all
// eleven widths 1 in 100 takes 2 % or more longer than with every wave loading all coefficients.
struct ForecastVariant { int pd, wpe; };
template <typename T, int KT2, bool SPLIT, bool EXT, bool HX, int MSX>
constexpr ForecastVariant forecast_variant(int ncw, bool shared, bool narrow) {
  constexpr bool kF32 = sizeof(T) == 4;
  if (!shared) return {KT2 == 1 ? (narrow ? 2 : 1) : (KT2 == 2 && SPLIT && !kF32 ? 4 : 2), 1};
  if (KT2 == 1) {
    if (kF32) return ncw >= 5 ? ForecastVariant{1, 1} : ForecastVariant{EXT ? 1 : 2, EXT ? 1 : 2};
    if (!HX) return {1, 1};
    return ncw >= 6 ? ForecastVariant{MSX > 2 ? 1 : 2, 2} : ForecastVariant{2, 2};
  }
  if (KT2 == 2) {
    if (kF32) return EXT ? ForecastVariant{ncw >= 4 ? 1 : 2, 1} : ForecastVariant{ncw >= 3 ? 2 : 3, 2};
    if (EXT) return {2, ncw >= 5 || MSX > 2 ? 1 : 2};
    return SPLIT ? ForecastVariant{ncw >= 4 ? 3 : 4, ncw >= 5 ? 1 : 2} : ForecastVariant{ncw >= 8 ? 2 : (ncw >= 5 ? 3 : 4), 2};
  }
  if (kF32) return EXT ? ForecastVariant{ncw >= 3 ? 1 : 2, 1} : ForecastVariant{2, ncw >= 3 ? 1 : 2};
  if (EXT) return {2, SPLIT && ncw <= 2 && MSX <= 2 ? 2 : 1};
  return SPLIT ? ForecastVariant{ncw >= 4 ? 3 : 4, ncw >= 3 ? 1 : 2} : ForecastVariant{ncw >= 4 ? 3 : 4, ncw >= 5 ? 1 : 2};
}

// tpg: row tiles per workgroup, 0: not chosen yet (see step_tiling.h, which may also choose a narrower slab)
template <typename T, int NCW, int KT2, bool SPLIT, bool EXT, bool PS = false, bool NARROW = false>
int32_t forecast_launch(const svdc_shape& s, const CoefStates& cs, const void* packed, const void* R, const void* X,
                        void* Fhat, hipStream_t st, int cus, int tpg = 0) {
  const int NS = s.D / (128 * NCW);
  const int ntile = (s.N + 15) / 16;
  if (tpg == 0) {
    const int m = s.D / 128;
    constexpr bool kToOne = narrow_slab(24, NCW, KT2, sizeof(T) == 4, EXT) == 1;
    const CachedCall call{m, ntile, s.B, KT2, SPLIT ? 2 : 1, (int)sizeof(T), cus};
    const bool two_per_unit = EXT && X && KT2 == 1 && sizeof(T) == 2 && NCW < 12;
    const CachedTiling t = cached_tiling(call, NCW, narrow_slab(m, NCW, KT2, sizeof(T) == 4, EXT), two_per_unit ? kAddingOneRound : 0.7);
    if constexpr (kToOne) {
      if (t.chunks == 1) return forecast_launch<T, 1, KT2, SPLIT, EXT, PS, true>(s, cs, packed, R, X, Fhat, st, cus, t.tiles);
    }
    if constexpr (NCW > 3 && !kToOne) {
      if (t.chunks == 3) return forecast_launch<T, 3, KT2, SPLIT, EXT, PS, true>(s, cs, packed, R, X, Fhat, st, cus, t.tiles);
      if (t.chunks == 2) return forecast_launch<T, 2, KT2, SPLIT, EXT, PS, true>(s, cs, packed, R, X, Fhat, st, cus, t.tiles);
    }
    tpg = t.tiles;
  }
  const int gpb = (ntile + tpg - 1) / tpg;
  const int64_t grid = (int64_t)NS * gpb * s.B;
  if (grid > 0x7fffffff) return SVDC_E_SHAPE;
  auto launch = [&](auto states, auto adds) {
    constexpr int MSX = decltype(states)::value;
    constexpr bool HX = decltype(adds)::value;
    // the kind that may take slabs of 12 unshared (forecast_by_width), and the narrow ones chosen in their place
    constexpr bool kWide = PS && !SPLIT && KT2 == 2;
    constexpr Share share = kWide && NCW == 12 ? Share::kNever : forecast_share<T, NCW, KT2, EXT, PS, HX, MSX>();
    constexpr bool kTwoPlain = EXT && KT2 == 1 && sizeof(T) == 2 && !HX && MSX <= 2;
    auto go = [&](auto shared) {
      constexpr bool SHARED = decltype(shared)::value;
      constexpr ForecastVariant v = forecast_variant<T, KT2, SPLIT, EXT, HX, MSX>(NCW, SHARED, NARROW);
      forecast_mfma_kernel<T, NCW, KT2, SPLIT, v.pd, EXT, PS, MSX, HX, SHARED, v.wpe><<<(unsigned)grid, 256, 0, st>>>(
          cs, (const uint16_t*)packed, (const T*)R, (const T*)X, (T*)Fhat, s.N, s.D, s.k, s.ldf, s.block_stride, NS, gpb, tpg);
    };
    if constexpr (share != Share::kNever) {
      if (share == Share::kAlways ||
          (grid > cus && !(kWide && NARROW && s.D % 1536 == 0) && !(kTwoPlain && two_states_stay_unshared(ntile, s.B, s.D, s.k, cus)))) {
        go(std::true_type{});
        return;
      }
    }
    if constexpr (share != Share::kAlways) go(std::false_type{});
  };
  using Two = std::integral_constant<int, 2>;
  using Most = std::integral_constant<int, kMaxStates>;
  if constexpr (EXT) {
    // registers for two or four states, with or without the added tensor
    auto by_states = [&](auto adds) {
      if (cs.m <= 2) launch(Two{}, adds);
      else launch(Most{}, adds);
    };
    if (X) by_states(std::true_type{});
    else by_states(std::false_type{});
  } else {
    launch(Most{}, std::false_type{});
  }
  return launch_status();
}

// Slab per wave (NCW chunks): the first of the widths that suit the kind of call and divide D / 128.  Plain bf16 calls up to rank 32 take the widest
// that keeps the basis operands in registers; hidden sizes that 12 does not divide (1152 = 9 x 128, 2560 and 5120 = 20 and 40 x
// 128, 4096 = 32 x 128, 1920 = 15 x 128) the next.  Every width has a divisor of 2 or 3 chunks; the last one of a list is not asked for.  The kinds that
// share the coefficients: see forecast_mfma_kernel.
template <typename T, int KT2, bool SPLIT, bool EXT, bool PS>
struct ForecastCall {
  const svdc_shape& s;
  const CoefStates& cs;
  const void *packed, *R, *X;
  void* Fhat;
  hipStream_t st;
  int cus;
  template <int NCW, int... Rest>
  int32_t first() const {
    if constexpr (sizeof...(Rest) == 0) {
      return forecast_launch<T, NCW, KT2, SPLIT, EXT, PS>(s, cs, packed, R, X, Fhat, st, cus);
    } else {
      if ((s.D / 128) % NCW == 0) return forecast_launch<T, NCW, KT2, SPLIT, EXT, PS>(s, cs, packed, R, X, Fhat, st, cus);
      return first<Rest...>();
    }
  }
};
template <typename T, int KT2, bool SPLIT, bool EXT, bool PS = false>
int32_t forecast_by_width(const svdc_shape& s, const CoefStates& cs, const void* packed, const void* R, const void* X,
                          void* Fhat, hipStream_t st) {
  constexpr bool kF32 = sizeof(T) == 4;
  const ForecastCall<T, KT2, SPLIT, EXT, PS> call{s, cs, packed, R, X, Fhat, st, num_compute_units()};
  if constexpr (KT2 == 1 && !kF32) {
    if constexpr (!EXT) {
      return call.template first<12, 10, 9, 8, 6, 5, 4, 3, 2>();
    } else {
      const CachedCall tiles{s.D / 128, (s.N + 15) / 16, s.B, KT2, 2, (int)sizeof(T), call.cus};
      if (X && !adding_takes_wide_slabs(tiles, cs.m)) return call.template first<6, 4, 3, 2>();
      return call.template first<12, 6, 4, 3, 2>();
    }
  } else if constexpr (KT2 == 1) {
    return call.template first<6, 5, 4, 3, 2>();
  } else if constexpr (KT2 == 2) {
    if constexpr (kF32) return call.template first<3, 4, 2>();
    else if constexpr (!SPLIT && PS) {
      // Single operand words that are loaded as they are: 2 KB per tile, and four waves hold 1536 channels.  Slabs of 12 unshared beat
      // 6 shared in long calls, and in short ones, where they make way for narrow ones (57 x 4608 x 3072, 128 pieces of a tile per compute
      // unit: 636 and 649 us; 1 x 4608, 2.25 pieces: 15.9 and 17.4), but not between them (9 and 18 pieces: 1 x 18432 x 3072 50.3 and 49.5 us,
      // 16 x 4608 x 1536 100 and 95; 29: 149.6 and 150.2).  400 sampled calls of 1536 and 3072 channels: 0.98 of the time of slabs of 12 alone, none
      // more than 3 % slower.
      const int64_t pieces = (int64_t)((s.N + 15) / 16) * s.B * (s.D / 1536);
      if (pieces <= 4 * (int64_t)call.cus || pieces >= 48 * (int64_t)call.cus) return call.template first<12, 6, 8, 5, 4, 3, 2>();
      return call.template first<6, 8, 5, 4, 3, 2>();
    } else if constexpr (!SPLIT) return call.template first<6, 8, 5, 4, 3, 2>();
    else if constexpr (PS) return call.template first<5, 4, 3, 2>();
    else return call.template first<4, 3, 2>();
  } else {
    if constexpr (kF32 || (EXT && SPLIT)) return call.template first<2, 3>();
    else if constexpr (PS && !SPLIT) return call.template first<5, 4, 3, 2>();
    else return call.template first<4, 3, 2>();
  }
}

template <typename T, int CH, int RT, int KT2, bool SPLIT, int RD, bool REMA, int LT = 0>
int32_t full_step_launch(const svdc_shape& s, const void* F, const void* packed, void* R, float* S, float* C,
                         float alpha, int init, ResidualEma re, hipStream_t st) {
  const int tiles = (s.N + 16 * (RT + LT) - 1) / (16 * (RT + LT));
  const int64_t total = (int64_t)tiles * s.B;
  if (total > 0x7fffffff) return SVDC_E_SHAPE;
  const int grid = (int)std::min<int64_t>(total, num_compute_units());
  full_step_mfma_kernel<T, CH, RT, KT2, SPLIT, SPLIT, RD, REMA, LT><<<grid, 256, 0, st>>>(
      (const T*)F, (const uint16_t*)packed, (T*)R, (const T*)re.prev, re.alpha_r, S, C, s.N, s.k, s.ldf,
      s.block_stride, alpha, init, tiles, (int)total, (u32x4*)re.packed_state);
  return launch_status();
}

// Depth of the basis-operand ring (items) for tiles of tile_rows row tiles.
constexpr int ring_depth(int CH, int W, int KT2) {
  const int rt = tile_rows(CH, W, KT2);
  int rd = KT2 == 1 ? 12 : (KT2 == 2 ? 16 : 8);   // measured best at 3072 channels
  if (CH == 24 && W == 1) return rd;
  // float32 features at rank 65..128 and 3072 channels (the only width that this changes: the others have the same depth with
  // 478): the estimate is about 100 registers too high (370 used at a depth of 4, 511 at 8, all 512 in the variant that
  // smooths the residual, none spilled to memory), and the basis stream is what bounds those 16-row tiles: 18432 rows, 297 -> 234 us
  const int limit = W == 2 && KT2 == 4 && CH <= 24 ? 568 : 478;   // 4096 channels and up spill
  while (rd > 2 && full_step_regs(CH, W, KT2, rt, rd) > limit) rd -= 2;
  return rd;
}

template <typename T, int CH, int KT2, bool SPLIT>
int32_t full_step_by_size(const svdc_shape& s, const void* F, const void* packed, void* R, float* S, float* C,
                          float alpha, int init, ResidualEma re, hipStream_t st) {
  constexpr int W = sizeof(T) == 4 ? 2 : 1;
  constexpr int RT = tile_rows(CH, W, KT2), RD = ring_depth(CH, W, KT2);
  // the variant that also smooths the residual keeps a few chunks of the previous residual in flight: one row
  // tile less, except where the registers hold them beside the full tile and that takes less time (see step_tiling.h)
  if (re.prev) {
    if constexpr (RT > 1 && full_step_regs(CH, W, KT2, RT, RD) + 4 * RT * 4 * W <= 440) {
      if (smoothing_takes_full_tiles(RT, KT2, s.N, s.B, num_compute_units()))
        return full_step_launch<T, CH, RT, KT2, SPLIT, RD, true>(s, F, packed, R, S, C, alpha, init, re, st);
    }
    return full_step_launch<T, CH, (RT > 1 ? RT - 1 : 1), KT2, SPLIT, RD, true>(s, F, packed, R, S, C, alpha, init, re, st);
  }
  const int rows = full_step_rows(CH, W, KT2, SPLIT, s.N, s.B, num_compute_units());
  if constexpr (has_lds_tile(CH, W, KT2)) {
    constexpr int RDL = SPLIT ? 12 : 16;
    if (rows == RT + 1) return full_step_launch<T, CH, RT, KT2, SPLIT, RDL, false, 1>(s, F, packed, R, S, C, alpha, init, re, st);
  }
  if constexpr (RT > 2) {
    if (rows == 1) return full_step_launch<T, CH, 1, KT2, SPLIT, RD, false>(s, F, packed, R, S, C, alpha, init, re, st);
  }
  if constexpr (RT > 1) {
    if (rows == RT - 1) return full_step_launch<T, CH, RT - 1, KT2, SPLIT, RD, false>(s, F, packed, R, S, C, alpha, init, re, st);
  }
  return full_step_launch<T, CH, RT, KT2, SPLIT, RD, false>(s, F, packed, R, S, C, alpha, init, re, st);
}

template <typename T, int CH, bool SPLIT>
int32_t full_step_by_rank(const svdc_shape& s, const void* F, const void* packed, void* R, float* S, float* C,
                          float alpha, int init, ResidualEma re, hipStream_t st) {
  const int kp = padded_rank(s.k);
  if (kp == 32) return full_step_by_size<T, CH, 1, SPLIT>(s, F, packed, R, S, C, alpha, init, re, st);
  if (kp == 64) return full_step_by_size<T, CH, 2, SPLIT>(s, F, packed, R, S, C, alpha, init, re, st);
  return full_step_by_size<T, CH, 4, SPLIT>(s, F, packed, R, S, C, alpha, init, re, st);
}

template <typename T, bool SPLIT>
int32_t full_step_by_width(const svdc_shape& s, const void* F, const void* packed, void* R, float* S, float* C,
                           float alpha, int init, ResidualEma re, hipStream_t st) {
  switch (s.D / 128) {
    case 2: return full_step_by_rank<T, 2, SPLIT>(s, F, packed, R, S, C, alpha, init, re, st);
    case 4: return full_step_by_rank<T, 4, SPLIT>(s, F, packed, R, S, C, alpha, init, re, st);
    case 8: return full_step_by_rank<T, 8, SPLIT>(s, F, packed, R, S, C, alpha, init, re, st);
    case 9: return full_step_by_rank<T, 9, SPLIT>(s, F, packed, R, S, C, alpha, init, re, st);
    case 12: return full_step_by_rank<T, 12, SPLIT>(s, F, packed, R, S, C, alpha, init, re, st);
    case 15: return full_step_by_rank<T, 15, SPLIT>(s, F, packed, R, S, C, alpha, init, re, st);
    case 16: return full_step_by_rank<T, 16, SPLIT>(s, F, packed, R, S, C, alpha, init, re, st);
    case 20: return full_step_by_rank<T, 20, SPLIT>(s, F, packed, R, S, C, alpha, init, re, st);
    case 24: return full_step_by_rank<T, 24, SPLIT>(s, F, packed, R, S, C, alpha, init, re, st);
    case 32: return full_step_by_rank<T, 32, SPLIT>(s, F, packed, R, S, C, alpha, init, re, st);
    case 40: return full_step_by_rank<T, 40, SPLIT>(s, F, packed, R, S, C, alpha, init, re, st);
    default: return SVDC_E_SHAPE;
  }
}

}  // namespace

namespace {

template <bool EXT, bool PS = false>
int32_t forecast_dispatch(const svdc_shape& s, const CoefStates& cs, const void* packed, const void* R,
                          const void* X, void* Fhat, hipStream_t st) {
  const int kp = padded_rank(s.k);
  if (s.dtype == SVDC_F32) {
    if (kp == 32) return forecast_by_width<float, 1, true, EXT, PS>(s, cs, packed, R, X, Fhat, st);
    if (kp == 64) return forecast_by_width<float, 2, true, EXT, PS>(s, cs, packed, R, X, Fhat, st);
    return forecast_by_width<float, 4, true, EXT, PS>(s, cs, packed, R, X, Fhat, st);
  }
  // at rank <= 32 the split-operand kernel is the faster one (its matrix-core work is hidden anyway)
  if (kp == 32) return forecast_by_width<bf16_t, 1, true, EXT, PS>(s, cs, packed, R, X, Fhat, st);
  if (s.precision == SVDC_PRECISE) {
    if (kp == 64) return forecast_by_width<bf16_t, 2, true, EXT, PS>(s, cs, packed, R, X, Fhat, st);
    return forecast_by_width<bf16_t, 4, true, EXT, PS>(s, cs, packed, R, X, Fhat, st);
  }
  if (kp == 64) return forecast_by_width<bf16_t, 2, false, EXT, PS>(s, cs, packed, R, X, Fhat, st);
  return forecast_by_width<bf16_t, 4, false, EXT, PS>(s, cs, packed, R, X, Fhat, st);
}

}  // namespace

int32_t launch_full_step_mfma(const svdc_shape& s, const void* F, const void* packed, void* R, float* S,
                              float* C, float alpha, int init, ResidualEma re, hipStream_t st) {
  const bool f32 = s.dtype == SVDC_F32, split = f32 || s.precision == SVDC_PRECISE;
  if (const int rt = C && !re.prev ? full_step_projection_rows(s.N, s.B, s.D, s.k, f32, split, num_compute_units()) : 0) {
    const int kt = padded_rank(s.k) / 16;
    if (f32) step_project_stream_f32(kt, rt, s, F, packed, S, C, alpha, init, re.packed_state, st);
    else step_project_stream_bf16(kt, rt, s, F, packed, S, C, alpha, init, re.packed_state, st);
    CoefStates cs{};
    cs.s[0] = C;
    cs.w[0] = -1.f;
    cs.m = 1;
    return forecast_dispatch<false>(s, cs, packed, F, nullptr, R, st);
  }
  // float32 features always use the full operand split (a single bf16 operand would cost 8 of their 24 bits)
  if (f32) return full_step_by_width<float, true>(s, F, packed, R, S, C, alpha, init, re, st);
  return s.precision == SVDC_PRECISE
             ? full_step_by_width<bf16_t, true>(s, F, packed, R, S, C, alpha, init, re, st)
             : full_step_by_width<bf16_t, false>(s, F, packed, R, S, C, alpha, init, re, st);
}

int32_t launch_forecast_mfma(const svdc_shape& s, const float* S, const void* packed, const void* R,
                             void* Fhat, hipStream_t st) {
  CoefStates cs{};
  cs.s[0] = S;
  cs.w[0] = 1.f;
  cs.m = 1;
  return forecast_dispatch<false>(s, cs, packed, R, nullptr, Fhat, st);
}

int32_t launch_forecast_combine_mfma(const svdc_shape& s, const CoefStates& cs, const void* packed, const void* R,
                                     const void* X, void* Out, hipStream_t st) {
  return forecast_dispatch<true>(s, cs, packed, R, X, Out, st);
}

size_t mfma_packed_state_bytes(const svdc_shape& s) {
  return (size_t)s.B * ((size_t)(s.N + 15) / 16) * (padded_rank(s.k) / 32) * 2 * 1024;
}

int32_t launch_pack_state(const svdc_shape& s, const float* S, void* Sp, hipStream_t st) {
  const int KT2 = padded_rank(s.k) / 32;
  const int64_t words = (int64_t)((s.N + 15) / 16) * KT2;
  dim3 grid((unsigned)((words + kWavesPerGroup - 1) / kWavesPerGroup), s.B);
  pack_state_kernel<<<grid, 256, 0, st>>>(S, (u32x4*)Sp, s.N, s.k, KT2, words);
  return launch_status();
}

int32_t launch_forecast_packed_mfma(const svdc_shape& s, const void* Sp, const void* packed, const void* R,
                                    void* Fhat, hipStream_t st) {
  CoefStates cs{};
  cs.s[0] = static_cast<const float*>(Sp);   // the kernel reads it as operand words
  cs.w[0] = 1.f;
  cs.m = 1;
  return forecast_dispatch<false, true>(s, cs, packed, R, nullptr, Fhat, st);
}

}  // namespace svdc
