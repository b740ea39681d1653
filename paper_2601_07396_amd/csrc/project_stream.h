// Y = F Q, or the coefficients C = F V of a full step, for one group of 16-row tiles per workgroup, both operands streamed through
// registers (gfx950): kernel, its variants by tile height and the rule that picks one.  Included by one translation unit per
// storage type.
#pragma once
#include <algorithm>
#include <type_traits>

#include "fit_operands.h"
#include "svdc_internal.h"

namespace svdc {
namespace {

// ---------------------------------------------------------------------------
// project, streamed: the NW waves of a workgroup take different channels of the same RT row tiles and keep RT x KT accumulators;
// pieces of F and operand words of Q pass through a ring of DEPTH slots of CS chunks of 32 channels, the next slot's loads
// requested as soon as a slot is used, with no barrier until the waves' sums meet in LDS (in the order of the waves: the same
// bits every run).  Operand roles and output layouts as in fit_project_rows_kernel.
// What bounds it: F from HBM, the operand words of Q out of L2, once per workgroup, which queue in the same return path of the
// compute unit, and the latency of the last loads.  With every unit busy for the same number of rounds a call takes
// rounds x (RT + 1.25) (stream_rows), so the height is chosen for even rounds: 18432 rows on 256 units are 231 tiles of 80 rows, where 128
// rows left 112 units idle and 64 rows took two rounds.  4608 / 18432 / 20 x 4608 rows of 3072 channels, us, against waves that
// split the rows or hold slabs of Q (KT = 4 and less) in registers: float32 width 128 67 / 103 / 349 -> 34 / 67 / 312, width 64
// 27 / 86 / 289 -> 26 / 53 / 245; bf16 split width 128 53 / 68 / 225 -> 28 / 47 / 216, width 64 24 / 51 -> 20 / 37; bf16 plain
// width 128 44 / 47 -> 20 / 37, width 64 15.1 / 40 / 131 -> 14.8 / 30 / 126.
// What becomes of a tile of the product is up to Out:
//   FitOut<FRO>  Y as operand words of the back-projection or as float32 rows; FRO: also accumulates sum F^2 (for ||F||_F^2)
//   StepOut      coefficients C and the state S of a full step; operand roles exchanged, so that a lane has four
//                neighbouring coefficients of one row
// ---------------------------------------------------------------------------
template <bool FRO>
struct FitOut {
  static constexpr bool kNorm = FRO, kRowInLane = false;
  float* Y;
  u32x4* Yp;
  double* fro_acc;
  int l, ldy;
  // s: rows 4 g + i of the tile, column 16 jt + r
  template <typename T, int KT>
  __device__ __forceinline__ void store(const f32x4& s, int b, int tile, int jt, int N, int r, int g) const {
    const int row = 16 * tile + 4 * g, nsteps = (N + 31) / 32;
    if (Yp) {
      // packed output for the back-projection: a tile is one half of the words of a 32-row step
      if (tile / 2 >= nsteps) return;
      const int64_t word = ((int64_t)b * nsteps + tile / 2) * KT + jt;
      store_y_half(FPiece<T>{}, Yp, word, tile & 1, s, row, N);
      if ((tile & 1) == 0 && 16 * (tile + 1) >= N)        // no tile has the other half of the last step: zeros
        store_y_half(FPiece<T>{}, Yp, word, 1, s, row + 16, N);
      return;
    }
    const int j = 16 * jt + r;
#pragma unroll
    for (int e = 0; e < 4; ++e)
      if (row + e < N && j < l) Y[((int64_t)b * N + row + e) * ldy + j] = s[e];
  }
};
struct StepOut {
  static constexpr bool kNorm = false, kRowInLane = true;
  float *S, *C;         // C nullable
  float alpha;
  int init, k;
  uint2* Sp;            // nullable: the new state as operand words of the cached step too (negated, see pack_state_kernel)
  // s: row r of the tile, columns 16 jt + 4 g + i
  template <typename T, int KT>
  __device__ __forceinline__ void store(const f32x4& s, int b, int tile, int jt, int N, int r, int g) const {
    const int row = 16 * tile + r, j = 16 * jt + 4 * g, ntile = (N + 15) / 16;
    if (tile >= ntile) return;
    f32x4 snew = {0.f, 0.f, 0.f, 0.f};
    if (row < N && j < k) {                                // k is a multiple of 4
      const int64_t at = ((int64_t)b * N + row) * k + j;
      snew = s;
      if (!init) {
        const f32x4 old = *reinterpret_cast<const f32x4*>(S + at);
#pragma unroll
        for (int i = 0; i < 4; ++i) snew[i] = ema(old[i], s[i], alpha);
      }
      *reinterpret_cast<f32x4*>(S + at) = snew;
      if (C) *reinterpret_cast<f32x4*>(C + at) = s;
    }
    if (Sp) {
      uint2* w = Sp + ((((int64_t)b * ntile + tile) * (KT / 2) + jt / 2) * 2 * 64 + (threadIdx.x & 63)) * 2 + jt % 2;
      const uint32_t h0 = pack_bf16(-snew[0], -snew[1]), h1 = pack_bf16(-snew[2], -snew[3]);
      w[0] = make_uint2(h0, h1);
      w[2 * 64] = make_uint2(pack_bf16(-snew[0] - bf16_lo(h0), -snew[1] - bf16_hi(h0)), pack_bf16(-snew[2] - bf16_lo(h1), -snew[3] - bf16_hi(h1)));
    }
  }
};

// q_block: elements from one block's operand words to the next one's.  RUN: the waves take runs of that many slots in turn; 0: one share each.
template <typename T, int KT, int RT, int NW, int DEPTH, int CS, bool SPLIT, int WPE, int RUN, typename Out>
__global__ __launch_bounds__(64 * NW, WPE) void project_stream_kernel(const T* __restrict__ F, const uint16_t* __restrict__ Qp, int64_t q_block, Out out,
                                                                      int N, int D, int64_t ldf, int64_t bstride, int groups_per_block) {
  constexpr bool FRO = Out::kNorm;
  constexpr int NP = SPLIT ? 2 : 1;           // operand parts (high, low)
  constexpr int G = NW * KT >= 64 ? 1 : 2;    // row tiles that meet in LDS at a time (64 KB)
  __shared__ f32x4 part[NW][G][KT][64];
  __shared__ double norm[NW];
  const int b = blockIdx.x / groups_per_block, rg = blockIdx.x % groups_per_block;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), lane = threadIdx.x & 63, r = lane & 15, g = lane >> 4;
  const int64_t per = (int64_t)D * KT * 16;
  // the slots of CS chunks that are this wave's (D / 32 is a multiple of 4)
  const int all = D / (32 * CS), begin = wave * all / NW, n = (wave + 1) * all / NW - begin, first = RUN ? wave * RUN : begin;
  const u32x4* Qhi = reinterpret_cast<const u32x4*>(Qp + b * q_block) + (int64_t)first * CS * KT * 64 + lane;
  const u32x4* Qlo = Qhi + per / 8;
  const int tile0 = rg * RT;
  const T* rows[RT];
#pragma unroll
  for (int t = 0; t < RT; ++t)
    rows[t] = F + (int64_t)b * bstride + (int64_t)min((tile0 + t) * 16 + r, N - 1) * ldf + 32 * CS * first + 8 * g;

  struct Slot {
    FPiece<T> f[RT][CS];
    u32x4 q[CS][KT][NP];
  };
  Slot ring[DEPTH];
  f32x4 acc[RT][KT];
#pragma unroll
  for (int t = 0; t < RT; ++t)
#pragma unroll
    for (int jt = 0; jt < KT; ++jt) acc[t][jt] = f32x4{0.f, 0.f, 0.f, 0.f};
  // bf16: the two 64-byte halves of a 128-byte line belong to neighbouring chunks and are requested together where CS = 2
  auto load = [&](Slot& s, int slot) {
    const int i = RUN ? slot / max(RUN, 1) * NW * RUN + slot % max(RUN, 1) : slot;
#pragma unroll
    for (int t = 0; t < RT; ++t)
#pragma unroll
      for (int c = 0; c < CS; ++c) s.f[t][c].load(rows[t] + 32 * (CS * i + c));
#pragma unroll
    for (int c = 0; c < CS; ++c)
#pragma unroll
      for (int jt = 0; jt < KT; ++jt) {
        const int64_t w = ((int64_t)CS * i + c) * KT + jt;
        s.q[c][jt][0] = Qhi[w * 64];
        if (SPLIT) s.q[c][jt][NP - 1] = Qlo[w * 64];
      }
  };
  float ssq[RT] = {};      // per tile: rows beyond N leave the sum at the end, not in the loop
  auto use = [&](const Slot& s) {
#pragma unroll
    for (int c = 0; c < CS; ++c) {
      u32x4 fh[RT], fl[RT];
#pragma unroll
      for (int t = 0; t < RT; ++t) s.f[t][c].operands(&fh[t], &fl[t]);
#pragma unroll
      for (int jt = 0; jt < KT; ++jt) {
        auto times = [&](const u32x4(&f)[RT], const u32x4& q) {
#pragma unroll
          for (int t = 0; t < RT; ++t) acc[t][jt] = Out::kRowInLane ? mfma16(q, f[t], acc[t][jt]) : mfma16(f[t], q, acc[t][jt]);
        };
        times(fh, s.q[c][jt][0]);
        if (FPiece<T>::kTwoParts) times(fl, s.q[c][jt][0]);
        if (SPLIT) times(fh, s.q[c][jt][NP - 1]);
      }
      if (FRO) {
#pragma unroll
        for (int t = 0; t < RT; ++t) ssq[t] += s.f[t][c].sumsq();
      }
    }
  };
#pragma unroll
  for (int u = 0; u < DEPTH; ++u)
    if (u < n) load(ring[u], u);
  int i = 0;
  for (; i + 2 * DEPTH <= n; i += DEPTH) {    // no condition inside, so that only a slot's own loads are waited for
#pragma unroll
    for (int u = 0; u < DEPTH; ++u) {
      use(ring[u]);
      load(ring[u], i + u + DEPTH);
      __builtin_amdgcn_sched_barrier(0);
    }
  }
#pragma unroll
  for (int u = 0; u < DEPTH; ++u) {
    if (i + u < n) use(ring[u]);
    if (i + u + DEPTH < n) load(ring[u], i + u + DEPTH);
  }
#pragma unroll
  for (int u = 0; u < DEPTH; ++u)
    if (i + u + DEPTH < n) use(ring[u]);

  if (FRO) {
    double s = 0.0;
#pragma unroll
    for (int t = 0; t < RT; ++t)
      if ((tile0 + t) * 16 + r < N) s += (double)ssq[t];
    s = wave_sum(s);
    if (lane == 0) norm[wave] = s;
  }

#pragma unroll
  for (int t0 = 0; t0 < RT; t0 += G) {
#pragma unroll
    for (int tt = 0; tt < G; ++tt)
#pragma unroll
      for (int jt = 0; jt < KT; ++jt)
        if (t0 + tt < RT) part[wave][tt][jt][lane] = acc[t0 + tt][jt];
    __syncthreads();
    if constexpr (FRO) {
      if (t0 == 0 && out.fro_acc && threadIdx.x == 0) {
        // one atomic per workgroup: all of a block's add to one word (one per wave: 1152 of them took 5 us of 4608 rows' 25)
        double s = norm[0];
#pragma unroll
        for (int w = 1; w < NW; ++w) s += norm[w];
        atomicAdd(out.fro_acc + b, s);
      }
    }
    for (int item = wave; item < G * KT; item += NW) {
      const int tt = item / KT, jt = item % KT;
      if (t0 + tt >= RT) break;
      f32x4 s = part[0][tt][jt][lane];
#pragma unroll
      for (int w = 1; w < NW; ++w) s += part[w][tt][jt][lane];
      out.template store<T, KT>(s, b, tile0 + t0 + tt, jt, N, r, g);
    }
    if (t0 + G < RT) __syncthreads();
  }
}

// Waves, ring slots and chunks per slot for 1 to 6 row tiles: eight waves, two per SIMD to hide each other's waits, or four with twice the
// registers, whichever was timed faster, at 15 shapes and without the squares; each within 3 % of the best of 7 to 15 variants.
// norm: where the squares' sums would not fit beside them, so that no variant uses scratch (with the rows tested at every use 22 of the 48
// with squares did, 8 to 916 bytes a lane).  The last product of a fit of one block of 3072 channels, us, before and now: 23000 float32 rows
// width 32 75 -> 45, width 128 91 -> 67; 18432 width 128 72 -> 53; 12000 bf16 rows width 16 47 -> 18, width 64 38 -> 24.
struct StreamVariant {
  int waves, depth, chunks;
};
template <typename T, bool SPLIT>
constexpr StreamVariant stream_variant(int kt, int rt, bool norm) {
  if (norm && std::is_same<T, float>::value) {
    if ((kt == 2 && rt == 6) || (kt == 8 && rt == 2) || (kt == 4 && rt == 4)) return {8, 1, 1};
    if (kt == 8 && rt == 6) return {4, 1, 1};
  }
  if (norm && !std::is_same<T, float>::value && kt == 1 && rt == 4) return {4, 2, 2};
  const int x = kt == 1 ? 0 : (kt == 2 ? 1 : (kt == 4 ? 2 : 3));
  constexpr StreamVariant f32[4][6] = {
      {{8, 4, 1}, {8, 4, 1}, {8, 3, 1}, {4, 3, 1}, {8, 2, 1}, {4, 2, 1}},
      {{8, 4, 1}, {8, 3, 1}, {8, 3, 1}, {4, 3, 1}, {8, 2, 1}, {8, 2, 1}},
      {{8, 3, 1}, {8, 1, 2}, {8, 2, 1}, {4, 2, 1}, {8, 1, 1}, {8, 1, 1}},
      {{8, 2, 1}, {8, 1, 2}, {8, 1, 1}, {4, 2, 1}, {4, 2, 1}, {4, 2, 1}}};
  constexpr StreamVariant plain[4][6] = {
      {{8, 6, 2}, {8, 6, 2}, {8, 6, 2}, {4, 4, 2}, {4, 3, 2}, {4, 3, 2}},
      {{8, 4, 2}, {8, 3, 2}, {8, 4, 2}, {4, 3, 2}, {4, 3, 2}, {4, 2, 2}},
      {{8, 3, 2}, {8, 3, 2}, {8, 2, 2}, {4, 2, 2}, {4, 2, 2}, {4, 3, 2}},
      {{8, 2, 2}, {8, 2, 2}, {8, 3, 1}, {4, 2, 1}, {4, 2, 2}, {4, 2, 2}}};
  constexpr StreamVariant split[4][6] = {
      {{8, 4, 2}, {8, 3, 2}, {8, 5, 2}, {4, 3, 2}, {8, 3, 2}, {8, 2, 2}},
      {{8, 3, 2}, {8, 2, 2}, {8, 3, 2}, {4, 2, 2}, {8, 2, 2}, {8, 2, 2}},
      {{8, 3, 1}, {8, 2, 2}, {8, 3, 1}, {4, 3, 1}, {8, 1, 1}, {8, 1, 1}},
      {{8, 2, 1}, {8, 2, 1}, {4, 3, 1}, {4, 2, 1}, {4, 2, 1}, {4, 1, 1}}};
  return std::is_same<T, float>::value ? f32[x][rt - 1] : (SPLIT ? split[x][rt - 1] : plain[x][rt - 1]);
}

// A full step adds the channels up in the order of full_step_mfma_kernel, four waves and a chunk at a time, so that its results do not
// depend on which of the two a call takes (only one with a buffer for C comes here).  Ring slots for padded rank 32, 64, 128; 4608 x 3072
// float32 rows at rank 128 with eight waves 33 us, with four 37, elsewhere within 5 %.  A depth of 2 at six float32 tiles of rank 128 spilled: full
// step of 24000 x 1536 133 -> 128 us, 20 x 4608 x 2048 539 -> 522.
template <typename T, bool SPLIT>
constexpr StreamVariant step_variant(int kt, int rt) {
  const int x = kt == 2 ? 0 : (kt == 4 ? 1 : 2);
  constexpr int f32[3][6] = {{4, 3, 3, 3, 2, 2}, {4, 3, 2, 2, 3, 2}, {2, 2, 3, 2, 2, 1}};
  constexpr int split[3][6] = {{4, 4, 3, 3, 2, 2}, {4, 4, 3, 3, 2, 3}, {2, 4, 3, 2, 2, 1}};
  constexpr int plain[3][6] = {{4, 4, 4, 4, 3, 3}, {4, 4, 4, 4, 3, 3}, {4, 4, 3, 2, 3, 3}};
  return {4, std::is_same<T, float>::value ? f32[x][rt - 1] : (SPLIT ? split[x][rt - 1] : plain[x][rt - 1]), 1};
}

template <typename Out>
struct StreamCall {
  const svdc_shape& s;
  const void *F, *Qp;
  int64_t q_block;
  Out out;
  hipStream_t st;
};

template <typename T, int KT, int RT, bool SPLIT, typename Out>
void stream_launch(const StreamCall<Out>& c) {
  constexpr StreamVariant v = Out::kRowInLane ? step_variant<T, SPLIT>(KT, RT) : stream_variant<T, SPLIT>(KT, RT, Out::kNorm);
  // registers of the accumulators and the ring: two waves per SIMD where they fit
  constexpr int regs = 4 * RT * KT + v.depth * v.chunks * (RT * (int)sizeof(FPiece<T>) / 4 + KT * (SPLIT ? 8 : 4));
  constexpr int wpe = v.waves == 8 || regs <= (Out::kRowInLane ? 220 : 232) ? 2 : 1;
  const int groups = ((c.s.N + 15) / 16 + RT - 1) / RT;
  auto launch = [&](auto run) {
    project_stream_kernel<T, KT, RT, v.waves, v.depth, v.chunks, SPLIT, wpe, decltype(run)::value, Out><<<(unsigned)((int64_t)groups * c.s.B), 64 * v.waves, 0, c.st>>>(
        (const T*)c.F, (const uint16_t*)c.Qp, c.q_block, c.out, c.s.N, c.s.D, c.s.ldf, c.s.block_stride, groups);
  };
  // Plain operands of width 64 at the height of large calls: the waves take 128 channels in turn, the order in which kernels that hold slabs of 512
  // channels add up, so that the bits of such fits are theirs (Y is rounded to bf16 before its next use, and in another order a rounding flips now
  // and then: R of 57 x 4608 x 3072 moved by 6e-4).  57 x 4608 x 3072, a whole fit 2894 us, with one share for each wave 2882.
  if constexpr (!SPLIT && KT == 4 && RT == 5) {
    static_assert(v.waves == 4 && 4 % v.chunks == 0, "slabs of 4 waves x 4 chunks");
    if (c.s.D % 512 == 0) return launch(std::integral_constant<int, 4 / v.chunks>{});
  }
  launch(std::integral_constant<int, 0>{});
}
template <typename T, int KT, bool SPLIT, typename Out>
void stream_by_rows(int rt, const StreamCall<Out>& c) {
  switch (rt) {
    case 1: return stream_launch<T, KT, 1, SPLIT>(c);
    case 2: return stream_launch<T, KT, 2, SPLIT>(c);
    case 3: return stream_launch<T, KT, 3, SPLIT>(c);
    case 4: return stream_launch<T, KT, 4, SPLIT>(c);
    case 5: return stream_launch<T, KT, 5, SPLIT>(c);
    default: return stream_launch<T, KT, 6, SPLIT>(c);
  }
}
// kt: 1, 2, 4 or 8; a step comes here with those of at least MIN
template <typename T, bool SPLIT, int MIN = 1, typename Out>
void stream_by_width(int kt, int rt, const StreamCall<Out>& c) {
  if constexpr (MIN <= 1) {
    if (kt == 1) return stream_by_rows<T, 1, SPLIT>(rt, c);
  }
  if constexpr (MIN <= 2) {
    if (kt == 2) return stream_by_rows<T, 2, SPLIT>(rt, c);
  }
  if constexpr (MIN <= 4) {
    if (kt == 4) return stream_by_rows<T, 4, SPLIT>(rt, c);
  }
  stream_by_rows<T, 8, SPLIT>(rt, c);
}

}  // namespace
}  // namespace svdc
