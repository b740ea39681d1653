// Channel slab and row tiles per workgroup of the cached step, row tiles of the full step: host arithmetic only, apart from the launcher so that it
// can be checked without a GPU.
#pragma once
#include <stdint.h>

#include <algorithm>
#include <cmath>

namespace svdc {

// What a cached step launches: slabs of `chunks` x 128 channels, `tiles` row tiles of 16 per workgroup.
struct CachedTiling {
  int chunks, tiles;
};

// One launch: m = D / 128 chunks of channels, ntile row tiles, B blocks; kt2 = padded rank / 32, parts = 2 where the basis
// operands have a high and a low part and 1 otherwise, elem = bytes of a feature, cus compute units.
struct CachedCall {
  int m, ntile;
  int64_t B;
  int kt2, parts, elem, cus;

  int64_t groups(int tiles) const { return (ntile + tiles - 1) / tiles; }
  int64_t workgroups(CachedTiling t) const { return (int64_t)(m / t.chunks) * groups(t.tiles) * B; }
  // share of the machine's workgroup slots, over whole rounds, that do work
  double fill(CachedTiling t) const {
    const double rounds = (double)workgroups(t) / cus;
    return rounds / std::ceil(rounds) * ((double)ntile / ((double)t.tiles * groups(t.tiles)));
  }
  // Rounds x (row tiles + basis operands of the slab), in units of the features of one bf16 row tile and chunk (4 KB in,
  // 4 KB out).  The operands of a chunk are 8 KB per part and 32 coefficients and come out of L2 about twice as fast; the
  // matrix instructions add a twentieth per 32 coefficients and product.
  double cost(CachedTiling t) const {
    const int64_t rounds = (workgroups(t) + cus - 1) / cus;
    const double tile = elem / 2 + 0.05 * kt2 * (parts == 2 ? 3 : 1), basis = 0.5 * kt2 * parts;
    return (double)rounds * t.chunks * (std::min(t.tiles, ntile) * tile + basis);
  }
};

// The slab that a cached step may take in the place of its widest one of `chunks`, 0: none.  3 or 2 chunks; float32 rows above rank 32 go down to one chunk
// with several states, whose loads a short call waits for (us with 2 or 3 chunks and with one: 1 x 273 x 1152
// rank 48, two states 5.1 and 3.7, 2 x 404 x 512 rank 124 4.6 and 4.0; 700 calls of up to 30 MB), and at rank 128 where 3 chunks are the widest slab (1 x 439 x
// 1152: 5.1 and 4.3).
constexpr int narrow_slab(int m, int chunks, int kt2, bool f32, bool several_states) {
  if (f32 && kt2 > 1 && chunks > 1 && (several_states || (kt2 == 4 && chunks == 3))) return 1;
  return chunks <= 3 ? 0 : (m % 3 == 0 ? 3 : (m % 2 == 0 ? 2 : 0));
}

// Every workgroup loads the operands of its slab once and uses them for each of its row tiles, so a call that fills the
// machine takes 6 to 16 of them, the number whose grid fills whole rounds best (a grid of e.g. 16.03 x the compute units
// costs a 17th, nearly empty round): with fewer the operands outweigh the features, and rounding better gains little
// (28 x 1548 x 1920 float32, rank 96: 335 us with one tile, 243 us like this; two states 2 x 22551 x 4096 bf16, rank 96:
// 1278 and 828 us).
// A call for which even the best of these fills less than 0.7 leaves compute units idle (one block of 4608 x 3072 rows:
// 96 workgroups of 1536 channels).  It may take fewer tiles, and a slab of 3 or 2 chunks (`narrow`, 0 if there is none)
// instead of the widest one (narrow_slab), where that costs less: 23 -> 13 us for that block at rank 32, 23 -> 17 us at rank 64.  Not
// where many small workgroups would only load operands (43 x 129 x 2048, rank 128: 29 us wide, 46 us narrow); over 460
// sampled calls of up to two rounds this is within 4 % of the best of all choices.
// one_round: the fill that a call of at most one workgroup per unit needs to keep the widest slab.  0.9 where a unit holds two workgroups and bf16 rows
// have a tensor added, rank <= 32 (kAddingOneRound): below it half of the places for workgroups are empty (us at 0.7 and like this: 12 x 749 x 1536, four states 25.6 and
// 23.3, 8 x 534 x 2048, two states 16.5 and 15.2; of 900 calls 13 change, all faster, by 8 %).  Elsewhere
// it is mixed: of 835 calls of one state above rank 32, 46 change, 32 to less time and 14 to more, 3.5 % less on average.
inline CachedTiling cached_tiling(const CachedCall& call, int chunks, int narrow, double one_round = 0.7) {
  CachedTiling best{chunks, 16};
  for (int cand = 15; cand >= 6; --cand)
    if (call.fill({chunks, cand}) > call.fill(best) + 1e-9) best.tiles = cand;
  if (call.fill(best) >= (call.workgroups(best) <= call.cus ? one_round : 0.7)) return best;
  double least = 0.85 * call.cost(best);
  const int few = chunks > 3 || narrow > 0 ? narrow : chunks;
  for (int cand = std::min(16, call.ntile); few > 0 && cand >= 1; --cand) {
    const double c = call.cost({few, cand});
    if (c < least) {
      least = c;
      best = {few, cand};
    }
  }
  return best;
}

constexpr double kAddingOneRound = 0.9;

// Whether a cached step that adds a tensor (bf16, rank <= 32) takes slabs of 12 chunks, one workgroup per compute unit whose waves each load all
// coefficients, instead of slabs of 6 that share them, two workgroups per unit.  Wide ones are 2 to 4 % faster in long calls of well-filled rounds (from 40
// row tiles of 1536 channels per unit: 57 x 4608 x 3072 rank 32, two states 945 and 969 us), and above two states, where a third or fifth round of the
// others is a half-empty one (4 x 6865 x 3072, four states: 1.11 of the wide ones' time; 10 blocks of 1607 rows 1.04); elsewhere up to 17 % slower (19 x
// 4608 x 3072: 327 and 323 us).  Over 475 sampled calls of one and more rounds this takes 0.2 % longer on average than the better of the two, slabs of 6
// alone 0.8 %, of 12 alone 2.7 %.
inline bool adding_takes_wide_slabs(const CachedCall& call, int states) {
  if (call.m % 12 != 0) return false;
  const CachedTiling wide = cached_tiling(call, 12, 0), half = cached_tiling(call, 6, 0);
  if (call.m / 12 * call.ntile * call.B >= 40 * (int64_t)call.cus && call.fill(wide) >= 0.96) return true;
  const int64_t rounds = (call.workgroups(half) + call.cus - 1) / call.cus;
  return states > 2 && call.fill(wide) >= 0.7 && (rounds == 3 || rounds == 5);
}

// Whether the waves of a cached step of one or two states (bf16, nothing added) each load all coefficients in a long call: up to rank 16 those are one load
// per state and tile, and with rows of a power of two of channels the waves that a barrier keeps in step lose more than the loads cost (2 to 6 % from 25 row
// tiles of 1536 channels per unit, 9 sampled calls; 4 x 12079 x 4096 rank 8 165 -> 176 us); shorter calls, other widths and higher ranks gain 2 to 10 %.
inline bool two_states_stay_unshared(int ntile, int64_t B, int D, int k, int cus) {
  return k <= 16 && (D & (D - 1)) == 0 && ntile * B * D >= (int64_t)25 * 1536 * cus;
}

// Whether the full step of a small call takes tiles of 16 rows: where they fit into one round of the machine (a second round
// costs more than a taller tile: 4608 x 3072 rows, rank 32: 24 us with tall tiles, 30 us), unless most of the machine then
// streams operands that no L2 (4 MB) holds: each tile reads all basis operands of its block twice.  Against tiles
// one step below the full height: 4 x 700 x 3072 23 -> 17 us, 28 x 128 x 1152 at rank 32 11.0 -> 8.7 us; but 28 x 125 x 1152
// at rank 64 (8.3 MB) 18.2 -> 22.3 us and 26 x 128 x 1920 (12.8 MB) 23.4 -> 33.2 us.  Of 234 calls sampled up to one round
// none is slower with this rule.
inline bool full_step_takes_single_tiles(int64_t tiles16, int64_t operand_bytes, int cus) {
  return tiles16 <= cus && (operand_bytes <= (int64_t)3 << 20 || 8 * tiles16 <= 5 * (int64_t)cus);
}

// Row tiles per workgroup tile (RT) of the full step, with a basis-operand ring of RD items, for a feature width of
// CH * 128 channels, W = 1 (bf16) or 2 (float32) registers per channel pair and KT2 = padded rank / 32.
// Every basis byte is read once per tile, so the tile should have as many rows as the 512 registers of a lane
// allow: estimate = row pieces + accumulators + coefficient operands + ring + addressing and temporaries.
constexpr int full_step_regs(int CH, int W, int KT2, int RT, int RD) {
  return RT * CH * 4 * W + 2 * KT2 * RT * 4 + RT * KT2 * 12 + RD * 8 + (W == 2 ? RT * 8 + 70 : 0) + 46 +
         (KT2 == 4 ? 40 : 0);
}
constexpr int tile_rows(int CH, int W, int KT2) {
  if (CH == 24 && W == 1) return KT2 == 1 ? 3 : 2;   // measured at 3072 channels (FLUX, HunyuanVideo)
  for (int rt = 4; rt > 1; --rt)   // 2 KT2 rt <= 16: the reduction buffer (4 KB per accumulator) stays within 64 KB of LDS
    if (full_step_regs(CH, W, KT2, rt, 8) <= 450 && 2 * KT2 * rt <= 16) return rt;
  return 1;
}
// Whether a workgroup tile can have one more row tile in LDS (LT): bf16 at 3072 channels, rank 33..64.  Measured at the HunyuanVideo
// shape: 4 % (split operands) to 8 % (single operands) less time per launch, 8-10 % on a single 18432-row block.  At rank <= 32 the
// packed-basis stream is small enough that a fourth tile gains nothing, at rank 128 the LDS tile only replaces the second register tile at
// equal speed.
constexpr bool has_lds_tile(int CH, int W, int KT2) { return CH == 24 && W == 1 && KT2 == 2; }

// Row tiles that a full step (without smoothing) takes at a time, the one in LDS included.
// A taller tile can leave more of the last round of the persistent grid empty, so the choice of the LDS tile compares rounds x tile height x
// cost per row (0.92 of the register-only tile's).  A launch with fewer tiles than compute units leaves units idle: such small
// problems take tiles one step smaller (their packed-basis traffic does not matter at that size), and tiles of 16 rows where the rule above allows.
inline int full_step_rows(int CH, int W, int KT2, bool split, int N, int64_t B, int cus) {
  const int RT = tile_rows(CH, W, KT2);
  auto tile_count = [&](int ra) { return (int64_t)((N + 16 * ra - 1) / (16 * ra)) * B; };
  if (has_lds_tile(CH, W, KT2)) {
    auto rounds = [&](int ra) { return (double)((tile_count(ra) + cus - 1) / cus); };
    if (tile_count(RT + 1) >= cus && rounds(RT + 1) * (RT + 1) * 0.92 <= rounds(RT) * RT) return RT + 1;
  }
  if (RT > 2 && full_step_takes_single_tiles(tile_count(1), B * CH * 128 * (32 * KT2) * 2 * (split ? 2 : 1), cus)) return 1;
  return RT > 1 && tile_count(RT) < cus ? RT - 1 : RT;
}

// Whether the full step that smooths the residual takes rt row tiles of 16 at a time, for which the previous residual
// still fits beside them, or one less: the persistent grid takes rounds x (rt + x), x = the basis stream in row tiles.
// Timed at 250 sampled calls (bf16, the widths and ranks where there is a choice: 256 to 1152 channels at rank 32, 256 at
// rank 64, 256 to 1536 at rank 128; 1 to 12 rounds): a round of 4 tiles takes 1.33 of one of 3 at rank 32 and 1.38 at
// rank 64, of 2 tiles 1.42 (split operands) to 1.47 of one of 1 at rank 128, which is x = 0.3 per 32 coefficients, split or
// not.  Short calls scatter by 8 % around that, so the taller tile has to promise as much: with it none of the 250 is
// slower than one tile less, and they take 11 % less time on average (28 blocks of 1024 x 1152 in two rounds of 64 rows
// instead of three of 48: 60.7 -> 57.7 us).
inline bool smoothing_takes_full_tiles(int rt, int kt2, int N, int64_t B, int cus) {
  auto cost = [&](int r) {
    const int64_t tiles = (int64_t)((N + 16 * r - 1) / (16 * r)) * B;
    return (double)((tiles + cus - 1) / cus) * (r + 0.3 * kt2);
  };
  return cost(rt) < 0.92 * cost(rt - 1);
}

// Row tiles of 16 that a workgroup of the streamed projection (project_stream.h) takes, 1 to 6, in calls of B blocks of ntile: those of the
// least rounds x (rows + x).  The operands of the basis or sketch that a workgroup reads once cost it as much as x = 1.25 tiles, at every width
// and for both storage types: over 14 shapes and 12 kinds of operands (1 x 300 x 1024 to 57 x 4608 x 3072) the choice is within
// 3 % of the best height.
constexpr double kStreamOperands = 1.25;
inline int64_t stream_rounds(int rt, int ntile, int64_t B, int cus) { return ((ntile + rt - 1) / rt * B + cus - 1) / cus; }
inline int stream_rows(int ntile, int64_t B, int cus) {
  auto cost = [&](int rt) { return (double)stream_rounds(rt, ntile, B, cus) * (rt + kStreamOperands); };
  int best = 1;
  for (int rt = 2; rt <= 6; ++rt)
    if (cost(rt) < cost(best)) best = rt;
  return best;
}

// Whether a bf16 projection of a fit, B blocks of ntile row tiles of 16 with kt tiles of 16 columns, has enough of them for the kernels that keep or share
// Q (fit_mfma_kernels.hip) in the place of the streamed one: 16 per compute unit; up to width 64 calls of 8 to 16 take the streamed one 2 to 6 % less of a
// whole fit.  At width 128 a unit holds two workgroups of 8 tiles, and one round of those pays from 12 tiles per unit on (3 x 9179 x 5120, plain: 77 us,
// streamed 94; 20 x 3000 x 1024 1.5 % of the fit, 15 x 3837 x 768 6 %), with up to 1024 channels, where the streamed waves' sums weigh more, from 8 on (4 x
// 14777 x 1024: 28 and 43 us); above 1024 channels 8 to 12 tiles are streamed 1 to 5 % faster, and calls just beyond the round 3 %.  260 fits of 4 to
// 20 tiles per unit timed both ways.
inline bool projection_is_large(int ntile, int64_t B, int kt, int D, int cus) {
  const int64_t tiles = ntile * B;
  if (tiles >= 16 * (int64_t)cus) return true;
  return kt == 8 && tiles >= (D <= 1024 ? 8 : 12) * (int64_t)cus && (ntile + 7) / 8 * B <= 2 * (int64_t)cus;
}

// Whether a full step that has a buffer for its coefficients runs as two launches, the streamed projection (C and S) and a cached step's
// kernel with -C for its state (R = F - C V^T), instead of one that keeps its rows on chip.  F is read twice, but neither launch
// streams a basis past 16 or 32 rows at a time: 18432 x 3072 float32 at rank 128 235 -> 190 us, 57 x 4608 x 3072 bf16 at rank 128 2117 ->
// 1645, 1 x 4608 at rank 64 45 -> 37 and rank 128 75 -> 51, 2 x 14626 x 4096 float32 at rank 128 781 -> 400 us; but 57 x 4608 x 3072 bf16 at rank
// 32 871 -> 1020, rank 64 1174 -> 1223.  Both sides are estimated in us for 256 compute units: one launch a + d rounds (b rows + c), two launches
// a + d (b + c rounds (rows + 1.25) + e tiles per unit), d = D / 1024, fitted to 1423 calls timed both ways (1 to 57 blocks, 200 to 24000
// rows, ranks 33 to 128, the widths of the kernel), with margins because the estimates meet the time within 6 to 18 %; calls of less than a tile
// of 16 rows per compute unit scatter more.  Of 769 other calls that go this way, timed both ways with inputs in turn, each takes 0.31 to 1.00
// of the single launch's time, 0.69 on average.  float32 rows of 5120 channels go this way at any rank, of 4096
// from rank 65 on or with a tile per compute unit: the single launch spills registers there (118 calls, 1.04 to 3.1 times the
// time).  Single operands (SVDC_FAST) do from rank 65 and 1536 channels on.
struct OneLaunch {
  int rows;             // row tiles of 16 that the single launch takes
  int64_t tiles;        // workgroup tiles of that height in all blocks
};
inline bool full_step_may_take_two_launches(int D, int k, bool f32, bool split) {
  if (k <= 32) return f32 && D >= 5120;
  return k > 64 ? D >= (split ? 512 : 1536) : split && D >= 1536;
}
inline bool full_step_in_two_launches(OneLaunch one, int N, int64_t B, int D, int k, bool f32, bool split, int cus) {
  const int ntile = (N + 15) / 16, rt = stream_rows(ntile, B, cus);
  if (f32 && (D >= 5120 || (D >= 4096 && (k > 64 || ntile * B >= cus)))) return true;
  struct Fit { double a, b, c; } p;
  struct Fit2 { double a, b, c, e; } q;
  if (k > 64) {
    p = f32 ? Fit{1.66, 17.05, 0.0} : (split ? Fit{3.62, 7.22, 5.40} : Fit{2.44, 6.82, 1.33});
    q = f32 ? Fit2{7.35, 0.21, 2.30, 11.74} : (split ? Fit2{7.94, 0.28, 1.93, 7.20} : Fit2{6.22, 0.0, 1.31, 6.16});
  } else {
    p = f32 ? Fit{2.06, 9.87, 1.42} : Fit{2.81, 5.26, 1.80};
    q = f32 ? Fit2{5.54, 0.0, 1.66, 9.75} : Fit2{6.15, 0.46, 0.99, 5.62};
  }
  const double d = D / 1024.0;
  // channels that slabs of 4 x 128 do not divide: narrower slabs of the second launch
  if (D % 512 != 0) q.e *= 1.15;
  const double single = p.a + d * (double)((one.tiles + cus - 1) / cus) * (p.b * one.rows + p.c);
  const double twice = q.a + d * (q.b + q.c * (double)stream_rounds(rt, ntile, B, cus) * (rt + kStreamOperands) + q.e * ((double)ntile * B / cus));
  return twice < (rt == 1 ? 0.8 : (f32 || k > 64 ? 0.97 : 0.94)) * single;
}

// Row tiles of the projection of a full step with a buffer for C that takes two launches, 0 where it takes one.
inline int full_step_projection_rows(int N, int64_t B, int D, int k, bool f32, bool split, int cus) {
  // beyond 2^26 row tiles (a terabyte of the narrowest rows that come here) a grid could have more than 2^31 workgroups: the single launch refuses those
  if (!full_step_may_take_two_launches(D, k, f32, split) || ((int64_t)N + 15) / 16 * B > (int64_t)1 << 26) return 0;
  const int rows = full_step_rows(D / 128, f32 ? 2 : 1, k <= 32 ? 1 : (k <= 64 ? 2 : 4), split, N, B, cus);
  const int64_t tiles = (int64_t)((N + 16 * rows - 1) / (16 * rows)) * B;
  return full_step_in_two_launches({rows, tiles}, N, B, D, k, f32, split, cus) ? stream_rows((N + 15) / 16, B, cus) : 0;
}

// The general steps (general_kernels.hip) run on the float32 matrix cores, 16 rows per workgroup, or on the bf16 ones with
// float32 values as three parts, 16 RT rows.  The rules below compare estimates of both (us, 256 compute units): rounds of workgroups
// or workgroups per unit x (a constant + chunks of 32 channels per wave x (rows + padded rank x work)).
// Fitted to half of 7184 calls timed with every choice (1 to 57 blocks, 34 to 40000 rows, 488 to 4480 channels, ranks 17 to 128).
// Over all of them, share of the calls in parts, their time against the float32 instructions, and how many of them are slower by
// more than 1.5 % and 0.2 us: full step of bf16 rows 81 %, 0.83, 1.2 %; with smoothing 55 %, 0.84, 1.7 %; of float32 rows 34 %, 0.88,
// 3.0 %; cached step of bf16 rows 55 %, 0.86, 3.0 %; of float32 rows 5 %, 0.94, 7 %.  (Choosing without a mistake would take 0.852 of
// the time of all full steps of bf16 rows, this takes 0.857.)  The margins are where few calls lose; the estimates meet the time
// within 8 to 11 %.
// The limits come first, so that a call outside them does not ask for the compute units (a fiftieth of the smallest calls).  Ranks
// up to 16 would be padded to 32 (20 x 900 x 1000, rank 16: 29 us on the float32 instructions, 36 in parts); with few channels the
// constants overlap with other workgroups (57 x 3874 x 72 float32: 170 and 250 us).

// Row tiles RT with which the general full step runs in parts, 0: on the float32 instructions.  Float32 rows and smoothing together
// do not fit the registers; one tile of either is never better than the float32 instructions by these estimates.
inline bool full_step_may_take_parts(int D, int k, bool f32, bool smoothing) {
  return k > 16 && k <= 128 && D > 480 && !(f32 && smoothing);
}
inline int full_step_parts_rows(int N, int64_t B, int D, int k, bool f32, bool smoothing, int cus) {
  const double chunks = ((D + 31) / 32) / 8.0, kt2 = (k + 31) / 32;
  auto rounds = [&](int rt) { return (double)(((int64_t)((N + 16 * rt - 1) / (16 * rt)) * B + cus - 1) / cus); };
  const double rows = f32 ? 0.84 : smoothing ? 0.44 : 0.25, margin = f32 || smoothing ? 0.85 : 1.0;
  double least = margin * ((f32 ? 4.6 : 6.0) + rounds(1) * (1.1 + chunks * (rows + (f32 ? 1.67 : 1.58) * kt2)));
  int best = 0;
  for (int rt = f32 || smoothing ? 2 : 1; rt <= 3; ++rt) {
    const double t = f32 ? rounds(rt) * (11 + chunks * (0.5 * kt2 + rt * (0.5 + 1.02 * kt2)))
                         : 2.5 + rounds(rt) * (5.2 + chunks * (kt2 + rt * ((smoothing ? 0.46 : 0.2) + 0.56 * kt2)));
    if (t < least) {
      least = t;
      best = rt;
    }
  }
  return best;
}

// Shares of the channels in the general cached step: until there are about four workgroups per compute unit, at least two chunks of
// 32 channels for each of the four waves.
inline int cached_shares(int64_t tiles, int64_t B, int D, bool parts, int cus) {
  const int64_t want = (4 * (int64_t)cus + tiles * B - 1) / (tiles * B), most = parts ? (D + 63) / 64 / 4 : (D + 31) / 32 / 8;
  return (int)std::max<int64_t>(1, std::min(want, most));
}

// Whether the general cached step runs in parts, 32 rows per workgroup.  Never with a tensor to add: there parts took 1.11
// of the time over 900 calls (2 x 2566 x 632, rank 32: 10.1 and 16.5 us; its registers spilled).
// Several states are combined once per row tile and share of the channels, of which the parts have more: float32 rows gain
// nothing then (280 calls: 1.002 of the time) and stay, bf16 rows have to promise more (418 calls: 18 slower by up to 15 % with the
// margin of one state).
inline bool cached_step_may_take_parts(int D, int k, bool f32, int states, bool add) {
  return k > (f32 ? 48 : 16) && k <= 128 && D > 480 && !add && !(f32 && states > 1);
}
inline bool cached_step_takes_parts(int N, int64_t B, int D, int k, bool f32, int states, int cus) {
  const double chunks = ((D + 31) / 32) / 4.0, kt = (k + 15) / 16, kt2 = (k + 31) / 32;
  struct Load { double groups, chunks; };       // workgroups per compute unit, chunks per wave
  auto load = [&](int64_t tiles, bool parts) {
    const int shares = cached_shares(tiles, B, D, parts, cus);
    return Load{(double)((tiles * B * shares + cus - 1) / cus), chunks / shares};
  };
  const Load p = load((N + 31) / 32, true), f = load((N + 15) / 16, false);
  // V passes through LDS in pieces of 32 columns up to rank 32 and of 64 beyond
  const double column = 0.127 * kt + 0.049 * (k <= 32 ? 2 : (k + 63) / 64 * 4);
  const double parts = 4.3 + 1.7 * kt2 + (f32 ? p.groups * (0.78 + p.chunks * (1.28 + 0.33 * kt2))
                                              : p.groups * (0.53 + p.chunks * (0.5 + 0.37 * kt2)));
  const double plain = 3.3 + 0.53 * kt + (f32 ? f.groups * (0.6 + f.chunks * (0.28 + column))
                                              : f.groups * (0.26 + f.chunks * (0.21 + column)));
  return parts < (f32 ? 0.91 : states > 1 ? 0.9 : 0.97) * plain;
}

// Rows of a slice, a multiple of 16 and at least 64, for the partial Gram matrices of a fit: `tiles` workgroups per slice (64 x 64 tiles of l x l, all blocks), room
// for `most` slices.  l <= 64: three workgroups fit on a compute unit, and as many slices as fill one round of that are taken.  Above, the 344 registers of
// the kernel allow one, and its start and end (the waves' sums, 32 KB of partial matrix) take it as long as 300 rows: the number of slices whose
// rounds x (rows + 300) is least.  us with rounds of two per unit, and like this, l = 128: 3 x 5120 rows 25.1 -> 17.1, 3 x 9179 30.4 -> 24.9, 4 x 14777 56 -> 43,
// 20 x 3000 46 -> 41; over 37 sizes (l = 16 to 192) timed at up to 17 numbers of slices the choice is within 1 % of the best on average, 7 % at worst.
inline int gram_slice_rows(int rows, int l, int64_t tiles, int64_t most, int cus) {
  auto slice = [&](int64_t n) { return std::max(64, (int)((rows + n - 1) / n + 15) / 16 * 16); };
  if (l <= 64) return slice(std::min(most, std::max<int64_t>(1, 3 * cus / tiles)));
  int64_t least = INT64_MAX;
  int best = 0;
  for (int64_t n = 1; n <= most && n <= (rows + 63) / 64; ++n) {
    const int r = slice(n);
    const int64_t cost = ((rows + r - 1) / r * tiles + cus - 1) / cus * (r + 300);
    if (cost < least) least = cost, best = r;
  }
  return best;
}

}  // namespace svdc
