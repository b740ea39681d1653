// Cholesky factor of the Gram matrices of the basis fit, with the inverse of its diagonal blocks (float64, gfx950).
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

#include <type_traits>

#include "svdc_device.h"
#include "svdc_internal.h"

namespace svdc {
namespace {

// A pivot of the Cholesky factorisation below kRankTol x the largest diagonal entry of the Gram matrix means that a
// column of the sketch depends on the others to within (1e-6)^2, the round-off of the float32 sketch itself: the
// matrix has numerical rank < l.  The shift keeps the factorisation going (the result stays orthonormal, directions
// beyond the numerical rank are arbitrary) and the block's status word reports it.
constexpr double kRankTol = 1e-12;

constexpr int kCholBlock = 64;    // columns whose inverse is formed together

// x of the lanes of row Q (of four rows of 16 lanes), in every row: v_permlane16_swap exchanges the odd rows of its first
// operand with the even rows of its second, v_permlane32_swap the upper half with the lower one.
template <int Q>
__device__ __forceinline__ double from_row(double x) {
  auto word = [](uint32_t w) {
    const auto a = __builtin_amdgcn_permlane16_swap(w, w, false, false);
    const uint32_t h = a[Q & 1];
    const auto c = __builtin_amdgcn_permlane32_swap(h, h, false, false);
    return (int)c[Q >> 1];
  };
  return __hiloint2double(word((uint32_t)__double2hiint(x)), word((uint32_t)__double2loint(x)));
}
// x of lane J of the same row of 16 lanes (row_newbcast)
template <int J>
__device__ __forceinline__ double from_lane(double x) {
  return __builtin_amdgcn_update_dpp(x, x, 0x150 + J, 0xf, 0xf, true);      // one v_mov_b64_dpp
}

__device__ __forceinline__ double wave_max(double x) {
  auto dpp = [](double v, auto ctrl) {
    const int lo = __double2loint(v), hi = __double2hiint(v);
    constexpr int C = decltype(ctrl)::value;
    return __hiloint2double(__builtin_amdgcn_update_dpp(hi, hi, C, 0xf, 0xf, true),
                            __builtin_amdgcn_update_dpp(lo, lo, C, 0xf, 0xf, true));
  };
  x = fmax(x, dpp(x, std::integral_constant<int, 0xB1>{}));     // quad_perm [1,0,3,2]
  x = fmax(x, dpp(x, std::integral_constant<int, 0x4E>{}));     // quad_perm [2,3,0,1]
  x = fmax(x, dpp(x, std::integral_constant<int, 0x141>{}));    // row_half_mirror
  x = fmax(x, dpp(x, std::integral_constant<int, 0x140>{}));    // row_mirror
  return fmax(fmax(from_row<0>(x), from_row<1>(x)), fmax(from_row<2>(x), from_row<3>(x)));
}

// 16 x 16 tile A = L' D L'^T by one wave, with U = L'^-1.  Lane (m = lane % 16, kq = lane / 16) holds A[m][4 c + kq] in a[c],
// which for a symmetric matrix is the result layout of the float64 matrix instruction; lo and u receive L' (without its
// unit diagonal) and U in the same places, drow the pivot of row m.  Column j of the
// elimination is brought to every row of lanes, its pivot and row j to every lane of a row: no LDS and no barrier.
struct TileFactor {
  double a[4], lo[4], u[4], drow;
  bool dependent;
  template <int J>
  __device__ __forceinline__ void column(int m, int kq, int w, double pivot_floor) {
    constexpr int cj = J / 4, gj = J % 4;
    const double y = from_row<gj>(a[cj]);
    const double p = from_lane<J>(y);
    dependent |= J < w && p < pivot_floor;
    const double d = fmax(p, 1e-300);
    // 1 / d: the hardware's estimate (about 2^-23) and one step of third order
    double x = __builtin_amdgcn_rcp(d);
    const double e1 = fma(-d, x, 1.0);
    x = fma(x, fma(e1, e1, e1), x);
    const double below = m > J ? y : 0.0, f = -(below * x);
    // the two factors of A first: the same bits on both sides of the diagonal, which (f times the row) would drift apart until what
    // rows and columns of a small pivot say differs by more than the pivots of dependent columns
#pragma unroll
    for (int c = cj; c < 4; ++c)
      if (4 * c + 3 > J) a[c] = fma(-(below * from_lane<J>(a[c])), x, a[c]);
#pragma unroll
    for (int c = 0; c <= cj; ++c) u[c] = fma(f, from_lane<J>(u[c]), u[c]);
    if (kq == gj) lo[cj] = -f;
    if (m == J) drow = d;
  }
  __device__ __forceinline__ void run(int m, int kq, int w, double pivot_floor) {
#pragma unroll
    for (int c = 0; c < 4; ++c) {
      lo[c] = 0.0;
      u[c] = m == 4 * c + kq ? 1.0 : 0.0;
    }
    drow = 1.0;
    dependent = false;
    column<0>(m, kq, w, pivot_floor); column<1>(m, kq, w, pivot_floor);
    column<2>(m, kq, w, pivot_floor); column<3>(m, kq, w, pivot_floor);
    column<4>(m, kq, w, pivot_floor); column<5>(m, kq, w, pivot_floor);
    column<6>(m, kq, w, pivot_floor); column<7>(m, kq, w, pivot_floor);
    column<8>(m, kq, w, pivot_floor); column<9>(m, kq, w, pivot_floor);
    column<10>(m, kq, w, pivot_floor); column<11>(m, kq, w, pivot_floor);
    column<12>(m, kq, w, pivot_floor); column<13>(m, kq, w, pivot_floor);
    column<14>(m, kq, w, pivot_floor); column<15>(m, kq, w, pivot_floor);
  }
};

// X = A L'^-T for 16 rows in the result layout (row 4 v + lane / 16, column lane % 16), by substitution: column J is final when its
// turn comes, and every lane takes it times L'[m][J] from its own.  l[J] = L'[m][J0 + J] of the lane's column m, zero from m on.
// Not as a product with the inverse: where a panel holds columns of the matrix' own scale and columns that depend on them to 1e-7, that
// is A times 1e7 / A, of whose sum all but a few digits cancel, and the error can exceed the shift that holds the pivots of the
// next panels up: negative ones in 1 to 4 of 100 matrices of rank 10, none in 6000 like this.
template <int J0, int J = 0>          // columns J0 .. J0 + 7
__device__ __forceinline__ void substitute(f64x4& x, const double (&l)[8]) {
#pragma unroll
  for (int v = 0; v < 4; ++v) x[v] = fma(-from_lane<J0 + J>(x[v]), l[J], x[v]);
  if constexpr (J < 7) substitute<J0, J + 1>(x, l);
}

// l[J] / diagonal entry J0 + J, which that lane has the reciprocal of: rows of L to rows of the unit triangle
template <int J0, int J = 0>
__device__ __forceinline__ void unit_columns(double (&l)[8], double rinv) {
  l[J] *= from_lane<J0 + J>(rinv);
  if constexpr (J < 7) unit_columns<J0, J + 1>(l, rinv);
}

__device__ __forceinline__ double rsqrt_f64(double d) {
  const double r = __builtin_amdgcn_rsq(d);      // the hardware's estimate and one step of third order
  const double e = fma(-(d * r), r, 1.0);
  return fma(r * e, fma(0.375, e, 0.5), r);
}

// ---------------------------------------------------------------------------
// Cholesky factor of a diagonal block of at most 16 NT columns, and the inverses of its diagonal blocks of 64, by one
// workgroup of 2 NT waves (one for NT = 1):
//   A = G[c0 .. c0 + w, same] + shift I - sum_{c < c0} L[., c] L[., c]^T  =  L L^T,       Minv = (blocks of 64 of L)^-T
// (the finished columns of its rows come transposed from the upper triangle of G: G[c][r] = L[r][c]).
// The matrix lives in registers as 16 x 16 tiles in the result layout of v_mfma_f64_16x16x4_f64, negated: the first NT waves
// own a diagonal tile each, the others share the rest and the tiles of the inverse.  Right-looking, a panel of 16 columns at a time:
//   the wave of the diagonal tile factors it and forms D = L_pp^-1                       (TileFactor)
//   L_ip = A_ip L_pp^-T by substitution,   M_pj = -D sum_{k < p} L_pk M_kj by a product; only these pass through LDS
//   A_ij -= L_ip L_jp^T,   the sums of the inverse grow by L_ip M_pj
// What bounds it is a chain: of 34000 clocks at 64 columns 6000 go by before the first pivot, 3500 in the 16 pivots of each
// panel (40 instructions a column), and another 3500 a panel in the substitution, the product and the barriers between one
// tile's pivots and the next one's (with a product instead of the substitution and two moves instead of one for a lane's
// double: as much).  So the diagonal tiles have waves of their own, which update the next tile first and go on while the
// others finish; the square roots and all stores wait until the end.  Measured inside a fit: 4.6 us at 8 columns, 16 us at 64,
// 37 us at 128, against 5.4, 24 and 61 us (in three launches) with panels of 4 columns in blocks of 4 x 4 per thread.
//   NT = 1: l <= 16; 4: blocks of 64 columns; 8: 65 to 128 columns at once
//   w <= 16 NT; columns from w on are padded with the identity.  Lower triangle of the block of G = L; of the upper part the
//   blocks of 64 on the diagonal are zeroed and the others receive L^T.
//   Minv   out  (want_inv) row-major [w x w] at row stride ldm; NT = 8: blocks of 64 at row stride ldm, 64 * 64 doubles apart;
//          block b at Minv + b * m_bstride
//   slot   the shift: computed from the diagonal of G and stored when c0 = 0, read otherwise (nullable when there is one
//          block only)
// ---------------------------------------------------------------------------
template <int NT>
__global__ __launch_bounds__(NT == 1 ? 64 : 128 * NT) void chol_tiles_kernel(double* G, int l, int c0, int w, double* Minv, int64_t m_bstride,
                                                             int ldm, int want_inv, double* slot, int64_t slot_bstride,
                                                             double rel_shift, int32_t* info) {
  constexpr int LT = 20;                              // row stride of a tile: operand reads without bank conflicts
  constexpr int TS = 16 * LT;
  constexpr int NA = NT * (NT - 1) / 2, NH = NT >= 4 ? NT / 4 : 0, NM = 6 * NH, NS = (NA + NM) / NT;
  static_assert((NA + NM) % NT == 0, "the tiles off the diagonal are dealt out evenly");
  __shared__ __align__(16) double panel[NT][TS];      // L_ip
  __shared__ __align__(16) double lpp[TS], rsv[16];   // unit triangle of the diagonal tile, without its diagonal, and 1 / sqrt(pivots)
  __shared__ double pivot[NT][16];
  __shared__ __align__(16) double dinv[2][TS];        // D
  __shared__ __align__(16) double mrow[2][3][TS];     // sums, then M_pj, j < p in the same block of 64
  __shared__ double s_shift;
  const int b = blockIdx.x, t = threadIdx.x, lane = t & 63, m = lane & 15, kq = lane >> 4;
  const int wave = __builtin_amdgcn_readfirstlane(t >> 6);
  double* g = G + (int64_t)b * l * l;
  double* gd = g + (int64_t)c0 * l + c0;
  double* mi = Minv + (int64_t)b * m_bstride;
  const int np = (w + 15) / 16;

  // the tiles of this wave: (ti, tj) of the matrix, or of the inverse (inv)
  const bool pivots = wave < NT;                      // owner of a diagonal tile, or of NS others
  int ti[NS > 0 ? NS : 1], tj[NS > 0 ? NS : 1];
  bool inv[NS > 0 ? NS : 1];
#pragma unroll
  for (int s = 0; s < NS; ++s) {
    int x = s * NT + wave - NT;
    inv[s] = x >= NA;
    if (pivots) {
      ti[s] = tj[s] = NT;                             // beyond np: none
    } else if (inv[s]) {                              // row by row: the tiles of a row go to different waves
      const int h = (x - NA) / 6;
      int i = 1;
      x = (x - NA) % 6;
      while (x >= i) { x -= i; ++i; }
      ti[s] = 4 * h + i;
      tj[s] = 4 * h + x;
    } else {                                          // column by column, likewise
      int j = 0;
      while (x >= NT - 1 - j) { x -= NT - 1 - j; ++j; }
      ti[s] = j + 1 + x;
      tj[s] = j;
    }
  }
  auto load = [&](int i, int j) {
    f64x4 x;
#pragma unroll
    for (int v = 0; v < 4; ++v)
      x[v] = gd[(int64_t)min(16 * i + 4 * v + kq, w - 1) * l + min(16 * j + m, w - 1)];
    return x;
  };
  f64x4 acc[NS > 0 ? NS : 1], diag = load(wave % NT, wave % NT);
#pragma unroll
  for (int s = 0; s < NS; ++s) acc[s] = inv[s] || pivots ? f64x4{0.0, 0.0, 0.0, 0.0} : load(ti[s], tj[s]);

  if (c0 == 0) {
    if (t < kWave) {
      double mx = 0.0;
      for (int i = t; i < l; i += kWave) mx = fmax(mx, g[(int64_t)i * l + i]);
      mx = wave_max(mx);
      if (t == 0) {
        s_shift = mx * rel_shift;
        if (slot) slot[(int64_t)b * slot_bstride] = mx * rel_shift;
      }
    }
  } else if (t == 0) {
    s_shift = slot[(int64_t)b * slot_bstride];
  }
  __syncthreads();
  const double shift = s_shift, pivot_floor = shift * (kRankTol / rel_shift);
  auto negate = [&](f64x4& x, int i, int j) {
#pragma unroll
    for (int v = 0; v < 4; ++v) {
      const int r = 16 * i + 4 * v + kq, c = 16 * j + m;
      if (r >= w || c >= w) x[v] = r == c ? -1.0 : 0.0;     // identity padding
      else x[v] = -(r == c ? x[v] + shift : x[v]);
    }
  };
  negate(diag, wave % NT, wave % NT);
#pragma unroll
  for (int s = 0; s < NS; ++s)
    if (!inv[s] && !pivots) negate(acc[s], ti[s], tj[s]);
  if constexpr (NT == 4) {
    // earlier columns: sum_c L[i][c] L[j][c], operands as they lie in the upper triangle (c0 is a multiple of 64)
    if (c0 > 0) {
      auto subtract = [&](f64x4& x, int i, int j) {
        const double* pi = g + (int64_t)kq * l + c0 + min(16 * i + m, w - 1);
        const double* pj = g + (int64_t)kq * l + c0 + min(16 * j + m, w - 1);
        const bool in_i = 16 * i + m < w, in_j = 16 * j + m < w;
        for (int k0 = 0; k0 < c0; k0 += 32) {
          double av[8], bv[8];
#pragma unroll
          for (int e = 0; e < 8; ++e) {
            av[e] = pi[(int64_t)(k0 + 4 * e) * l];
            bv[e] = pj[(int64_t)(k0 + 4 * e) * l];
          }
#pragma unroll
          for (int e = 0; e < 8; ++e)
            x = __builtin_amdgcn_mfma_f64_16x16x4f64(in_i ? av[e] : 0.0, in_j ? bv[e] : 0.0, x, 0, 0, 0);
        }
      };
      if (wave < np) subtract(diag, wave, wave);
#pragma unroll
      for (int s = 0; s < NS; ++s)
        if (!inv[s] && ti[s] < np) subtract(acc[s], ti[s], tj[s]);
    }
  }

  // acc + X Y^T (rows of both contiguous), or acc + X Y
  // (two chains of two matrix instructions: one waits 64 clocks for the other)
  auto product = [&](const double* X, const double* Y, int yk, int ym, const f64x4& x) {
    double xv[4], yv[4];
#pragma unroll
    for (int k4 = 0; k4 < 4; ++k4) {
      xv[k4] = X[m * LT + 4 * k4 + kq];
      yv[k4] = Y[(4 * k4 + kq) * yk + m * ym];
    }
    f64x4 p = __builtin_amdgcn_mfma_f64_16x16x4f64(xv[0], yv[0], x, 0, 0, 0);
    f64x4 q = __builtin_amdgcn_mfma_f64_16x16x4f64(xv[1], yv[1], f64x4{0.0, 0.0, 0.0, 0.0}, 0, 0, 0);
    p = __builtin_amdgcn_mfma_f64_16x16x4f64(xv[2], yv[2], p, 0, 0, 0);
    q = __builtin_amdgcn_mfma_f64_16x16x4f64(xv[3], yv[3], q, 0, 0, 0);
    return p + q;
  };
  auto times_t = [&](const double* X, const double* Y, const f64x4& x) { return product(X, Y, 1, LT, x); };
  auto times = [&](const double* X, const double* Y, const f64x4& x) { return product(X, Y, LT, 1, x); };
  auto put = [&](double* T, const f64x4& x, double sign) {
#pragma unroll
    for (int v = 0; v < 4; ++v) T[(4 * v + kq) * LT + m] = sign * x[v];
  };

  double dd[4];                                       // D of the wave's diagonal tile
  bool dependent = false;
  for (int p = 0; p < np; ++p) {
    const int par = p & 1;
    if (wave == p) {
      TileFactor f;
#pragma unroll
      for (int c = 0; c < 4; ++c) f.a[c] = -diag[c];
      f.run(m, kq, w - 16 * p, pivot_floor);
      const double rs = rsqrt_f64(f.drow);
#pragma unroll
      for (int c = 0; c < 4; ++c) {
        dd[c] = f.u[c] * rs;
        dinv[par][m * LT + 4 * c + kq] = dd[c];
        lpp[m * LT + 4 * c + kq] = f.lo[c];
        diag[c] = f.lo[c];
      }
      rsv[m] = rs;                                    // the four rows of lanes hold the same
      pivot[p][m] = f.drow;
      dependent = f.dependent;
    }
    __syncthreads();
#pragma unroll
    for (int s = 0; s < NS; ++s) {
      if (!inv[s] && tj[s] == p && ti[s] < np) {
        f64x4 x = -acc[s];
        double l8[8];                                 // half of a row at a time (registers)
#pragma unroll
        for (int j = 0; j < 8; ++j) l8[j] = lpp[m * LT + j];
        substitute<0>(x, l8);
#pragma unroll
        for (int j = 0; j < 8; ++j) l8[j] = lpp[m * LT + 8 + j];
        substitute<8>(x, l8);
        acc[s] = x * rsv[m];
        put(panel[ti[s]], acc[s], 1.0);
      }
      if (inv[s] && ti[s] == p && want_inv) {
        acc[s] = -times(dinv[par], mrow[par][tj[s] % 4], f64x4{0.0, 0.0, 0.0, 0.0});
        __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
        put(mrow[par][tj[s] % 4], acc[s], 1.0);
      }
    }
    if (p + 1 == np) break;
    __syncthreads();
    if (wave > p && wave < np) diag = times_t(panel[wave], panel[wave], diag);
#pragma unroll
    for (int s = 0; s < NS; ++s) {
      if (ti[s] <= p || ti[s] >= np) continue;
      if (!inv[s]) {
        if (tj[s] <= p) continue;
        acc[s] = times_t(panel[ti[s]], panel[tj[s]], acc[s]);
      } else if (want_inv && tj[s] <= p && ti[s] / 4 == p / 4) {
        acc[s] = times(panel[ti[s]], tj[s] == p ? dinv[par] : mrow[par][tj[s] % 4], acc[s]);
        if (ti[s] == p + 1) put(mrow[par ^ 1][tj[s] % 4], acc[s], 1.0);
      }
    }
  }

  // everything is still in registers: the factor, its zeros or transposes above the diagonal, the inverses
  if (wave < np) {
    if (info && dependent && lane == 0) atomicOr(info + b, SVDC_FIT_RANK_DEFICIENT);
    double* mh = mi + (int64_t)(wave / 4) * (kCholBlock * kCholBlock);
#pragma unroll
    for (int c = 0; c < 4; ++c) {
      const int r = 16 * wave + m, cc = 16 * wave + 4 * c + kq;
      if (r < w && cc < w) {
        const double d = pivot[wave][4 * c + kq], sq = d * rsqrt_f64(d);
        gd[(int64_t)r * l + cc] = r == cc ? sq : (r > cc ? diag[c] * sq : 0.0);
        if (want_inv) mh[(int64_t)(cc % kCholBlock) * ldm + r % kCholBlock] = dd[c];
      }
    }
  }
#pragma unroll
  for (int s = 0; s < NS; ++s) {
    if (ti[s] >= np || (inv[s] && !want_inv)) continue;
    const int r0 = 16 * ti[s] + kq, c = 16 * tj[s] + m;
    double* low = inv[s] ? mi + (int64_t)(ti[s] / 4) * (kCholBlock * kCholBlock - (int64_t)kCholBlock * (ldm + 1)) : gd;
    const int64_t ld = inv[s] ? ldm : l;
    // the inverse is stored transposed; blocks of 64 of the factor off the diagonal keep their transpose too
    const bool below = !inv[s], above = inv[s] || ti[s] / 4 != tj[s] / 4;
#pragma unroll
    for (int v = 0; v < 4; ++v) {
      const int r = r0 + 4 * v;
      if (r < w) {
        low[r * ld + c] = below ? acc[s][v] : 0.0;
        low[c * ld + r] = above ? acc[s][v] : 0.0;
      }
    }
  }
}

}  // namespace
}  // namespace svdc
