// Basis reuse across prompts and re-basing of the coefficient state (Sec. 3.3, Fig. 1(b)).
// All three kernels touch only the D x k bases and the N x k states, never the features.
#include <type_traits>

#include "svdc_device.h"
#include "svdc_internal.h"

namespace svdc {

namespace {

constexpr int kMaxRank = 128;    // overlap / re-basing work up to this rank

// v_mfma_f32_16x16x4_f32: lane (r = lane % 16, g = lane / 16) holds A[m = r][kk = g], B[kk = g][n = r] and the four
// results D[m = 4 g + i][n = r].
__device__ __forceinline__ f32x4 mfma_f32(float a, float b, const f32x4& c) {
  return __builtin_amdgcn_mfma_f32_16x16x4f32(a, b, c, 0, 0, 0);
}

// M[b][i][j] = sum_d V_old[b][d][i] * V_new[b][d][j], a 16 x 16 tile of M per workgroup, grid (tiles, B).  What bounds
// it is the latency of the loads: a tile's contraction over D rows of 64 bytes from each basis is spread over the 16
// waves of the workgroup (float32 matrix instructions, 16 independent loads in flight per wave), whose partial sums
// are added in wave order.  One wave per row of the tile walking over all D channels through LDS, as this was done
// before, took 201 us at 3072 channels, rank 32, one block (242 us for 57, 362 us at rank 64); this takes 9.6 us
// (28 and 13 us).  D is a multiple of 4 (svdc_shape); columns beyond k are clamped, their results are not stored.
// kOvWaves: 16, or 4 where many tiles fill the machine and the contraction is short (at most 256 channels): 300 blocks of
// 48 x 48 11.6 -> 5.9 us, of 80 x 80 33.4 -> 20.0 us (8.3 and 26.7 us by one thread per 1 x 8 elements of M).
template <int kOvWaves>
__global__ __launch_bounds__(64 * kOvWaves) void basis_overlap_kernel(const float* __restrict__ Vo,
                                                                      const float* __restrict__ Vn, float* M, int D,
                                                                      int k) {
  __shared__ f32x4 part[kOvWaves][64];
  const int b = blockIdx.y, tiles = (k + 15) / 16;
  const int i0 = (blockIdx.x / tiles) * 16, j0 = (blockIdx.x % tiles) * 16;
  const int wave = threadIdx.x >> 6, lane = threadIdx.x & 63, r = lane & 15, g = lane >> 4;
  const float* vo = Vo + (int64_t)b * D * k + min(i0 + r, k - 1);
  const float* vn = Vn + (int64_t)b * D * k + min(j0 + r, k - 1);
  // steps of 4 channels, wave w takes w, w + 16, ...; two accumulators
  f32x4 acc0 = {0.f, 0.f, 0.f, 0.f}, acc1 = {0.f, 0.f, 0.f, 0.f};
  const int nstep = D / 4;
  constexpr int U = 8;
  int st = wave;
  for (; st + (U - 1) * kOvWaves < nstep; st += U * kOvWaves) {
    float x[U], y[U];
#pragma unroll
    for (int u = 0; u < U; ++u) {
      const int64_t at = (int64_t)(4 * (st + u * kOvWaves) + g) * k;
      x[u] = vo[at];
      y[u] = vn[at];
    }
#pragma unroll
    for (int u = 0; u < U; u += 2) {
      acc0 = mfma_f32(x[u], y[u], acc0);
      acc1 = mfma_f32(x[u + 1], y[u + 1], acc1);
    }
  }
  for (; st < nstep; st += kOvWaves) {
    const int64_t at = (int64_t)(4 * st + g) * k;
    acc0 = mfma_f32(vo[at], vn[at], acc0);
  }
  part[wave][lane] = f32x4{acc0[0] + acc1[0], acc0[1] + acc1[1], acc0[2] + acc1[2], acc0[3] + acc1[3]};
  __syncthreads();
  const int t = threadIdx.x;
  if (t >= 256) return;
  const int row = t >> 4, col = t & 15;                 // element of the tile; it sits in lane (col, row / 4), word row % 4
  float s = 0.f;
#pragma unroll
  for (int w = 0; w < kOvWaves; ++w) s += part[w][(row >> 2) * 16 + col][row & 3];
  if (i0 + row < k && j0 + col < k) M[((int64_t)b * k + i0 + row) * k + j0 + col] = s;
}

// S_out[row][j] = sum_i S_in[row][i] * M[i][j] on the float32 matrix cores, KT = ceil(k / 16).  M sits in LDS (row stride
// 16 KT + 4 floats: the four rows that the lane groups of an operand read fall into different banks); a wave brings a
// tile of 16 rows of S into registers before it writes any of it, so S_out may be S_in.  The contraction index of
// step (s, e) is i = 16 s + 4 g + e, so that a lane's four steps are one 16-byte piece of its row (VEC: k a multiple of 4
// and 16-byte aligned states; otherwise four loads).  It streams S: 27 -> 4.9 us at 4608 x 32 and 97 -> 18 us for 57
// such blocks (3.7 TB/s) against one wave per row with a chain of k dependent LDS reads and multiply-adds.
template <int KT, bool VEC>
__global__ __launch_bounds__(256) void rebase_state_kernel(const float* __restrict__ M, const float* Sin, float* Sout,
                                                           int N, int k, int tiles_per_wave) {
  extern __shared__ float m[];          // [16 KT][LS]
  constexpr int LS = 16 * KT + 4;
  const int wave = threadIdx.x >> 6, lane = threadIdx.x & 63, r = lane & 15, g = lane >> 4;
  const int b = blockIdx.y;
  const float* mg = M + (int64_t)b * k * k;
  for (int e = threadIdx.x; e < 16 * KT * 16 * KT; e += 256) {
    const int i = e / (16 * KT), j = e % (16 * KT);
    m[i * LS + j] = (i < k && j < k) ? mg[i * k + j] : 0.f;
  }
  __syncthreads();
  for (int q = 0; q < tiles_per_wave; ++q) {
    const int row0 = ((blockIdx.x * tiles_per_wave + q) * 4 + wave) * 16;
    if (row0 >= N) return;
    const float* src = Sin + ((int64_t)b * N + min(row0 + r, N - 1)) * k;
    float a[KT][4];
#pragma unroll
    for (int s = 0; s < KT; ++s) {
      const int i = 16 * s + 4 * g;
      if constexpr (VEC) {
        f32x4 x = {0.f, 0.f, 0.f, 0.f};
        if (i < k) x = *reinterpret_cast<const f32x4*>(src + i);
#pragma unroll
        for (int e = 0; e < 4; ++e) a[s][e] = x[e];
      } else {
#pragma unroll
        for (int e = 0; e < 4; ++e) a[s][e] = i + e < k ? src[i + e] : 0.f;
      }
    }
    f32x4 acc[KT];
#pragma unroll
    for (int jt = 0; jt < KT; ++jt) acc[jt] = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int s = 0; s < KT; ++s)
#pragma unroll
      for (int e = 0; e < 4; ++e)
#pragma unroll
        for (int jt = 0; jt < KT; ++jt)
          acc[jt] = mfma_f32(a[s][e], m[(16 * s + 4 * g + e) * LS + 16 * jt + r], acc[jt]);
#pragma unroll
    for (int jt = 0; jt < KT; ++jt)
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        const int row = row0 + 4 * g + i;
        if (row < N && 16 * jt + r < k) Sout[((int64_t)b * N + row) * k + 16 * jt + r] = acc[jt][i];
      }
  }
}

// Fig. 1(b): cosine similarity times magnitude similarity for every pair of basis directions and for the two
// singular-value vectors, float64 sums.  A workgroup takes C columns of both bases, 16 (or 4 or 1 for ranks that have no
// more): neighbouring threads read consecutive floats of a row, the groups of C threads take the rows in turn.  (One wave per
// column read 4 bytes of every row: 89 us at 3072 channels, rank 32, one block, 150 us for 57, against 7.3 and 18 us.)
// kSimThreads: 1024, or 256 where a thread then has at most 8 rows, or 32 if many workgroups fill the machine (300 blocks of
// 320 x 1 with 16 columns and 1024 threads 4.8 us, of 1504 x 1 8.2 us; like this 4.0 and 4.2).
template <int kSimThreads, int C>
__global__ __launch_bounds__(kSimThreads) void basis_similarity_kernel(const float* __restrict__ Va,
                                                                       const float* __restrict__ sa,
                                                                       const float* __restrict__ Vb,
                                                                       const float* __restrict__ sb, float* sim_dir,
                                                                       float* sim_sigma, int D, int k) {
  constexpr int kRowGroups = kSimThreads / C, kWaves = kSimThreads / 64;
  __shared__ double part[kWaves][C][3];
  const int b = blockIdx.y, wave = threadIdx.x >> 6, lane = threadIdx.x & 63, c = threadIdx.x % C;
  const int j = blockIdx.x * C + c;
  const float* va = Va + (int64_t)b * D * k + min(j, k - 1);
  const float* vb = Vb + (int64_t)b * D * k + min(j, k - 1);
  auto score = [](double dot, double na2, double nb2, bool take_abs) -> float {
    if (!(na2 > 0.0) || !(nb2 > 0.0)) return 0.f;
    const double na = sqrt(na2), nb = sqrt(nb2);
    const double co = (take_abs ? fabs(dot) : dot) / (na * nb);
    return (float)(co * (na < nb ? na / nb : nb / na));
  };
  double dot = 0.0, na = 0.0, nb = 0.0;
#pragma unroll 8
  for (int d = threadIdx.x / C; d < D; d += kRowGroups) {
    const double x = va[(int64_t)d * k], y = vb[(int64_t)d * k];
    dot += x * y; na += x * x; nb += y * y;
  }
#pragma unroll
  for (int o = C; o < kWave; o <<= 1) {       // the row groups of a wave
    dot += __shfl_xor(dot, o, kWave); na += __shfl_xor(na, o, kWave); nb += __shfl_xor(nb, o, kWave);
  }
  if (lane < C) { part[wave][c][0] = dot; part[wave][c][1] = na; part[wave][c][2] = nb; }
  __syncthreads();
  if (threadIdx.x < C && j < k) {
    dot = na = nb = 0.0;
    for (int w = 0; w < kWaves; ++w) { dot += part[w][c][0]; na += part[w][c][1]; nb += part[w][c][2]; }
    sim_dir[(int64_t)b * k + j] = score(dot, na, nb, true);
  }
  if (blockIdx.x == 0 && wave == 1 && sim_sigma) {
    dot = na = nb = 0.0;
    for (int i = lane; i < k; i += kWave) {
      const double x = sa[(int64_t)b * k + i], y = sb[(int64_t)b * k + i];
      dot += x * y; na += x * x; nb += y * y;
    }
    dot = wave_sum(dot); na = wave_sum(na); nb = wave_sum(nb);
    if (lane == 0) sim_sigma[b] = score(dot, na, nb, false);
  }
}

}  // namespace

bool rebase_rank_supported(int k) { return k >= 1 && k <= kMaxRank; }

int32_t launch_basis_overlap(const svdc_shape& s, const float* V_old, const float* V_new, float* M, hipStream_t st) {
  const int tiles = (s.k + 15) / 16;
  const dim3 grid(tiles * tiles, s.B);
  if (s.D <= 256 && (int64_t)grid.x * s.B >= num_compute_units())
    basis_overlap_kernel<4><<<grid, 256, 0, st>>>(V_old, V_new, M, s.D, s.k);
  else
    basis_overlap_kernel<16><<<grid, 1024, 0, st>>>(V_old, V_new, M, s.D, s.k);
  return launch_status();
}

namespace {

template <int KT>
int32_t rebase_launch(const svdc_shape& s, const float* M, const float* S_in, float* S_out, hipStream_t st) {
  const size_t lds = (size_t)16 * KT * (16 * KT + 4) * sizeof(float);
  // M of rank 65..128 is 37-66 KB: two row tiles per wave for each copy of it
  const int tiles_per_wave = KT > 4 ? 2 : 1;
  const bool vec = s.k % 4 == 0 && ((reinterpret_cast<uintptr_t>(S_in) | reinterpret_cast<uintptr_t>(S_out)) & 15) == 0;
  auto launch = [&](auto kernel) -> int32_t {
    if (lds > 48 * 1024 && hipFuncSetAttribute((const void*)kernel, hipFuncAttributeMaxDynamicSharedMemorySize,
                                               (int)lds) != hipSuccess)
      return SVDC_E_HIP;
    const int rows = 64 * tiles_per_wave;
    kernel<<<dim3((s.N + rows - 1) / rows, s.B), 256, lds, st>>>(M, S_in, S_out, s.N, s.k, tiles_per_wave);
    return launch_status();
  };
  return vec ? launch(rebase_state_kernel<KT, true>) : launch(rebase_state_kernel<KT, false>);
}

}  // namespace

int32_t launch_rebase_state(const svdc_shape& s, const float* M, const float* S_in, float* S_out, hipStream_t st) {
  switch ((s.k + 15) / 16) {
    case 1: return rebase_launch<1>(s, M, S_in, S_out, st);
    case 2: return rebase_launch<2>(s, M, S_in, S_out, st);
    case 3: return rebase_launch<3>(s, M, S_in, S_out, st);
    case 4: return rebase_launch<4>(s, M, S_in, S_out, st);
    case 5: return rebase_launch<5>(s, M, S_in, S_out, st);
    case 6: return rebase_launch<6>(s, M, S_in, S_out, st);
    case 7: return rebase_launch<7>(s, M, S_in, S_out, st);
    default: return rebase_launch<8>(s, M, S_in, S_out, st);
  }
}

int32_t launch_basis_similarity(const svdc_shape& s, const float* V_a, const float* sigma_a, const float* V_b,
                                const float* sigma_b, float* sim_dir, float* sim_sigma, hipStream_t st) {
  auto launch = [&](auto columns) {
    constexpr int C = decltype(columns)::value;
    const dim3 grid((s.k + C - 1) / C, s.B);
    const int64_t rows = ((int64_t)s.D * C + 255) / 256;       // of each of 256 threads
    if (rows <= 8 || (rows <= 32 && (int64_t)grid.x * s.B >= num_compute_units()))
      basis_similarity_kernel<256, C><<<grid, 256, 0, st>>>(V_a, sigma_a, V_b, sigma_b, sim_dir, sim_sigma, s.D, s.k);
    else
      basis_similarity_kernel<1024, C><<<grid, 1024, 0, st>>>(V_a, sigma_a, V_b, sigma_b, sim_dir, sim_sigma, s.D, s.k);
  };
  if (s.k == 1) launch(std::integral_constant<int, 1>{});
  else if (s.k <= 4) launch(std::integral_constant<int, 4>{});
  else launch(std::integral_constant<int, 16>{});
  return launch_status();
}

}  // namespace svdc
