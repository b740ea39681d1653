// Host-side declarations shared between the translation units of libsvdcache.
#pragma once
#include <hip/hip_runtime.h>
#include <stddef.h>
#include <stdint.h>

#include "../../include/svdcache.h"

namespace svdc {

// Compute units of the current device (a partition of a card has fewer than the 256 of a whole one); every rule of a launch
// that depends on how much of the machine a grid fills asks for it.
inline int num_compute_units() {
  int dev = 0, n = 0;
  if (hipGetDevice(&dev) != hipSuccess) return 256;
  if (hipDeviceGetAttribute(&n, hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess || n <= 0) return 256;
  return n;
}

inline int32_t launch_status() { return hipGetLastError() == hipSuccess ? SVDC_OK : SVDC_E_HIP; }

// Coefficient states of a forecaster that is linear in them: C_hat = sum_{i < m} w[i] * s[i] (device pointers,
// each [B, N, k] float32).  Passed to kernels by value.
constexpr int kMaxStates = SVDC_MAX_STATES;
struct CoefStates {
  const float* s[kMaxStates];
  float w[kMaxStates];
  int m;
};

// ---- general (any-shape) kernels: general_kernels.hip -----------------------
// Optional smoothing of the residual state: R = (1 - alpha_r) prev + alpha_r (F - C V^T); prev == nullptr: plain.
struct ResidualEma {
  const void* prev = nullptr;
  float alpha_r = 1.f;
  void* packed_state = nullptr;   // matrix-core full step only: second output of the new state, as operand words
};
int32_t launch_full_step_general(const svdc_shape& s, const void* F, const float* V, void* R, float* S,
                                 float* C, float alpha, int init, ResidualEma re, hipStream_t st);
// Out = (sum_m w_m S_m) V^T + R [+ X]   (X nullable)
int32_t launch_forecast_general(const svdc_shape& s, const CoefStates& cs, const float* V, const void* R,
                                const void* X, void* Out, hipStream_t st);
// rank selection by retained energy and truncation of a fitted basis to per-block ranks
int32_t launch_select_rank(int B, int k, const float* sigma, const float* fro2, float tau, int32_t* k_star,
                           int32_t* reached, hipStream_t st);
int32_t launch_truncate_basis(const svdc_shape& s, float* V, float* sigma, const int32_t* k_star, hipStream_t st);

// ---- basis reuse and re-basing: basis_kernels.hip ------------------------------------------
bool rebase_rank_supported(int k);
int32_t launch_basis_overlap(const svdc_shape& s, const float* V_old, const float* V_new, float* M, hipStream_t st);
int32_t launch_rebase_state(const svdc_shape& s, const float* M, const float* S_in, float* S_out, hipStream_t st);
int32_t launch_basis_similarity(const svdc_shape& s, const float* V_a, const float* sigma_a, const float* V_b,
                                const float* sigma_b, float* sim_dir, float* sim_sigma, hipStream_t st);

// ---- matrix-core kernels: mfma_kernels.hip -----------------------------------
bool mfma_shape_supported(const svdc_shape& s);
size_t mfma_packed_bytes(const svdc_shape& s);
int32_t launch_pack_basis(const svdc_shape& s, const float* V, void* packed, hipStream_t st);
int32_t launch_full_step_mfma(const svdc_shape& s, const void* F, const void* packed, void* R, float* S,
                              float* C, float alpha, int init, ResidualEma re, hipStream_t st);
int32_t launch_forecast_mfma(const svdc_shape& s, const float* S, const void* packed, const void* R,
                             void* Fhat, hipStream_t st);
// Coefficient state as the cached step's operand words (bf16 high + low parts of -S, tiled per 16 rows)
size_t mfma_packed_state_bytes(const svdc_shape& s);
int32_t launch_pack_state(const svdc_shape& s, const float* S, void* Sp, hipStream_t st);
int32_t launch_forecast_packed_mfma(const svdc_shape& s, const void* Sp, const void* packed, const void* R,
                                    void* Fhat, hipStream_t st);
int32_t launch_forecast_combine_mfma(const svdc_shape& s, const CoefStates& cs, const void* packed, const void* R,
                                     const void* X, void* Out, hipStream_t st);

// ---- basis fit: fit_kernels.hip ------------------------------------------------
struct FitPlan {
  int l;          // sketch width
  int q;          // power iterations
  uint64_t seed;
  int max_sweeps; // cap on the Jacobi sweeps
  size_t off_Q, off_Z, off_Y, off_G, off_Gp, off_M, off_W, off_misc, off_info, off_jcnt, off_Qp, total;
  bool mfma;      // products with F on the matrix cores
};
bool make_fit_plan(const svdc_shape& s, const svdc_fit_params* p, FitPlan* plan);
int32_t run_fit(const svdc_shape& s, const FitPlan& plan, const void* F, float* V, float* sigma, float* fro2,
                void* workspace, hipStream_t st);

// ---- matrix-core products of the basis fit: fit_mfma_kernels.hip ------------------------
bool fit_mfma_supported(const svdc_shape& s, int l);
size_t fit_mfma_packed_q_bytes(const svdc_shape& s, int l);
// Where the operand words of Q go (projection layout): per column range (sketches wider than 128 are multiplied as two, 128 and the rest) its
// 16-column tiles KT and byte offset.  Per block the hi part, D * 16 KT elements, then the lo part; in each, word (cg, jt) of 64
// lanes x 8 bf16, lane (r, g), e  ->  Q[d = 32 cg + 8 g + e][j = 16 jt + r], 0 for columns beyond the range.
struct PackedQ {
  char* p = nullptr;
  int ranges = 0;
  int kt[2] = {0, 0};
  int64_t offset[2] = {0, 0};
};
PackedQ fit_mfma_packed_q(const svdc_shape& s, int l, void* Qp);
// Bytes of Y in the operand layout of the back-projection (written by fit_mfma_project when asked): rounded to bf16, one
// part, for bf16 features; bf16 high and low parts, two, for float32 features
size_t fit_mfma_packed_y_bytes(const svdc_shape& s, int l, int parts);
// Y = F Q;  fro_acc (nullable) += ||F||_F^2;  split: bf16 high + low parts of Q.
// Ypacked != nullptr (bf16 features: plain operands only): the result goes there in packed form and Y is not written.
void fit_mfma_project(const svdc_shape& s, int l, const void* F, const void* Qp, float* Y, void* Ypacked,
                      double* fro_acc, bool split, hipStream_t st);
// The streamed form of it, kt tiles of 16 columns and rt row tiles per workgroup (project_f32.hip, project_bf16.hip); last: accumulates
// ||F||_F^2, and for bf16 features takes both parts of Q (the others are plain).
void fit_project_stream_f32(int kt, int rt, const svdc_shape& s, int l, int ldy, const void* F, const void* Qp, float* Y, void* Yp, bool last,
                            double* fro_acc, hipStream_t st);
void fit_project_stream_bf16(int kt, int rt, const svdc_shape& s, int l, int ldy, const void* F, const void* Qp, float* Y, void* Yp, bool last,
                             double* fro_acc, hipStream_t st);
// The same with a packed basis in the place of the sketch: C = F V (nullable) and the state S (and its operand words Sp, nullable) of a
// full step.  kt from 2 on for float32 features, 4 for bf16 ones, 8 with single operands.
void step_project_stream_f32(int kt, int rt, const svdc_shape& s, const void* F, const void* packed, float* S, float* C, float alpha, int init,
                             void* Sp, hipStream_t st);
void step_project_stream_bf16(int kt, int rt, const svdc_shape& s, const void* F, const void* packed, float* S, float* C, float alpha, int init,
                              void* Sp, hipStream_t st);
// Z = F^T Y, with Y as float32 rows or (Ypacked != nullptr) in the packed form; z_clear: Z holds zeros already
void fit_mfma_backproject(const svdc_shape& s, int l, const void* F, const float* Y, const void* Ypacked, float* Z,
                          bool z_clear, hipStream_t st);
// whether the product of a power iteration accumulates into Z (several row groups), which then has to hold zeros; packed: Y's form
bool fit_mfma_backproject_accumulates(const svdc_shape& s, int l, bool packed);

}  // namespace svdc
