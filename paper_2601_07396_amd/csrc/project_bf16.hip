// Streamed projection for bf16 features: plain operands, or the sketch and the basis in two parts.
#include "project_stream.h"

namespace svdc {

void fit_project_stream_bf16(int kt, int rt, const svdc_shape& s, int l, int ldy, const void* F, const void* Qp, float* Y, void* Yp, bool last,
                            double* fro_acc, hipStream_t st) {
  const int64_t q_block = (int64_t)2 * s.D * kt * 16;
  const StreamCall<FitOut<true>> norm{s, F, Qp, q_block, {Y, (u32x4*)Yp, fro_acc, l, ldy}, st};
  const StreamCall<FitOut<false>> plain{s, F, Qp, q_block, {Y, (u32x4*)Yp, nullptr, l, ldy}, st};
  if (last) stream_by_width<bf16_t, true>(kt, rt, norm);
  else stream_by_width<bf16_t, false>(kt, rt, plain);
}

void step_project_stream_bf16(int kt, int rt, const svdc_shape& s, const void* F, const void* packed, float* S, float* C, float alpha, int init,
                             void* Sp, hipStream_t st) {
  const StreamCall<StepOut> c{s, F, packed, (int64_t)4 * s.D * kt * 16, {S, C, alpha, init, s.k, (uint2*)Sp}, st};
  if (s.precision == SVDC_PRECISE) stream_by_width<bf16_t, true, 4>(kt, rt, c);
  else stream_by_width<bf16_t, false, 8>(kt, rt, c);
}

}  // namespace svdc
