// Streamed projection of the basis fit for float32 features (both operands in two bf16 parts).
#include "project_stream.h"

namespace svdc {

void fit_project_stream_f32(int kt, int rt, const svdc_shape& s, int l, int ldy, const void* F, const void* Qp, float* Y, void* Yp, bool last,
                            double* fro_acc, hipStream_t st) {
  const StreamCall c{s, l, ldy, F, Qp, Y, (u32x4*)Yp, fro_acc, st};
  if (last) stream_by_width<float, true, true>(kt, rt, c);
  else stream_by_width<float, true, false>(kt, rt, c);
}

}  // namespace svdc
