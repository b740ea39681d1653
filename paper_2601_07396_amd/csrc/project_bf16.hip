// Streamed projection of the basis fit for bf16 features: plain sketch operands, or (the last product) in two parts.
#include "project_stream.h"

namespace svdc {

void fit_project_stream_bf16(int kt, int rt, const svdc_shape& s, int l, int ldy, const void* F, const void* Qp, float* Y, void* Yp, bool last,
                             double* fro_acc, hipStream_t st) {
  const StreamCall c{s, l, ldy, F, Qp, Y, (u32x4*)Yp, fro_acc, st};
  if (last) stream_by_width<bf16_t, true, true>(kt, rt, c);
  else stream_by_width<bf16_t, false, false>(kt, rt, c);
}

}  // namespace svdc
