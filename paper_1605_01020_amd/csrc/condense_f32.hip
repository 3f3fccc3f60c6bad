// Element condensation, FP32 storage and FP32 MFMA with FP32 accumulation
// (section 2.2.1, eq. LS).
#include "condense_gemm.h"

namespace iedg {
hipError_t condense_run_f32(const CondenseWork<float>& w, int lw, int ct, hipStream_t s) {
  return condense_run<float, 0>(w, lw, ct, s);
}
}  // namespace iedg
