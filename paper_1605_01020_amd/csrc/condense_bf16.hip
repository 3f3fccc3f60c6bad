// Element condensation, FP32 storage, BF16 MFMA operands with FP32
// accumulation (section 2.2.1, eq. LS).
#include "condense_gemm.h"

namespace iedg {
hipError_t condense_run_bf16(const CondenseWork<float>& w, int lw, int ct, hipStream_t s) {
  return condense_run<float, 1>(w, lw, ct, s);
}
}  // namespace iedg
