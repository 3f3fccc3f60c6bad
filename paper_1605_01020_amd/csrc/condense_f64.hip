// Element condensation, FP64 storage and MFMA (section 2.2.1, eq. LS).
#include "condense_gemm.h"

namespace iedg {
hipError_t condense_run_f64(const CondenseWork<double>& w, int lw, int ct, hipStream_t s) {
  return condense_run<double, 0>(w, lw, ct, s);
}
}  // namespace iedg
