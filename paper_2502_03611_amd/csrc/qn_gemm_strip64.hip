// FP64 instances of the strip-form mode products.
#include "qn_gemm_strip.h"

namespace qn {
hipError_t launch_strip64(bool rows, int kind, const StripArgs& a, hipStream_t st) {
  return rows ? strip::right<double>(a, kind, true, st) : strip::left<double>(a, kind, st);
}
}  // namespace qn
