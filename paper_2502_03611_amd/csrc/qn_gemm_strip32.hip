// FP32 instances of the strip-form mode products.
#include "qn_gemm_strip.h"

namespace qn {
hipError_t launch_strip32(bool rows, int kind, bool in64, const StripArgs& a, hipStream_t st) {
  return rows ? strip::right<float>(a, kind, in64, st) : strip::left<float>(a, kind, st);
}
}  // namespace qn
