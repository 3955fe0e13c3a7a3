// m2l_sym_f64.hip -- the reflection-reduced M2L on the FP64 matrix cores
// (FP64 plans, p >= 4).
#include "m2l_sym_kernel.h"

namespace fmm {
hipError_t launch_m2l_sym_f64(fmm_plan_s* P, hipStream_t s) {
  switch (P->p) {
    case 4: return sym::run<4, double>(P, s);
    case 5: return sym::run<5, double>(P, s);
    case 6: return sym::run<6, double>(P, s);
    case 7: return sym::run<7, double>(P, s);
    case 8: return sym::run<8, double>(P, s);
    case 9: return sym::run<9, double>(P, s);
    case 10: return sym::run<10, double>(P, s);
    case 11: return sym::run<11, double>(P, s);
    case 12: return sym::run<12, double>(P, s);
  }
  return hipErrorInvalidValue;
}
}  // namespace fmm
