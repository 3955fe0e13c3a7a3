// m2l_sym_f32.hip -- the reflection-reduced M2L on the FP32 matrix cores
// (FMM_M2L_F32, p >= 4).
#include "m2l_sym_kernel.h"

namespace fmm {
hipError_t launch_m2l_sym_f32(fmm_plan_s* P, hipStream_t s) {
  switch (P->p) {
    case 4: return sym::run<4, float>(P, s);
    case 5: return sym::run<5, float>(P, s);
    case 6: return sym::run<6, float>(P, s);
    case 7: return sym::run<7, float>(P, s);
    case 8: return sym::run<8, float>(P, s);
    case 9: return sym::run<9, float>(P, s);
    case 10: return sym::run<10, float>(P, s);
    case 11: return sym::run<11, float>(P, s);
    case 12: return sym::run<12, float>(P, s);
  }
  return hipErrorInvalidValue;
}
}  // namespace fmm
