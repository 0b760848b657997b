// The stage kernel's FP32 instantiations.
#include "stage_kernel.h"

namespace wacm {

template <>
hipError_t stage_run<float>(int mode, int bs, const StageArgs<float>& a, const wacm_schedule& s,
                            hipStream_t st) {
  return stage_run_t<float>(mode, bs, a, s, st);
}

}  // namespace wacm
