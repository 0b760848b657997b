// The stage kernel's FP64 instantiations.
#include "stage_kernel.h"

namespace wacm {

template <>
hipError_t stage_run<double>(int mode, int bs, const StageArgs<double>& a, const wacm_schedule& s,
                            hipStream_t st) {
  return stage_run_t<double>(mode, bs, a, s, st);
}

}  // namespace wacm
