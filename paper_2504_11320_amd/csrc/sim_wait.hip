// sim_wait.hip -- instantiates the WAIT kernel (Algorithm 1) with constant
// arrival rates.
#include "sim_wait_impl.h"

namespace wsim {

hipError_t launch_wait(int max_m, const KArgs &A, hipStream_t s) {
  // arrival lists, time-varying rates, per-batch traces and per-stage caps
  // run in the general instantiation
  if (A.any_trace || A.any_tv || A.btrace != nullptr || A.any_caps)
    return launch_wait_tv(max_m, A, s);
  if (A.unit_n) return launch_wait_k<false, true, false>(max_m, A, s);
  return launch_wait_k<false, false, false>(max_m, A, s);
}

}  // namespace wsim
