// sim_nested.hip -- instantiates the Nested WAIT simulation kernel (Algorithm
// 2) for constant arrival rates and arrival lists, and picks a launch's kernel.
#include "sim_nested_impl.h"

namespace wsim {

hipError_t launch_nested(int max_m, int max_seg, const KArgs &A, hipStream_t s) {
  // time-varying rates, per-batch traces and per-stage caps run in the
  // general instantiation
  if (A.any_tv || A.btrace != nullptr || A.any_caps) return launch_nested_tv(max_m, max_seg, A, s);
  // the kernel for unit thresholds draws every arrival: launches in which a
  // job replays an arrival list run in the one for any thresholds
  if (A.unit_n && !A.any_trace) return launch_nested_unit(max_m, max_seg, A, s);
  return launch_nested_k<false>(max_m, max_seg, A, s);
}

}  // namespace wsim
