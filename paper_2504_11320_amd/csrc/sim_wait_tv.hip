// sim_wait_tv.hip -- instantiates the WAIT kernel (Algorithm 1) for launches
// with time-varying arrival rates, arrival lists, per-stage caps or a
// per-batch trace.
#include "sim_wait_impl.h"

namespace wsim {

hipError_t launch_wait_tv(int max_m, const KArgs &A, hipStream_t s) {
  if (A.any_trace) return launch_wait_k<true, false, true>(max_m, A, s);
  return launch_wait_k<true, false, false>(max_m, A, s);
}

}  // namespace wsim
