// sim_fcfs_tv.hip -- instantiates the FCFS kernel for known output lengths for
// launches with time-varying arrival rates, arrival lists or a per-batch trace.
#include "sim_fcfs_impl.h"

namespace wsim {

hipError_t launch_fcfs_tv(int max_m, const KArgs &A, hipStream_t s) {
  if (A.any_trace) return launch_fcfs_k<true, true>(max_m, A, s);
  return launch_fcfs_k<true, false>(max_m, A, s);
}

}  // namespace wsim
