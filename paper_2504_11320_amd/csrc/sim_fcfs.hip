// sim_fcfs.hip -- instantiates the FCFS kernel for known output lengths
// (Section 4.1) with constant arrival rates.
#include "sim_fcfs_impl.h"

namespace wsim {

hipError_t launch_fcfs(int max_m, const KArgs &A, hipStream_t s) {
  // arrival lists, time-varying rates and per-batch traces run in the general
  // instantiation
  if (A.any_trace || A.any_tv || A.btrace != nullptr) return launch_fcfs_tv(max_m, A, s);
  return launch_fcfs_k<false, false>(max_m, A, s);
}

}  // namespace wsim
