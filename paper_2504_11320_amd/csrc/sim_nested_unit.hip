// sim_nested_unit.hip -- instantiates the Nested WAIT kernel for unit
// thresholds and constant arrival rates.
#include "sim_nested_unit_impl.h"

namespace wsim {

hipError_t launch_nested_unit(int max_m, int max_seg, const KArgs &A, hipStream_t s) {
  // what the kernel does not read would be left out without an error
  if (!A.unit_n || A.any_trace || A.any_tv || A.any_caps || A.btrace != nullptr)
    return hipErrorInvalidValue;
  const int G = nested_group_width(max_m, max_seg);
  // the host's replica list holds 64 / G replicas per wavefront
  if (A.lanes != 64 / G || A.n_list % 64 != 0) return hipErrorInvalidValue;
  if (G == 4) return launch_unit_g<4>(A, s);
  if (G == 8) return launch_unit_g<8>(A, s);
  if (G == 16) return launch_unit_g<16>(A, s);
  if (G == 32) return launch_unit_g<32>(A, s);
  return launch_unit_g<64>(A, s);
}

}  // namespace wsim
