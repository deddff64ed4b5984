// Whole-loop kernels with one workgroup per problem that may select on one pass over the keys in steps
// whose scores nobody sees (RowEstimates in owner_body.h).  Kernels of their own: the
// others - layers that select together, slots by rank - do not carry the code.
#include "owner_body.h"

namespace finch {

hipError_t launch_owner_loop_once_bf16(int head_dim, const LaunchParams& p, const int* step_first, int n_steps, int n_slots,
                                       hipStream_t s) {
  return launch_owner_loop_impl<false, true>(head_dim, p, step_first, n_steps, n_slots, s);
}

hipError_t set_max_lds_owner_once(size_t bytes) {
  return set_max_lds_kernels(bytes, [](int d, int q, bool rot, auto f) { with_loop_kernel<false, true>(d, q, rot, f); });
}

}  // namespace finch

#ifdef FINCH_PHASE_TIMERS
// Phase-timer build only: as finch_debug_phases, for the kernels of this file.
extern "C" int finch_debug_phases_once(unsigned long long* out, int reset) {
  if (reset) {
    const unsigned long long zero[8] = {0};
    return static_cast<int>(hipMemcpyToSymbol(HIP_SYMBOL(finch::finch_phase_ticks), zero, sizeof(zero)));
  }
  return static_cast<int>(hipMemcpyFromSymbol(out, HIP_SYMBOL(finch::finch_phase_ticks), sizeof(unsigned long long) * 8));
}
#endif
