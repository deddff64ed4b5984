// Kernels with one workgroup per problem whose rows include the chunk's own tokens
// (the paper's ablation of the conditioning: document-only or document + prompt
// self-attention, with the causal mask and the Method's normalisation step).  The
// code is in owner_body.h.
#include "owner_body.h"

namespace finch {

hipError_t launch_owner_doc_bf16(int head_dim, const LaunchParams& p, int stages, hipStream_t s) {
  return launch_owner_impl<true>(head_dim, p, stages, s);
}

hipError_t launch_owner_loop_doc_bf16(int head_dim, const LaunchParams& p, const int* step_first,
                                      int n_steps, int n_slots, hipStream_t s) {
  return launch_owner_loop_impl<true, false>(head_dim, p, step_first, n_steps, n_slots, s);
}

hipError_t set_max_lds_owner_doc(size_t bytes) { return set_max_lds_owner_impl<true>(bytes); }

}  // namespace finch

#ifdef FINCH_PHASE_TIMERS
// Phase-timer build only: as finch_debug_phases, for the kernels of this file.
extern "C" int finch_debug_phases_doc(unsigned long long* out, int reset) {
  if (reset) {
    const unsigned long long zero[8] = {0};
    return static_cast<int>(hipMemcpyToSymbol(HIP_SYMBOL(finch::finch_phase_ticks), zero, sizeof(zero)));
  }
  return static_cast<int>(hipMemcpyFromSymbol(out, HIP_SYMBOL(finch::finch_phase_ticks), sizeof(unsigned long long) * 8));
}
#endif
