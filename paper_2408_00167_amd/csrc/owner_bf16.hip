// Kernels with one workgroup per problem, rows from the prompt only (the method's
// own conditioning; Method: prompt-guided sub-matrix).  The code is in owner_body.h.
#include <algorithm>

#include "owner_body.h"

namespace finch {

// Dynamic LDS the kernels need for `row_chunk` staged prompt rows (a multiple of 32, at most
// kOwnerMaxRowChunk): the rows, then the larger of {pass-1 statistics + lse + block counter} and the
// selection scratch.  That is as large as the batch's candidates and kept rows (n_max, r_max;
// nothing if only scores are wanted) ask for, at most kOwnerSelectBytes: the kernels for narrow heads
// and few rows have registers for two workgroups a compute unit, and 60 KB for each leave room for one.
// 1024 problems, 64 channels, 700 candidates: scores 39.3 us with room for any selection, 30.3 with
// what is needed; whole steps 58.6 and 45.2 (128 registers in place of 143 among it).
size_t owner_lds_bytes(int head_dim, int row_chunk, int n_max, int r_max, bool rank_order, bool stages) {
  const size_t q = static_cast<size_t>(row_chunk) * (head_dim * 2 + 16);
  const size_t scoring = static_cast<size_t>(row_chunk) * (kOwnWaves * 8 + 4) + 16;
  if (!stages) return q + scoring;
  const size_t kept = (static_cast<size_t>(r_max) + kSelIdxPad) * 4;
  const size_t keys = static_cast<size_t>(std::min(n_max, kOwnThreads * kSelRegKeys)) * 4;
  size_t want = std::max(sizeof(SelLds) + kept, scoring) + 16 + keys;  // (see own_sel_keys)
  if (rank_order) {
    size_t records = 64;
    while (records < static_cast<size_t>(std::min(r_max, kOwnerRankRows))) records <<= 1;
    want = std::max(want, sizeof(SelLds) + kept + 8 + 8 * records);
  }
  return q + std::max(scoring, std::min(want, sizeof(SelLds) + kOwnerSelectBytes));
}

hipError_t launch_owner_bf16(int head_dim, const LaunchParams& p, int stages, hipStream_t s) {
  return launch_owner_impl<false>(head_dim, p, stages, s);
}

hipError_t launch_owner_loop_bf16(int head_dim, const LaunchParams& p, const int* step_first, int n_steps,
                                  int n_slots, hipStream_t s) {
  if (p.est_words > 0) return launch_owner_loop_once_bf16(head_dim, p, step_first, n_steps, n_slots, s);
  return launch_owner_loop_impl<false, false>(head_dim, p, step_first, n_steps, n_slots, s);
}

hipError_t set_max_lds_owner(size_t bytes) {
  const hipError_t e = set_max_lds_owner_impl<false>(bytes);
  return e == hipSuccess ? set_max_lds_owner_once(bytes) : e;
}

}  // namespace finch

#ifdef FINCH_PHASE_TIMERS
extern "C" int finch_debug_phases_once(unsigned long long* out, int reset);
// Phase-timer build only: the totals of the kernels for prompt rows only (of this file and of
// owner_once_bf16.hip together) on the current device, 8 words of wall-clock ticks (10 ns); reset != 0
// clears them instead.
extern "C" int finch_debug_phases(unsigned long long* out, int reset) {
  if (reset) {
    const unsigned long long zero[8] = {0};
    const int e = finch_debug_phases_once(out, reset);
    return e ? e : static_cast<int>(hipMemcpyToSymbol(HIP_SYMBOL(finch::finch_phase_ticks), zero, sizeof(zero)));
  }
  unsigned long long once[8];
  int e = finch_debug_phases_once(once, 0);
  if (!e) e = static_cast<int>(hipMemcpyFromSymbol(out, HIP_SYMBOL(finch::finch_phase_ticks), sizeof(unsigned long long) * 8));
  for (int i = 0; !e && i < 8; ++i) out[i] += once[i];
  return e;
}
#endif
